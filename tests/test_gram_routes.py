"""Which FP64 projections take the library's product: by the launches of the host code on a host
stand-in for HIP, on both sides of the limits (strides of 2 MiB and of more, tiles of 128 columns)."""
import pytest

from tests import _host


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return _host.build_stub(tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("n,library,own", [
    ((64, 64, 64), [513, 600], [100, 384, 500, 512]),                             # 2 MiB
    ((64, 128, 64), [353, 384, 449, 512, 513], [100, 300, 352, 385, 400, 448]),   # 4 MiB
    ((96, 128, 64), [384, 500, 1000], [256, 400]),                                # 6 MiB
    ((64, 96, 64), [], [384, 500, 512, 600, 900]),                                # 3 MiB
    ((72, 72, 72), [], [384, 600]),
])
def test_routes(stub, n, library, own):
    out = _host.run(stub, "tests.gram_routes_child", *n, *library, *own)
    assert {int(a): int(b) for a, b in (line.split() for line in out.splitlines())} == {**dict.fromkeys(library, 1),
                                                                                      **dict.fromkeys(own, 0)}
