"""A switch of the projector route that fails for want of memory leaves the handle on its route, with
its tables: the library's host code runs on a host stand-in for HIP whose k-th allocation fails, for
every k, and the kernels launched afterwards are those launched before."""
import pytest

from tests import _host


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return _host.build_stub(tmp_path_factory.mktemp("stub"))


# handles as created have the band pass beside the records; to the records: from the band pass alone
@pytest.mark.parametrize("precision,to_stencil", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_failed_switch(stub, precision, to_stencil):
    assert int(_host.run(stub, "tests.route_switch_child", precision, to_stencil)) > 2
