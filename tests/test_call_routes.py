"""Which calls of a handle as created take the band pass: by the kernels that the library's host code
launches on a host stand-in for HIP, on both sides of every limit of the rule."""
import pytest

from tests import _host

FP64, MIXED = 0, 1


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return _host.build_stub(tmp_path_factory.mktemp("stub"))


# problem, precision, max_ns, {ns: (band pass in a single application, in a filter)}
@pytest.mark.parametrize("problem,precision,max_ns,calls", [
    # no overlap, few points touched: from 2^23 values on, whatever the handle could hold
    ("sparse", FP64, 400, {1: (0, 0), 8: (0, 0), 131: (0, 0), 132: (1, 1), 400: (1, 1)}),
    ("sparse", MIXED, 400, {1: (0, 0), 131: (0, 0), 132: (0, 1), 400: (0, 1)}),
    ("sparse", FP64, 131, {131: (0, 0)}),
    # more touched: never for single applications; mixed filters from 2^27 values
    ("dense", FP64, 400, {1: (0, 0), 131: (0, 0), 132: (0, 1), 400: (0, 1)}),
    ("dense", MIXED, 400, {1: (0, 0), 132: (0, 0), 400: (0, 0)}),
    # overlapping supports: from four orbitals on
    ("overlap", FP64, 60, {1: (0, 0), 3: (0, 0), 4: (1, 1), 60: (1, 1)}),
    ("overlap", FP64, 8, {8: (0, 0)}),  # fewer than 2^18 values
    ("overlap", MIXED, 60, {1: (0, 0), 3: (0, 0), 4: (0, 1), 60: (0, 1)}),
    ("overlap", MIXED, 3, {3: (0, 0)}),
    # a few overlapping points: from 3 2^20 values in FP64, four orbitals in mixed filters
    ("weak", FP64, 120, {1: (0, 0), 62: (0, 0), 63: (1, 1), 120: (1, 1)}),
    ("weak", MIXED, 120, {3: (0, 0), 4: (0, 1)}),
    # 2^14 to 2^15 points without overlap: with 2^20 values in the widest call
    ("small", FP64, 60, {3: (0, 0), 6: (1, 1), 60: (1, 1)}),
    ("small", FP64, 40, {40: (0, 0)}),
])
def test_routes(stub, problem, precision, max_ns, calls):
    out = _host.run(stub, "tests.call_routes_child", problem, precision, max_ns, *calls).splitlines()
    touched, scattered, nd = map(int, out[0].split())
    assert {"sparse": scattered == 0 and 5 * touched <= nd, "dense": scattered == 0 and 5 * touched > nd,
            "overlap": scattered >= 512, "weak": 0 < scattered < 512, "small": scattered == 0 and 1 << 14 <= nd < 1 << 15}[problem]
    got = {int(ns): (int(a), int(f)) for ns, a, f in (line.split() for line in out[1:])}
    assert got == calls
