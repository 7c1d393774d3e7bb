"""Every allocation of a route switch fails once; see test_route_switch_failures.py."""
import sys

from paper_2302_09708_amd import inputs
from tests._host import Host


def main(stub, precision, to_stencil):
    prob = inputs.small_problem(n=(27, 30, 26), h=(0.3, 0.3, 0.3), bc=(0, 0, 1), n_atoms=20, nproj_per_atom=4, seed=17)
    h = Host(stub, prob, int(precision), 60)
    if int(to_stencil):
        h.h.chefsi_set_projector_pass(False)
    what = [("apply", 6), ("filter", 6), ("apply", 60), ("filter", 60), ("apply", 2)]
    before, size = [h.kernels(*w) for w in what], h.h.device_bytes()
    failed = 0
    for k in range(1, 100):
        h.stub.stub_fail(k)
        st = h.status(lambda: h.h.chefsi_set_projector_pass(bool(int(to_stencil))))
        h.stub.stub_fail(0)
        if st == 0:
            break
        failed += 1
        assert st == h.cs.ERR_OOM, st
        assert [h.kernels(*w) for w in what] == before, f"another route after failed allocation {k}"
        assert h.stub.stub_null_tables() == 0, f"null tables after failed allocation {k}"
        assert h.h.device_bytes() == size, f"device bytes after failed allocation {k}"
    assert failed > 2
    after = [h.kernels(*w) for w in what]
    assert h.stub.stub_null_tables() == 0
    assert after != before
    assert any("nl_band" in n for n in after[1]) == (not int(to_stencil))
    print(failed)


if __name__ == "__main__":
    main(*sys.argv[1:])
