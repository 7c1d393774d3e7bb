"""Projector routes of one handle's calls, by the kernels launched; see test_call_routes.py."""
import sys

import numpy as np

from paper_2302_09708_amd import inputs
from tests._host import Host


def lattice(n, m):
    """m^3 atoms far enough apart that no point lies in two supports (h = 0.3)."""
    size = np.array(n) * 0.3
    pos = np.array([[(a + 0.5) / m * s for a, s in zip(i, size)] for i in np.ndindex(m, m, m)])
    h, bc = (0.3, 0.3, 0.3), (0, 0, 0)
    sp, si, npj, chi, gam = inputs.kb_projectors(n, h, bc, pos, 4)
    return inputs.Problem(n, h, bc, 12, np.zeros(int(np.prod(n))), pos, sp, si, npj, chi, gam, name="lattice")


PROBLEMS = {
    "sparse": lambda: lattice((40, 40, 40), 1),            # 0.8 % of 64000 points touched
    "dense": lambda: lattice((40, 40, 40), 3),             # 22 %
    "overlap": lambda: inputs.small_problem(n=(27, 30, 26), h=(0.3, 0.3, 0.3), bc=(0, 0, 1), n_atoms=20, nproj_per_atom=4,
                                            seed=17),
    "weak": lambda: inputs.small_problem(n=(42, 40, 30), h=(0.3, 0.3, 0.3), bc=(0, 0, 0), n_atoms=6, nproj_per_atom=4,
                                         seed=5),
    "small": lambda: inputs.small_problem(n=(27, 30, 26), h=(0.3, 0.3, 0.3), bc=(0, 0, 1), n_atoms=1, nproj_per_atom=4,
                                          seed=17),
}


def main(stub, problem, precision, max_ns, *widths):
    prob = PROBLEMS[problem]()
    entries = np.zeros(prob.nd, dtype=int)
    for k in range(prob.n_atoms):
        np.add.at(entries, prob.supp_idx[prob.supp_ptr[k]:prob.supp_ptr[k + 1]], prob.nproj[k])
    print((entries > 0).sum(), (entries > 4).sum(), prob.nd)
    h = Host(stub, prob, int(precision), int(max_ns))
    for ns in map(int, widths):
        band = [any("nl_band_kernel" in k for k in h.kernels(w, ns)) for w in ("apply", "filter")]
        both = [any("nl_project" in k or "nl_scatter" in k for k in h.kernels(w, ns)) for w in ("apply", "filter")]
        assert band != both, (band, both)
        assert all(b != r for b, r in zip(band, both))
        print(ns, *map(int, band))
    assert h.stub.stub_null_tables() == 0


if __name__ == "__main__":
    main(*sys.argv[1:])
