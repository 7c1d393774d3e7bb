"""FP64 projections by the library's product or the own kernel; see test_gram_routes.py."""
import sys

from paper_2302_09708_amd import inputs
from tests._host import Host


def main(stub, nx, ny, nz, *widths):
    prob = inputs.small_problem(n=(int(nx), int(ny), int(nz)), h=(0.3, 0.3, 0.3), bc=(0, 0, 0), n_atoms=0, nproj_per_atom=0)
    h = Host(stub, prob, 0, 1000)
    for ns in map(int, widths):
        names = h.kernels("project", ns)
        own, library = any("gram_both" in k for k in names), any("dgemm" in k for k in names)
        assert own != library, names
        print(ns, int(library))


if __name__ == "__main__":
    main(*sys.argv[1:])
