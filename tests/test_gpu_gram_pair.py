"""Split-bf16 projection over units of 256 x (128 + 128) results at the edges of its units,
row groups and FP32 sums, against the FP64 products of the same blocks.

Tolerance (element-wise): 3.1 2^-16 from the split (representation of both operands and the
dropped lo lo product) plus K 2^-24 from an FP32 sum of K terms, times sum |x y|; an FP32
sum spans at most 16384 rows."""
import numpy as np
import pytest

from paper_2302_09708_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    from paper_2302_09708_amd import chefsi
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    chefsi.load()
    return chefsi


# rows and widths: one odd and one even count of column blocks, a last block of one column, a
# K chunk of an odd number of 16 rows, chunks longer than one FP32 sum, a last stage of one row
@pytest.mark.parametrize("n,ns", [((60, 61, 71), 577), ((64, 64, 65), 640), ((97, 75, 49), 641), ((73, 70, 93), 513),
                                  ((60, 60, 100), 1281)])
def test_units(cs, n, ns):
    print(f"gram pair n {n} ns {ns}", flush=True)
    prob = inputs.small_problem(n=n, h=(0.3, 0.3, 0.3), bc=(0, 0, 1), n_atoms=3, nproj_per_atom=4, seed=5)
    h = cs.Handle(prob, precision=cs.MIXED, max_ns=ns)
    ws = cs.workspace(h, ns)
    g = torch.Generator(device="cuda")
    g.manual_seed(77)
    X = torch.randn((ns, prob.nd), generator=g, device="cuda", dtype=torch.float32)
    Y = torch.empty_like(X)
    h.chefsi_apply_h(X, Y, ns, ws)
    Hs = torch.empty((ns, ns), dtype=torch.float64, device="cuda")
    Ms = torch.empty_like(Hs)
    h.chefsi_project(X, ns, Hs, Ms, ws)
    first = (Hs.clone(), Ms.clone())
    h.chefsi_project(X, ns, Hs, Ms, ws)
    assert torch.equal(Hs, first[0]) and torch.equal(Ms, first[1])
    assert torch.equal(Hs, Hs.T) and torch.equal(Ms, Ms.T)
    tol = 3.1 * 2.0 ** -16 + min(prob.nd, 16384) * 2.0 ** -24
    X64 = X.double()
    for got, other in ((Ms, X64), (Hs, Y.double())):
        err = torch.triu((got - X64 @ other.T).abs())  # C(i, j), i <= j, from row i of X
        assert bool((err <= tol * (X64.abs() @ other.abs().T)).all())
    h.close()
