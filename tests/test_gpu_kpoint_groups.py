"""The complex band pass in groups of eight and of four orbitals: an orbital's sums do not depend
on the group it is in, so a wide block's columns are those of a narrow one, bit for bit."""
import numpy as np
import pytest

from oracle import kpoint as ok
from paper_2302_09708_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    from paper_2302_09708_amd import chefsi
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    chefsi.load()
    return chefsi


# few and many projectors per point (regions full by points, by entries, by projectors)
@pytest.mark.parametrize("n_atoms,nproj", [(2, 1), (40, 4), (90, 4)])
def test_groups(cs, n_atoms, nproj):
    print(f"k-point groups {n_atoms} atoms x {nproj}", flush=True)
    prob = inputs.small_problem(n=(30, 26, 28), h=(0.3, 0.3, 0.3), bc=(0, 0, 1), n_atoms=n_atoms, nproj_per_atom=nproj,
                                seed=31)
    k, img, wide = (0.4, -0.7, 0.0), inputs.support_images(prob), 1201
    hw, hn = cs.KPoint(prob, k, img, max_ns=wide), cs.KPoint(prob, k, img, max_ns=5)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    X = torch.randn((wide, prob.nd), generator=g, device="cuda", dtype=torch.complex128)
    Y = torch.empty_like(X)
    hw.apply_h(X, Y, wide, hw.workspace(wide))
    wn = hn.workspace(5)
    for v in (0, 600, wide - 5):
        Yn = torch.empty((5, prob.nd), dtype=torch.complex128, device="cuda")
        hn.apply_h(X[v:v + 5].clone(), Yn, 5, wn)
        assert torch.equal(Yn, Y[v:v + 5])
    x = X[:5].cpu().numpy().T
    ref = ok.apply_h_k(prob, img, k, x)
    assert np.abs(Y[:5].cpu().numpy().T - ref).max() <= 1e-12 * np.abs(ref).max()
    hw.close()
    hn.close()
