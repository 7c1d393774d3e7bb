"""The split-bf16 rotation around whole and ragged 32-column stages, even and odd in number."""
import numpy as np
import pytest

from paper_2302_09708_amd import inputs
from tests._gpu import dev, dev_square, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U16, U24 = 2.0 ** -16, 2.0 ** -24


@pytest.fixture(scope="module")
def cs():
    from paper_2302_09708_amd import chefsi
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    chefsi.load()
    return chefsi


# points: below one wave's 64, one block's 256, and four beyond
@pytest.mark.parametrize("n", [(7, 7, 1), (8, 8, 4), (13, 5, 4)])
@pytest.mark.parametrize("ns", [31, 32, 33, 63, 64, 65, 96, 128, 129, 160])
def test_stages(cs, n, ns):
    print(f"rotate {n} ns {ns}", flush=True)
    prob = inputs.small_problem(n=n, bc=(1, 1, 1), n_atoms=0, nproj_per_atom=0, seed=1)
    if ns > prob.nd:
        pytest.skip("fewer points than orbitals")
    rng = np.random.default_rng(ns)
    X = rng.standard_normal((prob.nd, ns)).astype(np.float32).astype(np.float64)
    Z = rng.standard_normal((ns, ns))
    h = cs.Handle(prob, precision=cs.MIXED, max_ns=ns)
    ws = cs.workspace(h, ns)
    ws.fill_(0xff)
    Xd = dev(X, "float32")
    h.chefsi_rotate(Xd, dev_square(Z), ns, ws)
    torch.cuda.synchronize()
    ref = X @ Z
    # three of the four products of two-term splits (3.1 2^-16 of |X| |Z|), FP32 sums of ns terms
    # and the stored result's rounding
    bound = (3.1 * U16 + ns * U24) * (np.abs(X) @ np.abs(Z)) + U24 * np.abs(ref)
    assert np.all(np.abs(host(Xd) - ref) <= bound)
    h.close()
