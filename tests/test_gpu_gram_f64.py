"""FP64 projection matrices at the edges of the Gram kernel's tiles, K chunks and dispatch."""
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


def _project(cs, prob, X, ns):
    """(Hs, Ms, Y) of block X: Y = H X is the block Hs is formed from."""
    h = cs.Handle(prob, precision=cs.FP64, max_ns=ns)
    ws = cs.workspace(h, ns)
    ws.fill_(0xff)  # NaN in every double: nothing may be read that was not written
    Hs = torch.full((ns, ns), float("nan"), device="cuda", dtype=torch.float64)
    Ms, Y = torch.full_like(Hs, float("nan")), torch.empty_like(X)
    h.chefsi_project(X, ns, Hs, Ms, ws)
    h.chefsi_apply_h(X, Y, ns, ws)
    h.close()
    return Hs.cpu().numpy(), Ms.cpu().numpy(), Y.cpu().numpy()


# below one step, one ragged step, whole steps, a chunk's remainder; an odd column stride
@pytest.mark.parametrize("n", [(5, 5, 7), (8, 8, 8), (11, 13, 15), (24, 22, 23)])
def test_tile_edges(cs, n):
    prob = inputs.small_problem(n=n, h=(0.5, 0.5, 0.5), bc=(1, 1, 1), n_atoms=1, nproj_per_atom=4, seed=5)
    for ns in (1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128, 129, 200, 257):
        if ns > prob.nd:
            continue
        print(f"gram f64 {n} ns {ns}", flush=True)
        X = torch.from_numpy(np.random.default_rng(ns).standard_normal((ns, prob.nd))).cuda()
        Hs, Ms, Y = _project(cs, prob, X, ns)
        x = X.cpu().numpy()
        # two FP64 sums of nd products, each within nd 2^-53 |x|^T |y| of the exact one
        for C, y in ((Hs, Y), (Ms, x)):
            ref = x @ y.T
            bound = 2 * prob.nd * 2.0**-53 * (np.abs(x) @ np.abs(y).T)
            up = np.triu(np.ones_like(ref, dtype=bool))
            assert (np.abs(C - ref) <= bound)[up].all()
            assert np.array_equal(C, C.T)


@pytest.mark.parametrize("ns", [512, 513])
def test_strides_of_2_mib(cs, ns):
    """64^3 points: the columns of 513 orbitals go to the library's product, of 512 do not."""
    print(f"gram f64 64^3 ns {ns}", flush=True)
    prob = inputs.small_problem(n=(64, 64, 64), h=(0.5, 0.5, 0.5), bc=(0, 0, 0), n_atoms=1, nproj_per_atom=1, seed=5)
    g = torch.Generator(device="cuda")
    g.manual_seed(ns)
    X = torch.randn((ns, prob.nd), generator=g, device="cuda", dtype=torch.float64)
    Hs, Ms, Y = _project(cs, prob, X, ns)
    x = X.cpu().numpy()
    for C, y in ((Hs, Y), (Ms, x)):
        cols = [0, 1, 63, 64, 300, 511, ns - 1]
        ref, size = x @ y[cols].T, np.abs(x) @ np.abs(y[cols]).T
        for k, j in enumerate(cols):
            assert (np.abs(C[:j + 1, j] - ref[:j + 1, k]) <= 2 * prob.nd * 2.0**-53 * size[:j + 1, k]).all()
        assert np.array_equal(C, C.T)
