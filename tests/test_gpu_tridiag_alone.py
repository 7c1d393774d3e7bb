"""The tridiagonalisation where a wait between its workgroups is not met: the wait's bound is set to
one look from the host, so the launch gives up and one workgroup does the reduction again.

Tolerances as for any backward stable reduction: Q T Q^T - A and Q^T Q - I are at most about n eps
|A| and n eps; the factor 10 covers the constants."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = 2.0 ** -52
LAUNCH = "_ZN6chefsi14launch_tridiagEPdiS0_S0_S0_PvPiP12ihipStream_tj"  # chefsi::launch_tridiag


@pytest.fixture(scope="module")
def cs():
    from paper_2302_09708_amd import chefsi
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    chefsi.load()
    return chefsi


def _q(v, tau):
    """H_{n-1} ... H_1 with H_m = I - tau[m-1] u u^T, u = (column m above the superdiagonal, 1, 0 ...)."""
    n = v.shape[0]
    q = np.eye(n)
    for m in range(n - 1, 0, -1):
        u = np.zeros(n)
        u[:m - 1] = v[:m - 1, m]
        u[m - 1] = 1.0
        q -= tau[m - 1] * np.outer(q @ u, u)
    return q


@pytest.mark.parametrize("n", [129, 130, 257, 600, 1025, 1408])
@pytest.mark.parametrize("polls", [1, 40])
def test_reduction_after_an_unmet_wait(cs, n, polls):
    print(f"tridiag alone n {n} polls {polls}", flush=True)
    launch = getattr(cs.load(), LAUNCH)
    launch.argtypes = [ctypes.c_void_p, ctypes.c_int] + [ctypes.c_void_p] * 6 + [ctypes.c_uint]
    rng = np.random.Generator(np.random.PCG64(n + polls))
    a = rng.standard_normal((n, n))
    a = a + a.T
    a[: n // 3, n // 3:] = 0.0  # columns that need no reflector
    a[n // 3:, : n // 3] = 0.0
    A = torch.from_numpy(a.copy()).cuda()
    D, E, tau = (torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3))
    msg = torch.empty(8 * n, dtype=torch.int64, device="cuda")
    info = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert launch(A.data_ptr(), n, D.data_ptr(), E.data_ptr(), tau.data_ptr(), msg.data_ptr(), info.data_ptr(), 0,
                  polls) == 0
    torch.cuda.synchronize()
    assert int(info[0]) == 0
    v = A.cpu().numpy().T  # column-major
    d, e, t = (x.cpu().numpy() for x in (D, E, tau))
    q = _q(v, t)
    T = np.diag(d) + np.diag(e[:-1], 1) + np.diag(e[:-1], -1)
    scale = np.linalg.norm(a, 2)
    assert np.abs(q.T @ q - np.eye(n)).max() <= 10.0 * n * EPS
    assert np.abs(q @ T @ q.T - a).max() <= 10.0 * n * EPS * scale
