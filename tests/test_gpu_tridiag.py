"""Subspace eigensolve at the edges of its tridiagonalisation kernel: row widths around every
64-wide chunk count, one workgroup and several, columns that need no reflector, and solves
that run side by side.

Tolerances: a backward stable solve of a scaled pencil moves the eigenvalues by at most about
n eps cond(Ms) |Hs| / min Ms, and the same bounds Z^T Ms Z - I and the residual; the factor
10 covers the constants of the stages (Cholesky, two triangular solves, eigensolve)."""
import threading

import numpy as np
import pytest
import scipy.linalg

from paper_2302_09708_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def cs():
    from paper_2302_09708_amd import chefsi
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    chefsi.load()
    return chefsi


def _pencil(n, kind, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    a = rng.standard_normal((n, 2 * n + 8)) / np.sqrt(2 * n + 8)
    ms = a @ a.T
    if kind == "diagonal":  # no reflector in any column
        return np.diag(rng.uniform(-1.0, 20.0, n)), np.diag(rng.uniform(0.5, 2.0, n))
    h = rng.standard_normal((n, n))
    h = h + h.T
    if kind == "blocks":  # blocks of three: columns whose part above the diagonal is zero
        i = np.arange(n) // 3
        h[i[:, None] != i[None, :]] = 0.0
        ms = np.eye(n)
    return h, ms


def _solve(cs, handle, h, ms, ws, stream=None):
    n = h.shape[0]
    Hs = torch.from_numpy(h.copy()).cuda()
    Ms = torch.from_numpy(ms.copy()).cuda()
    D = torch.empty(n, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    handle.chefsi_eigh(Hs, Ms, D, n, ws, stream=stream)
    torch.cuda.synchronize()
    return D.cpu().numpy(), Hs.cpu().numpy()  # row j = eigenvector j


SIZES = [1, 2, 3, 63, 64, 65, 127, 128, 129, 130, 255, 256, 257, 384, 385, 512, 513, 640, 641, 832, 833, 1024, 1025, 1216,
         1217, 1408]


@pytest.mark.parametrize("n,kind", [(n, k) for n in SIZES for k in ("full", "blocks", "diagonal")
                                    if k == "full" or n <= 641])
def test_sizes(cs, n, kind):
    print(f"eigh n {n} {kind}", flush=True)
    h, ms = _pencil(n, kind, 900 + n)
    prob = inputs.small_problem(n=(12, 12, 12), n_atoms=0, nproj_per_atom=0, seed=1)
    handle = cs.Handle(prob, precision=cs.FP64, max_ns=n)
    ws = cs.workspace(handle, n)
    d, z = _solve(cs, handle, h, ms, ws)
    d2, z2 = _solve(cs, handle, h, ms, ws)
    assert np.array_equal(d, d2) and np.array_equal(z, z2)
    ref = scipy.linalg.eigh(h, ms, eigvals_only=True)
    lam = np.linalg.eigvalsh(ms)
    tol = 10.0 * n * EPS * (lam[-1] / lam[0])
    scale = np.linalg.norm(h, 2) / lam[0]
    assert np.all(np.diff(d) >= 0.0)
    assert np.abs(d - ref).max() <= tol * scale
    assert np.abs(z @ ms @ z.T - np.eye(n)).max() <= tol
    assert np.abs(z @ h - d[:, None] * (z @ ms)).max() <= tol * scale * np.sqrt(lam[-1])
    handle.close()


def test_side_by_side(cs):
    """Four threads on their own streams and handles: every solve's bits are those of the solve
    alone, whatever shares the GPU."""
    ns = [40, 150, 300, 400]
    prob = inputs.small_problem(n=(12, 12, 12), n_atoms=0, nproj_per_atom=0, seed=1)
    jobs = []
    for n in ns:
        handle = cs.Handle(prob, precision=cs.FP64, max_ns=n)
        h, ms = _pencil(n, "full", 70 + n)
        jobs.append((handle, torch.from_numpy(h).cuda(), torch.from_numpy(ms).cuda(), cs.workspace(handle, n),
                     torch.cuda.Stream()))

    def run(job, times, out):
        handle, h, ms, ws, stream = job
        with torch.cuda.stream(stream):
            for _ in range(times):
                Hs, Ms = h.clone(), ms.clone()
                D = torch.empty(h.shape[0], dtype=torch.float64, device="cuda")
                handle.chefsi_eigh(Hs, Ms, D, h.shape[0], ws, stream=stream)
                out.append((D, Hs))
        stream.synchronize()

    alone = []
    for job in jobs:
        out = []
        run(job, 1, out)
        alone.append(out[0])
    torch.cuda.synchronize()
    outs = [[] for _ in jobs]
    threads = [threading.Thread(target=run, args=(job, 8, out)) for job, out in zip(jobs, outs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for (d, z), out in zip(alone, outs):
        assert len(out) == 8
        for d2, z2 in out:
            assert torch.equal(d, d2) and torch.equal(z, z2)
    for job in jobs:
        job[0].close()
