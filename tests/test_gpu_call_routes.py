"""Calls on both sides of the limit from which a handle as created takes the band pass: against the
oracle, and bit for bit those of a handle on that route alone; a bound on a wide handle."""
import numpy as np
import pytest

from oracle import chefsi as oc
from oracle.hamiltonian import apply_h
from paper_2302_09708_amd import inputs
from tests._gpu import dev, host, stencil_scale

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    from paper_2302_09708_amd import chefsi
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    chefsi.load()
    return chefsi


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_both_sides(cs, prec):
    """40^3 points, one atom: from 132 orbitals on (2^23 values)."""
    print(f"call routes {prec}", flush=True)
    prob = inputs.small_problem(n=(40, 40, 40), h=(0.3, 0.3, 0.3), bc=(0, 0, 0), n_atoms=1, nproj_per_atom=4, seed=3)
    dt, p = ("float64", cs.FP64) if prec == "fp64" else ("float32", cs.MIXED)
    ns, degree = 132, 3
    X = np.random.default_rng(8).standard_normal((prob.nd, ns)).astype(dt)
    lo, cut, hi = oc.spectral_bounds(prob)
    ref = apply_h(prob, X.astype(np.float64))
    fref = oc.chebyshev_filter(prob, X.astype(np.float64), degree, lo, cut, hi)
    tol = 1e-12 if prec == "fp64" else 2e-6

    def run(handle, k):
        ws = cs.workspace(handle, k)
        Y = torch.zeros(k, prob.nd, dtype=getattr(torch, dt), device="cuda")
        handle.chefsi_apply_h(dev(X[:, :k], dt), Y, k, ws)
        F = dev(X[:, :k], dt)
        handle.chefsi_filter(F, k, degree, lo, cut, hi, ws)
        return Y, F

    h = cs.Handle(prob, precision=p, max_ns=ns)
    got = {k: run(h, k) for k in (131, 132)}
    forced = {}
    for in_stencil in (True, False):
        h.chefsi_set_projector_pass(in_stencil)
        forced[in_stencil] = {k: run(h, k) for k in (131, 132)}
    for k, (y, f) in got.items():
        assert np.abs(host(y) - ref[:, :k]).max() <= tol * stencil_scale(prob) * np.abs(X).max()
        assert np.abs(host(f) - fref[:, :k]).max() <= tol * degree * np.abs(X).max()
        assert torch.equal(y, forced[not (k == 132 and prec == "fp64")][k][0])
        assert torch.equal(f, forced[k != 132][k][1])
    h.close()


def test_bound_on_a_wide_handle(cs):
    """The Lanczos bound takes one orbital: the records, whatever the handle is wide enough for."""
    prob = inputs.small_problem(n=(27, 30, 26), h=(0.3, 0.3, 0.3), bc=(0, 0, 1), n_atoms=20, nproj_per_atom=4, seed=17)
    v = torch.from_numpy(np.random.default_rng(2).standard_normal(prob.nd)).cuda()
    out = []
    for max_ns in (1, 60):
        h = cs.Handle(prob, precision=cs.FP64, max_ns=max_ns)
        ws = torch.empty(h.chefsi_lanczos_workspace_bytes(), dtype=torch.uint8, device="cuda")
        out.append(h.chefsi_lanczos_bound(v, 12, ws))
        h.close()
    (l0, t0, a0, b0), (l1, t1, a1, b1) = out
    assert l0 == l1 and t0 == t1 and np.array_equal(a0, a1) and np.array_equal(b0, b1)
