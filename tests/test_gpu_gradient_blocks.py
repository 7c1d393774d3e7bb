"""The force and stress kernels: what the LDS kernel's idle threads read, several orbitals a block (a
block takes atoms x orbitals / 1024 of them, at most 16) with a shorter last run, and the kernel with
cached loads where one support is too large for LDS.

FP64 sums in another order than the oracle's: 1e-11 of the largest component, as in the calls' own
parity tests."""
import numpy as np
import pytest

from oracle.forces import kinetic_stress, nonlocal_forces, nonlocal_stress
from paper_2302_09708_amd import inputs
from tests.test_gpu_gradient_sums import _with_projectors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    from paper_2302_09708_amd import chefsi
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    chefsi.load()
    return chefsi


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_values_outside_the_stencils(cs, bad):
    """A non-finite orbital value that no support point's derivative reads leaves the results as they are
    (the corner of the support's box, where threads without a point used to form one)."""
    print(f"gradient blocks {bad}", flush=True)
    prob = inputs.small_problem(n=(24, 25, 26), h=(0.3, 0.3, 0.3), bc=(1, 0, 1), n_atoms=1, nproj_per_atom=4, seed=3)
    r, n = prob.fd_order // 2, prob.n
    xyz = np.array(np.unravel_index(prob.supp_idx, n[::-1])).T[:, ::-1]
    corner = xyz.min(axis=0)
    read = np.zeros(n[::-1], dtype=bool)
    for d in range(3):
        for p in range(-r, r + 1):
            q = xyz.copy()
            q[:, d] += p
            if prob.bc[d] == 0:
                q[:, d] %= n[d]
            q = q[(q[:, d] >= 0) & (q[:, d] < n[d])]
            read[q[:, 2], q[:, 1], q[:, 0]] = True
    assert not read[corner[2], corner[1], corner[0]] and len(prob.supp_idx) % 512 != 0
    ns = 5
    X = inputs.initial_block(prob.nd, ns, 31).T
    occ = np.linspace(2.0, 0.5, ns)
    disp = np.random.Generator(np.random.PCG64(4)).uniform(-1.5, 1.5, (len(prob.supp_idx), 3))
    h = cs.Handle(prob, precision=cs.FP64, max_ns=ns)
    ws = torch.empty(h.chefsi_forces_workspace_bytes(ns), dtype=torch.uint8, device="cuda")
    Xd = torch.from_numpy(np.ascontiguousarray(X.T)).cuda()
    Xd[2, np.flatnonzero(~read.reshape(-1))] = bad
    assert not torch.isfinite(Xd[2, corner[0] + n[0] * (corner[1] + n[1] * corner[2])])
    for got, ref in ((h.chefsi_nonlocal_forces(Xd, ns, occ, ws), nonlocal_forces(prob, X, occ)),
                     (h.chefsi_nonlocal_stress(Xd, ns, occ, disp, ws), nonlocal_stress(prob, X, occ, disp))):
        assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max()
    h.close()


def _compare(cs, prob, ns, prec):
    X = inputs.initial_block(prob.nd, ns, 4100 + ns).T
    if prec == "mixed":
        X = X.astype(np.float32).astype(np.float64)
    occ = np.linspace(2.0, 0.25, ns)
    disp = np.random.Generator(np.random.PCG64(ns)).uniform(-1.5, 1.5, (len(prob.supp_idx), 3))
    h = cs.Handle(prob, precision=cs.FP64 if prec == "fp64" else cs.MIXED, max_ns=ns)
    ws = torch.empty(h.chefsi_forces_workspace_bytes(ns), dtype=torch.uint8, device="cuda")
    ws.fill_(0xff)  # NaN in every double
    Xd = torch.from_numpy(np.ascontiguousarray(X.T)).to(device="cuda", dtype=torch.float64 if prec == "fp64" else torch.float32)
    for got, ref in ((h.chefsi_nonlocal_forces(Xd, ns, occ, ws), nonlocal_forces(prob, X, occ)),
                     (h.chefsi_kinetic_stress(Xd, ns, occ, ws), kinetic_stress(prob, X, occ)),
                     (h.chefsi_nonlocal_stress(Xd, ns, occ, disp, ws), nonlocal_stress(prob, X, occ, disp))):
        assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max()
    h.close()


# 3, 5 and 16 orbitals a block; remainders of 2, 1 and 7; one, two and three passes of projectors
@pytest.mark.parametrize("order,n,bc,atoms,ns", [
    (12, (20, 18, 16), (0, 0, 1), 16, 200),
    (6, (16, 21, 18), (1, 0, 0), 21, 251),
    (8, (18, 17, 20), (0, 1, 0), 64, 263),
])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_several_orbitals_a_block(cs, order, n, bc, atoms, ns, prec):
    print(f"gradient blocks order {order} n {n} atoms {atoms} ns {ns} {prec}", flush=True)
    prob = inputs.small_problem(n=n, h=(0.4, 0.42, 0.38), bc=bc, fd_order=order, n_atoms=atoms, nproj_per_atom=1, seed=order)
    counts = [(4, 1, 5, 0, 8, 9, 2)[k % 7] for k in range(atoms)]
    prob = _with_projectors(prob, counts, 60 + order)
    assert np.diff(prob.supp_ptr).max() <= 1536 and np.diff(prob.supp_ptr).min() == 0
    _compare(cs, prob, ns, prec)


# one support of more than 1536 points sends every atom to the kernel with cached loads
@pytest.mark.parametrize("order,ns", [(2, 1), (4, 7), (6, 8), (8, 9), (10, 17), (12, 5)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_large_supports(cs, order, ns, prec):
    print(f"gradient blocks, large support, order {order} ns {ns} {prec}", flush=True)
    prob = inputs.small_problem(n=(19, 18, 20), h=(0.2, 0.21, 0.19), bc=(0, 1, 0), fd_order=order, n_atoms=5, nproj_per_atom=1,
                                seed=order)
    prob = _with_projectors(prob, (4, 7, 0, 1, 5), 70 + order)
    assert np.diff(prob.supp_ptr).max() > 1536
    _compare(cs, prob, ns, prec)
