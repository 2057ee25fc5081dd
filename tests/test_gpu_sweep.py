"""Short vectors: a block runs a whole sweep (kg_sweep.hip).  The sizes where it
can go wrong: one wavefront, ragged rows (D not a multiple of 64), the change
from four to five wavefronts (where wavefront 0 computes the scalars for all),
the largest block, and costates that come in several launches."""

import numpy as np
import pytest
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec
from oracle import grape, model, pe
import workloads

pytestmark = pytest.mark.gpu

# oracle (FP64) against complex128 / complex64: the bounds of the one-block calls,
# see test_gpu_fused
TOL = {torch.complex128: 1e-10, torch.complex64: 1e-4}


def _check(r, ref, tol):
    assert abs(float(r.F) - ref.F) <= tol * max(abs(ref.F), 1e-12)
    assert np.linalg.norm(r.grad.cpu().numpy() - ref.grad) <= tol * np.linalg.norm(ref.grad)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("L,m,ckpt,centred", [(2, 3, 0, False), (6, 8, 0, True), (7, 9, 4, False),
                                              (8, 20, 3, True), (9, 10, 0, True), (10, 5, 0, False),
                                              (10, 5, 2, True)])
def test_full_space_gradient(L, m, ckpt, centred, dtype):
    rng = np.random.default_rng(40 + L)
    N = 9
    ch = model.Chain(L, 1.0, 0.7, workloads.HC_SX, 1)
    u = rng.uniform(-1.0, 1.0, N)
    psi0 = workloads.random_phase_state(rng, 1 << L)
    f = workloads.random_phase_state(rng, 1 << L)
    ref = (grape.gradient_centred if centred else grape.gradient)(ch, u, psi0, f, 0.05, m)
    h = kg.XXZ(L, 1.0, 0.7, kg.KG_HC_SX, 1)
    r = kg.grape_gradient(h, torch.tensor(u, device="cuda"), 0.05, kg.Krylov(m), dev_vec(psi0, dtype),
                          dev_vec(f, dtype), ckpt_every=ckpt, centred=centred)
    _check(r, ref, TOL[dtype])


# dims 10 (one ragged wavefront), 144 (three), 280 and 472 (five and eight, wavefront 0's scalars)
@pytest.mark.parametrize("L,K", [(6, 3), (24, 2), (16, 3), (12, 6)])
def test_reduced_gradient(L, K):
    t = workloads.pe_task(L, K, 7, dt=0.1)
    B = kg.ReducedBasis(L, K)
    P = pe.PEChain(L, K, t.J, t.Delta, t.hc_sites)
    rng = np.random.default_rng(L)
    psi0, f = workloads.random_state(rng, B.dim), workloads.random_state(rng, B.dim)
    ref = grape.gradient(P, t.u, psi0, f, t.dt, t.m)
    h = kg.XXZ(L, t.J, t.Delta, kg.KG_HC_SZ, t.hc_sites)
    r = kg.grape_gradient_pe(h, B, torch.tensor(t.u, device="cuda"), t.dt, kg.Krylov(t.m),
                             dev_vec(psi0), dev_vec(f))
    _check(r, ref, 1e-10)


def test_costates_in_several_launches():
    """More slices than half the workspace's free area holds costates: the gradient
    equals the checkpointed one, whose segments fit, bit for bit."""
    L, m, N = 10, 4, 700
    h, k = kg.XXZ(L, 1.0, 0.5), kg.Krylov(m)
    ws = kg.Workspace(h, k, torch.complex128)
    assert ws.nbytes // 2 < N * 16 * h.D
    rng = np.random.default_rng(3)
    u = torch.tensor(rng.uniform(-1.0, 1.0, N), device="cuda")
    psi0 = dev_vec(workloads.random_phase_state(rng, h.D))
    f = dev_vec(workloads.random_phase_state(rng, h.D))
    a = kg.grape_gradient(h, u, 0.05, k, psi0, f, workspace=ws, centred=True)
    b = kg.grape_gradient(h, u, 0.05, k, psi0, f, ckpt_every=26, centred=True)
    assert torch.equal(a.F, b.F) and torch.equal(a.grad, b.grad)
