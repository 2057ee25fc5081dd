"""One launch per Lanczos step (kg_step.hip), against the oracle at the sizes
where it can go wrong: the smallest and largest vectors that take it, each
tile of its table, Krylov dimensions around the groups of four and eight window
vectors and of rows with more than 64 pairs of values, both window policies."""

import numpy as np
import pytest
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec, host, rel_err
from oracle import krylov, model
import workloads

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128
# as the other Krylov calls: rounding of the vectors over m steps
TOL = {C128: 1e-12, C64: 1e-5}


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("L,m,reorth", [(11, 2, True), (11, 5, True), (11, 64, True), (12, 6, False),
                                        (13, 9, True), (13, 10, True), (13, 34, True),
                                        (14, 17, True), (16, 18, True), (17, 6, True), (17, 3, False),
                                        (18, 10, True)])
def test_against_oracle(L, m, reorth, dtype):
    rng = np.random.default_rng(100 * L + m)
    hc = workloads.HC_SZ if m % 2 else workloads.HC_SX
    sites = (1 | (1 << (L - 1))) if m % 2 else 1 << (L // 2)
    v = workloads.random_state(rng, 1 << L) * 1.7
    if dtype == C64:
        v = v.astype(np.complex64).astype(np.complex128)
    ref = krylov.expv(lambda x: model.apply_h(L, 1.0, 0.6, hc, sites, 0.4, x), v, 0.3, m, reorth)
    h = kg.XXZ(L, 1.0, 0.6, hc, sites)
    out = kg.krylov_expv(h, 0.4, 0.3, dev_vec(v, dtype), kg.Krylov(m, reorth))
    assert rel_err(host(out), ref) <= TOL[dtype]


def test_in_place_and_breakdown():
    """v_out = v_in; and a basis that ends early (the all-up state is an eigenstate)
    stops the later launches."""
    L = 12
    h = kg.XXZ(L, 1.0, 0.5, kg.KG_HC_SZ, 1)
    k = kg.Krylov(8)
    rng = np.random.default_rng(5)
    v = dev_vec(workloads.random_state(rng, 1 << L))
    out = kg.krylov_expv(h, 0.2, 0.3, v, k)
    w = v.clone()
    kg.krylov_expv(h, 0.2, 0.3, w, k, out=w)
    assert torch.equal(w, out)
    e = torch.zeros(1 << L, dtype=C128, device="cuda")
    e[0] = 2.0
    m_eff = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = kg.krylov_expv(h, 0.2, 0.3, e, k, m_eff=m_eff)
    assert int(m_eff) == 1
    E = 0.125 * (L - 1) + 0.2 * 0.5
    assert abs(complex(got[0].cpu()) - 2.0 * np.exp(-0.3j * E)) < 1e-14
    assert float(got[1:].abs().max()) == 0.0
    z = kg.krylov_expv(h, 0.2, 0.3, torch.zeros_like(e), k, m_eff=m_eff)
    assert int(m_eff) == 0 and float(z.abs().max()) == 0.0


def test_paired_sweeps_equal_one_stream():
    """The store-all gradient with both sweeps side by side (odd and even slice
    counts, two slices) is the sequential one bit for bit, states included."""
    import os
    rng = np.random.default_rng(8)
    for L, N, centred, dtype in [(11, 2, False, C128), (11, 7, True, C64), (12, 8, False, C64),
                                 (19, 3, True, C64)]:
        h, k = kg.XXZ(L, 1.0, 0.7), kg.Krylov(6)
        u = torch.tensor(rng.uniform(-1.0, 1.0, N), device="cuda")
        psi0 = dev_vec(workloads.random_phase_state(rng, h.D), dtype)
        f = dev_vec(workloads.random_phase_state(rng, h.D), dtype)
        a = kg.grape_gradient(h, u, 0.05, k, psi0, f, centred=centred)
        os.environ["KG_ONE_STREAM"] = "1"
        try:
            b = kg.grape_gradient(h, u, 0.05, k, psi0, f, centred=centred)
        finally:
            del os.environ["KG_ONE_STREAM"]
        assert torch.equal(a.F, b.F) and torch.equal(a.grad, b.grad) and torch.equal(a.states, b.states)
        p = torch.stack([psi0, psi0 * 0.5])
        t = torch.stack([f, f])
        a = kg.grape_gradient_columns(h, u, 0.05, k, p, t, centred=centred)
        os.environ["KG_ONE_STREAM"] = "1"
        try:
            b = kg.grape_gradient_columns(h, u, 0.05, k, p, t, centred=centred)
        finally:
            del os.environ["KG_ONE_STREAM"]
        assert torch.equal(a.F, b.F) and torch.equal(a.grad, b.grad)


# dims 1716 and 6470: a ragged last tile, padded tiles without rows, odd dimensions
@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("L,K,m,ckpt", [(14, 7, 6, 0), (15, 6, 9, 2), (16, 8, 10, 0)])
def test_reduced_basis(L, K, m, ckpt, dtype):
    from oracle import grape, pe
    t = workloads.pe_task(L, K, 5, dt=0.1, m=m)
    B = kg.ReducedBasis(L, K)
    P = pe.PEChain(L, K, t.J, t.Delta, t.hc_sites)
    rng = np.random.default_rng(L + m)
    psi0, f = workloads.random_state(rng, B.dim), workloads.random_state(rng, B.dim)
    ref = grape.gradient_centred(P, t.u, psi0, f, t.dt, m)
    h = kg.XXZ(L, t.J, t.Delta, kg.KG_HC_SZ, t.hc_sites)
    r = kg.grape_gradient_pe(h, B, torch.tensor(t.u, device="cuda"), t.dt, kg.Krylov(m),
                             dev_vec(psi0, dtype), dev_vec(f, dtype), ckpt_every=ckpt,
                             variant="centred")
    tol = 1e-10 if dtype == C128 else 1e-4
    assert abs(float(r.F) - ref.F) <= tol * ref.F
    assert np.linalg.norm(host(r.grad) - ref.grad) <= tol * np.linalg.norm(ref.grad)
