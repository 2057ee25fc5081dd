"""The tiled passes (A, B and the pairs A C A P) forced onto vectors that other forms
serve by default, against the oracle: every tile size, window sizes up to the largest,
both window policies, gathered neighbours; and the sizes that take them by themselves.
Tolerances as the other Krylov calls (rounding of the vectors over m steps)."""

import numpy as np
import pytest
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec, host, rel_err, tile_bits, tiled_only
from oracle import grape, krylov, model, pe
import workloads

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128
TOL = {C128: 1e-12, C64: 1e-5}


def call(L, m, reorth, t, v, dtype):
    hc = workloads.HC_SZ if m % 2 else workloads.HC_SX
    sites = (1 | (1 << (L - 1))) if m % 2 else 1 << (L // 2)
    v = v.astype(np.complex64).astype(np.complex128)
    ref = krylov.expv(lambda x: model.apply_h(L, 1.0, 0.6, hc, sites, 0.4, x), v, t, m, reorth)
    out = kg.krylov_expv(kg.XXZ(L, 1.0, 0.6, hc, sites), 0.4, t, dev_vec(v, dtype), kg.Krylov(m, reorth))
    return host(out), ref


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("reorth", [True, False])
@pytest.mark.parametrize("L,m", [(8, 7), (9, 33), (10, 24), (11, 63), (11, 64), (13, 16), (13, 17), (14, 64),
                                 (17, 24)])
def test_windows(L, m, reorth, dtype):
    v = workloads.random_state(np.random.default_rng(100 * L + m), 1 << L) * 1.7
    with tiled_only():
        out, ref = call(L, m, reorth, 0.6, v, dtype)
    assert rel_err(out, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("tb", [6, 7, 8, 9, 10, 11, 12])
def test_tiles(tb, dtype):
    v = workloads.random_state(np.random.default_rng(tb), 1 << 14)
    for m, reorth in [(16, True), (17, True), (20, False)] + ([(64, True)] if tb >= 11 else []):
        with tile_bits(tb):
            out, ref = call(14, m, reorth, 0.8, v, dtype)
        assert rel_err(out, ref) <= TOL[dtype]


def test_the_switches_change_the_form():
    """A forced call is not the default one bit for bit (the forms round differently)."""
    L = 13
    v = dev_vec(workloads.random_state(np.random.default_rng(0), 1 << L), C64)
    h, k = kg.XXZ(L, 1.0, 0.6), kg.Krylov(12)
    a = kg.krylov_expv(h, 0.4, 0.6, v, k)
    with tiled_only():
        b = kg.krylov_expv(h, 0.4, 0.6, v, k)
    with tile_bits(9):
        c = kg.krylov_expv(h, 0.4, 0.6, v, k)
    assert not torch.equal(a, b) and not torch.equal(a, c)
    assert torch.equal(a, kg.krylov_expv(h, 0.4, 0.6, v, k))


def reduced(L, K, m, N, dt, dtype, P, B):
    t = workloads.pe_task(L, K, N, dt=dt, m=m)
    rng = np.random.default_rng(L + m)
    psi0, f = workloads.random_state(rng, B.dim), workloads.random_state(rng, B.dim)
    psi0, f = (x.astype(np.complex64).astype(np.complex128) for x in (psi0, f))
    ref, _ = grape.forward(P, t.u, psi0, dt, m, keep=False)
    r = kg.grape_gradient_pe(kg.XXZ(L, t.J, t.Delta, kg.KG_HC_SZ, t.hc_sites), B,
                             torch.tensor(t.u, device="cuda"), dt, kg.Krylov(m), dev_vec(psi0, dtype),
                             dev_vec(f, dtype))
    return rel_err(host(r.states).reshape(N, -1)[-1], ref)


@pytest.mark.parametrize("L,K,ms", [(16, 8, (7, 8, 9, 24)), (15, 6, (12, 13))])
def test_reduced_basis_forced(L, K, ms):
    t = workloads.pe_task(L, K, 2)
    P, B = pe.PEChain(L, K, t.J, t.Delta, t.hc_sites), kg.ReducedBasis(L, K)
    for m in ms:
        for dtype in (C128, C64):
            with tiled_only():
                assert reduced(L, K, m, 2, 0.3, dtype, P, B) <= 2 * TOL[dtype]


def test_reduced_basis():
    """352,716 orbits: the pairs over gathered neighbours, by themselves."""
    L, K = 22, 11
    t = workloads.pe_task(L, K, 1)
    P, B = pe.PEChain(L, K, t.J, t.Delta, t.hc_sites), kg.ReducedBasis(L, K)
    for m in (8, 9):
        for dtype in (C128, C64):
            assert reduced(L, K, m, 1, 0.3, dtype, P, B) <= TOL[dtype]
