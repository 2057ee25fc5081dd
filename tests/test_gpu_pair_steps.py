"""Two Lanczos steps per pass over the window (full re-orthogonalisation of vectors
on the tiled passes, m >= 8), against the oracle: odd and even m (an even m takes its
first step alone), whole tiles, tiles longer than the vector, the largest window, and
a basis that ends at either step of a pair."""

import numpy as np
import pytest
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec, host, rel_err, tile_bits, tiled_only
from oracle import krylov, model
import workloads

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128
# as the other Krylov calls: rounding of the vectors over m steps
TOL = {C128: 1e-12, C64: 1e-5}


def both(L, m, u, t, v, dtype, **kw):
    hc = workloads.HC_SZ if m % 2 else workloads.HC_SX
    sites = (1 | (1 << (L - 1))) if m % 2 else 1 << (L // 2)
    if dtype == C64:
        v = v.astype(np.complex64).astype(np.complex128)
    ref = krylov.expv(lambda x: model.apply_h(L, 1.0, 0.6, hc, sites, u, x), v, t, m, True)
    out = kg.krylov_expv(kg.XXZ(L, 1.0, 0.6, hc, sites), u, t, dev_vec(v, dtype), kg.Krylov(m), **kw)
    return host(out), ref


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("L,m", [(5, 8), (6, 9), (8, 8), (8, 9), (9, 10), (9, 33), (10, 24), (10, 63),
                                 (10, 64), (19, 8), (19, 13)])
def test_against_oracle(L, m, dtype):
    rng = np.random.default_rng(100 * L + m)
    v = workloads.random_state(rng, 1 << L) * 1.7
    with tiled_only():
        out, ref = both(L, m, 0.4, 0.5, v, dtype)
    assert rel_err(out, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("tb", [6, 7, 8, 9, 10])
def test_every_tile(tb, dtype):
    rng = np.random.default_rng(tb)
    v = workloads.random_state(rng, 1 << 10)
    with tiled_only(), tile_bits(tb):
        out, ref = both(10, 16 + tb % 2, 0.3, 1.5, v, dtype)
    assert rel_err(out, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("m", [12, 13])
@pytest.mark.parametrize("L", [6, 7, 8, 9])
def test_basis_ends_inside_a_pair(L, m, dtype):
    """One flipped spin at the end of the chain spans an invariant space of dimension L
    under the S^z control: the basis ends after L vectors, at the first step of a pair
    or at its second."""
    h = kg.XXZ(L, 1.0, 0.5, kg.KG_HC_SZ, 1)
    v = np.zeros(1 << L, dtype=np.complex128)
    v[1] = 1.5
    ref = krylov.expv(lambda x: model.apply_h(L, 1.0, 0.5, workloads.HC_SZ, 1, 0.7, x), v, 0.6, m, True)
    m_eff = torch.zeros(1, dtype=torch.int32, device="cuda")
    with tiled_only():
        out = host(kg.krylov_expv(h, 0.7, 0.6, dev_vec(v, dtype), kg.Krylov(m), m_eff=m_eff))
    assert int(m_eff) == L
    assert rel_err(out, ref) <= TOL[dtype]
    with tiled_only():
        z = kg.krylov_expv(h, 0.7, 0.6, dev_vec(0.0 * v, dtype), kg.Krylov(m), m_eff=m_eff)
    assert int(m_eff) == 0 and float(z.abs().max()) == 0.0
    v[2] = np.nan
    with tiled_only():
        n = kg.krylov_expv(h, 0.7, 0.6, dev_vec(v, dtype), kg.Krylov(m))
    assert bool(torch.isnan(torch.view_as_real(n)).any())


@pytest.mark.parametrize("dtype", [C128, C64])
def test_reduced_basis(dtype):
    """Vectors that fill no whole tile, gathered neighbours (dimension 352,716)."""
    L, K = 22, 11
    B = kg.ReducedBasis(L, K)
    h = kg.XXZ(L, 1.0, 0.6, kg.KG_HC_SZ, 1 | 1 << (L - 1))
    rng = np.random.default_rng(3)
    psi0 = dev_vec(workloads.random_phase_state(rng, B.dim), dtype)
    f = dev_vec(workloads.random_phase_state(rng, B.dim), dtype)
    u = torch.tensor([0.3, -0.2, 0.5], dtype=torch.float64, device="cuda")
    # m = 7 takes one step per pass; three short slices are converged at both
    a = kg.grape_gradient_pe(h, B, u, 0.02, kg.Krylov(7), psi0, f, variant="centred")
    for m in (8, 9):
        b = kg.grape_gradient_pe(h, B, u, 0.02, kg.Krylov(m), psi0, f, variant="centred")
        tol = 1e-9 if dtype == C128 else 1e-4
        assert abs(float(a.F) - float(b.F)) <= tol * float(a.F)
        assert float((a.grad - b.grad).norm()) <= tol * float(a.grad.norm())
