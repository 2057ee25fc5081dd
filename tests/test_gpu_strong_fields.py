"""Krylov calls whose diagonal entries |alpha_k| exceed the off-diagonal ones
(strong S^z control, strong anisotropy, product states), where a recurrence for
H u_k, or a subtraction deferred past the rounding of a vector, would lose
accuracy by |alpha_k| / beta_k a step.  Compared with the same m-step propagator in
FP64, on the same input.

Each of the m stored vectors is rounded once, by 2^-24 or 2^-53 of its norm,
independently: sqrt(m) roundings, times 4 for the H v sums and t ||H||."""

import numpy as np
import pytest
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec, host, rel_err
from oracle import grape, krylov, model, pe
import workloads

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128
SX, SZ = workloads.HC_SX, workloads.HC_SZ


def bound(m, dtype):
    return 4.0 * np.sqrt(m) * 2.0 ** (-24 if dtype == C64 else -53)


def domain_wall(L):
    v = np.zeros(1 << L, dtype=np.complex128)
    v[int("0" * (L // 2) + "1" * (L - L // 2), 2)] = 1.0
    return v


# one block per call: four wavefronts, one
SHORT = [(8, 1.0, 0.5, SZ, 1, -60.0, 1.0, 30, True), (8, 1.0, 0.5, SZ, 1, 100.0, 1.0, 24, True),
         (8, 0.2, 20.0, SX, 1, 1.0, 4.0, 24, True), (6, 1.0, 3.0, SZ, 1, 40.0, 0.4, 20, False),
         (9, 1.0, 0.5, SZ, 0b100000001, 70.0, 0.5, 15, True)]


@pytest.mark.parametrize("L,J,delta,kind,sites,u,t,m,reorth", SHORT)
def test_one_block(L, J, delta, kind, sites, u, t, m, reorth):
    v = domain_wall(L)
    ref = krylov.expv(lambda x: model.apply_h(L, J, delta, kind, sites, u, x), v, t, m, reorth)
    out = kg.krylov_expv(kg.XXZ(L, J, delta, kind, sites), u, t, dev_vec(v, C64), kg.Krylov(m, reorth))
    assert rel_err(host(out), ref) <= bound(m, C64)


# one launch per step: short windows and long ones, a vector beyond the one-block form's LDS
LONG = [(12, 1.0, 0.5, SZ, 1, 100.0, 1.0, 30, True), (11, 1.0, 0.5, SZ, 1, -60.0, 1.0, 30, True),
        (12, 0.2, 20.0, SX, 1, 1.0, 1.0, 24, True), (12, 1.0, 10.0, SX, 1, 1.0, 1.0, 40, False),
        (9, 1.0, 0.5, SZ, 1, 70.0, 0.5, 30, True), (14, 1.0, 4.0, SX, 1 << 5, 3.0, 0.5, 18, True),
        (17, 1.0, 0.5, SZ, 0b10001, 50.0, 0.3, 14, True)]


@pytest.mark.parametrize("L,J,delta,kind,sites,u,t,m,reorth", LONG)
def test_one_launch_per_step(L, J, delta, kind, sites, u, t, m, reorth):
    v = domain_wall(L)
    ref = krylov.expv(lambda x: model.apply_h(L, J, delta, kind, sites, u, x), v, t, m, reorth)
    out = kg.krylov_expv(kg.XXZ(L, J, delta, kind, sites), u, t, dev_vec(v, C64), kg.Krylov(m, reorth))
    assert rel_err(host(out), ref) <= bound(m, C64)


@pytest.mark.parametrize("L,delta,kind,u,t,m", [(11, 2.0, SZ, 12.0, 0.4, 24), (12, 6.0, SX, 2.0, 0.3, 20),
                                                (16, 1.0, SZ, 8.0, 0.2, 16)])
def test_one_launch_per_step_c128(L, delta, kind, u, t, m):
    v = domain_wall(L)
    ref = krylov.expv(lambda x: model.apply_h(L, 1.0, delta, kind, 1, u, x), v, t, m, True)
    out = kg.krylov_expv(kg.XXZ(L, 1.0, delta, kind, 1), u, t, dev_vec(v, C128), kg.Krylov(m))
    assert rel_err(host(out), ref) <= 8.0 * bound(m, C128)     # both sides round in FP64


@pytest.mark.parametrize("dtype", [C64, C128])
@pytest.mark.parametrize("L,K,u,t,m", [(14, 7, 30.0, 0.2, 20), (16, 8, 15.0, 0.3, 16)])
def test_reduced_basis_steps(L, K, u, t, m, dtype):
    """The states of a forward sweep in the reduced basis, from the task's product state."""
    B, sites, N = kg.ReducedBasis(L, K), 1 | (1 << (L - 1)), 3
    P = pe.PEChain(L, K, 1.0, 3.0, sites)
    psi0, f = np.zeros(B.dim, complex), workloads.random_state(np.random.default_rng(1), B.dim)
    psi0[B.dim // 3] = 1.0
    us = u * np.array([1.0, -1.0, 0.5])
    ref, _ = grape.forward(P, us, psi0, t, m, keep=False)
    r = kg.grape_gradient_pe(kg.XXZ(L, 1.0, 3.0, kg.KG_HC_SZ, sites), B, torch.tensor(us, device="cuda"), t,
                             kg.Krylov(m), dev_vec(psi0, dtype), dev_vec(f, dtype))
    got = host(r.states).reshape(N, -1)[-1]
    assert rel_err(got, ref) <= N * (1.0 if dtype == C64 else 8.0) * bound(m, dtype)


@pytest.mark.parametrize("L,u,delta,pos,sites", [
    (6, -12.0, -3.0, 3, 0b1), (6, 5.0, 0.5, 3, 0b1001), (6, 17.0, 2.0, 3, 0b1), (7, -40.0, -3.0, 0, 0b1001),
    (7, -3.0, 0.5, 3, 0b1001), (7, 5.0, 2.0, 3, 0b1), (7, 5.0, 4.0, 3, 0b1)])
def test_basis_closes(L, u, delta, pos, sites):
    """One flipped spin under S^z controls: an invariant space of dimension L, found in
    complex64 too."""
    v = np.zeros(1 << L, dtype=np.complex128)
    v[1 << pos] = 1.5
    m_eff = torch.zeros(1, dtype=torch.int32, device="cuda")
    ref = krylov.expv(lambda x: model.apply_h(L, 1.0, delta, SZ, sites, u, x), v, 0.3, 13, True)
    out = kg.krylov_expv(kg.XXZ(L, 1.0, delta, SZ, sites), u, 0.3, dev_vec(v, C64), kg.Krylov(13), m_eff=m_eff)
    assert int(m_eff) == L
    assert rel_err(host(out), ref) <= bound(13, C64)


def test_bang_bang_gradient():
    """Twenty slices of +-50: the rounding of a slice's state is carried on by unitaries,
    so the bound of the states is that of a call times the slices."""
    L, N, m, dt = 8, 20, 20, 0.5
    ch = model.Chain(L, 2.0, 0.5, SZ, 1)
    u = 50.0 * np.where(np.arange(N) % 3 == 0, -1.0, 1.0)
    rng = np.random.default_rng(4)
    psi0, f = domain_wall(L), workloads.random_state(rng, 1 << L)
    f = f.astype(np.complex64).astype(np.complex128)
    ref, _ = grape.forward(ch, u, psi0, dt, m, keep=False)
    r = kg.grape_gradient(kg.XXZ(L, 2.0, 0.5, SZ, 1), torch.tensor(u, device="cuda"), dt, kg.Krylov(m),
                          dev_vec(psi0, C64), dev_vec(f, C64))
    got = host(r.states).reshape(N, -1)
    assert rel_err(got[-1], ref) <= N * bound(m, C64)
