"""More Krylov vectors asked for than the invariant space of the input holds.

A product state under S^z controls spans the sector of its magnetisation at most.
Once the basis fills it, the next vector is rounding noise: the call either ends
there or goes on in directions that carry no weight, and the result stays that of
the exact propagator either way.  Noise of eps ||H|| re-enters through t ||H|| of
propagation: with ||H|| t <= 20 that is below 1e-5 in complex64 and 1e-11 in
complex128."""

import numpy as np
import pytest
import scipy.linalg as sla
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec, host, rel_err, tiled_only
from oracle import model
import workloads

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128
TOL = {C128: 1e-11, C64: 1e-5}


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("m", [29, 30])
@pytest.mark.parametrize("bits", ["00011", "01100", "10010", "11100", "01101", "00111", "00001"])
def test_sector_of_a_short_chain(bits, m, dtype):
    L, sites = 5, 0b10001
    v = np.zeros(1 << L, dtype=np.complex128)
    v[int(bits, 2)] = 1.0
    for u, delta in [(51.3, -1.5), (-24.2, 2.5), (12.7, 1.7), (-12.2, 3.15), (0.4, 0.5)]:
        H = model.xxz_dense(L, 1.0, delta) + u * model.hc_dense(L, workloads.HC_SZ, sites)
        ref = sla.expm(-0.3j * H) @ v
        with tiled_only():
            out = kg.krylov_expv(kg.XXZ(L, 1.0, delta, kg.KG_HC_SZ, sites), u, 0.3, dev_vec(v, dtype),
                                 kg.Krylov(m))
        assert rel_err(host(out), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [C128, C64])
@pytest.mark.parametrize("m", [27, 32])
@pytest.mark.parametrize("u,delta,t", [(0.7, 0.5, 0.4), (30.0, 1.2, 0.3), (-12.0, -2.5, 0.8)])
def test_one_magnon_of_a_long_chain(u, delta, t, m, dtype):
    """One flipped spin among 19: a space of dimension 19, exactly solvable."""
    L, sites = 19, 1 | (1 << 9)
    states = [1 << (L - 1 - i) for i in range(L)]           # the flipped spin at site i + 1
    H = np.zeros((L, L))
    for i in range(L):
        walls = 1 if i in (0, L - 1) else 2
        up = [0.5 - (1.0 if i == s else 0.0) for s in (0, 9)]   # S^z of the control sites
        H[i, i] = 0.25 * delta * (L - 1 - 2 * walls) + u * sum(up)
        if i + 1 < L:
            H[i, i + 1] = H[i + 1, i] = 0.5
    v = np.zeros(1 << L, dtype=np.complex128)
    v[states[7]] = 1.0
    ref = np.zeros_like(v)
    ref[states] = sla.expm(-1j * t * H)[:, 7]
    out = kg.krylov_expv(kg.XXZ(L, 1.0, delta, kg.KG_HC_SZ, sites), u, t, dev_vec(v, dtype), kg.Krylov(m))
    assert rel_err(host(out), ref) <= TOL[dtype]
