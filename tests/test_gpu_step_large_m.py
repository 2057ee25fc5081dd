"""One launch per step where its blocks need more than 64 KiB of LDS: the largest
windows at the largest tiles, full space and reduced basis.  Tolerances as the other
Krylov calls (rounding over m steps)."""

import numpy as np
import pytest
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec, host, rel_err
from oracle import krylov, model, pe
import workloads

pytestmark = pytest.mark.gpu

C64, C128 = torch.complex64, torch.complex128
TOL = {C128: 1e-12, C64: 1e-5}


@pytest.mark.parametrize("dtype", [C128, C64])
def test_largest_window_full_space(dtype):
    L, m = 18, 64
    rng = np.random.default_rng(1)
    v = workloads.random_state(rng, 1 << L).astype(np.complex64).astype(np.complex128)
    ref = krylov.expv(lambda x: model.apply_h(L, 1.0, 0.6, workloads.HC_SX, 1, 0.4, x), v, 2.0, m, True)
    out = kg.krylov_expv(kg.XXZ(L, 1.0, 0.6), 0.4, 2.0, dev_vec(v, dtype), kg.Krylov(m))
    assert rel_err(host(out), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [C128, C64])
def test_largest_window_reduced_basis(dtype):
    L, K, m = 21, 10, 60                                   # 176,484 orbits
    sites = 1 | (1 << (L - 1))
    B, P = kg.ReducedBasis(L, K), pe.PEChain(L, K, 1.0, 0.6, sites)
    rng = np.random.default_rng(2)
    v = workloads.random_state(rng, B.dim).astype(np.complex64).astype(np.complex128)
    f = workloads.random_state(rng, B.dim)
    ref = krylov.expv(lambda x: P.apply(0.3, x), v, 1.5, m, True)
    r = kg.grape_gradient_pe(kg.XXZ(L, 1.0, 0.6, kg.KG_HC_SZ, sites), B,
                             torch.tensor([0.3], dtype=torch.float64, device="cuda"), 1.5, kg.Krylov(m),
                             dev_vec(v, dtype), dev_vec(f, dtype))
    assert rel_err(host(r.states).reshape(-1), ref) <= TOL[dtype]
