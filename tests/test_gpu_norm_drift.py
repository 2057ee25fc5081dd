"""The norm of a propagated state over many slices.  Every slice is a unitary up to
rounding: a few roundings of its scalars, independent from slice to slice, so that
the norm wanders by about sqrt(N) of them.  A scale that is off by a unit in the last
place in the same direction every time would show as N of them."""

import numpy as np
import pytest
import torch

import paper_2010_03598_amd as kg
from gpu_util import dev_vec, host
import workloads

pytestmark = pytest.mark.gpu


# one block per sweep (four and eight wavefronts, two rows a thread), one launch per step
@pytest.mark.parametrize("L,m,N", [(8, 10, 400), (9, 9, 400), (10, 7, 400), (11, 12, 300), (12, 24, 300)])
def test_norm(L, m, N):
    rng = np.random.default_rng(L)
    u = rng.uniform(-1.0, 1.0, N)
    psi0, f = workloads.random_state(rng, 1 << L), workloads.random_state(rng, 1 << L)
    r = kg.grape_gradient(kg.XXZ(L, 1.0, 0.5), torch.tensor(u, device="cuda"), 0.05, kg.Krylov(m),
                          dev_vec(psi0), dev_vec(f))
    last = host(r.states).reshape(N, -1)[-1]
    norm = lambda x: np.sqrt(np.sum(x.real.astype(np.longdouble) ** 2 + x.imag.astype(np.longdouble) ** 2))
    drift = float(abs(norm(last) / norm(np.asarray(psi0)) - 1))
    assert drift <= 4.0 * np.sqrt(N) * 2.0 ** -53
