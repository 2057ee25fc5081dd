"""Workspace sizes hold the vectors that the calls use and no more."""

import ctypes

import pytest

from paper_2010_03598_amd import _lib


def nbytes(L, m, prec):
    h = _lib.KgXxz(L, _lib.KG_HC_SX, 1.0, 0.5, 1)
    k = _lib.KgKrylov(m, 1, 0.0)
    return _lib.load().kg_workspace_bytes(ctypes.byref(h), ctypes.byref(k), prec)


@pytest.mark.parametrize("prec,amp", [(_lib.KG_C128, 16), (_lib.KG_C64, 8)])
@pytest.mark.parametrize("m", [1, 2, 20])
def test_tiled_sizes(m, prec, amp):
    """Beyond 2^18 amplitudes: two slots of m vectors, a costate and fixed tables."""
    fixed = {nbytes(L, m, prec) - (2 * m + 1) * (amp << L) for L in range(19, 25)}
    assert len(fixed) == 1 and 0 < fixed.pop() < 16 << 20


@pytest.mark.parametrize("L", [12, 15, 18])
def test_single_pass_sizes(L):
    """Up to 2^18: one vector a slot more in complex128, three in complex64."""
    for prec, amp, extra in [(_lib.KG_C128, 16, 1), (_lib.KG_C64, 8, 3)]:
        fixed = nbytes(24, 20, prec) - 41 * (amp << 24)
        assert nbytes(L, 20, prec) == fixed + (41 + 2 * extra) * (amp << L)
