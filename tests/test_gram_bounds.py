"""The rounding bounds of the carried correlations' shortlist, as the library
computes them (host code, no GPU), against the exact counts of operations of
the products they bound."""
from __future__ import annotations

import ctypes

import pytest

from paper_0809_1833_amd import mp


class Bounds(ctypes.Structure):
    _fields_ = [(k, ctypes.c_float) for k in ("pass_", "col", "step", "carry", "dot")]


def _fn(name, *argtypes):
    fn = getattr(mp.library(), name)
    fn.restype, fn.argtypes = Bounds, list(argtypes)
    return fn


U = 2.0 ** -24


@pytest.mark.parametrize("one", [False, True])
def test_dot_bound_covers_every_column_length(one):
    """Two lane chains over the halves of a column (the ragged FP32 form: one
    over all of it) in 16-byte pieces, then the sums of the lanes (6, and one
    between the chains): each lane's chain has 4 ceil(pieces / 64) terms."""
    if one:
        fn = _fn("_ZN2mp15gram_bounds_oneEld", ctypes.c_int64, ctypes.c_double)
    else:
        fn = _fn("_ZN2mp11gram_boundsEldb", ctypes.c_int64, ctypes.c_double, ctypes.c_bool)
    short = []
    for n in range(1, 16385):
        ld4 = (n + 63) // 64 * 16
        chain = ld4 if one else ld4 // 2
        roundings = 4 * ((chain + 63) // 64) + 7
        b = fn(n, 1.0) if one else fn(n, 1.0, False)
        if b.dot < roundings * U / (1 - roundings * U):
            short.append((n, roundings, b.dot / U))
    assert not short, (len(short), short[:5])


def test_pass_bounds_cover_the_chains():
    """Chains of 32 rows (FP64: 16), a rounding per product, one of the result;
    from an FP64 dictionary also one of each operand and of the coefficient."""
    fn = _fn("_ZN2mp11gram_boundsEldb", ctypes.c_int64, ctypes.c_double, ctypes.c_bool)
    for n in (1, 15, 16, 17, 31, 32, 33, 64, 100, 4096, 16384):
        for f64 in (False, True):
            b = fn(n, 1.0, f64)
            chain = min((n + 63) // 64 * 64, 16 if f64 else 32)
            need = (chain + 2 + (3 if f64 else 0)) * U
            assert b.pass_ >= need and b.col >= need
            assert b.carry >= U and (f64 or b.step >= U)
