"""F, PSL and C of walks that are started (given and random pivots, several to a
call), changed by forced flips and restored, at the lengths where the segments
of the sums (powers of two from 256 shifts) and the words of the bits end,
against exact sums over the correlation of the bits read back."""
import math

import numpy as np
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_09801_amd import libpsl
    c = libpsl.Context(0)
    yield c
    c.close()


def _check(st, L):
    f = np.fft.rfft(si.to_pm1(st["pivot"], L).astype(np.float64), 1 << (2 * L - 1).bit_length())
    C = np.rint(np.fft.irfft(f * f.conj())[:L]).astype(np.int64)
    assert np.array_equal(st["C"], C)
    assert st["psl_pivot"] == np.abs(C[1:]).max()
    # |C|^4 < 2^53 is exact; a compensated sum of n non-negative terms is within
    # 2 u + n^2 u^2 of it (u = 2^-53), the segments' sums once more
    F = math.fsum(float(v) ** 4 for v in np.abs(C[1:]))
    assert abs(st["F_pivot"] - F) <= 4 * 2.0 ** -53 * F


@pytest.mark.parametrize("L", [3, 63, 64, 65, 129, 257, 258, 1024, 1025, 1026, 2049, 4097, 33000, 131071])
def test_started_flipped_restored(ctx, L):
    bits = [si.random_bits(L, L), si.random_bits(L, L + 7)]
    ids = ctx.init_walks(L, 2, 1, alpha1=4, n_lmt=1, init_bits=bits) + ctx.init_walks(L, 2, 5, alpha1=4, n_lmt=1)
    for w in ids:
        st = ctx.read_walk(w)
        _check(st, L)
        assert st["value_local"] == st["F_pivot"] and st["psl_best"] == st["psl_pivot"]
    for w, b in zip(ids, bits):
        assert np.array_equal(ctx.read_walk(w)["pivot"], b)
    assert not np.array_equal(ctx.read_walk(ids[2])["pivot"], ctx.read_walk(ids[3])["pivot"]) or L < 64
    ck = ctx.checkpoint(ids[0])
    start = ctx.read_walk(ids[0])
    for j in (0, L // 2, L - 1):
        before = ctx.read_walk(ids[0])["pivot"].copy()
        ctx.apply_flip(ids[0], j)
        st = ctx.read_walk(ids[0])
        _check(st, L)
        assert np.flatnonzero(si.to_pm1(st["pivot"], L) != si.to_pm1(before, L)).tolist() == [j]
    ctx.restore(ids[0], ck)
    st = ctx.read_walk(ids[0])
    _check(st, L)
    assert st["F_pivot"] == start["F_pivot"] and np.array_equal(st["C"], start["C"])
    ctx.free_walks(ids)
