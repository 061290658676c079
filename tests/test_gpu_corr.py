"""The correlation of Eq. (2) at the sizes where its two forms meet and where
the matrix form's tiles (4096 shifts), chunks (32 positions) and parts end,
against an exact correlation (whole numbers: equal)."""
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


def _corr(bits, L):
    # FP64 FFT of +-1 values: errors far below 1/2, so rounding is exact
    f = np.fft.rfft(si.to_pm1(bits, L).astype(np.float64), 1 << (2 * L - 1).bit_length())
    return np.rint(np.fft.irfft(f * f.conj())[:L]).astype(np.int32)


@pytest.mark.parametrize("L", [4095, 4096, 4097, 4127, 8191, 8192, 8193, 12289, 40009, 131071, 300001, 1048575])
def test_init_correlation(ctx, L):
    bits = [si.random_bits(L, L), si.biased_bits(L, 3, 0.1)] if L < 200000 else [si.random_bits(L, L)]
    ids = ctx.init_walks(L, len(bits), 1, n_lmt=1, init_bits=bits)
    for w, b in zip(ids, bits):
        C = ctx.read_walk(w)["C"]
        assert np.array_equal(C, _corr(b, L))
    ck = ctx.checkpoint(ids[0])
    ck["pivot"] = si.random_bits(L, L + 1)      # a restore with a pivot that is not local_best
    ctx.restore(ids[0], ck)
    assert np.array_equal(ctx.read_walk(ids[0])["C"], _corr(ck["pivot"], L))
    ctx.free_walks(ids)


def test_large_rand_flip_rebuild(ctx):
    """FLIP_lmt above the one-flip rebuild's 64, short and long walks in one batch."""
    ids = []
    for L in (1001, 4096, 9001, 33000):
        ids += ctx.init_walks(L, 1, L, n_lmt=64, flip_lmt=90, switch_period=1)
    ctx.step_batch(ids, 3)
    for w in ids:
        g = ctx.read_walk(w)
        C = _corr(g["pivot"], g["L"])
        assert np.array_equal(g["C"], C) and g["psl_pivot"] == np.abs(C[1:]).max()
    ctx.free_walks(ids)
