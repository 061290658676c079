"""The correlation's two forms by launch: the matrix form on the shortest walks it
can take (launches of many), the popcount form up to its longest (few walks), and
what a start that takes the latter costs."""
import time

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


# walks of a launch: the last count with at most 16384 chunks of work, and the next
@pytest.mark.parametrize("L,n", [(4096, 252), (4096, 253), (4097, 260), (4127, 260), (8191, 63), (8192, 64), (8193, 65),
                                 (12289, 28), (12289, 29), (16384, 15), (16384, 16), (36863, 3), (36863, 4), (36864, 1),
                                 (36865, 2)])
def test_both_forms(ctx, L, n):
    bits = [si.random_bits(L, L), si.biased_bits(L, 3, 0.1), si.all_plus_bits(L)]
    ids = ctx.init_walks(L, n, 1, n_lmt=1, flip_lmt=1, init_bits=[bits[i % 3] for i in range(n)])
    want = [_corr(b, L) for b in bits]
    for i in sorted({0, 1 % n, 2 % n, n // 2, n - 1}):
        assert np.array_equal(ctx.read_walk(ids[i])["C"], want[i % 3])
    ctx.free_walks(ids)


@pytest.mark.parametrize("Ls", [[1001, 4096, 9001, 33000], [300, 4096, 5001, 70001], [4096] * 130 + [16384] * 8])
def test_large_rand_flips_in_mixed_batches(ctx, Ls):
    ids = []
    for i, L in enumerate(Ls):
        ids += ctx.init_walks(L, 1, i, n_lmt=64, flip_lmt=90, switch_period=1)
    ctx.step_batch(ids, 3)
    for w in ids[:3] + ids[-2:]:
        g = ctx.read_walk(w)
        C = _corr(g["pivot"], g["L"])
        assert np.array_equal(g["C"], C) and g["psl_pivot"] == np.abs(C[1:]).max()
    ctx.free_walks(ids)


def test_a_start_of_moderate_length(ctx):
    """A walk of 8193 elements starts in about the time of one of 4095, on which
    there is no choice (34 and 34 us; the matrix form's three launches: 51)."""
    best = {}
    for L in (4095, 8193):
        best[L] = 1e9
        for _ in range(60):
            t = time.perf_counter()
            ids = ctx.init_walks(L, 1, 3, n_lmt=1)
            best[L] = min(best[L], time.perf_counter() - t)
            ctx.free_walks(ids)
    assert best[8193] <= 1.3 * best[4095], best
