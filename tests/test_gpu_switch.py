"""Phase switches of walks with more segments than blocks that rebuild them: C, F
and PSL of the new pivot after each switch, at the counts of segments and flips
where the rule turns, and what such a step costs."""
import math
import time

import numpy as np
import pytest

import oracle
import seeded_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_2107_09801_amd import libpsl
    c = libpsl.Context(0)
    yield c
    c.close()


def _check(st, L):
    n = 1 << (2 * L - 1).bit_length()
    f = np.fft.rfft(si.to_pm1(st["pivot"], L).astype(np.float64), n)
    C = np.rint(np.fft.irfft(f * f.conj(), n)[:L]).astype(np.int64)
    assert np.array_equal(st["C"], C)
    a = np.abs(C[1:])
    assert st["psl_pivot"] == a.max() and st["unimproved"] == 0
    # a compensated sum of n terms: 2 u + n^2 u^2, the segments' sums once more
    F = math.fsum(oracle.power_table(st["alpha"], L + 8)[a])
    assert abs(st["F_pivot"] - F) <= 4 * 2.0 ** -53 * F and st["value_local"] == st["F_pivot"]


@pytest.mark.parametrize("L,n,flips", [(262144, 1, 10), (262145, 1, 10), (524287, 1, 16), (524287, 1, 17), (524288, 1, 1),
                                       (1048575, 1, 10), (1048575, 1, 0), (1048575, 1, 64), (1048575, 2, 5), (300000, 5, 16)])
def test_switched_pivots(ctx, L, n, flips):
    ids = ctx.init_walks(L, n, 3, alpha1=4, alpha2=7, n_lmt=70, switch_period=1, flip_lmt=flips)
    for _ in range(3):
        ctx.step_batch(ids, 1)
        _check(ctx.read_walk(ids[-1]), L)


def test_a_switching_step_of_a_long_walk(ctx):
    """A switch rebuilds C in about the time of the rest of a step."""
    best = {}
    for period in (0, 1):
        ids = ctx.init_walks(1048575, 1, 3, n_lmt=256, switch_period=period, flip_lmt=10)
        ctx.step_batch(ids, 5)
        best[period] = 1e9
        for _ in range(5):
            t = time.perf_counter()
            ctx.step_batch(ids, 20)
            best[period] = min(best[period], (time.perf_counter() - t) / 20)
        ctx.free_walks(ids)
    assert best[1] <= 2 * best[0], best
