"""Evaluations and batches that cannot use the layout of the one before (another
N_lmt, other walks): right, and not much slower than without the matrix path, whose
memory a layout hands to the next."""
import time

import numpy as np
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_2107_09801_amd import libpsl
    c = libpsl.Context(0)
    yield c
    c.close()


def _eval(ctx, w, start, n):
    import torch
    F = torch.empty(n, dtype=torch.float64, device="cuda:0")
    P = torch.empty(n, dtype=torch.int32, device="cuda:0")
    ch = ctx.eval_neighbourhood(w, start, n, F, P)
    return ch["i_best"], F.cpu().numpy(), P.cpu().numpy()


def test_layouts_in_turn_equal_fresh_ones(ctx):
    """Each layout after a smaller, larger, equal and much larger one, matrix and
    table, against contexts that make no other."""
    from paper_2107_09801_amd import libpsl
    calls = [(600, 600), (5001, 5001), (5001, 700), (300, 300), (5001, 4000), (131071, 6912), (600, 512), (131071, 600),
             (2049, 2049), (131071, 512)]
    ids = {}
    for L in sorted({L for L, _ in calls}):
        (ids[L],) = ctx.init_walks(L, 1, 1, n_lmt=1, init_bits=[si.random_bits(L, L)])
    for L, n in calls + calls[::-1]:
        i, F, P = _eval(ctx, ids[L], L // 3, n)
        with libpsl.Context(0) as one:
            (w,) = one.init_walks(L, 1, 1, n_lmt=1, init_bits=[si.random_bits(L, L)])
            j, F1, P1 = _eval(one, w, L // 3, n)
        assert i == j and np.array_equal(F, F1) and np.array_equal(P, P1), (L, n)


def test_a_new_layout_costs_what_the_tables_do(ctx):
    from paper_2107_09801_amd import libpsl
    L = 1048575
    (w,) = ctx.init_walks(L, 1, 3, n_lmt=1)
    best = {}
    for mode in (-1, 0):
        ctx.set_option(libpsl.OPT_SPLIT, mode)
        best[mode] = 1e9
        for _ in range(12):
            t = time.perf_counter()
            for n in (600, 599, 601, 598):
                ctx.eval_neighbourhood(w, 5, n)
            best[mode] = min(best[mode], time.perf_counter() - t)
    assert best[-1] <= 1.4 * best[0], best


def test_a_new_batch_costs_what_the_tables_do(ctx):
    """Layouts of 1024 short walks, one after another, each with a step."""
    from paper_2107_09801_amd import libpsl
    ids = ctx.init_walks(600, 1024, 3)
    best = {}
    for mode in (-1, 0):
        best[mode] = 1e9
        for _ in range(12):
            t = time.perf_counter()
            ctx.set_option(libpsl.OPT_SPLIT, mode)          # drops the kept layouts
            ctx.step_batch(ids, 1)
            best[mode] = min(best[mode], time.perf_counter() - t)
    assert best[-1] <= 1.6 * best[0], best
