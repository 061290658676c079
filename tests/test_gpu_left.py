"""Walks whose near-peak list overflows, so that a step leaves them to the table
evaluation: no matrix products where no step could use them, table evaluations
spread over the launch, and the large launches' forms (more than 256 combine
blocks; flat and persistent, every number of wavefronts)."""
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


def _equal(a, b):
    assert all(np.array_equal(a[k], b[k]) for k in ("pivot", "best", "local_best", "C"))
    assert all(a[k] == b[k] for k in ("t", "alpha", "psl_pivot", "psl_best", "last_k", "unimproved"))
    assert abs(a["value_local"] - b["value_local"]) <= 1e-13 * b["value_local"]


def test_no_products_with_the_list_switched_off(ctx):
    """PSL_OPT_NEAR_LIMIT 0: the time of the products (events around them) is that
    of no launch; a launch over this walk takes more than 0.1 ms."""
    from paper_2107_09801_amd import libpsl
    ctx.set_option(libpsl.OPT_NEAR_LIMIT, 0)
    (w,) = ctx.init_walks(131071, 1, 3)
    ctx.step_batch([w], 2)
    ctx.timing_enable()
    ctx.step_batch([w], 5)
    t = ctx.timing_read()
    assert t["steps"] == 5 and t["lin_ms"] / 5 < 0.05


@pytest.mark.parametrize("L,n_lmt", [(131071, 512), (65535, 6912), (1048575, 512)])
def test_a_left_walk_costs_few_table_steps(ctx, L, n_lmt):
    """All elements alike: the nine smallest shifts are near the peak, so that every
    step overflows a list of one."""
    from paper_2107_09801_amd import libpsl
    per = []
    for opt, value in ((libpsl.OPT_NEAR_LIMIT, 1), (libpsl.OPT_SPLIT, 0)):
        ctx.set_option(opt, value)
        (w,) = ctx.init_walks(L, 1, 3, n_lmt=n_lmt, init_bits=[si.all_plus_bits(L)])
        ctx.step_batch([w], 2)
        best = 1e9
        for _ in range(3):
            t = time.perf_counter()
            ctx.step_batch([w], 10)
            best = min(best, (time.perf_counter() - t) / 10)
        per.append(best)
        ctx.set_option(opt, -1)
    assert per[0] <= 6 * per[1], per


@pytest.mark.parametrize("L,n_lmt,n", [(512, 512, 1), (600, 512, 2), (1021, 1021, 1), (4099, 300, 1), (9001, 5000, 3),
                                       (65535, 512, 1), (65535, 6912, 1), (131071, 700, 2), (65535, 65535, 1), (131071, 131071, 1)])
@pytest.mark.parametrize("limit", [1, 3])
def test_left_walks_make_the_table_steps(ctx, L, n_lmt, n, limit):
    """Random pivots, whose lists overflow in some steps, and alike elements, whose
    do in all."""
    from paper_2107_09801_amd import libpsl
    bits = [si.random_bits(L, L + n), si.all_plus_bits(L), si.biased_bits(L, 5, 0.2)][:n]
    if n == 1 and limit == 3:
        bits = [si.all_plus_bits(L)]
    states = []
    for opts in (((libpsl.OPT_SPLIT, 1), (libpsl.OPT_NEAR_LIMIT, limit)), ((libpsl.OPT_SPLIT, 0),)):
        for o, v in opts:
            ctx.set_option(o, v)
        ids = ctx.init_walks(L, n, 11, alpha1=4, alpha2=10, n_lmt=n_lmt, switch_period=4, init_bits=bits)
        ctx.step_batch(ids, 9)
        states.append([ctx.read_walk(w) for w in ids])
        for o, _ in opts:
            ctx.set_option(o, -1)
    for a, b in zip(*states):
        _equal(a, b)


@pytest.mark.parametrize("limit", [1, 3])
@pytest.mark.parametrize("shape", [None, (16, 1, 2), (16, 1, 1), (8, 0, 0), (8, 1, 3), (4, 0, 0), (4, 1, 6)])
def test_left_walks_of_large_launches(ctx, tmp_path, shape, limit):
    """512 walks of 600 elements (1536 combine blocks, 16 wavefronts by default),
    with a limit that some or all of them overflow."""
    from paper_2107_09801_amd import libpsl
    lg = lambda x: int(x).bit_length() - 1
    states = []
    for mode in (1, 0):
        c = libpsl.Context(0)
        c.set_option(libpsl.OPT_SPLIT, mode)
        if mode:
            c.set_option(libpsl.OPT_NEAR_LIMIT, limit)
            if shape:
                f = tmp_path / "shape.txt"
                f.write_text("%d %d %d %d\n" % ((lg(600) << 24 | lg(600) << 16 | lg(512) << 8,) + shape))
                c.tune_load(str(f))
        ids = c.init_walks(600, 512, 77, alpha1=4, alpha2=13, switch_period=3, flip_lmt=10)
        c.step_batch(ids, 7)
        states.append([c.read_walk(w) for w in ids[::7]])
        c.close()
    for a, b in zip(*states):
        _equal(a, b)
