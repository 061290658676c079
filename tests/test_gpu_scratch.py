"""Device memory of the matrix path: its scratch follows the neighbourhood, not
the sequence, and a batch whose scratch cannot be had is evaluated from the
tables instead of being refused. Kept layouts give way to walks and to serving."""
import numpy as np
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

STATE = ("pivot", "C", "best", "local_best")
MB = 1 << 20


@pytest.fixture()
def ctx():
    from paper_2107_09801_amd import libpsl
    c = libpsl.Context(0)
    yield c
    c.close()


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info(0)[0]


def _fill(leave):
    """Tensors, in a list, that leave about `leave` bytes of device memory free (what
    is reported free after an allocation can be more than was before it less its size)."""
    import torch
    torch.cuda.empty_cache()
    hold = []
    while _free() > leave + 32 * MB:
        try:
            hold.append(torch.empty(_free() - leave, dtype=torch.uint8, device="cuda:0"))
        except torch.OutOfMemoryError:      # less is free than is reported
            break
    return hold


def _drop(hold):
    import torch
    hold.clear()
    torch.cuda.empty_cache()


def _same(a, b):
    assert all(np.array_equal(a[k], b[k]) for k in STATE)
    assert all(a[k] == b[k] for k in ("t", "psl_pivot", "psl_best", "last_k"))
    assert abs(a["value_local"] - b["value_local"]) <= 1e-13 * b["value_local"]


@pytest.mark.parametrize("L,n_lmt", [(1048575, 512), (1048575, 6912), (262143, 700)])
def test_scratch_of_a_limited_neighbourhood(ctx, L, n_lmt):
    """Digits and prefix sums take 40 bytes per shift; the partial sums of the
    neighbourhood's tiles and of the table evaluation a few MB more."""
    (w,) = ctx.init_walks(L, 1, 3, n_lmt=n_lmt)
    ctx.init_walks(2, 1, 3)
    before = _free()
    ctx.step_batch([w], 1)
    assert before - _free() <= 40 * L + 96 * MB


def _room(ctx):
    """Walk slots for the tests: later starts do not grow the walk array, which would
    drop the kept layouts."""
    for n in (300, 301):
        ctx.free_walks(ctx.init_walks(2, n, 3))


# 700 MB of digits and prefix sums, where the table evaluation takes about 50
BATCH = dict(L=262143, n=64, seed=5, alpha1=4, alpha2=10, n_lmt=512, switch_period=3)


def test_steps_without_room_for_the_matrix_scratch(ctx):
    from paper_2107_09801_amd import libpsl
    states = []
    for full in (False, True):
        ids = ctx.init_walks(**BATCH)
        ctx.set_option(libpsl.OPT_SPLIT, -1 if full else 0)
        hold = _fill(400 * MB) if full else []
        try:
            ctx.step_batch(ids, 4)
        finally:
            _drop(hold)
        states.append([ctx.read_walk(w) for w in ids[::9]])
        ctx.free_walks(ids)
    for a, b in zip(*states):
        _same(a, b)


def test_walks_start_in_memory_that_kept_layouts_hold(ctx):
    _room(ctx)
    ids = ctx.init_walks(**BATCH)
    ctx.step_batch(ids, 1)
    hold = _fill(64 * MB)
    try:
        more = ctx.init_walks(**dict(BATCH, seed=99))      # 140 MB of slabs
        ctx.step_batch(ids[:1] + more[:1], 2)
    finally:
        _drop(hold)
    assert ctx.read_walk(more[0])["t"] == 2 and ctx.read_walk(ids[0])["t"] == 3


def test_serving_starts_in_memory_that_kept_layouts_hold(ctx):
    _room(ctx)
    ctx.init_walks(1048575, 1, 3, n_lmt=1)                  # the power tables of the longest walk
    ids = ctx.init_walks(**BATCH)
    ctx.step_batch(ids, 1)
    hold = _fill(64 * MB)
    try:
        ctx.serve_start(400 * MB, 4)
        t = ctx.serve_submit(1001, 1, 3)
        ctx.serve_stop()
        assert ctx.serve_poll(t)["steps"] == 3
    finally:
        _drop(hold)


@pytest.mark.parametrize("L", [513, 769, 1025, 12289, 16640])
def test_neighbourhoods_across_a_short_last_tile(ctx, L):
    """Neighbourhoods that start in every kind of tile and wrap: the partial sums'
    places count tiles from the neighbourhood's first."""
    import torch
    from paper_2107_09801_amd import libpsl
    (w,) = ctx.init_walks(L, 1, 1, alpha1=4, alpha2=13, init_bits=[si.random_bits(L, L)])
    for start, n in ((L - 1, 1), (L - 2, 2), (L - 2, 513), (255, 258), (256, 512), (L - 257, 259), (L - 2, L),
                     (300, L), (511, L - 255), (L // 2, L - 1)):
        res = []
        for mode in (1, 0):
            ctx.set_option(libpsl.OPT_SPLIT, mode)
            F = torch.empty(n, dtype=torch.float64, device="cuda:0")
            P = torch.empty(n, dtype=torch.int32, device="cuda:0")
            ch = ctx.eval_neighbourhood(w, start % L, n, F, P)
            res.append((ch, F.cpu().numpy(), P.cpu().numpy()))
        (a, F, P), (b, Ft, Pt) = res
        assert np.array_equal(P, Pt) and np.max(np.abs(F - Ft) / Ft) <= 1e-13, (start, n)
        assert all(a[k] == b[k] for k in ("i_best", "j_best", "j_psl", "psl_min", "psl_k")), (start, n)
