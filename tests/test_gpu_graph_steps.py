"""Calls of any length with graph replay (graphs hold up to eight steps, longer
captures replace shorter ones, remainders are launched one by one) make the
steps that plain launches make: every state equal after every call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_09801_amd import libpsl
    c = libpsl.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("Ls,flip", [([1021], 5), ([300, 700, 4097], 3), ([9001], 90), ([16383, 257], 70)])
def test_calls_of_any_length(ctx, Ls, flip):
    mk = lambda: [w for L in Ls for w in ctx.init_walks(L, 1, 31 + L, n_lmt=0, switch_period=4, flip_lmt=flip)]
    eager, graph, other = mk(), mk(), ctx.init_walks(300, 2, 7, n_lmt=0)
    for steps in (1, 2, 7, 8, 9, 20, 3, 16, 1):
        ctx.step_batch(eager, steps)
        ctx.step_batch(graph, steps, graph=True)
        ctx.step_batch(other, 1)          # eager work between replays
        ctx.sync()
        for a, b in zip(eager, graph):
            ga, gb = ctx.read_walk(a), ctx.read_walk(b)
            for key in ("pivot", "C", "best", "local_best"):
                assert np.array_equal(ga[key], gb[key]), (steps, key)
            for key in ("t", "psl_best", "alpha", "unimproved", "q", "last_k", "value_local", "F_pivot"):
                assert ga[key] == gb[key], (steps, key)
    ctx.free_walks(eager + graph + other)
