"""Batches that mix matrix and table walks, the table evaluation's launch shapes
on walks that would take the matrix path, what the autotuner times, and the
evaluation call's other forms: without allocations, and into memory that kernels
cannot write."""
import ctypes

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


def _run(c, Ls, steps=9, n=2):
    ids = []
    for L in Ls:
        ids += c.init_walks(L, n, 57 + L, n_lmt=0, switch_period=4, flip_lmt=min(5, L))
    c.step_batch(ids, steps)
    states = [c.read_walk(w) for w in ids]
    c.free_walks(ids)
    return states


def _equal(got, want, tag=None):
    for a, b in zip(got, want):
        assert all(np.array_equal(a[k], b[k]) for k in ("pivot", "C", "best", "local_best")), tag
        assert all(a[k] == b[k] for k in ("t", "alpha", "psl_pivot", "psl_best", "last_k", "unimproved")), tag
        assert abs(a["value_local"] - b["value_local"]) <= 1e-13 * b["value_local"], tag


MIXED = [2, 65, 257, 511, 512, 1001, 3000, 9000]


@pytest.fixture(scope="module")
def want():
    from paper_2107_09801_amd import libpsl
    with libpsl.Context(0) as c:
        c.set_option(libpsl.OPT_SPLIT, 0)
        return _run(c, MIXED)


@pytest.mark.parametrize("shape", [(16, 0, 0), (16, 1, 1), (16, 1, 2), (8, 0, 0), (8, 1, 3), (4, 0, 0), (4, 1, 6)])
@pytest.mark.parametrize("route", ["table", "matrix", "left"])
def test_mixed_batch_in_every_launch_shape(ctx, tmp_path, want, shape, route):
    """table: no matrix walk; matrix: those of 512 elements and more; left: these
    too, but some of them evaluated from the tables."""
    from paper_2107_09801_amd import libpsl
    lg = lambda x: int(x).bit_length() - 1
    nl = sorted(L for L in MIXED for _ in range(2))
    key = lg(max(nl)) << 24 | lg(nl[len(nl) // 2]) << 16 | lg(len(nl)) << 8 | 1
    f = tmp_path / "shape.txt"
    f.write_text("%d %d %d %d\n" % ((key,) + shape))
    ctx.set_option(libpsl.OPT_SPLIT, 0 if route == "table" else 1)
    if route == "left":
        ctx.set_option(libpsl.OPT_NEAR_LIMIT, 2)
    ctx.tune_load(str(f))
    _equal(_run(ctx, MIXED), want, (shape, route))


@pytest.mark.parametrize("Ls", [[65, 511, 2049], [257, 16383], [300] * 40 + [5000], [2, 512]])
def test_mixed_batches(ctx, Ls):
    from paper_2107_09801_amd import libpsl
    ctx.set_option(libpsl.OPT_SPLIT, 0)
    table = _run(ctx, Ls)
    ctx.set_option(libpsl.OPT_SPLIT, 1)
    _equal(_run(ctx, Ls), table)


@pytest.mark.parametrize("L,n_lmt", [(16383, 0), (131071, 6912)])
def test_autotune_times_the_table_evaluation(ctx, L, n_lmt):
    """The tuned shape is the table evaluation's: its times are the same whether or
    not the batch's steps would take the matrix path."""
    from paper_2107_09801_amd import libpsl
    ids = ctx.init_walks(L, 1, 3, n_lmt=n_lmt)
    a = ctx.autotune(ids)
    ctx.set_option(libpsl.OPT_SPLIT, 0)
    b = ctx.autotune(ids)
    for k in ("default_ms", "eval_ms"):
        assert 0.6 < a[k] / b[k] < 1.7, (k, a[k], b[k])


@pytest.mark.parametrize("L,alpha,start,n", [(300, 4, 7, 300), (512, 13, 511, 512), (1001, 4, 17, 1001), (2049, 16, 0, 600),
                                             (16383, 13, 5, 16383), (16383, 4, 16000, 511), (131071, 10, 131000, 6912),
                                             (131071, 4, 9, 131071), (1048575, 4, 77, 1024)])
@pytest.mark.parametrize("limit", [-1, 1])
def test_noalloc_gives_the_same_bits(ctx, L, alpha, start, n, limit):
    """The call without allocations: the same evaluation, so the same F to the last
    bit, on either path."""
    import torch
    from paper_2107_09801_amd import libpsl
    ctx.set_option(libpsl.OPT_NEAR_LIMIT, limit)
    (w,) = ctx.init_walks(L, 1, 1, alpha1=alpha, n_lmt=1, init_bits=[si.random_bits(L, L + alpha)])
    res = []
    for call in (ctx.eval_neighbourhood, ctx.eval_neighbourhood_noalloc, ctx.eval_neighbourhood_noalloc):
        F = torch.empty(n, dtype=torch.float64, device="cuda:0")
        P = torch.empty(n, dtype=torch.int32, device="cuda:0")
        res.append((call(w, start, n, F, P), F.cpu().numpy(), P.cpu().numpy()))
    for ch, F, P in res[1:]:
        assert np.array_equal(F, res[0][1]) and np.array_equal(P, res[0][2]) and ch == res[0][0]


@pytest.mark.parametrize("L,n", [(300, 300), (1001, 1001), (16383, 700)])
def test_evaluation_into_host_memory(ctx, L, n):
    """Output arrays in pageable host memory, which a kernel cannot write, are copied
    to; so are pinned ones."""
    import torch
    from paper_2107_09801_amd import libpsl
    (w,) = ctx.init_walks(L, 1, 9, n_lmt=1)
    F = torch.empty(n, dtype=torch.float64, device="cuda:0")
    P = torch.empty(n, dtype=torch.int32, device="cuda:0")
    want = ctx.eval_neighbourhood(w, 3, n, F, P)
    for pin in (True, False):
        Fh = torch.zeros(n, dtype=torch.float64, pin_memory=pin)
        Ph = torch.zeros(n, dtype=torch.int32, pin_memory=pin)
        ch = libpsl.Choice()
        ctx._check(libpsl.lib().psl_eval_neighbourhood(ctx._h, w, 3, n, Fh.data_ptr(), Ph.data_ptr(), ctypes.byref(ch)))
        assert torch.equal(Fh, F.cpu()) and torch.equal(Ph, P.cpu()) and ch.as_dict() == want
