"""Device memory of the matrix path: its scratch follows the neighbourhood, not
the sequence."""
import numpy as np
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

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


@pytest.mark.parametrize("L,n_lmt", [(1048575, 512), (1048575, 6912), (262143, 700)])
def test_scratch_of_a_limited_neighbourhood(ctx, L, n_lmt):
    """Digits and prefix sums take 40 bytes per shift; the partial sums of the
    neighbourhood's tiles and of the table evaluation a few MB more."""
    (w,) = ctx.init_walks(L, 1, 3, n_lmt=n_lmt)
    ctx.init_walks(2, 1, 3)
    before = _free()
    ctx.step_batch([w], 1)
    assert before - _free() <= 40 * L + 96 * MB


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
