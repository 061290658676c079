"""F of the matrix path against exact sums of the same table values, within the
bound its signed sums have, from the shortest walks it takes (where tiles, guards
and edges are tightest and |C_k| is smallest against the flip's 4) on.

F_j = sum T(|C_k|) + prefix differences + matrix sums. Every part is a sum of
fewer than 64 rounded additions per path from a term to F_j, so with
S_j the sum of the absolute values of all terms that go into it (both prefix
sums whole, all coefficients) its error is at most 64 u S_j, u = 2^-53, plus U / 2 for each
of the L - 1 rounded coefficients, U the quantum."""
import math

import numpy as np
import pytest

import oracle
import seeded_inputs as si

pytestmark = pytest.mark.gpu

U53 = 2.0 ** -53


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_09801_amd import libpsl
    c = libpsl.Context(0)
    yield c
    c.close()


def _reference(s, C, alpha, j):
    """(F_j, PSL_j, bound on the matrix path's error)."""
    L = len(s)
    T = oracle.power_table(alpha, L + 8)
    k = np.arange(1, L)
    c = C[1:].astype(np.int64)
    right = np.where(j + k < L, s[np.minimum(j + k, L - 1)], 0)
    left = np.where(j - k >= 0, s[np.maximum(j - k, 0)], 0)
    cj = c - 2 * s[j] * (right + left)
    F = math.fsum(T[np.abs(cj)])
    t = lambda d: T[np.abs(c + d)]
    m, M = min(j, L - 1 - j), max(j, L - 1 - j)
    both, one = k <= m, (k > m) & (k <= M)
    pre = np.abs(t(-2 * s[j]) - t(0))
    S = t(0).sum() + pre[k <= M].sum() + pre[both].sum()
    S += (np.abs(t(-4) - t(0)) + np.abs(t(4) - t(-4)))[both].sum() + np.abs(t(2) - t(-2))[one].sum()
    P = int(np.abs(c).max())
    big = max(T[P + 4] - T[abs(P - 4)], T[P + 2] - T[abs(P - 2)])
    quantum = 2.0 ** (math.frexp(big)[1] - 1 - 66)
    return F, int(np.abs(cj).max()), 64 * U53 * S + 0.5 * (L - 1) * quantum


def _low_psl(ctx, L):
    """The best sequence of a short search."""
    (w,) = ctx.init_walks(L, 1, 7 * L, alpha1=4, alpha2=10, ls_lmt=200, flip_lmt=5)
    ctx.step_batch([w], 1500)
    bits = ctx.read_walk(w)["best"].copy()
    ctx.free_walks([w])
    return bits


LENGTHS = [512, 513, 543, 544, 575, 599, 639, 640, 641, 767, 768, 769, 1023, 1024, 1025, 1100, 1279, 1281, 1535, 2047]


@pytest.mark.parametrize("L", LENGTHS)
@pytest.mark.parametrize("low", [False, True])
def test_matrix_error_within_its_bound(ctx, L, low):
    import torch
    from paper_2107_09801_amd import libpsl
    bits = _low_psl(ctx, L) if low else si.random_bits(L, 3 * L)
    s = si.to_pm1(bits, L).astype(np.int64)
    C = oracle.corr(si.to_pm1(bits, L))
    for alpha in (1, 4, 13, 16):
        (w,) = ctx.init_walks(L, 1, 1, alpha1=alpha, n_lmt=1, init_bits=[bits])
        for start, n in ((L - 1, L), (0, 1), (254, 3), (L - 2, 2), (L // 2 - 2, 5)):
            ctx.set_option(libpsl.OPT_SPLIT, 1)
            F = torch.empty(n, dtype=torch.float64, device="cuda:0")
            P = torch.empty(n, dtype=torch.int32, device="cuda:0")
            try:
                ctx.eval_neighbourhood(w, start, n, F, P)
            finally:
                ctx.set_option(libpsl.OPT_SPLIT, -1)
            F, P = F.cpu().numpy(), P.cpu().numpy()
            for i in np.unique(np.linspace(0, n - 1, 23).astype(int)):
                Fr, Pr, tol = _reference(s, C, alpha, (start + 1 + int(i)) % L)
                assert P[i] == Pr and abs(F[i] - Fr) <= tol, (alpha, start, n, int(i), F[i], Fr, tol)
        ctx.free_walks([w])


@pytest.mark.parametrize("kind", ["plus", "alternating", "biased"])
@pytest.mark.parametrize("alpha", [1, 2, 13])
def test_largest_digit_sums(ctx, kind, alpha):
    """The longest walks with the largest |C_k|, where the sums of the digit columns
    come nearest to what FP32 holds exactly."""
    import torch
    from paper_2107_09801_amd import libpsl
    L, n = 1048575, 520
    bits = {"plus": si.all_plus_bits(L), "alternating": si.alternating_bits(L), "biased": si.biased_bits(L, 3, 0.1)}[kind]
    (w,) = ctx.init_walks(L, 1, 1, alpha1=alpha, n_lmt=1, init_bits=[bits])
    for start in (0, L // 2 - 260, L - 300):
        res = []
        for mode in (1, 0):
            ctx.set_option(libpsl.OPT_SPLIT, mode)
            F = torch.empty(n, dtype=torch.float64, device="cuda:0")
            P = torch.empty(n, dtype=torch.int32, device="cuda:0")
            ctx.eval_neighbourhood(w, start, n, F, P)
            res.append((F.cpu().numpy(), P.cpu().numpy()))
        ctx.set_option(libpsl.OPT_SPLIT, -1)
        (F, P), (Ft, Pt) = res
        # the coefficients add up to less than 3 F here: 64 u (1 + 4 x 3) + 1e-14
        assert np.array_equal(P, Pt) and np.max(np.abs(F - Ft) / Ft) <= 1.1e-13
    ctx.free_walks([w])
