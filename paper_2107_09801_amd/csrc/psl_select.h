// psl_select.h -- device code: F and PSL per candidate from the partial sums,
// and Algorithm 1's selection, flags and bookkeeping (k_combine and k_select in
// psl_kernels.hip, k_combine_left in psl_eval.hip).
#pragma once
#include "psl_dev_util.h"
#include "psl_device.h"

#include <climits>

namespace psl {

struct ChoiceDev {
    uint32_t i_best, j_best;
    double F_best, F_min;
    uint32_t j_psl;
    int32_t psl_min;
    int32_t psl_k;
    uint32_t flags;         // CHOICE_AMBIG_ARGMIN
    uint32_t table;         // 1: no choice yet, the walk is left to the table evaluation
};

constexpr int kCombThreads = 256;
constexpr int kCombBatch = 16;      // split loads a combine lane keeps in flight
constexpr uint64_t kCombFuseBlocks = 256;   // most combine blocks of a launch that selects in its last blocks

// Candidates [lo, hi) of combine block b of `blocks`: contiguous ranges in
// scan order, a multiple of the block's candidates per pass (kCombThreads / G)
// long, so a block's minimum covers a contiguous run of scan indices.
__device__ __forceinline__ void comb_range(uint32_t n, uint32_t blocks, uint32_t G, uint32_t b, uint32_t &lo,
                                           uint32_t &hi)
{
    const uint32_t cpb = kCombThreads / G;
    const uint32_t chunk = ((n + blocks - 1) / blocks + cpb - 1) / cpb * cpb;
    lo = min(n, b * chunk);
    hi = min(n, lo + chunk);
}

__device__ __forceinline__ void sel_merge(double &f, int32_t &p, uint32_t &i, double of, int32_t op,
                                          uint32_t oi)
{
    f = of < f ? of : f;
    if (op < p || (op == p && oi < i)) {
        p = op;
        i = oi;
    }
}

// The wavefront's smallest F, and its first smallest PSL (PSLs are not negative).
__device__ __forceinline__ void sel_wave(double &f, int32_t &p, uint32_t &i)
{
    f = wave_least(f);
    const uint64_t v = wave_least(((uint64_t)(uint32_t)p << 32) | i);
    p = (int32_t)(v >> 32);
    i = (uint32_t)v;
}

// The scan of Algorithm 1 over the combined F and PSL of one walk (batch
// position bi), its ambiguity flags and, pure == 0, the rest of the iteration
// but for the C update, by a block of NT threads.
//
// Selection: the move is the first candidate in scan order within
// F_min*(1+tau); the best-PSL neighbour is the first with the minimum PSL. On a
// strict PSL improvement psl_best and solution_best = pivot with j_psl flipped.
// Ambiguity:
//   ARGMIN: some scanned neighbour's F lies within amb = margin*F_min of the
//     band edge thr = F_min*(1+tau) (|F - thr| <= amb): a different rounding
//     of Eq. (5) could move it across the edge and change the move;
//   COMPARE (steps only): the move's F lies strictly within margin*v_local of
//     v_local*(1-tau) or of v_local*(1+tau), the edges of the three-way
//     comparison with the local best.
// Every F of a combine block is at least that block's minimum and the blocks
// cover the scan order in runs, so the first band member is in the first block
// whose minimum is in the band, and only the blocks whose minimum is at most
// thr + amb are read (usually the one that holds F_min): one pass over them
// gives both.
// Bookkeeping: the move's bit, the three-way comparison with v_local, the
// unimproved counter, the local best, and the phase switch (Rand_flip of the
// local best and the exponent swap; the walk joins the batch's pending list,
// whose C, F and PSL the C update then rebuilds). The C update runs after it
// (k_apply), from bits that equal the pre-move pivot's at every position but j:
// the pivot's, or on a switch the local best's (which are then the move's
// pivot, if the move improved; if it did not, C is rebuilt from C of the local
// best anyway).
// pure != 0: the choice record goes to out[bi] and the walk stays unchanged.
//
// Everything is latency here: the walk's fields are read at the start, and what
// the parts hand on stays in LDS (through global memory, one after the other,
// the same work took 5 us more of a single walk's step). Minima go through lane
// permutations. Of the 13.7 us of a combine with its selection at L = 16383 (14.9
// with butterflies through LDS and the prefix sums loaded after the lanes' sums)
// the candidates take 4, the blocks' count with its release 2, the selection 4.
struct FinishLds {
    SelPart w[16];
    uint64_t near[16];
    uint32_t first[16];
    double Fb;
    int32_t Pb;
    int hit[16];
    int improve, improved, sw;
    uint32_t kb, jp;
    uint32_t pos[1024];
};

template <int NT>
__device__ __forceinline__ void finish_walk(FinishLds &sh, WalkDev &w, const BatchEntry &be, uint32_t bi,
                                            uint32_t comb_blocks, uint32_t comb_group, int pure, ChoiceDev *out,
                                            uint32_t *pend, double margin)
{
    constexpr int kWaves = NT / 64;
    static_assert(kCombMaxBlocks <= NT && kWaves <= 16, "one combine block per thread");
    const uint32_t t = threadIdx.x;
    if (pure == 1 && be.lsplit && !be.ss->use) {
        if (t == 0) out[bi].table = 1;
        return;
    }
    const int lane = (int)t & 63, wave = (int)t >> 6;
    double fmin = INFINITY;
    int32_t pmin = INT_MAX;
    uint32_t ipmin = UINT_MAX;
    if (t < comb_blocks) {
        const SelPart r = be.red[t];
        fmin = r.f;
        pmin = r.p;
        ipmin = r.i;
    }
    const uint32_t n = be.fixed ? be.n_lmt : w.n_lmt;
    const uint32_t start = be.fixed ? be.start : step_start(w);
    const uint32_t L = w.L;
    const double vl = w.value_local;
    const int32_t psl_best = w.psl_best;
    const uint32_t unimproved0 = w.unimproved, ls_lmt = w.ls_lmt, period = w.switch_period;
    const uint64_t step = w.t;
    const uint32_t trace_cap = w.trace_cap, alpha = w.alpha;
    const double my_f = fmin;           // this thread's combine block minimum
    // block minima: within each wavefront, then across the wavefronts (the
    // minimum F and the first minimum (PSL, index) do not depend on the order)
    sel_wave(fmin, pmin, ipmin);
    if (lane == 0) sh.w[wave] = SelPart{fmin, pmin, ipmin};
    __syncthreads();
    SelPart r = sh.w[0];
    for (int x = 1; x < kWaves; ++x) sel_merge(r.f, r.p, r.i, sh.w[x].f, sh.w[x].p, sh.w[x].i);
    const double Fmin = r.f;
    const int32_t Pmin = r.p;
    const uint32_t iPmin = r.i;
    const double thr = Fmin * (1.0 + kTau), amb = margin * Fmin;

    // the combine blocks to read, one 64-bit mask per wavefront
    const uint64_t m = __ballot(t < comb_blocks && (my_f <= thr || my_f - thr <= amb));
    if (lane == 0) sh.near[wave] = m;
    __syncthreads();
    uint32_t ifirst = UINT_MAX;         // this thread's first candidate in the band, its F and PSL
    double Fi = 0.0;
    int32_t Pi = 0;
    int hit = 0;
    for (int q = 0; q < kWaves; ++q) {
        for (uint64_t bits = sh.near[q]; bits; bits &= bits - 1) {      // the same for every thread of the block
            const uint32_t b = 64u * (uint32_t)q + (uint32_t)__builtin_ctzll(bits);
            uint32_t lo, hi;
            comb_range(n, comb_blocks, comb_group, b, lo, hi);
            for (uint32_t i0 = lo; i0 < hi; i0 += 4 * NT) {
                double v[4];
                int32_t pv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t i = i0 + (uint32_t)u * NT + t;
                    v[u] = i < hi ? be.F[i] : INFINITY;
                    pv[u] = i < hi ? be.P[i] : 0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double g = v[u] - thr;
                    hit |= (g < 0.0 ? -g : g) <= amb;
                    const uint32_t i = i0 + (uint32_t)u * NT + t;
                    if (v[u] <= thr && i < ifirst) {
                        ifirst = i;
                        Fi = v[u];
                        Pi = pv[u];
                    }
                }
            }
        }
    }
    uint32_t ib = ifirst;
    ib = (uint32_t)wave_least((uint64_t)ib);
    hit = __any(hit);
    if (lane == 0) {
        sh.first[wave] = ib;
        sh.hit[wave] = hit;
    }
    __syncthreads();
    ib = sh.first[0];
    hit = sh.hit[0];
    for (int x = 1; x < kWaves; ++x) {
        ib = min(ib, sh.first[x]);
        hit |= sh.hit[x];
    }
    // with finite F the block holding F_min is in the band, so a member was
    // found; otherwise only the reads stay in bounds
    if (ib < n) {
        if (ifirst == ib) {
            sh.Fb = Fi;
            sh.Pb = Pi;
        }
    } else {
        ib = iPmin < n ? iPmin : 0u;
        if (t == 0) {
            sh.Fb = be.F[ib];
            sh.Pb = be.P[ib];
        }
    }
    __syncthreads();
    if (t == 0) {
        const uint32_t kb = (uint32_t)(((uint64_t)start + 1u + ib) % L);
        const uint32_t jp = (uint32_t)(((uint64_t)start + 1u + iPmin) % L);
        const double Fb = sh.Fb;
        const int32_t Pb = sh.Pb;
        be.near[0] = 0;           // the evaluation has read it; the next step appends to it
        sh.improve = sh.improved = sh.sw = 0;
        if (pure) {
            ChoiceDev c;
            c.i_best = ib; c.j_best = kb; c.F_best = Fb; c.F_min = Fmin;
            c.j_psl = jp; c.psl_min = Pmin; c.psl_k = Pb; c.flags = hit ? CHOICE_AMBIG_ARGMIN : 0u;
            c.table = 0;
            out[bi] = c;
        } else {
            // three-way comparison of the move with v_local (Algorithm 1)
            uint32_t fl = 0;
            const double elo = vl * (1.0 - kTau), ehi = vl * (1.0 + kTau), band = margin * vl;
            if (Fb < elo) fl = STEP_IMPROVED;
            else if (Fb > ehi) fl = STEP_WORSE;
            int32_t best = psl_best;
            if (Pmin < psl_best) {
                best = Pmin;
                w.psl_best = Pmin;
                fl |= STEP_PSL_IMPROVED;
                sh.improve = 1;
            }
            if (hit) fl |= STEP_AMBIG_ARGMIN;
            if ((Fb - elo < band && elo - Fb < band) || (Fb - ehi < band && ehi - Fb < band)) fl |= STEP_AMBIG_COMPARE;
            uint32_t unimproved = unimproved0;
            int sw = 0;
            if (fl & STEP_IMPROVED) {
                sh.improved = 1;
                unimproved = 0;
                w.value_local = Fb;
            } else if (fl & STEP_WORSE) {
                unimproved += 1;
                if (period == 0 && unimproved > ls_lmt) sw = 1;
            }
            if (period > 0 && ((step + 1u) % period) == 0) sw = 1;
            if (sw) fl |= STEP_SWITCHED;
            w.unimproved = unimproved;
            w.start = start;
            w.k = kb;
            w.i_best = ib;
            w.value_step = Fb;
            w.F_min = Fmin;
            w.psl_k = Pb;
            w.j_psl = jp;
            w.psl_min = Pmin;
            w.F_pivot = Fb;
            w.psl_pivot = Pb;
            w.flags = fl;
            if (trace_cap) {
                TraceEntry e;
                e.t = step;
                e.start = start;
                e.k = kb;
                e.value_step = Fb;
                e.psl_k = Pb;
                e.psl_best = best;
                e.alpha = sw ? (alpha == w.alpha1 ? w.alpha2 : w.alpha1) : alpha;
                e.flags = fl;
                w.trace[step % trace_cap] = e;
            }
            w.t = step + 1;
            sh.sw = sw;
            sh.kb = kb;
            sh.jp = jp;
        }
    }
    if (pure) return;
    __syncthreads();
    const uint32_t kb = sh.kb;
    // solution_best from the pre-move pivot, then the move, then local_best
    // from the new pivot
    if (sh.improve) {
        copy_words(w.best, w.pivot, w.nw, t, NT, sh.jp >> 6, 1ull << (sh.jp & 63u));
        __syncthreads();                // before the bit flips
    }
    if (t == 0) w.pivot[kb >> 6] ^= 1ull << (kb & 63u);
    if (!sh.improved && !sh.sw) return;
    __syncthreads();
    if (sh.improved) copy_words(w.local_best, w.pivot, w.nw, t, NT, UINT32_MAX, 0);
    if (!sh.sw) return;
    __syncthreads();
    copy_words(w.pivot, w.local_best, w.nw, t, NT, UINT32_MAX, 0);
    __syncthreads();
    if (t == 0) {
        uint32_t cnt = 0;
        for (uint64_t a = 0; cnt < w.flip_lmt && a < (1ull << 24); ++a) {
            const uint64_t ctr = (2ull << 60) | (w.q << 24) | a;
            const uint32_t pos = (uint32_t)(draw(w.seed, ctr) % (uint64_t)L);
            bool dup = false;
            for (uint32_t x = 0; x < cnt; ++x) dup |= (sh.pos[x] == pos);
            if (dup) continue;
            sh.pos[cnt] = pos;
            w.flips[cnt] = pos;
            ++cnt;
            w.pivot[pos >> 6] ^= 1ull << (pos & 63u);
        }
        w.n_flips = cnt;
        w.alpha = (w.alpha == w.alpha1) ? w.alpha2 : w.alpha1;
        w.q += 1;
        w.pending = 1;
        pend[1 + atomicAdd(&pend[0], 1u)] = bi;
    }
}

// The largest |C'_k| of element j's flip over the near-peak shifts list[g],
// list[g + G], ..
__device__ __forceinline__ uint32_t near_peak(const uint32_t *__restrict__ list, uint32_t n, const int32_t *__restrict__ C,
                                              const uint32_t *__restrict__ w32, int L, int j, uint32_t g, uint32_t G)
{
    const uint32_t sj = (w32[j >> 5] >> (j & 31)) & 1u;
    int peak = 0;
#pragma unroll 4
    for (uint32_t q = g; q < n; q += G) {
        const int k = (int)list[q];
        int c = C[k];
        const int pr = j + k, pl = j - k;            // the guard words hold every index
        const uint32_t wr = w32[pr >> 5], wl = w32[pl >> 5];
        if (pr < L) c += (((wr >> (pr & 31)) & 1u) ^ sj) ? 2 : -2;
        if (pl >= 0) c += (((wl >> (pl & 31)) & 1u) ^ sj) ? 2 : -2;
        peak = max(peak, c < 0 ? -c : c);
    }
    return (uint32_t)peak;
}

// F and PSL per candidate from the partials, for block b of a walk's `blocks`; the
// block leaves its smallest F and its first smallest PSL in be.red. Form: from
// ks table partials per candidate, from the matrix sums, or as this step chose.
// EARLY: the prefix sums are loaded first. A group of G lanes
// (a power of two, at most 64) shares a candidate: lane g adds splits g,
// g+G, ... in order, then the group adds its lanes' sums in a fixed order for
// a given split count and G (G = 1 adds the splits in order). For G <= 4 a
// group is G adjacent lanes (a butterfly); for G >= 8 a block pass takes
// cpb = 256 / G <= 32 candidates, lane t of the block has candidate t mod cpb
// and split lane t / cpb, so that one load of a wavefront reads cpb
// consecutive partials of each of 64 / cpb splits; the sums go through a
// butterfly over the wavefront's split lanes, then the four wavefronts' sums
// are added in wavefront order.
struct CombLds {
    double f[4][32];
    uint32_t m[4][32];
    SelPart r[kCombThreads / 64];
    uint32_t last;
    FinishLds fin;
};
enum class Form { table, matrix, either };
template <bool EARLY, Form FORM>
__device__ __forceinline__ void combine_part(CombLds &sh, WalkDev &w, const BatchEntry &be, const Tables &tabs, int G,
                                             uint32_t blocks, uint32_t b, uint32_t ks)
{
    const uint32_t n = be.fixed ? be.n_lmt : w.n_lmt;
    const double *T = tabs.T[w.alpha];
    const uint32_t cpb = kCombThreads / (uint32_t)G;      // candidates per block pass
    const bool wide = G >= 8;
    const uint32_t g = wide ? threadIdx.x / cpb : threadIdx.x & (uint32_t)(G - 1);
    const uint32_t ci = wide ? threadIdx.x % cpb : threadIdx.x / (uint32_t)G;   // candidate in the pass
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert(kCombThreads == 256, "four wavefronts per combine block");
    // matrix path: F_j from the prefix sums and the matrix sums (psl_split.hip),
    // PSL_j from the near-peak shifts here
    const bool split = FORM == Form::matrix || (FORM == Form::either && be.lsplit != 0 && be.ss->use != 0);
    const double U = split ? be.ss->U : 0.0, total = split ? be.ss->total : 0.0;
    const uint32_t start = be.fixed ? be.start : step_start(w);
    const uint32_t L = w.L;
    const uint32_t j_first = (start + 1u) % L;
    const uint32_t n_near = split ? be.near[0] : 0;

    double fmin = INFINITY;
    int32_t pmin = INT_MAX;
    uint32_t ipmin = UINT_MAX;
    uint32_t lo, hi;
    comb_range(n, blocks, (uint32_t)G, b, lo, hi);
    for (uint32_t i0 = lo; i0 < hi; i0 += cpb) {
        const uint32_t i = i0 + ci;
        double f = 0.0;
        uint32_t m = 0;
        // the prefix sums of F_j = sum_k T(|C_k|) + sum_{m<k<=M} (T(|C_k-+2|) - T(|C_k|))
        // + U (matrix sums), m = min(j, L-1-j), M = max(j, L-1-j), -2 for
        // s_j = +1; lane 0 of a group has them. In small launches they are loaded
        // first, beside the other lanes' loads; in large ones last, for fewer
        // registers (1024 walks at L = 131071 with five values: 2.6 ms per step, loaded
        // first 2.9; with these two 2.3)
        double pv[2] = {}, po[2] = {};
        auto prefixes = [&]() {
            const uint32_t j = (uint32_t)(((uint64_t)start + 1u + i) % L);
            const uint32_t mj = min(j, L - 1 - j), Mj = max(j, L - 1 - j);
            const int p1 = get_bit(w.pivot, j) ? 1 : 0;
            split_prefix(be, L, p1, Mj, pv[0], po[0]);
            split_prefix(be, L, p1, mj, pv[1], po[1]);
        };
        if (split) {
            if (i < hi) {
                const uint32_t j = (uint32_t)(((uint64_t)start + 1u + i) % L);
                if (EARLY && g == 0) prefixes();
                const double *part = be.lpart + mx_place(L, j_first, j);
                for (uint32_t x = g; x <= be.lsplit; x += (uint32_t)G) f += part[(size_t)x * be.lrow];
                m = near_peak(be.near + 1, n_near, w.C, reinterpret_cast<const uint32_t *>(w.pivot), (int)L, (int)j, g,
                              (uint32_t)G);
            }
        } else if (i < hi) {
            // up to kCombBatch of this lane's splits are loaded before they
            // are added (in split order)
            for (uint32_t x0 = g; x0 < ks; x0 += (uint32_t)G * kCombBatch) {
                double v[kCombBatch];
                uint32_t mv[kCombBatch];
#pragma unroll
                for (int u = 0; u < kCombBatch; ++u) {
                    const uint32_t x = x0 + (uint32_t)u * (uint32_t)G;
                    if (x < ks) {
                        v[u] = be.Fpart[(size_t)x * n + i];
                        mv[u] = be.Mpart[(size_t)x * n + i];
                    }
                }
#pragma unroll
                for (int u = 0; u < kCombBatch; ++u) {
                    if (x0 + (uint32_t)u * (uint32_t)G < ks) {
                        f += v[u];
                        m = max(m, mv[u]);
                    }
                }
            }
        }
        if (wide) {
            for (int o = (int)cpb; o < 64; o <<= 1) {
                f += __shfl_xor(f, o);
                m = max(m, (uint32_t)__shfl_xor((int)m, o));
            }
            if ((uint32_t)lane < cpb) {
                sh.f[wave][lane] = f;
                sh.m[wave][lane] = m;
            }
            __syncthreads();
            if (g == 0) {           // wavefront 0, lanes below cpb
                f = sh.f[0][lane];
                m = sh.m[0][lane];
                for (int x = 1; x < 4; ++x) {
                    f += sh.f[x][lane];
                    m = max(m, sh.m[x][lane]);
                }
            }
            __syncthreads();        // the next pass rewrites the rows
        } else {
            for (int o = G >> 1; o > 0; o >>= 1) {
                f += __shfl_xor(f, o);
                m = max(m, (uint32_t)__shfl_xor((int)m, o));
            }
        }
        if (g == 0 && i < hi) {
            // the near-peak path stores the PSL itself; the dense path the
            // high word of T(PSL), which is at least hi32(T(1)) = 0x3FF00000
            // because |C'_{L-1}| = 1 for every sequence
            const int32_t p = m < 0x3FF00000u ? (int32_t)m : table_inverse(T, tabs.n, m);
            if (split) {
                if (!EARLY) prefixes();
                f = total + ((pv[0] + po[0]) - (pv[1] + po[1])) + U * f;
            }
            be.F[i] = f;
            be.P[i] = p;
            fmin = f < fmin ? f : fmin;
            if (p < pmin) { pmin = p; ipmin = i; }
        }
    }
    sel_wave(fmin, pmin, ipmin);
    if (lane == 0) sh.r[wave] = SelPart{fmin, pmin, ipmin};
    __syncthreads();
    if (threadIdx.x == 0) {
        SelPart r = sh.r[0];
        for (int x = 1; x < kCombThreads / 64; ++x) sel_merge(r.f, r.p, r.i, sh.r[x].f, sh.r[x].p, sh.r[x].i);
        be.red[b] = r;
    }
}

// Whether the block is the last of `blocks` to come here (counted in done[bi],
// which it returns to 0 for the next launch). Each block's count is a
// device-scope release of what it stored, and the last block acquires it all.
__device__ __forceinline__ bool last_block(CombLds &sh, uint32_t *done, uint32_t bi, uint32_t blocks)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t last = 1;
        if (blocks > 1) {
            const uint32_t before =
                __hip_atomic_fetch_add(&done[bi], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            last = before == blocks - 1 ? 1u : 0u;
            if (last) done[bi] = 0;
        }
        sh.last = last;
    }
    __syncthreads();
    if (!sh.last) return false;
    if (blocks > 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return true;
}

// The launches that make their selection in the last combine blocks.
inline bool comb_small(uint32_t nb, uint32_t comb_blocks) { return (uint64_t)nb * comb_blocks <= kCombFuseBlocks; }

}  // namespace psl
