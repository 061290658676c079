// psl_kernels.hip -- gfx950 kernels of libpsl around the neighbourhood
// evaluation (which lives in psl_eval.hip): power tables, init (the
// correlations of Eq. (2) are psl_corr.hip's), the phase-switch rebuild, the per-step chunk sums
// and near-peak list the evaluation reads, the selection of Algorithm 1's
// scan, the O(L) flip of Section 3 and the step's bookkeeping.
#include "psl_chunks.h"
#include "psl_dev_util.h"
#include "psl_device.h"
#include "psl_launch.h"
#include "psl_select.h"

#include <algorithm>
#include <climits>

namespace psl {

// ------------------------------------------------------- power tables

__global__ void k_power_table(double *T, uint32_t n, uint32_t alpha)
{
    uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    double x = (double)c, p = x;
    for (uint32_t a = 1; a < alpha; ++a) p = p * x;
    T[c] = p;
}

// ------------------------------------------------------------- init

// A walk's start: block (x, b) zeroes its part of walk b's slab (the pivot sits
// between zeroed guard words, see guard_words) and block (0, b) writes the
// walk's record. One launch for a batch; a memset and a copy per walk took 15 us
// of host time each.
constexpr uint32_t kInitSpan = 16384;      // bytes of a slab per block
__global__ __launch_bounds__(256) void k_init_slabs(WalkDev *walks, const InitRec *recs)
{
    const InitRec &rec = recs[blockIdx.y];
    if (blockIdx.x == 0) {
        constexpr uint32_t kWords = sizeof(WalkDev) / 4;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(&rec.dev);
        uint32_t *dst = reinterpret_cast<uint32_t *>(&walks[rec.slot]);
        for (uint32_t i = threadIdx.x; i < kWords; i += 256) dst[i] = src[i];
    }
    const uint64_t lo = (uint64_t)blockIdx.x * kInitSpan;
    if (lo >= rec.bytes) return;
    uint4 *p = reinterpret_cast<uint4 *>(reinterpret_cast<char *>(rec.slab) + lo);
    const uint32_t n = (uint32_t)((rec.bytes - lo < kInitSpan ? rec.bytes - lo : kInitSpan) / 16);
    for (uint32_t i = threadIdx.x; i < n; i += 256) p[i] = make_uint4(0, 0, 0, 0);
}

// The initial pivots: the given bits (rec.given, in words of the staged bits) or
// Rand(L, SEED); then local_best = best = pivot.
__global__ void k_init_bits(WalkDev *walks, const InitRec *recs, const uint64_t *bits)
{
    const InitRec &rec = recs[blockIdx.y];
    const WalkDev &w = walks[rec.slot];
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= w.nw) return;
    uint64_t v;
    if (rec.given != kNoBits) {
        v = bits[rec.given + i];
    } else {
        v = draw(w.seed, i);
        if (i == w.nw - 1 && (w.L & 63u)) v &= (1ull << (w.L & 63u)) - 1ull;
    }
    w.pivot[i] = v;
    w.local_best[i] = v;
    w.best[i] = v;
}

// The pending list of a batch: pend[0] = count, pend[1..] = batch positions
// of the walks whose step ended in a phase switch (the bookkeeping appends,
// the selection of the next step clears the count).
//
// C of a switched pivot from C of local_best: the FLIP_lmt one-element flips
// in draw order, where flip f sees local_best with flips 0..f-1 applied.
// Element x of that sequence differs from local_best only if x is an earlier
// flip position, and flip f reads elements p_f and p_f +- k; so for every k
// outside D = {|p_f - p_g| : g < f} the update can read local_best's bits
// directly, and the shifts in D take the sequential bits.
__device__ __forceinline__ int32_t switch_flip_delta(const uint64_t *lb, uint32_t L, uint32_t k, uint32_t p, int sp)
{
    int d = 0;
    if (p + k < L) d += get_bit(lb, p + k) ? -1 : 1;
    if (k <= p) d += get_bit(lb, p - k) ? -1 : 1;
    return -2 * sp * d;
}

// C_k of the switched pivot for a shift k in D, from c = C_k of local_best: each
// flip reads the elements as the earlier flips left them.
__device__ __forceinline__ int32_t switch_corr_seq(const uint64_t *lb, int32_t c, uint32_t L, uint32_t k,
                                                   const uint32_t *fl, uint32_t nf)
{
    for (uint32_t h = 0; h < nf; ++h) {
        // element x after flips 0..h-1
        auto bit = [&](uint32_t x) {
            uint32_t v = get_bit(lb, x);
            for (uint32_t e = 0; e < h; ++e) v ^= (fl[e] == x) ? 1u : 0u;
            return v;
        };
        const uint32_t p = fl[h];
        const int sp = bit(p) ? -1 : 1;
        int d = 0;
        if (p + k < L) d += bit(p + k) ? -1 : 1;
        if (k <= p) d += bit(p - k) ? -1 : 1;
        c -= 2 * sp * d;
    }
    return c;
}

// The sum of T(|C_k|) (sum + comp) and the maximum |C_k| over a block's
// threads (lanes by a butterfly, then wavefronts in order) into pair u of the
// walk's chunk arrays.
constexpr int kPendThreads = 256;
struct PendLds {
    double s[kPendThreads / 64], c[kPendThreads / 64];
    uint32_t m[kPendThreads / 64];
};
__device__ __forceinline__ void pend_store(PendLds &sh, double ts, double tc, uint32_t tm, const BatchEntry &be, uint32_t u)
{
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    // every lane of the butterfly ends with the same sums
    for (int o = 32; o > 0; o >>= 1) {
        const double ps = __shfl_xor(ts, o), pc = __shfl_xor(tc, o);
        const uint32_t pm = (uint32_t)__shfl_xor((int)tm, o);
        nsum_add(ts, tc, ps);
        tc += pc;
        tm = max(tm, pm);
    }
    if (lane == 0) {
        sh.s[wave] = ts;
        sh.c[wave] = tc;
        sh.m[wave] = tm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double us = 0.0, uc = 0.0;
        uint32_t um = 0;
        for (int x = 0; x < kPendThreads / 64; ++x) {
            nsum_add(us, uc, sh.s[x]);
            uc += sh.c[x];
            um = max(um, sh.m[x]);
        }
        be.S0[2 * u] = us;
        be.S0[2 * u + 1] = uc;
        be.M0[u] = um;
    }
}

// Pending walks whose Rand_flip is too large for the one-flip rebuild, after
// k_corr: the sums of T(|C_k|) of their new pivot, in work units of kPendUnit
// shifts dealt round-robin over the grid, walk after walk.
__global__ __launch_bounds__(kPendThreads) void k_pending(WalkDev *walks, const BatchEntry *batch, Tables tabs,
                                                          const uint32_t *pend)
{
    __shared__ PendLds sh;
    const uint32_t np = pend[0];
    const uint32_t G = gridDim.x;
    uint32_t base = 0;                  // units of the earlier pending walks
    for (uint32_t q = 0; q < np; ++q) {
        const BatchEntry be = batch[pend[1 + q]];
        WalkDev &w = walks[be.slot];
        if (w.n_flips <= kFlipIncremental) continue;
        const uint32_t L = w.L;
        const uint32_t nu = (L - 1 + kPendUnit - 1) / kPendUnit;
        const double *T = tabs.T[w.alpha];
        for (uint32_t u = (blockIdx.x + G - base % G) % G; u < nu; u += G) {
            const uint32_t k_lo = 1 + u * kPendUnit, k_hi = min(L, k_lo + kPendUnit);
            double ts = 0.0, tc = 0.0;
            uint32_t tm = 0;
            for (uint32_t k = k_lo + threadIdx.x; k < k_hi; k += kPendThreads) {
                const int32_t c = w.C[k];
                const uint32_t a = (uint32_t)(c < 0 ? -c : c);
                nsum_add(ts, tc, T[a]);
                tm = max(tm, a);
            }
            __syncthreads();            // the previous unit is done with the LDS
            pend_store(sh, ts, tc, tm, be, u);
        }
        base += nu;
    }
}

// The sums of a walk's n segments or units (pend_store) in order, by one
// wavefront: lane l adds l, l + 64, ..., then the lanes in a fixed butterfly.
// Every lane ends with the walk's F and PSL.
__device__ __forceinline__ void pend_sum(const BatchEntry &be, uint32_t n, int lane, double &F, uint32_t &m)
{
    double s = 0.0, c = 0.0;
    m = 0;
#pragma unroll 4
    for (uint32_t x = (uint32_t)lane; x < n; x += 64) {
        nsum_add(s, c, be.S0[2 * x]);
        c += be.S0[2 * x + 1];
        m = max(m, be.M0[x]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double ps = __shfl_xor(s, o), pc = __shfl_xor(c, o);
        const uint32_t pm = (uint32_t)__shfl_xor((int)m, o);
        nsum_add(s, c, ps);
        c += pc;
        m = max(m, pm);
    }
    F = s + c;
}

// A walk that switched phase starts over from its new pivot's F and PSL.
__device__ __forceinline__ void pend_done(WalkDev &w, double F, uint32_t m)
{
    w.F_pivot = F;
    w.psl_pivot = (int32_t)m;
    w.value_local = F;
    w.unimproved = 0;
    w.pending = 0;
}

// One wavefront per pending walk that k_pending took (k_apply finishes the others).
__global__ __launch_bounds__(64) void k_pending_fin(WalkDev *walks, const BatchEntry *batch, const uint32_t *pend)
{
    const uint32_t np = pend[0];
    for (uint32_t q = blockIdx.x; q < np; q += gridDim.x) {
        const BatchEntry be = batch[pend[1 + q]];
        WalkDev &w = walks[be.slot];
        if (w.n_flips <= kFlipIncremental) continue;
        double F;
        uint32_t m;
        pend_sum(be, (w.L - 1 + kPendUnit - 1) / kPendUnit, (int)threadIdx.x, F, m);
        if (threadIdx.x == 0) pend_done(w, F, m);
    }
}

// F of the pivot (Eq. (5)) and its PSL (Eq. (3)) from C in two launches: the
// sums of the walk's segments, then (k_fit_fin) the segments' in order. The same
// C always gives the same F bits. One block per walk took 55 us of a forced flip
// at L = 40009.
constexpr int kFitBatch = 4;
__global__ __launch_bounds__(kPendThreads) void k_fit(const WalkDev *walks, const BatchEntry *batch, Tables tabs, SegMap map)
{
    __shared__ PendLds sh;
    uint32_t bi, seg;
    seg_of(map, blockIdx.x, bi, seg);
    const BatchEntry be = batch[bi];
    const WalkDev &w = walks[be.slot];
    const double *T = tabs.T[w.alpha];
    const uint32_t k0 = 1u + (seg << map.shift), k1 = min(w.L, k0 + (1u << map.shift));
    double ts = 0.0, tc = 0.0;
    uint32_t tm = 0;
    for (uint32_t k = k0 + threadIdx.x; k < k1; k += kFitBatch * kPendThreads) {
        uint32_t a[kFitBatch];
#pragma unroll
        for (int u = 0; u < kFitBatch; ++u) {
            const uint32_t kk = k + (uint32_t)u * kPendThreads;
            const int32_t c = kk < k1 ? w.C[kk] : 0;       // T[0] = 0
            a[u] = (uint32_t)(c < 0 ? -c : c);
        }
#pragma unroll
        for (int u = 0; u < kFitBatch; ++u) {
            nsum_add(ts, tc, T[a[u]]);
            tm = max(tm, a[u]);
        }
    }
    pend_store(sh, ts, tc, tm, be, seg);
}

// mode kFitInit: value_local, F_pivot, psl_pivot and psl_best; kFitPivot (a
// restore): F_pivot and psl_pivot.
__global__ __launch_bounds__(64) void k_fit_fin(WalkDev *walks, const BatchEntry *batch, uint32_t seg_shift, int mode)
{
    const BatchEntry be = batch[blockIdx.x];
    WalkDev &w = walks[be.slot];
    double F;
    uint32_t m;
    pend_sum(be, seg_count(w.L, seg_shift), (int)threadIdx.x, F, m);
    if (threadIdx.x == 0) {
        w.F_pivot = F;
        w.psl_pivot = (int32_t)m;
        if (mode == kFitInit) {
            w.value_local = F;
            w.psl_best = (int32_t)m;
        }
    }
}

// --------------------------------------------- neighbourhood evaluation

constexpr uint32_t kMaxGridY = 65535;      // walks per launch of the 2-D grids

// The chunk sums and near list of a step: one block per segment of the map.
__global__ __launch_bounds__(kChunkThreads) void k_chunks(const WalkDev *walks, BatchEntry *batch,
                                                          Tables tabs, SegMap map, uint32_t *pend, EvalCall call)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) eval_call(batch, call);
    // the previous step's pending list has been consumed; this step's
    // bookkeeping (in the selection) refills it
    if (pend && blockIdx.x == 0 && threadIdx.x == 0) pend[0] = 0;
    __shared__ ChunkLds sh;
    uint32_t b, seg;
    seg_of(map, blockIdx.x, b, seg);
    const BatchEntry be = batch[b];
    const WalkDev &w = walks[be.slot];
    chunk_segment(sh, be, w, tabs.T[w.alpha], map, seg);
}

// Suffix values of the step's chunk arrays, one wavefront per segment of the
// map: the segment's chunks (at most 128, two per lane) are scanned from the
// right with doubling steps, and the offset is the sum of the totals of the
// walk's later segments (a fixed butterfly over lanes). Each entry is a sum
// of the same chunk values, each in a fixed order.
constexpr int kSegScanThreads = 256;
__global__ __launch_bounds__(kSegScanThreads) void k_seg_scan(const WalkDev *walks, const BatchEntry *batch,
                                                              SegMap map)
{
    const uint32_t i = blockIdx.x * (kSegScanThreads / 64) + (threadIdx.x >> 6);
    if (i >= map.total) return;              // wave-uniform
    const int lane = threadIdx.x & 63;
    uint32_t b, seg;
    seg_of(map, i, b, seg);
    const BatchEntry be = batch[b];
    if (be.lsplit) return;                   // a matrix walk has no chunk arrays
    const WalkDev &w = walks[be.slot];
    const int nchunks = ((int)w.L - 1 + 31) / 32;
    const int cps = 1 << (map.shift - 5);    // chunks per segment
    const int c0 = (int)seg * cps;
    const int c1 = min(nchunks, c0 + cps);
    // totals of the later segments of this walk
    const uint32_t last = map.off ? map.off[b + 1] : (b + 1) * map.spw;
    double os = 0.0, oc = 0.0;
    uint32_t om = 0;
    for (uint32_t x = i + 1 + lane; x < last; x += 64) {
        nsum_add(os, oc, map.tot[x]);
        om = max(om, map.tmax[x]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double ps = __shfl_xor(os, o), pc = __shfl_xor(oc, o);
        const uint32_t pm = (uint32_t)__shfl_xor((int)om, o);
        nsum_add(os, oc, ps);
        oc += pc;
        om = max(om, pm);
    }
    // lane l holds chunks c0 + 2l, c0 + 2l + 1
    const int ca = c0 + 2 * lane, cb = ca + 1;
    const double va = ca < c1 ? be.S0[ca] : 0.0, vb = cb < c1 ? be.S0[cb] : 0.0;
    const uint32_t ma = ca < c1 ? be.M0[ca] : 0u, mb = cb < c1 ? be.M0[cb] : 0u;
    double ls = 0.0, lc = 0.0;
    nsum_add(ls, lc, vb);
    nsum_add(ls, lc, va);
    uint32_t lm = max(ma, mb);
    // inclusive suffix over lanes, then exclusive by one lane
    for (int d = 1; d < 64; d <<= 1) {
        const double ps = __shfl_down(ls, d), pc = __shfl_down(lc, d);
        const uint32_t pm = (uint32_t)__shfl_down((int)lm, d);
        if (lane + d < 64) {
            nsum_add(ls, lc, ps);
            lc += pc;
            lm = max(lm, pm);
        }
    }
    double es = __shfl_down(ls, 1), ec = __shfl_down(lc, 1);
    uint32_t em = (uint32_t)__shfl_down((int)lm, 1);
    if (lane == 63) {
        es = 0.0;
        ec = 0.0;
        em = 0;
    }
    // add the later segments, then this lane's chunks from the right
    nsum_add(es, ec, os);
    ec += oc;
    em = max(em, om);
    if (cb < c1) {
        nsum_add(es, ec, vb);
        em = max(em, mb);
        be.S0[cb] = es + ec;
        be.M0[cb] = em;
    }
    if (ca < c1) {
        nsum_add(es, ec, va);
        em = max(em, ma);
        be.S0[ca] = es + ec;
        be.M0[ca] = em;
    }
    if (c1 == nchunks && lane == 0) {
        be.S0[nchunks] = 0.0;
        be.M0[nchunks] = 0;
    }
}

// ------------------------------------------------------- selection

// Block blockIdx.x of a walk's gridDim.x (blockIdx.y = batch position, b0 that of
// blockIdx.y = 0). With TAIL the walk's last block to finish then makes its
// selection (finish_walk) and sets the ambiguity flags; done holds one zeroed
// counter per batch position.
template <bool TAIL>
__global__ __launch_bounds__(kCombThreads) void k_combine(WalkDev *walks, const BatchEntry *batch, Tables tabs,
                                                          int G, int pure, ChoiceDev *out, uint32_t *pend,
                                                          uint32_t *done, double margin, uint32_t b0)
{
    __shared__ CombLds sh;
    const BatchEntry be = batch[blockIdx.y];
    WalkDev &w = walks[be.slot];
    combine_part<TAIL, Form::either>(sh, w, be, tabs, G, gridDim.x, blockIdx.x, be.ksplit);
    const uint32_t bi = b0 + blockIdx.y;
    if (!TAIL || !last_block(sh, done, bi, gridDim.x)) return;
    finish_walk<kCombThreads>(sh.fin, w, be, bi, gridDim.x, (uint32_t)G, pure, out, pend, margin);
}

// The selection of a walk, its ambiguity flags and (pure == 0) its
// bookkeeping: one block per walk, after k_combine when the combine launch
// does not make them itself.
constexpr int kSelThreads = 256;
__global__ __launch_bounds__(kSelThreads) void k_select(WalkDev *walks, const BatchEntry *batch,
                                                        uint32_t comb_blocks, uint32_t comb_group, int pure,
                                                        ChoiceDev *out, uint32_t *pend, double margin)
{
    const BatchEntry be = batch[blockIdx.x];
    WalkDev &w = walks[be.slot];
    __shared__ FinishLds fin;
    finish_walk<kSelThreads>(fin, w, be, blockIdx.x, comb_blocks, comb_group, pure, out, pend, margin);
}


// ------------------------------------------------------------ flip

// Flip(pivot, j), part 1: C_k += -2 s_j (s_{j+k} + s_{j-k}) over the terms in
// bounds, read from the pivot before its bit changes. j_fixed < 0: the walk's
// recorded move.
constexpr int kApplyThreads = 256;

// The C update of shifts k0 + tid, k0 + tid + kApplyThreads, ... < k1. C and
// C_lb are separate arrays: each thread loads four shifts' C values and bit
// words before it stores any of them. The bit words of j + k and j - k are
// read whether or not those elements exist: the pivot's zero guard words
// (nw + 2 on each side) hold every index from -(L-1) to 2L-2.
constexpr int kApplyBatch = 4;
// With SUM (a forced flip) also the sum of T(|C_k|) and the maximum |C_k|.
template <bool SUM>
__device__ __forceinline__ void apply_range(int32_t *__restrict__ C, int32_t *__restrict__ C_lb,
                                            const uint64_t *__restrict__ b, uint32_t L, uint32_t j, int sj,
                                            bool lb, uint32_t k0, uint32_t k1, const double *__restrict__ T, double &ts,
                                            double &tc, uint32_t &tm)
{
    for (uint32_t k = k0 + threadIdx.x; k < k1; k += kApplyBatch * kApplyThreads) {
        int32_t cv[kApplyBatch];
        uint64_t wr[kApplyBatch], wl[kApplyBatch];
#pragma unroll
        for (int u = 0; u < kApplyBatch; ++u) {
            uint32_t kk = k + (uint32_t)u * kApplyThreads;
            kk = kk < k1 ? kk : k;                  // past the end: a valid shift, not stored
            const int32_t pl = (int32_t)j - (int32_t)kk;
            cv[u] = C[kk];
            wr[u] = b[(j + kk) >> 6];
            wl[u] = b[pl >> 6];                     // arithmetic shift: a guard word when pl < 0
        }
#pragma unroll
        for (int u = 0; u < kApplyBatch; ++u) {
            const uint32_t kk = k + (uint32_t)u * kApplyThreads;
            if (kk < k1) {
                int d = 0;
                if (j + kk < L) d += ((wr[u] >> ((j + kk) & 63u)) & 1u) ? -1 : 1;
                if (kk <= j) d += ((wl[u] >> ((j - kk) & 63u)) & 1u) ? -1 : 1;
                const int32_t c = cv[u] - 2 * sj * d;
                C[kk] = c;
                if (lb) C_lb[kk] = c;
                if (SUM) {
                    const uint32_t a = (uint32_t)(c < 0 ? -c : c);
                    nsum_add(ts, tc, T[a]);
                    tm = max(tm, a);
                }
            }
        }
    }
}


// The shifts k0 .. k1-1 (at most 2^kSegShiftMax) of a walk that switched phase
// after this move: C of the new pivot, by the FLIP_lmt one-flip updates from C of
// local_best (which the move makes of C if it improved), the sum of T(|C_k|) in
// the new exponent and the maximum |C_k|. The shifts of D in the range are
// marked in an LDS bitmap first. In one pass with the move's update (a pass and
// a launch of its own before: 5 us of a single walk's step, switching or not).
struct SwitchLds {
    uint32_t fl[kFlipIncremental];
    int sign[kFlipIncremental];         // of local_best's elements there
    uint32_t in[(1u << kSegShiftMax) / 32];
    PendLds pend;
};
__device__ __forceinline__ void switch_range(SwitchLds &sh, WalkDev &w, const BatchEntry &be, const double *T, uint32_t j,
                                             int sj, bool improved, uint32_t k0, uint32_t k1, uint32_t seg)
{
    const uint32_t L = w.L, nf = w.n_flips;
    const uint64_t *lb = w.local_best;
    if (threadIdx.x < nf) {
        const uint32_t p = w.flips[threadIdx.x];
        sh.fl[threadIdx.x] = p;
        sh.sign[threadIdx.x] = get_bit(lb, p) ? -1 : 1;
    }
    if (threadIdx.x < (1u << kSegShiftMax) / 32) sh.in[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t pr = threadIdx.x; pr < nf * nf; pr += kApplyThreads) {
        const uint32_t f = pr / nf, g = pr - f * nf;
        if (g >= f) continue;
        const uint32_t k = sh.fl[f] > sh.fl[g] ? sh.fl[f] - sh.fl[g] : sh.fl[g] - sh.fl[f];
        if (k >= k0 && k < k1) atomicOr(&sh.in[(k - k0) >> 5], 1u << ((k - k0) & 31u));
    }
    __syncthreads();
    double ts = 0.0, tc = 0.0;
    uint32_t tm = 0;
    for (uint32_t k = k0 + threadIdx.x; k < k1; k += kApplyThreads) {
        int32_t c;
        if (improved) {
            int d = 0;
            if (j + k < L) d += get_bit(lb, j + k) ? -1 : 1;
            if (k <= j) d += get_bit(lb, j - k) ? -1 : 1;
            c = w.C[k] - 2 * sj * d;
            w.C_lb[k] = c;
        } else {
            c = w.C_lb[k];
        }
        const uint32_t o = k - k0;
        if ((sh.in[o >> 5] >> (o & 31u)) & 1u)
            c = switch_corr_seq(lb, c, L, k, sh.fl, nf);
        else
#pragma unroll 4
            for (uint32_t f = 0; f < nf; ++f) c += switch_flip_delta(lb, L, k, sh.fl[f], sh.sign[f]);
        w.C[k] = c;
        const uint32_t a = (uint32_t)(c < 0 ? -c : c);
        nsum_add(ts, tc, T[a]);
        tm = max(tm, a);
    }
    pend_store(sh.pend, ts, tc, tm, be, seg);
}

// Of a walk whose F and PSL are new with this update (a switched phase, a forced
// flip) the last block to finish, counted in done[bi] (zero between launches),
// adds up the segments' sums. (A launch of its own for that took 3.6 us of a
// single walk's step, switching or not, and 4.5 us of a forced flip.) Each count
// is a device-scope release of the stored C, which the blocks of an XCD make one
// after another (about 40 ns each): with 16 flips at most, about kSwitchBlocks blocks of a
// launch take switched walks' segments, each several in turn. Steps that switch
// with 10 flips, N_lmt = 256, us, against a block per segment: one walk at
// L = 1048575 (2048 segments) 181 -> 141, four 290 -> 261, one at L = 524287
// 113 -> 100; with 64 flips, whose shifts in D cost most, 512 blocks took 1700 for 527.
constexpr uint32_t kSwitchBlocks = 1024, kSwitchFew = 16;
__global__ __launch_bounds__(kApplyThreads) void k_apply(WalkDev *walks, const BatchEntry *batch, Tables tabs,
                                                         int64_t j_fixed, SegMap map, uint32_t *done)
{
    __shared__ SwitchLds sh;
    __shared__ uint32_t s_last;
    uint32_t bi, seg;
    seg_of(map, blockIdx.x, bi, seg);
    const BatchEntry be = batch[bi];
    WalkDev &w = walks[be.slot];
    const uint32_t L = w.L;
    const uint32_t j = j_fixed >= 0 ? (uint32_t)j_fixed : w.k;
    // a forced flip reads the pivot before its bit changes; the step's move
    // comes after the bookkeeping, which flipped bit j, and on a phase switch
    // replaced the pivot: then the local best holds the pre-move bits at
    // every position but j (an improving move), or C is rebuilt from C of the
    // local best
    const bool moved = j_fixed < 0;
    const bool switched = moved && (w.flags & STEP_SWITCHED);
    const uint64_t *b = switched ? w.local_best : w.pivot;
    const int sj = (get_bit(b, j) != 0) != moved ? -1 : 1;      // s_j before the flip
    // the move improves on v_local: the new pivot becomes local_best
    const bool lb = moved && (w.flags & STEP_IMPROVED);
    const uint32_t k0 = 1u + (seg << map.shift);
    const uint32_t k1 = min(L, k0 + (1u << map.shift));
    const uint32_t n = seg_count(L, map.shift);
    uint32_t blocks = n;                // that count themselves
    double ts = 0.0, tc = 0.0;
    uint32_t tm = 0;
    if (!moved) {
        apply_range<true>(w.C, w.C_lb, b, L, j, sj, lb, k0, k1, tabs.T[w.alpha], ts, tc, tm);
        pend_store(sh.pend, ts, tc, tm, be, seg);
    } else if (switched && w.n_flips <= kFlipIncremental) {
        if (w.n_flips <= kSwitchFew) blocks = min(n, max(kSwitchBlocks / map.nb, 128u));
        if (seg >= blocks) return;
        for (uint32_t x = seg; x < n; x += blocks) {
            const uint32_t x0 = 1u + (x << map.shift);
            switch_range(sh, w, be, tabs.T[w.alpha], j, sj, lb, x0, min(L, x0 + (1u << map.shift)), x);
        }
    } else {
        apply_range<false>(w.C, w.C_lb, b, L, j, sj, lb, k0, k1, nullptr, ts, tc, tm);
        return;
    }
    if (threadIdx.x == 0) {             // it stored the segment's sums
        s_last = 1;
        if (blocks > 1) {
            s_last = __hip_atomic_fetch_add(&done[bi], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) == blocks - 1;
            if (s_last) done[bi] = 0;
        }
    }
    __syncthreads();
    if (!s_last || threadIdx.x >= 64) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    double F;
    uint32_t m;
    pend_sum(be, n, (int)threadIdx.x, F, m);
    if (threadIdx.x) return;
    if (moved) {
        pend_done(w, F, m);
    } else {
        w.F_pivot = F;
        w.psl_pivot = (int32_t)m;
        w.pivot[j >> 6] ^= 1ull << (j & 63u);
    }
}

// ------------------------------------------------------------ launches

hipError_t launch_power_table(double *T, uint32_t n, uint32_t alpha, hipStream_t s)
{
    k_power_table<<<(n + 255) / 256, 256, 0, s>>>(T, n, alpha);
    return hipGetLastError();
}

hipError_t launch_init(WalkDev *walks, const InitRec *recs, const uint64_t *bits, uint32_t nb, uint64_t max_bytes,
                       uint32_t max_nw, hipStream_t s)
{
    for (uint32_t b0 = 0; b0 < nb; b0 += kMaxGridY) {
        const uint32_t ny = std::min(kMaxGridY, nb - b0);
        k_init_slabs<<<dim3((uint32_t)((max_bytes + kInitSpan - 1) / kInitSpan), ny), 256, 0, s>>>(walks, recs + b0);
        k_init_bits<<<dim3((max_nw + 255) / 256, ny), 256, 0, s>>>(walks, recs + b0, bits);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_pending(WalkDev *walks, const BatchEntry *batch, uint32_t nb, uint64_t units,
                          const Tables &tabs, const uint32_t *pend, hipStream_t s)
{
    if (!pend) return hipErrorInvalidValue;
    // every unit of the batch's walks gets a block when all of them switch
    const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(4096, units));
    k_pending<<<grid, kPendThreads, 0, s>>>(walks, batch, tabs, pend);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_pending_fin<<<std::max<uint32_t>(1, std::min<uint32_t>(nb, 1024)), 64, 0, s>>>(walks, batch, pend);
    return hipGetLastError();
}

hipError_t launch_fit(WalkDev *walks, const BatchEntry *batch, uint32_t nb, const Tables &tabs, const SegMap &map,
                      int mode, hipStream_t s)
{
    if (map.total == 0 || map.nb != nb || map.shift < kSegShiftMin || map.shift > kSegShiftMax)
        return hipErrorInvalidValue;
    k_fit<<<map.total, kPendThreads, 0, s>>>(walks, batch, tabs, map);
    k_fit_fin<<<nb, 64, 0, s>>>(walks, batch, map.shift, mode);
    return hipGetLastError();
}

hipError_t launch_seg_scan(const WalkDev *walks, const BatchEntry *batch, const SegMap &map, hipStream_t s)
{
    constexpr uint32_t per = kSegScanThreads / 64;
    k_seg_scan<<<(map.total + per - 1) / per, kSegScanThreads, 0, s>>>(walks, batch, map);
    return hipGetLastError();
}

hipError_t launch_suffix(const WalkDev *walks, BatchEntry *batch, uint32_t nb, const Tables &tabs, const SegMap *map,
                         uint32_t *pend, int scan, const EvalCall &call, hipStream_t s)
{
    if (!map || map->total == 0 || map->nb != nb || map->shift < kSegShiftMin || map->shift > kSegShiftMax)
        return hipErrorInvalidValue;
    if (scan && (!map->tot || !map->tmax)) return hipErrorInvalidValue;
    SegMap m = *map;
    if (!scan) m.tot = nullptr, m.tmax = nullptr;
    k_chunks<<<m.total, kChunkThreads, 0, s>>>(walks, batch, tabs, m, pend, call);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !scan) return e;
    // suffix values segment by segment (evaluations in 16-wavefront blocks)
    return launch_seg_scan(walks, batch, m, s);
}

// A batch's counters and, of its matrix walks, the records after each
// coefficient's last: zeros. One block per walk.
__global__ __launch_bounds__(64) void k_batch_reset(const WalkDev *walks, const BatchEntry *batch, uint32_t *pend, uint32_t *done,
                                                    bool left)
{
    const BatchEntry be = batch[blockIdx.x];
    if (threadIdx.x == 0) {
        be.near[0] = 0;
        done[blockIdx.x] = 0;
        if (blockIdx.x == 0) pend[0] = 0;
    }
    if (left)
        for (uint32_t i = threadIdx.x; i < kCombMaxBlocks; i += 64) done[gridDim.x + kCombMaxBlocks * blockIdx.x + i] = 0;
    if (!be.lsplit) return;
    const uint32_t L = walks[be.slot].L;
    uint32_t *one = reinterpret_cast<uint32_t *>(be.dig_one + (size_t)split_chunks(L) * kRecBytes);
    uint32_t *both = reinterpret_cast<uint32_t *>(be.dig_both + (size_t)split_both_chunks(L) * 2 * kRecBytes);
    for (uint32_t i = threadIdx.x; i < kRecPad * kRecBytes / 4; i += 64) one[i] = 0;
    for (uint32_t i = threadIdx.x; i < kRecPad * 2 * kRecBytes / 4; i += 64) both[i] = 0;
}

hipError_t launch_batch_reset(const WalkDev *walks, const BatchEntry *batch, uint32_t nb, uint32_t *pend, uint32_t *done,
                              bool left, hipStream_t s)
{
    if (nb == 0) return hipSuccess;
    if (!pend || !done) return hipErrorInvalidValue;
    k_batch_reset<<<nb, 64, 0, s>>>(walks, batch, pend, done, left);
    return hipGetLastError();
}

hipError_t launch_select(WalkDev *walks, const BatchEntry *batch, uint32_t nb, uint32_t comb_blocks,
                         uint32_t comb_group, const Tables &tabs, int pure, void *out, uint32_t *pend,
                         uint32_t *done, double margin, hipStream_t s)
{
    if (comb_blocks < 1 || comb_blocks > kCombMaxBlocks) return hipErrorInvalidValue;
    if (comb_group < 1 || comb_group > 64 || (comb_group & (comb_group - 1))) return hipErrorInvalidValue;
    if (pure && (!out || nb != 1)) return hipErrorInvalidValue;
    if (nb == 0) return hipSuccess;
    // small launches make the selection in the combine launch (one launch
    // fewer); large ones in launches of their own, where the per-block
    // device-scope release of the fused form costs more than the launches
    const int tail = comb_blocks == 1 || (comb_small(nb, comb_blocks) && done) ? 1 : 0;
    for (uint32_t b0 = 0; b0 < nb; b0 += kMaxGridY) {
        (tail ? k_combine<true> : k_combine<false>)<<<dim3(comb_blocks, std::min(kMaxGridY, nb - b0)), kCombThreads, 0, s>>>(
            walks, batch + b0, tabs, (int)comb_group, pure, (ChoiceDev *)out, pend, done, margin, b0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (tail) return hipSuccess;
    k_select<<<nb, kSelThreads, 0, s>>>(walks, batch, comb_blocks, comb_group, pure, (ChoiceDev *)out, pend,
                                        margin);
    return hipGetLastError();
}

size_t choice_dev_size() { return sizeof(ChoiceDev); }

bool choice_dev_table(const void *p) { return ((const ChoiceDev *)p)->table != 0; }

void choice_dev_unpack(const void *p, uint32_t *i_best, uint32_t *j_best, double *F_best,
                       double *F_min, uint32_t *j_psl, int32_t *psl_min, int32_t *psl_k, uint32_t *flags)
{
    const ChoiceDev *c = (const ChoiceDev *)p;
    *i_best = c->i_best; *j_best = c->j_best; *F_best = c->F_best; *F_min = c->F_min;
    *j_psl = c->j_psl; *psl_min = c->psl_min; *psl_k = c->psl_k; *flags = c->flags;
}

hipError_t launch_apply(WalkDev *walks, const BatchEntry *batch, const SegMap &map, const Tables &tabs,
                        int64_t j_fixed, uint32_t *done, hipStream_t s)
{
    if (!done) return hipErrorInvalidValue;
    if (map.shift < kSegShiftMin || map.shift > kSegShiftMax) return hipErrorInvalidValue;
    if (map.total == 0) return hipSuccess;       // L = 1 has no shift to update
    k_apply<<<map.total, kApplyThreads, 0, s>>>(walks, batch, tabs, j_fixed, map, done);
    return hipGetLastError();
}

}  // namespace psl
