// psl_kernels.hip -- gfx950 kernels of libpsl around the neighbourhood
// evaluation (which lives in psl_eval.hip): power tables, init (the
// correlations of Eq. (2) are psl_corr.hip's), the phase-switch rebuild, the per-step chunk sums
// and near-peak list the evaluation reads, the selection of Algorithm 1's
// scan, the O(L) flip of Section 3 and the step's bookkeeping.
#include "psl_chunks.h"
#include "psl_dev_util.h"
#include "psl_device.h"
#include "psl_launch.h"

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
__device__ __forceinline__ int32_t switch_flip_delta(const uint64_t *lb, uint32_t L, uint32_t k, uint32_t p)
{
    const int sp = get_bit(lb, p) ? -1 : 1;
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
// whose C, F and PSL k_pending then rebuilds). The C update runs after it
// (k_apply), from bits that equal the pre-move pivot's at every position but j:
// the pivot's, or on a switch the local best's (which are then the move's
// pivot, if the move improved; if it did not, C is rebuilt from C of the local
// best anyway).
// pure != 0: the choice record goes to out[bi] and the walk stays unchanged.
//
// Everything is latency here: the walk's fields are read at the start, and what
// the parts hand on stays in LDS (through global memory, one after the other,
// the same work took 5 us more of a single walk's step).
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
    const double my_f = fmin;           // this thread's combine block minimum
    // block minima: within each wavefront, then across the wavefronts (the
    // minimum F and the first minimum (PSL, index) do not depend on the order)
    for (int o = 32; o > 0; o >>= 1) {
        const double of = __shfl_xor(fmin, o);
        const int32_t op = __shfl_xor(pmin, o);
        const uint32_t oi = (uint32_t)__shfl_xor((int)ipmin, o);
        sel_merge(fmin, pmin, ipmin, of, op, oi);
    }
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
    for (int o = 32; o > 0; o >>= 1) ib = min(ib, (uint32_t)__shfl_xor((int)ib, o));
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
            uint32_t unimproved = w.unimproved;
            int sw = 0;
            if (fl & STEP_IMPROVED) {
                sh.improved = 1;
                unimproved = 0;
                w.value_local = Fb;
            } else if (fl & STEP_WORSE) {
                unimproved += 1;
                if (w.switch_period == 0 && unimproved > w.ls_lmt) sw = 1;
            }
            if (w.switch_period > 0 && ((w.t + 1u) % w.switch_period) == 0) sw = 1;
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
            if (w.trace_cap) {
                TraceEntry e;
                e.t = w.t;
                e.start = start;
                e.k = kb;
                e.value_step = Fb;
                e.psl_k = Pb;
                e.psl_best = best;
                e.alpha = sw ? (w.alpha == w.alpha1 ? w.alpha2 : w.alpha1) : w.alpha;
                e.flags = fl;
                w.trace[w.t % w.trace_cap] = e;
            }
            w.t += 1;
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

// F and PSL per candidate from the k-split partials, spread over gridDim.x
// blocks per walk (blockIdx.y = batch position); each block leaves its
// smallest F and its first smallest PSL in be.red. A group of G lanes
// (a power of two, at most 64) shares a candidate: lane g adds splits g,
// g+G, ... in order, then the group adds its lanes' sums in a fixed order for
// a given split count and G (G = 1 adds the splits in order). For G <= 4 a
// group is G adjacent lanes (a butterfly); for G >= 8 a block pass takes
// cpb = 256 / G <= 32 candidates, lane t of the block has candidate t mod cpb
// and split lane t / cpb, so that one load of a wavefront reads cpb
// consecutive partials of each of 64 / cpb splits; the sums go through a
// butterfly over the wavefront's split lanes, then the four wavefronts' sums
// are added in wavefront order.
// With tail != 0 the walk's last block to finish then makes its selection
// (finish_walk); b0 = the batch position of
// blockIdx.y = 0; done holds one zeroed counter per batch position.
__global__ __launch_bounds__(kCombThreads) void k_combine(WalkDev *walks, const BatchEntry *batch, Tables tabs,
                                                          int G, int tail, int pure, ChoiceDev *out, uint32_t *pend,
                                                          uint32_t *done, double margin, uint32_t b0)
{
    const BatchEntry be = batch[blockIdx.y];
    WalkDev &w = walks[be.slot];
    const uint32_t n = be.fixed ? be.n_lmt : w.n_lmt;
    const uint32_t ks = be.ksplit;
    const double *T = tabs.T[w.alpha];
    const uint32_t cpb = kCombThreads / (uint32_t)G;      // candidates per block pass
    const bool wide = G >= 8;
    const uint32_t g = wide ? threadIdx.x / cpb : threadIdx.x & (uint32_t)(G - 1);
    const uint32_t ci = wide ? threadIdx.x % cpb : threadIdx.x / (uint32_t)G;   // candidate in the pass
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert(kCombThreads == 256, "four wavefronts per combine block");
    __shared__ double s_wf[4][32];
    __shared__ uint32_t s_wm[4][32];
    // matrix path: F_j from the prefix sums and the matrix sums (psl_split.hip),
    // PSL_j from the near-peak shifts here
    const bool split = be.lsplit != 0 && be.ss->use != 0;
    const double U = split ? be.ss->U : 0.0;
    const uint32_t start = be.fixed ? be.start : step_start(w);
    const uint32_t L = w.L;
    const uint32_t n_near = split ? be.near[0] : 0;

    double fmin = INFINITY;
    int32_t pmin = INT_MAX;
    uint32_t ipmin = UINT_MAX;
    uint32_t lo, hi;
    comb_range(n, gridDim.x, (uint32_t)G, blockIdx.x, lo, hi);
    for (uint32_t i0 = lo; i0 < hi; i0 += cpb) {
        const uint32_t i = i0 + ci;
        double f = 0.0;
        uint32_t m = 0;
        if (split) {
            if (i < hi) {
                const uint32_t j = (uint32_t)(((uint64_t)start + 1u + i) % L);
                for (uint32_t x = g; x <= be.lsplit; x += (uint32_t)G) f += be.lpart[(size_t)x * L + j];
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
                s_wf[wave][lane] = f;
                s_wm[wave][lane] = m;
            }
            __syncthreads();
            if (g == 0) {           // wavefront 0, lanes below cpb
                f = s_wf[0][lane];
                m = s_wm[0][lane];
                for (int x = 1; x < 4; ++x) {
                    f += s_wf[x][lane];
                    m = max(m, s_wm[x][lane]);
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
                // F_j = sum_{k<=m} T(|C_k|) + sum_{m<k<=M} T(|C_k-+2|) + sum_{k>M} T(|C_k|)
                //       + U (matrix sums), m = min(j, L-1-j), M = max(j, L-1-j), -2 for s_j = +1
                const uint32_t j = (uint32_t)(((uint64_t)start + 1u + i) % L);
                const uint32_t mj = min(j, L - 1 - j), Mj = max(j, L - 1 - j);
                const int p1 = get_bit(w.pivot, j) ? 1 : 0;
                f = split_prefix(be, L, 2, mj) + (split_prefix(be, L, p1, Mj) - split_prefix(be, L, p1, mj)) +
                    (split_prefix(be, L, 2, L - 1) - split_prefix(be, L, 2, Mj)) + U * f;
            }
            be.F[i] = f;
            be.P[i] = p;
            fmin = f < fmin ? f : fmin;
            if (p < pmin) { pmin = p; ipmin = i; }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double of = __shfl_xor(fmin, o);
        const int32_t op = __shfl_xor(pmin, o);
        const uint32_t oi = (uint32_t)__shfl_xor((int)ipmin, o);
        sel_merge(fmin, pmin, ipmin, of, op, oi);
    }
    __shared__ SelPart s_r[kCombThreads / 64];
    if (lane == 0) s_r[wave] = SelPart{fmin, pmin, ipmin};
    __syncthreads();
    if (threadIdx.x == 0) {
        SelPart r = s_r[0];
        for (int x = 1; x < kCombThreads / 64; ++x) sel_merge(r.f, r.p, r.i, s_r[x].f, s_r[x].p, s_r[x].i);
        be.red[blockIdx.x] = r;
    }
    if (!tail) return;
    // tail != 0: the walk's last block to finish (counted in done[bi], which
    // it returns to 0 for the next launch) makes the selection and sets the
    // ambiguity flags. Each block's count is a device-scope release of its F,
    // P and minimum, and the last block acquires them all.
    const uint32_t bi = b0 + blockIdx.y;
    __shared__ uint32_t s_last;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t last = 1;
        if (gridDim.x > 1) {
            const uint32_t before =
                __hip_atomic_fetch_add(&done[bi], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            last = before == gridDim.x - 1 ? 1u : 0u;
            if (last) done[bi] = 0;
        }
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    if (gridDim.x > 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __shared__ FinishLds fin;
    finish_walk<kCombThreads>(fin, w, be, bi, gridDim.x, (uint32_t)G, pure, out, pend, margin);
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
    uint32_t in[(1u << kSegShiftMax) / 32];
    PendLds pend;
};
__device__ __forceinline__ void switch_range(SwitchLds &sh, WalkDev &w, const BatchEntry &be, const double *T, uint32_t j,
                                             int sj, bool improved, uint32_t k0, uint32_t k1, uint32_t seg)
{
    const uint32_t L = w.L, nf = w.n_flips;
    const uint64_t *lb = w.local_best;
    if (threadIdx.x < nf) sh.fl[threadIdx.x] = w.flips[threadIdx.x];
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
            for (uint32_t f = 0; f < nf; ++f) c += switch_flip_delta(lb, L, k, sh.fl[f]);
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
// single walk's step, switching or not, and 4.5 us of a forced flip.)
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
    double ts = 0.0, tc = 0.0;
    uint32_t tm = 0;
    if (!moved) {
        apply_range<true>(w.C, w.C_lb, b, L, j, sj, lb, k0, k1, tabs.T[w.alpha], ts, tc, tm);
        pend_store(sh.pend, ts, tc, tm, be, seg);
    } else if (switched && w.n_flips <= kFlipIncremental) {
        switch_range(sh, w, be, tabs.T[w.alpha], j, sj, lb, k0, k1, seg);
    } else {
        apply_range<false>(w.C, w.C_lb, b, L, j, sj, lb, k0, k1, nullptr, ts, tc, tm);
        return;
    }
    const uint32_t n = seg_count(L, map.shift);
    if (threadIdx.x == 0) {             // it stored the segment's sums
        s_last = 1;
        if (n > 1) {
            s_last = __hip_atomic_fetch_add(&done[bi], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
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

__global__ void k_near_reset(const BatchEntry *batch, uint32_t nb, uint32_t *pend, uint32_t *done)
{
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < nb) batch[b].near[0] = 0;
    if (b < nb && done) done[b] = 0;
    if (b == 0 && pend) pend[0] = 0;
}

hipError_t launch_near_reset(const BatchEntry *batch, uint32_t nb, uint32_t *pend, uint32_t *done, hipStream_t s)
{
    k_near_reset<<<(nb + 255) / 256, 256, 0, s>>>(batch, nb, pend, done);
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
    const int tail = comb_blocks == 1 || ((uint64_t)nb * comb_blocks <= kCombFuseBlocks && done) ? 1 : 0;
    for (uint32_t b0 = 0; b0 < nb; b0 += kMaxGridY) {
        k_combine<<<dim3(comb_blocks, std::min(kMaxGridY, nb - b0)), kCombThreads, 0, s>>>(
            walks, batch + b0, tabs, (int)comb_group, tail, pure, (ChoiceDev *)out, pend, done, margin, b0);
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
