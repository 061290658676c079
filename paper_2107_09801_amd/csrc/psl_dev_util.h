// psl_dev_util.h -- small device helpers shared by the libpsl kernel sources
// (internal).
#pragma once

#include "psl_device.h"

namespace psl {

// Counter-based SplitMix64 (Steele, Lea & Flood 2014): output ctr+1 of the
// stream whose state starts at seed.
__device__ __forceinline__ uint64_t draw(uint64_t seed, uint64_t ctr)
{
    uint64_t z = seed + (ctr + 1u) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint32_t step_start(const WalkDev &w)
{
    return (uint32_t)(draw(w.seed, (1ull << 60) | w.t) % (uint64_t)w.L);
}

__device__ __forceinline__ uint32_t get_bit(const uint64_t *b, uint32_t i)
{
    return (uint32_t)((b[i >> 6] >> (i & 63u)) & 1u);
}

// dst[x] = src[x] for x < n (word flip_word also XORed with flip_mask), the
// threads of a block striding by nthreads. The two arrays never overlap;
// each thread issues eight loads before their stores instead of waiting on
// one load per word.
__device__ __forceinline__ void copy_words(uint64_t *__restrict__ dst, const uint64_t *__restrict__ src,
                                           uint32_t n, uint32_t tid, uint32_t nthreads, uint32_t flip_word,
                                           uint64_t flip_mask)
{
    uint32_t x = tid;
    for (; x + 7u * nthreads < n; x += 8u * nthreads) {
        uint64_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[x + (uint32_t)u * nthreads];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t y = x + (uint32_t)u * nthreads;
            dst[y] = y == flip_word ? v[u] ^ flip_mask : v[u];
        }
    }
    for (; x < n; x += nthreads) dst[x] = x == flip_word ? src[x] ^ flip_mask : src[x];
}

// High 32 bits of a non-negative double. Over the power table they are
// strictly increasing in |c| (consecutive entries differ by a factor of at
// least 1 + 2^-19 for alpha >= 2 and |c| <= 2^20 + 8; for alpha = 1 the
// entries are integers below 2^21, exact in 20 fraction bits), so the
// running maximum of T(|C'|) can be kept as a 32-bit unsigned maximum.
__device__ __forceinline__ uint32_t hi32(double v)
{
    return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32);
}

// Neumaier's compensated addition.
__device__ __forceinline__ void nsum_add(double &sum, double &comp, double x)
{
    double t = sum + x;
    if (fabs(sum) >= fabs(x)) comp += (sum - t) + x;
    else                      comp += (x - t) + sum;
    sum = t;
}

// Smallest c with hi32(T[c]) >= h: |c| from the high word of T(|c|).
__device__ __forceinline__ int32_t table_inverse(const double *T, uint32_t n, uint32_t h)
{
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        uint32_t mid = (lo + hi) >> 1;
        if (hi32(T[mid]) < h) lo = mid + 1;
        else                  hi = mid;
    }
    return (int32_t)lo;
}

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of work items so that the blocks of one walk share an L2.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nb)
{
    const uint32_t nx = 8;
    uint32_t q = nb / nx, r = nb % nx;
    uint32_t x = b % nx, local = b / nx;
    return x * q + (x < r ? x : r) + local;
}

// (walk, segment) of block i of an O(L) pass.
__device__ __forceinline__ void seg_of(const SegMap &m, uint32_t i, uint32_t &b, uint32_t &seg)
{
    if (!m.off) {
        b = i / m.spw;
        seg = i - b * m.spw;
        return;
    }
    uint32_t lo = 0, hi = m.nb - 1;      // the largest b with off[b] <= i
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (m.off[mid] <= i) lo = mid;
        else                 hi = mid - 1;
    }
    b = lo;
    seg = i - m.off[lo];
}

// The fields of an evaluation call into its plan's entry, by one thread of the
// call's first kernel.
__device__ __forceinline__ void eval_call(BatchEntry *batch, const EvalCall &call)
{
    if (!call.on) return;
    batch[0].start = call.start;
    batch[0].F = call.F;
    batch[0].P = call.P;
}

// v of the lane that lane-permuting control CTRL names (old where it names none,
// and outside the rows of ROWS): 0x110 + n the lane n before in the row of 16,
// 0x142 and 0x143 the last lane of the row, of the two rows, before.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_mov(uint64_t old, uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)old, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(old >> 32), (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t last_lane(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}
// The wavefront's smallest value, in every lane (all 64 active; no NaN): six
// register moves and comparisons, where a butterfly through LDS took 0.6 us.
__device__ __forceinline__ uint64_t wave_least(uint64_t v)
{
    auto least = [](uint64_t a, uint64_t b) { return a < b ? a : b; };
    v = least(v, dpp_mov<0x111, 0xF>(v, v));
    v = least(v, dpp_mov<0x112, 0xF>(v, v));
    v = least(v, dpp_mov<0x114, 0xF>(v, v));
    v = least(v, dpp_mov<0x118, 0xF>(v, v));
    v = least(v, dpp_mov<0x142, 0xA>(v, v));
    v = least(v, dpp_mov<0x143, 0xC>(v, v));
    return last_lane(v);
}
__device__ __forceinline__ double wave_least(double v)
{
    auto bits = [](double a) { return (uint64_t)__double_as_longlong(a); };
    auto least = [](double a, uint64_t b) { const double o = __longlong_as_double((long long)b); return o < a ? o : a; };
    v = least(v, dpp_mov<0x111, 0xF>(bits(v), bits(v)));
    v = least(v, dpp_mov<0x112, 0xF>(bits(v), bits(v)));
    v = least(v, dpp_mov<0x114, 0xF>(bits(v), bits(v)));
    v = least(v, dpp_mov<0x118, 0xF>(bits(v), bits(v)));
    v = least(v, dpp_mov<0x142, 0xA>(bits(v), bits(v)));
    v = least(v, dpp_mov<0x143, 0xC>(bits(v), bits(v)));
    return __longlong_as_double((long long)last_lane(bits(v)));
}

// Place of element j in a row of the matrix path's partial sums (BatchEntry::lpart):
// tiles count from the one of the neighbourhood's first element, j_first. (Rows
// of all L elements took 2.5 GB for one walk at L = 1048575 with N_lmt = 512,
// whose few tiles split 313 ways; these 2.6 MB.)
__device__ __forceinline__ uint32_t mx_place(uint32_t L, uint32_t j_first, uint32_t j)
{
    const uint32_t ntile = (L + kMxTile - 1) / kMxTile, t0 = j_first / kMxTile, t = j / kMxTile;
    return kMxTile * (t < t0 ? t + ntile - t0 : t - t0) + j % kMxTile;
}

// Prefix sum x (0 or 1, BatchEntry::pre) of a matrix walk over the shifts
// 1 .. k, in two parts to add: the one within the segment, and the segment's offset.
__device__ __forceinline__ void split_prefix(const BatchEntry &be, uint32_t L, int x, uint32_t k, double &in, double &off)
{
    const uint32_t seg = min(k >> be.seg_shift, seg_count(L, be.seg_shift) - 1u);
    in = be.pre[(size_t)x * L + k];
    off = be.segoff[3 * (size_t)seg + x];
}

}  // namespace psl
