// psl_chunks.h -- chunk sums and near-peak list of one segment of a walk
// (device code shared by the step's and the matrix path's first kernels).
#pragma once

#include "psl_dev_util.h"
#include "psl_device.h"

namespace psl {

// Per walk and step, from the pivot's C:
//  * chunk suffix sums S0[x] = sum_{1+32x <= k' < L} T(|C_k'|) and
//    M0[x] = max |C_k'| over the same range, x = 0..nchunks (the last entry
//    0). A candidate j leaves every C_k with k > max(j, L-1-j) unchanged
//    (both neighbours of the flipped element are out of bounds), so that
//    part of its F (and PSL) is read from them; the evaluation only needs
//    them at 32-shift chunk starts;
//  * the near-peak shift list: with P the pivot's PSL, every neighbour has
//    PSL >= P - 4 (one flip moves each C_k by at most 4), and a shift with
//    |C_k| <= P - 9 reaches at most P - 5, so a neighbour's PSL is the maximum
//    of |C'_k| over the shifts with |C_k| >= P - 8 alone. near[0] = count,
//    near[1..] = those shifts (any order), while the count fits kNearCap.
// Two kernels: k_chunks (several blocks per walk) writes per-chunk sums and
// maxima and appends to the near list; k_seg_scan turns the chunk values into
// suffix values in a fixed order, for the evaluation shapes that read those.
constexpr int kChunkThreads = 256;
// Octets o0, o0 + step, ... below o1 of one walk (an octet is 256 consecutive
// shifts, eight chunks), for the calling wavefront: four coalesced passes of
// 64 shifts put T(|C_k|) and |C_k| in the wavefront's LDS rows (sv, sa); then
// lane l adds the four consecutive values 4(l mod 8) .. +3 of chunk l / 8
// (left to right) and a three-level butterfly over the chunk's eight lanes
// finishes its sum and maximum, the same in all eight. The octet's total (a
// fixed tree over its chunks) goes into the wavefront's running total.
__device__ __forceinline__ void chunk_octs(const BatchEntry &be, const WalkDev &w, const double *T, int cut,
                                           int o0, int o1, int step, double *sv, int *sa,
                                           double &ws, double &wc, uint32_t &wm)
{
    const int L = (int)w.L;
    const int nchunks = (L - 1 + 31) / 32;
    const int lane = threadIdx.x & 63;
    for (int o = o0; o < o1; o += step) {
        // the four passes' C values, then their T values, are all loaded
        // before any is used (two waits per octet, not eight)
        int av[4];
        double tv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 1 + 256 * o + 64 * i + lane;
            const int32_t x = k < L ? w.C[k] : 0;
            av[i] = x < 0 ? -x : x;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 1 + 256 * o + 64 * i + lane;
            tv[i] = k < L ? T[av[i]] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 64 * i + lane;
            const int k = 1 + 256 * o + e;
            const int a = av[i];
            sv[e] = tv[i];
            sa[e] = a;
            const bool take = k < L && a >= cut;
            const uint64_t bal = __ballot(take);
            if (bal) {
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&be.near[0], (uint32_t)__popcll(bal));
                base = (uint32_t)__shfl((int)base, 0);
                const uint32_t q = base + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
                if (take && q < (uint32_t)kNearCap) be.near[1 + q] = (uint32_t)k;
            }
        }
        // the wavefront's rows are written before any lane reads them
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int r = 32 * (lane >> 3) + 4 * (lane & 7);
        double v = sv[r];
        v += sv[r + 1];
        v += sv[r + 2];
        v += sv[r + 3];
        int m = max(max(sa[r], sa[r + 1]), max(sa[r + 2], sa[r + 3]));
        for (int d = 1; d < 8; d <<= 1) {
            v += __shfl_xor(v, d);
            m = max(m, __shfl_xor(m, d));
        }
        const int c = 8 * o + (lane >> 3);
        if ((lane & 7) == 0 && c < nchunks) {
            be.S0[c] = v;
            be.M0[c] = (uint32_t)m;
        }
        // the octet's total over its chunk leaders (every lane ends with it)
        double ts = v, tc = 0.0;
        for (int d = 8; d < 64; d <<= 1) {
            const double ps = __shfl_xor(ts, d), pc = __shfl_xor(tc, d);
            nsum_add(ts, tc, ps);
            tc += pc;
            m = max(m, __shfl_xor(m, d));
        }
        nsum_add(ws, wc, ts);
        wc += tc;
        wm = max(wm, (uint32_t)m);
        // every lane has read the rows before the next octet overwrites them
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

struct ChunkLds {
    double v[kChunkThreads / 64][256];
    int a[kChunkThreads / 64][256];
    double s[kChunkThreads / 64], c[kChunkThreads / 64];
    uint32_t m[kChunkThreads / 64];
};

// Segment `seg` (block blockIdx.x of the map) of one walk.
__device__ __forceinline__ void chunk_segment(ChunkLds &sh, const BatchEntry &be, const WalkDev &w, const double *T,
                                              const SegMap &map, uint32_t seg)
{
    const int wave = (int)threadIdx.x >> 6;
    constexpr int kWaves = kChunkThreads / 64;
    const int nocts = ((int)w.L - 1 + 255) / 256;
    const int octs_per_seg = 1 << (map.shift - 8);
    const int o0 = (int)seg * octs_per_seg;
    const int o1 = min(nocts, o0 + octs_per_seg);
    // the near-peak cut (the pivot's PSL is kept current by every step)
    double ws = 0.0, wc = 0.0;
    uint32_t wm = 0;
    chunk_octs(be, w, T, w.psl_pivot - 8, o0 + wave, o1, kWaves, sh.v[wave], sh.a[wave], ws, wc, wm);
    if (map.tot) {
        // the segment's total (waves in order) for the segment-parallel scan
        if ((threadIdx.x & 63) == 0) {
            sh.s[wave] = ws;
            sh.c[wave] = wc;
            sh.m[wave] = wm;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double ts = 0.0, tc = 0.0;
            uint32_t tm = 0;
            for (int x = 0; x < kWaves; ++x) {
                nsum_add(ts, tc, sh.s[x]);
                tc += sh.c[x];
                tm = max(tm, sh.m[x]);
            }
            map.tot[blockIdx.x] = ts + tc;
            map.tmax[blockIdx.x] = tm;
        }
    }
}

}  // namespace psl
