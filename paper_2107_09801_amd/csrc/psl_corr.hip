// psl_corr.hip -- Eq. (2) from the packed pivot (gfx950): C_k = sum_i s_i s_{i+k}
// for every shift, O(L^2), at init, at a restore and after a Rand_flip too
// large for the one-flip rebuild.
//
// Long sequences, and many: on the matrix cores, as products of two +-1 matrices made
// from the sequence's bits in FP4. One block takes kCorrTile = 4096
// consecutive shifts and a range of the positions i, in 32-position chunks.
// The 16 rows of v_mfma_f32_16x16x128_f8f6f4 hold s at i + K0 + 32 n + 16 p + r
// (r the row; n = 0..7 and p = 0..1 one product each), the 16 columns s at
// i - 256 q (q the column), so that a product's entries are the shifts
// K0 + 256 q + 32 n + 16 p + r, all of them used. Lane group g of the operands
// has the chunk c0 + g N + s at step s: the row matrix of (n, p) depends on
// chunk + n only, so a step makes two new ones (a ring of eight) and one column
// matrix for its 16 products. A position outside the sequence is 0 in the
// matrices. Sums stay integers below 2^24, exact in FP32.
//
// What bounds it: a step is 16 products of 16 x 16 x 128 (16 cycles each) and
// about 40 vector instructions (4 cycles each): away from the sequence's ends the
// matrices need no masks, which took 30 more. 1024 walks at L = 131071 take 3.7
// ms, 14 ns per product and SIMD; alone, a product takes 7 to 10. One XOR
// and popcount per 32 products, the form of short sequences and small launches, is
// bound by vector issue, in small launches by the length of a block's sweep.
#include "psl_dev_util.h"
#include "psl_device.h"
#include "psl_launch.h"

#include <algorithm>

namespace psl {

// Shortest walk that the matrix form can take: its column words reach 120 words before the
// sequence, inside the guards from L = 3712 on.
constexpr uint32_t kCorrMxMinL = 4096;

// Which walks a correlation covers (launch_corr's mode).
__device__ __forceinline__ bool corr_takes(const WalkDev &w, int mode)
{
    return mode != 1 || (w.pending && w.n_flips > kFlipIncremental);
}

// C_k = (L-k) - 2 * #(s_i != s_{i+k}). A block owns 256 consecutive shifts
// k0..k0+255 and sweeps the sequence in LDS-staged segments of 32-bit words:
// word x of the sequence and the word at bit offset 32x + k (one funnel shift
// of two staged words) give 32 products per XOR and popcount.
constexpr int kCorrThreads = 256;
constexpr int kCorrSeg = 1024;        // staged 32-bit words per segment
__global__ __launch_bounds__(kCorrThreads) void k_corr(WalkDev *walks, const BatchEntry *batch, int mode,
                                                       uint32_t mx_L)
{
    WalkDev &w = walks[batch[blockIdx.y].slot];
    const uint32_t L = w.L;
    const uint32_t k0 = blockIdx.x * kCorrThreads;
    if (k0 >= L || L >= mx_L || !corr_takes(w, mode)) return;
    __shared__ uint32_t A[kCorrSeg];
    __shared__ uint32_t B[kCorrSeg + 16];
    const uint32_t *s32 = reinterpret_cast<const uint32_t *>(w.pivot);
    const uint32_t n32 = (L + 31) / 32;
    const uint32_t k = k0 + threadIdx.x;
    const uint32_t d = threadIdx.x, dq = d >> 5, dr = d & 31u;
    const uint32_t nprod = k < L ? L - k : 0;          // products of this shift
    const uint32_t nwb = (L - k0 + 31) / 32;           // words the block needs
    const uint32_t kq = k0 / 32;
    uint32_t diff = 0;
    for (uint32_t w0 = 0; w0 < nwb; w0 += kCorrSeg) {
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < kCorrSeg; t += kCorrThreads)
            A[t] = (w0 + t < n32) ? s32[w0 + t] : 0u;
        for (uint32_t t = threadIdx.x; t < kCorrSeg + 16; t += kCorrThreads)
            B[t] = (w0 + kq + t < n32) ? s32[w0 + kq + t] : 0u;
        __syncthreads();
        // this shift's products in the segment: bits 32*w0 .. nprod
        const uint32_t have = nprod > 32 * w0 ? nprod - 32 * w0 : 0;
        const uint32_t full = min((uint32_t)kCorrSeg, have / 32);
        for (uint32_t x = 0; x < full; ++x)
            diff += __popc(A[x] ^ __builtin_amdgcn_alignbit(B[x + dq + 1], B[x + dq], dr));
        if (full < (uint32_t)kCorrSeg && (have & 31u)) {
            const uint32_t x = full;
            const uint32_t v = A[x] ^ __builtin_amdgcn_alignbit(B[x + dq + 1], B[x + dq], dr);
            diff += __popc(v & ((1u << (have & 31u)) - 1u));
        }
    }
    if (k < L) {
        const int32_t c = (int32_t)nprod - 2 * (int32_t)diff;
        w.C[k] = c;
        if (mode == 0) w.C_lb[k] = c;
    }
}

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr uint32_t kCorrTile = 4096;     // shifts per wavefront
constexpr int kWordPad = 256;            // words before the sequence that the word offsets start from
constexpr int kMxThreads = 256;

// 32 sequence bits as +-1 in FP4 (1.0 = 0x2, the sign 0x8), shifts 4q + r of
// the chunk in nibble q of word r; v: the bits inside the sequence, others 0
// (their x is 0 too).
__device__ __forceinline__ void pm1_nibbles(uint32_t x, uint32_t v, uint32_t (&o)[4])
{
    constexpr uint32_t kS = 0x88888888u, kV = 0x22222222u;
    o[0] = ((x << 3) & kS) | ((v << 1) & kV);
    o[1] = ((x << 2) & kS) | (v & kV);
    o[2] = ((x << 1) & kS) | ((v >> 1) & kV);
    o[3] = (x & kS) | ((v >> 2) & kV);
}
// The same with every bit inside the sequence.
__device__ __forceinline__ void pm1_nibbles(uint32_t x, uint32_t (&o)[4])
{
    constexpr uint32_t kS = 0x88888888u, kV = 0x22222222u;
    o[0] = ((x << 3) & kS) | kV;
    o[1] = ((x << 2) & kS) | kV;
    o[2] = ((x << 1) & kS) | kV;
    o[3] = (x & kS) | kV;
}

// Block (x, y): tile y % tiles, positions' part y / tiles (Q chunks each) of walk
// (x + y) % walks: the longest parts of all walks start first, and the blocks of
// a walk and of a tile are dealt to all XCDs. (In steps of 8 one XCD got the first
// parts of every tile, the only ones that short tiles have, or all blocks of a
// walk: one walk at L = 1048575 398 us, now 257; 32 walks of a serving wave 5.0
// ms, now 1.5.) Four wavefronts take a quarter of the chunks each and add their
// sums in LDS: with a part per wavefront, added into C one by one, 64 walks at
// L = 65535 took 133 us (now 80). One part: C (and C_lb in mode 0) is stored;
// several: added into C, which is zero.
__global__ __launch_bounds__(kMxThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_corr_mx(
    WalkDev *walks, const BatchEntry *batch, int mode, uint32_t mx_L, int splits, int Q)
{
    WalkDev &w = walks[batch[(blockIdx.x + blockIdx.y) % gridDim.x].slot];
    if (!corr_takes(w, mode)) return;
    const int L = (int)w.L;
    const int tiles = (int)(gridDim.y / (uint32_t)splits);
    const int K0 = (int)kCorrTile * ((int)blockIdx.y % tiles);
    if (K0 >= L || L < (int)mx_L) return;
    // the block's chunks (those with a position i below L - K0), a quarter for each wavefront
    const int p0 = Q * ((int)blockIdx.y / tiles), p1 = min(p0 + Q, (L - K0 + 31) >> 5);
    if (p0 >= p1) return;
    __shared__ int sum[kCorrTile + 64];
    for (int x = (int)threadIdx.x; x < (int)kCorrTile + 64; x += kMxThreads) sum[x] = 0;
    __syncthreads();
    const int wq4 = (p1 - p0 + 3) >> 2;
    const int c0 = min(p1, p0 + wq4 * ((int)threadIdx.x >> 6)), c1 = min(p1, c0 + wq4);
    const int lane = (int)threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int N = (c1 - c0 + 3) >> 2, cb = c0 + g * N;
    const uint32_t *base = reinterpret_cast<const uint32_t *>(w.pivot) - kWordPad;
    auto word = [&](int i) {
        return *(const __attribute__((address_space(1))) uint32_t *)(base + (uint32_t)(i + kWordPad));
    };
    const int kw = K0 >> 5;                 // first word of the rows at chunk 0
    v4f acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
    // row matrix of (chunk + n) = u, p: bits 32 (kw + u) + 16 p + r ..; a chunk
    // past this part's last is taken by the column's mask
    uint32_t A[8][2][4];
    auto rows = [&](uint32_t hi, uint32_t lo, int u, uint32_t(&a)[2][4]) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t x = __builtin_amdgcn_alignbit(hi, lo, (uint32_t)r + 16u * p);
            const int nv = L - (32 * (kw + u) + 16 * p + r);
            const uint32_t v = nv >= 32 ? 0xFFFFFFFFu : nv > 0 ? (1u << nv) - 1u : 0u;
            pm1_nibbles(x, v, a[p]);
        }
    };
    // steps at which every lane's column chunk lies in 120 .. c1-1 and the next
    // row window inside the sequence
    const int inner0 = 120 - c0;
    const int inner1 = min(c1 - c0 - 3 * N, ((L - 63) >> 5) - kw - c0 - 3 * N - 7);
    uint32_t prev, wq[4], bq[4];
    {
        uint32_t x[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) x[i] = word(kw + cb + i);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            wq[k] = word(kw + cb + k + 9);
            bq[k] = word(cb + k - 8 * r);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) rows(x[u + 1], x[u], cb + u, A[u]);
        prev = x[8];
    }
    for (int s = 0; s < N;) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            if (s >= N) break;
            const uint32_t wn = wq[v & 3], xb = bq[v & 3];
            wq[v & 3] = word(kw + cb + s + 13);
            bq[v & 3] = word(cb + s + 4 - 8 * r);
            // the column's word: position 32 (chunk - 8 q), whole words before
            // the sequence 0, and 0 in chunks past this part
            const int c = cb + s;
            const bool on = c >= 8 * r && c < c1;
            const bool inner = s >= inner0 && s < inner1;
            uint32_t b[4];
            if (inner) pm1_nibbles(xb, b);
            else       pm1_nibbles(on ? xb : 0u, on ? 0xFFFFFFFFu : 0u, b);
            const v8i B = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], 0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t(&a)[4] = A[(v + (i >> 1)) & 7][i & 1];
                const v8i M = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], 0, 0, 0, 0};
                acc[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(M, B, acc[i], 4, 4, 0, 0, 0, 0);
            }
            if (inner) {
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    pm1_nibbles(__builtin_amdgcn_alignbit(wn, prev, (uint32_t)r + 16u * p), A[v][p]);
            } else {
                rows(wn, prev, cb + s + 8, A[v]);
            }
            prev = wn;
            ++s;
        }
    }
    // register j of product i, lane (g, q): shift 256 q + 16 i + 4 g + j of the
    // tile, in LDS 16 (q / 4) + q % 4 words further on: a wavefront's 64 lanes
    // then meet 64 banks
    const int at = 256 * r + 16 * (r >> 2) + (r & 3) + 4 * g;
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) atomicAdd(&sum[at + 16 * i + j], (int)acc[i][j]);
    __syncthreads();
    for (int x = (int)threadIdx.x; x < (int)kCorrTile && K0 + x < L; x += kMxThreads) {
        const int q = x >> 8, c = sum[x + 16 * (q >> 2) + (q & 3)];
        if (splits == 1) {
            w.C[K0 + x] = c;
            if (mode == 0) w.C_lb[K0 + x] = c;
        } else {
            atomicAdd(&w.C[K0 + x], c);
        }
    }
}

// Before and after the parts of k_corr_mx are added into C: C = 0; C_lb = C.
__global__ void k_corr_edge(WalkDev *walks, const BatchEntry *batch, int mode, uint32_t mx_L, int after)
{
    WalkDev &w = walks[batch[blockIdx.y].slot];
    if (!corr_takes(w, mode)) return;
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= w.L || w.L < mx_L) return;
    if (after) w.C_lb[k] = w.C[k];
    else       w.C[k] = 0;
}

hipError_t launch_corr(WalkDev *walks, const BatchEntry *batch, uint32_t nb, const CorrDims &d, int mode, hipStream_t s)
{
    constexpr uint32_t kMaxY = 65535;      // walks per launch of the 2-D grids
    // parts of the positions that give the launch about kBlocks blocks, each of
    // kMinPart chunks at least: a part more per tile costs 4096 atomic additions,
    // a part less leaves compute units idle. At 1024 / 2048 / 4096 blocks, us: one
    // walk at L = 1048575 257 / 240 / 252, 64 at L = 65535 80 / 86 / 112, 32 of L
    // up to 1048575 1520 / 1530 / 1530; parts of at least 512 chunks: one walk at
    // L = 131071 21 for 19, at L = 9001 18 for 15.
    constexpr uint32_t kBlocks = 1024, kMinPart = 256;
    const uint32_t most = (d.max_L + 31) / 32;
    const uint32_t Q = (uint32_t)std::min<uint64_t>(most, std::max<uint64_t>(kMinPart, (d.chunks + kBlocks - 1) / kBlocks));
    const uint32_t splits = (most + Q - 1) / Q, tiles = (d.max_L + kCorrTile - 1) / kCorrTile;
    // the shortest walk on the matrix cores: none in a launch with little work of
    // walks of moderate length, whose few tiles leave most compute units idle, where
    // a block of the popcount form has 256 shifts and no zeroed C to add to. Starts,
    // matrix / popcount, us: one walk at L = 4097 39 / 32, 16383 47 / 38, 32767
    // 48 / 45, 40009 48 / 50, 65535 47 / 61; 4 at 32767 (16384 chunks) 51 / 49, 8 at
    // 32767 51 / 62; 16 at 16383 (16384) 51 / 48, 32 54 / 64; 64 at 8193 (16448)
    // 62 / 55, at 12001 65 / 67; 256 at 4097 (16640) 77 / 79.
    constexpr uint32_t kMaxPopL = 36864, kMaxPopChunks = 16384;
    const uint32_t mx_L = d.max_L < kMaxPopL && d.chunks <= kMaxPopChunks ? UINT32_MAX : kCorrMxMinL;
    for (uint32_t b0 = 0; b0 < nb; b0 += kMaxY) {
        const uint32_t ny = std::min(kMaxY, nb - b0);
        if (d.min_L < mx_L) {
            const uint32_t len = std::min(d.max_L, mx_L - 1);
            k_corr<<<dim3((len + kCorrThreads - 1) / kCorrThreads, ny), kCorrThreads, 0, s>>>(walks, batch + b0, mode, mx_L);
        }
        if (d.max_L >= mx_L) {
            const dim3 all((d.max_L + 255) / 256, ny);
            if (splits > 1) k_corr_edge<<<all, 256, 0, s>>>(walks, batch + b0, mode, mx_L, 0);
            k_corr_mx<<<dim3(ny, tiles * splits), kMxThreads, 0, s>>>(walks, batch + b0, mode, mx_L, (int)splits, (int)Q);
            if (splits > 1 && mode == 0) k_corr_edge<<<all, 256, 0, s>>>(walks, batch + b0, mode, mx_L, 1);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace psl
