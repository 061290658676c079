// psl_split.hip -- the matrix evaluation of libpsl (gfx950).
//
// Eq. (5) summed over the neighbours of Algorithm 1, as products of 0/1
// matrices with coefficient vectors. For shift k with c = C_k and
// T(x) = T_alpha(|x|), the one-element flip of Section 3 gives
// C'_k = c + 4(x_R + x_L - 1) where both neighbours of j exist
// (k <= m_j = min(j, L-1-j)) and c + 2(2x - 1) where one does
// (m_j < k <= M_j = max(j, L-1-j)); x_R = 1 where s_j s_{j+k} = -1, x_L = 1
// where s_j s_{j-k} = -1. So
//   both: T(c-4) + XOR(x_R, x_L) (T(c) - T(c-4)) + AND(x_R, x_L) (T(c+4) - T(c-4)),
//   one:  T(c-2) + x (T(c+2) - T(c-2)),
// and F_j is a sum of prefix sums of the constant parts plus three 0/1
// matrices times coefficient vectors. The matrix cores take the matrices as
// FP4 (a bit of the sequence is a nibble of 0.5 or 1.0 after one masking
// operation) and the coefficients as exact fixed-point numbers in kDig
// balanced base-32 digits, each exact in FP6: the FP32 accumulators then hold
// exact integers, and only the rounding of a coefficient to the quantum U
// enters. This file holds the per-step preparation (coefficients, digits,
// prefix sums, scale and path choice) and the matrix kernel.
#include "psl_dev_util.h"
#include "psl_device.h"
#include "psl_launch.h"

#include <algorithm>
#include <climits>

namespace psl {

// The quantum of a step's coefficients: U = 2^e with every coefficient below
// 2^67 U. They grow with |c| (T is increasing and convex in |c|), so the
// largest is T(P+4) - T(P-4) at the pivot's PSL P (the maximum |C_k|).
__device__ __forceinline__ double split_scale(const double *__restrict__ T, int P)
{
    const int m4 = P >= 4 ? P - 4 : 4 - P, m2 = P >= 2 ? P - 2 : 2 - P;
    const double c4 = T[P + 4] - T[m4], c2 = T[P + 2] - T[m2];
    return ldexp(1.0, ilogb(c4 > c2 ? c4 : c2) - 66);
}

// The digits of one coefficient as FP6 codes, four per word (digit 4q + i in
// byte i of out[q]; digits 14 and 15 are 0). v = coefficient / U in three
// 30-bit words of six digits; adding 16 to every 5-bit field (kBias) turns
// the balanced digits d in -16..15 into plain fields d + 16. The FP6 (E2M3)
// code of n/8, n = 0..16, is n; of n/4 it is n + min(n, 8); 0x20 is the sign.
// Odd shifts meet 1.0 in the FP4 matrix and take d/8, even ones 0.5 and d/4.
constexpr int kBias = 0x21084210;

__device__ __forceinline__ uint32_t digit_codes(uint32_t v, bool even)
{
    const uint32_t neg = ~(v >> 4) & 0x01010101u;                   // d < 0
    const uint32_t mag = ((v ^ ((neg << 4) - neg)) & 0x0F0F0F0Fu) + neg;   // |d|
    const uint32_t big = ((mag >> 3) | (mag >> 4)) & 0x01010101u;   // |d| >= 8
    const uint32_t dbl = mag + ((mag & ~((big << 5) - big)) | (big << 3));
    return (even ? dbl : mag) | (neg << 5);
}

__device__ __forceinline__ void split_digits(double v, bool even, uint32_t (&out)[4])
{
    const double h2 = rint(v * 0x1p-60);
    const double r1 = fma(h2, -0x1p60, v);
    const double h1 = rint(r1 * 0x1p-30);
    const double r0 = fma(h1, -0x1p30, r1);
    int w0 = __double2int_rn(r0) + kBias, w1 = __double2int_rn(h1) + kBias, w2 = __double2int_rn(h2) + kBias;
    w1 += w0 >> 30;                     // the carries out of the six-digit words
    w0 &= 0x3FFFFFFF;
    w2 += w1 >> 30;
    w1 &= 0x3FFFFFFF;
    const uint32_t a = (uint32_t)w0, b = (uint32_t)w1, c = (uint32_t)w2;
    out[0] = (a & 31u) | ((a << 3) & 0x1F00u) | ((a << 6) & 0x1F0000u) | ((a << 9) & 0x1F000000u);
    out[1] = ((a >> 20) & 31u) | ((a >> 17) & 0x1F00u) | ((b << 16) & 0x1F0000u) | ((b << 19) & 0x1F000000u);
    out[2] = ((b >> 10) & 31u) | ((b >> 7) & 0x1F00u) | ((b >> 4) & 0x1F0000u) | ((b >> 1) & 0x1F000000u);
    out[3] = (c & 31u) | ((c << 3) & 0x1F00u) | 0x10100000u;
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = digit_codes(out[q], even);
}

// Per shift k of every split walk (one block per segment of the walk's shifts,
// in tiles of 256): the values T(|C_k - 4|), T(|C_k - 2|), T(|C_k + 2|),
// T(|C_k|) that k_split_scan turns into prefix sums, and the digit records.
// A record holds one 32-shift chunk (shifts 32c .. 32c+31) of one coefficient:
// 16 columns (digits) of 32 FP6 codes, the first 16 bytes of each column, then
// the last 8 of each (kRecBytes); slot 8 r + q of a column is shift 32c + 4q + r,
// the order in which the matrix kernel's masks leave the bits of a word. The
// threads leave the codes of a tile in LDS (one word per shift and four
// columns); then one thread per (coefficient, chunk, four columns) packs them.
constexpr int kPrepThreads = 256;
constexpr int kPrepStride = 36;         // words per chunk and four columns in LDS (32 and padding)
__global__ __launch_bounds__(kPrepThreads) void k_split_prep(const WalkDev *walks, const BatchEntry *batch,
                                                             Tables tabs, SegMap map)
{
    __shared__ __align__(16) uint32_t s_c[3][4][8 * kPrepStride];
    uint32_t b, seg;
    seg_of(map, blockIdx.x, b, seg);
    const BatchEntry be = batch[b];
    if (!be.lsplit) return;
    const WalkDev &w = walks[be.slot];
    const int L = (int)w.L;
    const double *__restrict__ T = tabs.T[w.alpha];
    const double inv = 1.0 / split_scale(T, w.psl_pivot);      // exact: U is a power of two
    const int half = (L - 1) / 2;                              // the largest m_j
    const int nbo = (int)split_both_chunks((uint32_t)L), nco = (int)split_chunks((uint32_t)L);
    const int k_end = (int)seg + 1 == (int)seg_count((uint32_t)L, map.shift) ? 32 * nco : (int)((seg + 1) << map.shift);
    const int t = (int)threadIdx.x;
    const int slot = (t >> 5) * kPrepStride + 8 * (t & 3) + ((t & 31) >> 2);
    double *__restrict__ pre = be.pre;
    for (int k0 = (int)(seg << map.shift); k0 < k_end; k0 += kPrepThreads) {
        const int k = k0 + t;
        const bool in = k >= 1 && k < L;
        const bool both = (k0 >> 5) < nbo;                     // some chunk of the tile has both-neighbour shifts
        const int c = in ? w.C[k] : 0;
        const int a4 = c + 4 < 0 ? -(c + 4) : c + 4, m4 = c - 4 < 0 ? 4 - c : c - 4;
        const int a2 = c + 2 < 0 ? -(c + 2) : c + 2, m2 = c - 2 < 0 ? 2 - c : c - 2;
        const double t0 = T[c < 0 ? -c : c], tp2 = T[a2], tm2 = T[m2];
        if (in) {
            pre[(size_t)L + k] = tm2;
            pre[2 * (size_t)L + k] = tp2;
            pre[3 * (size_t)L + k] = t0;
        }
        uint32_t d[4];
        split_digits(in ? (tp2 - tm2) * inv : 0.0, !(t & 1), d);
#pragma unroll
        for (int q = 0; q < 4; ++q) s_c[2][q][slot] = d[q];
        if (both) {
            const double tp4 = T[a4], tm4 = T[m4];
            if (in && k <= half) pre[k] = tm4;
            split_digits(in ? (t0 - tm4) * inv : 0.0, !(t & 1), d);
#pragma unroll
            for (int q = 0; q < 4; ++q) s_c[0][q][slot] = d[q];
            split_digits(in ? (tp4 - tm4) * inv : 0.0, !(t & 1), d);
#pragma unroll
            for (int q = 0; q < 4; ++q) s_c[1][q][slot] = d[q];
        }
        __syncthreads();
        // task e: coefficient e / 32, chunk (e / 4) % 8, columns 4 (e % 4) .. +3
        const int set = t >> 5, cc = (t >> 2) & 7, q = t & 3;
        const int ch = (k0 >> 5) + cc;
        if (t < 96 && ch < (set == 2 ? nco : nbo)) {
            const uint4 *src = reinterpret_cast<const uint4 *>(&s_c[set][q][cc * kPrepStride]);
            uint32_t o[4][6];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t x[4][4];                              // [column][4 codes in 24 bits]
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const uint4 v = src[4 * h + y];
                    // 16-bit lanes: columns 0 and 2, columns 1 and 3
                    const uint32_t e01 = (v.x & 0x00FF00FFu) | ((v.y & 0x00FF00FFu) << 6);
                    const uint32_t e23 = (v.z & 0x00FF00FFu) | ((v.w & 0x00FF00FFu) << 6);
                    const uint32_t f01 = ((v.x >> 8) & 0x00FF00FFu) | (((v.y >> 8) & 0x00FF00FFu) << 6);
                    const uint32_t f23 = ((v.z >> 8) & 0x00FF00FFu) | (((v.w >> 8) & 0x00FF00FFu) << 6);
                    x[0][y] = (e01 & 0xFFFFu) | ((e23 & 0xFFFFu) << 12);
                    x[1][y] = (f01 & 0xFFFFu) | ((f23 & 0xFFFFu) << 12);
                    x[2][y] = (e01 >> 16) | ((e23 >> 16) << 12);
                    x[3][y] = (f01 >> 16) | ((f23 >> 16) << 12);
                }
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    o[y][3 * h] = x[y][0] | (x[y][1] << 24);
                    o[y][3 * h + 1] = (x[y][1] >> 8) | (x[y][2] << 16);
                    o[y][3 * h + 2] = (x[y][2] >> 16) | (x[y][3] << 8);
                }
            }
            uint8_t *rec = set == 2 ? be.dig_one + (size_t)ch * kRecBytes
                                    : be.dig_both + ((size_t)ch * 2 + (size_t)set) * kRecBytes;
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                *reinterpret_cast<uint4 *>(rec + 16 * (4 * q + y)) = make_uint4(o[y][0], o[y][1], o[y][2], o[y][3]);
                *reinterpret_cast<uint2 *>(rec + 256 + 8 * (4 * q + y)) = make_uint2(o[y][4], o[y][5]);
            }
        }
        __syncthreads();
    }
}

// One block per (split walk, value array): the array becomes its inclusive
// prefix sums over k = 1..k (entry 0 = 0). Chunks of kScanChunk consecutive
// entries go through the block in order: each thread sums its kScanPer
// entries, the wavefronts scan their threads' totals and the block adds the
// wavefronts' totals before them, and the chunks' totals are carried with
// Neumaier's compensation. Every summand is non-negative, so each prefix is
// within a few dozen roundings of its exact value. Block (walk, 0) also
// stores the step's scale and path choice: the matrix path is taken when the
// near-peak list holds the PSL (sparse form) and the quantization error,
// at most (L-1) U, is below 1e-14 of a lower bound of every neighbour's F
// (T(P-4) for the pivot's PSL P, and at least 1); a walk that does not take
// it is counted in *tab, which the table evaluation looks at first.
constexpr int kScanThreads = 256;
constexpr int kScanPer = 4;
constexpr int kScanChunk = kScanThreads * kScanPer;
__global__ __launch_bounds__(kScanThreads) void k_split_scan(const WalkDev *walks, const BatchEntry *batch,
                                                             Tables tabs, uint32_t *tab)
{
    const uint32_t wb = blockIdx.x / 4, x = blockIdx.x % 4;
    const BatchEntry be = batch[wb];
    if (!be.lsplit) {
        if (x == 0 && threadIdx.x == 0) atomicAdd(tab, 1u);
        return;
    }
    const WalkDev &w = walks[be.slot];
    const int L = (int)w.L;
    const int K = x == 0 ? (L - 1) / 2 + 1 : L;     // T(|C_k - 4|) is summed over both-neighbour shifts only
    double *__restrict__ v = be.pre + (size_t)x * L;
    __shared__ double s_tot[kScanThreads / 64];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    auto load = [&](int base, double (&e)[kScanPer]) {
        const int k0 = base + (int)threadIdx.x * kScanPer;
#pragma unroll
        for (int i = 0; i < kScanPer; ++i) e[i] = k0 + i < K ? v[k0 + i] : 0.0;
    };
    double carry = 0.0, ccomp = 0.0;
    double cur[kScanPer], nxt[kScanPer];
    load(1, cur);
    for (int base = 1; base < K; base += kScanChunk) {
        if (base + kScanChunk < K) load(base + kScanChunk, nxt);
#pragma unroll
        for (int i = 1; i < kScanPer; ++i) cur[i] += cur[i - 1];
        // inclusive scan of the thread totals over the wavefront
        double t = cur[kScanPer - 1];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const double o = __shfl_up(t, d);
            if (lane >= d) t += o;
        }
        double excl = __shfl_up(t, 1);
        if (lane == 0) excl = 0.0;
        if (lane == 63) s_tot[wave] = t;
        __syncthreads();
        double off = carry + ccomp, tot = 0.0;
#pragma unroll
        for (int q = 0; q < kScanThreads / 64; ++q) {
            if (q < wave) off += s_tot[q];
            tot += s_tot[q];
        }
        off += excl;
        const int k0 = base + (int)threadIdx.x * kScanPer;
#pragma unroll
        for (int i = 0; i < kScanPer; ++i)
            if (k0 + i < K) v[k0 + i] = off + cur[i];
        nsum_add(carry, ccomp, tot);
        __syncthreads();                           // s_tot is rewritten by the next chunk
#pragma unroll
        for (int i = 0; i < kScanPer; ++i) cur[i] = nxt[i];
    }
    if (threadIdx.x == 0) {
        v[0] = 0.0;
        if (x == 0) {
            const double *__restrict__ T = tabs.T[w.alpha];
            const int P = w.psl_pivot;
            const double U = split_scale(T, P);
            const double flow = P > 4 ? T[P - 4] : 0.0;
            const bool exact_enough = (double)(L - 1) * U <= 1e-14 * (flow > 1.0 ? flow : 1.0);
            const bool sparse_psl = be.near[0] <= be.near_lim;
            SplitState st;
            st.U = U;
            st.use = exact_enough && sparse_psl ? 1u : 0u;
            st.pad = 0;
            *be.ss = st;
            if (!st.use) atomicAdd(tab, 1u);
        }
    }
}

hipError_t launch_split_prep(const WalkDev *walks, const BatchEntry *batch, uint32_t nb, const Tables &tabs,
                             const SegMap &map, uint32_t *tab, hipStream_t s)
{
    if (map.shift < kSegShiftMin || map.shift > kSegShiftMax || map.nb != nb || !tab) return hipErrorInvalidValue;
    if (nb == 0 || map.total == 0) return hipSuccess;
    k_split_prep<<<map.total, kPrepThreads, 0, s>>>(walks, batch, tabs, map);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_split_scan<<<4 * nb, kScanThreads, 0, s>>>(walks, batch, tabs, tab);
    return hipGetLastError();
}

// ------------------------------------------------------- matrix kernel

// One wavefront per work item (walk, tile of kMxTile = 256 consecutive
// elements, k-split). The tile's elements J0 + 32 b + 16 p + r (b = 0..7,
// p = 0..1, r = 0..15) are the rows of 16 products per step of
// v_mfma_f32_16x16x128_f8f6f4: lane l has row r = l % 16 (FP4 matrix) or
// column l % 16 (FP6 digits) and the 32 shifts of one chunk, lane group
// g = l / 16 having a chunk of its own. Element j and chunk c read the right
// window, bits j + 32c .. +31 of the sequence, and the left window, bits
// j - 32c, j - 32c - 1, ..; the right one depends on b + c and p only, the
// left one on b - c and p. So the four lane groups sweep four ranges of N
// chunks each (chunk c0 + g N + s at step s): a step then needs one new right
// and one new left window per p, kept in rings of eight, for its 16 products
// of a 16 x 128 matrix. Per product the wavefront makes four words of eight
// nibbles: (bits & 0x11111111) holds shifts 4q as 0.5, (bits & 0x22222222)
// shifts 4q + 1 as 1.0, and the same of (bits >> 2) shifts 4q + 2 and 4q + 3;
// the record's slot order and digit scales match.
//
// One-neighbour shifts come first, with the sequence's bits as they are (the
// matrix of a window is the same for all b + c, so it is masked once); then
// the rows with s_j = -1 change sign (their x is 1 minus the bit, and the
// combine takes T(c+2) as their constant part), and the both-neighbour shifts
// add XOR (which s_j does not change) and AND of the bits times s_j. Both go
// into the same accumulators: |digit| <= 16 over at most L-1 shifts, one
// coefficient each, stays within 2^24 units of 1/8, exact in FP32.
//
// Chunks in which some row of the tile has a bound (m_j) inside, and the up to
// three that do not fill a step, are taken by mx_edge: four consecutive
// chunks per step, every row's shifts outside its bounds masked.
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr uint32_t kM0 = 0x11111111u, kM1 = 0x22222222u;
constexpr int kBlk = kMxTile / 32;       // pairs of 16-row blocks of a tile
constexpr int kPad = 256;                // words before the sequence that the word offsets start from

__device__ __forceinline__ v4f mx_mfma(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, v8i B, v4f acc)
{
    const v8i A = {(int)x0, (int)x1, (int)x2, (int)x3, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, B, acc, 4, 2, 0, 0, 0, 0);
}

// (a ^ b) & m and (a ^ s) & (b ^ s), one operation each
__device__ __forceinline__ uint32_t xor_and(uint32_t a, uint32_t b, uint32_t m)
{
    return __builtin_amdgcn_bitop3_b32(a, b, m, 0x28);
}
__device__ __forceinline__ uint32_t and_signed(uint32_t a, uint32_t b, uint32_t s)
{
    return __builtin_amdgcn_bitop3_b32(a, b, s, 0x42);
}

// This lane's column of a digit record.
__device__ __forceinline__ v8i mx_rec(const uint8_t *__restrict__ base, uint32_t off16, uint32_t off8)
{
    const v4i a = *(const __attribute__((address_space(1))) v4i *)(base + off16);
    const v2i b = *(const __attribute__((address_space(1))) v2i *)(base + off8);
    return v8i{a.x, a.y, a.z, a.w, b.x, b.y, 0, 0};
}

struct MxLane {
    const uint32_t *w;      // kPad words before the sequence's first
    int J32;                // first word of the tile
    int r, g, col;
    uint32_t S[2 * kBlk];   // all ones where s_j = -1, per 16-row block
    __device__ __forceinline__ uint32_t word(int i) const
    {
        return *(const __attribute__((address_space(1))) uint32_t *)(w + (uint32_t)(i + kPad));
    }
};

// The both-neighbour products of chunks c0 + g N + s, s < N, all of whose
// shifts are at most every row's m_j.
__device__ __forceinline__ void mx_both(v4f (&acc)[2 * kBlk], const MxLane &ln, const uint8_t *__restrict__ dig, int c0,
                                        int N)
{
    const int cb = c0 + ln.g * N;
    const uint32_t shr = (uint32_t)ln.r, shl = (uint32_t)(31 - ln.r);
    uint32_t R[8][2], R2[8][2], W[8][2], W2[8][2];        // right and left windows, and shifted by 2
    uint32_t rprev, lprev, rq[4], lq[4];
    v8i bx[2], ba[2];
    uint32_t o16 = (uint32_t)cb * (2 * kRecBytes) + 16u * (uint32_t)ln.col;
    uint32_t o8 = (uint32_t)cb * (2 * kRecBytes) + 256u + 8u * (uint32_t)ln.col;
    bx[0] = mx_rec(dig, o16, o8);
    ba[0] = mx_rec(dig + kRecBytes, o16, o8);
    {
        uint32_t x[9], y[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            x[i] = ln.word(ln.J32 + cb + i);
            y[i] = ln.word(ln.J32 - cb - 1 + i);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            rq[k] = ln.word(ln.J32 + cb + k + 9);
            lq[k] = ln.word(ln.J32 - cb - k - 2);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) y[i] = __builtin_bitreverse32(y[i]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                R[u][p] = __builtin_amdgcn_alignbit(x[u + 1], x[u], shr + 16u * p);
                R2[u][p] = R[u][p] >> 2;
                W[u][p] = __builtin_amdgcn_alignbit(y[u], y[u + 1], shl - 16u * p);
                W2[u][p] = W[u][p] >> 2;
            }
        rprev = x[8];
        lprev = y[0];
    }
    for (int s = 0;;) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            if (s >= N) return;
            o16 += 2 * kRecBytes;
            o8 += 2 * kRecBytes;
            bx[(v + 1) & 1] = mx_rec(dig, o16, o8);
            ba[(v + 1) & 1] = mx_rec(dig + kRecBytes, o16, o8);
            const uint32_t rn = rq[v & 3], lw = lq[v & 3];
            rq[v & 3] = ln.word(ln.J32 + cb + s + 13);
            lq[v & 3] = ln.word(ln.J32 - cb - s - 6);
#pragma unroll
            for (int b = 0; b < kBlk; ++b) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int i = 2 * b + p, u = (v + b) & 7, x = (b - v) & 7;
                    acc[i] = mx_mfma(xor_and(R[u][p], W[x][p], kM0), xor_and(R[u][p], W[x][p], kM1),
                                     xor_and(R2[u][p], W2[x][p], kM0), xor_and(R2[u][p], W2[x][p], kM1), bx[v & 1],
                                     acc[i]);
                    const uint32_t t = and_signed(R[u][p], W[x][p], ln.S[i]);
                    const uint32_t t2 = and_signed(R2[u][p], W2[x][p], ln.S[i]);
                    acc[i] = mx_mfma(t & kM0, t & kM1, t2 & kM0, t2 & kM1, ba[v & 1], acc[i]);
                }
            }
            const uint32_t ly = __builtin_bitreverse32(lw);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                R[v][p] = __builtin_amdgcn_alignbit(rn, rprev, shr + 16u * p);
                R2[v][p] = R[v][p] >> 2;
                W[7 - v][p] = __builtin_amdgcn_alignbit(ly, lprev, shl - 16u * p);
                W2[7 - v][p] = W[7 - v][p] >> 2;
            }
            rprev = rn;
            lprev = ly;
            ++s;
        }
    }
}

// The one-neighbour products (right or left side) of chunks c0 + g N + s,
// s < N, all of whose shifts are past every row's m_j.
template <bool RIGHT>
__device__ __forceinline__ void mx_one(v4f (&acc)[2 * kBlk], const MxLane &ln, const uint8_t *__restrict__ dig, int c0,
                                       int N)
{
    const int cb = c0 + ln.g * N;
    const uint32_t sh = RIGHT ? (uint32_t)ln.r : (uint32_t)(31 - ln.r);
    uint32_t A[8][2][4];                    // the matrices of eight windows
    uint32_t prev, wq[4];
    v8i bq[4];
    uint32_t o16 = (uint32_t)cb * kRecBytes + 16u * (uint32_t)ln.col;
    uint32_t o8 = (uint32_t)cb * kRecBytes + 256u + 8u * (uint32_t)ln.col;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        bq[k] = mx_rec(dig, o16, o8);
        o16 += kRecBytes;
        o8 += kRecBytes;
    }
    auto make = [&](uint32_t hi, uint32_t lo, uint32_t(&a)[2][4]) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t win = __builtin_amdgcn_alignbit(hi, lo, RIGHT ? sh + 16u * p : sh - 16u * p);
            a[p][0] = win & kM0;
            a[p][1] = win & kM1;
            a[p][2] = (win >> 2) & kM0;
            a[p][3] = (win >> 2) & kM1;
        }
    };
    {
        uint32_t x[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) x[i] = ln.word(RIGHT ? ln.J32 + cb + i : ln.J32 - cb - 1 + i);
#pragma unroll
        for (int k = 0; k < 4; ++k) wq[k] = ln.word(RIGHT ? ln.J32 + cb + k + 9 : ln.J32 - cb - k - 2);
        if (!RIGHT) {
#pragma unroll
            for (int i = 0; i < 9; ++i) x[i] = __builtin_bitreverse32(x[i]);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) make(RIGHT ? x[u + 1] : x[u], RIGHT ? x[u] : x[u + 1], A[u]);
        prev = RIGHT ? x[8] : x[0];
    }
    for (int s = 0;;) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            if (s >= N) return;
            bq[(v + 2) & 3] = mx_rec(dig, o16, o8);
            o16 += kRecBytes;
            o8 += kRecBytes;
            uint32_t wn = wq[v & 3];
            wq[v & 3] = ln.word(RIGHT ? ln.J32 + cb + s + 13 : ln.J32 - cb - s - 6);
#pragma unroll
            for (int b = 0; b < kBlk; ++b) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int i = 2 * b + p;
                    const uint32_t(&a)[4] = A[RIGHT ? (v + b) & 7 : (b - v) & 7][p];
                    acc[i] = mx_mfma(a[0], a[1], a[2], a[3], bq[v & 3], acc[i]);
                }
            }
            if (!RIGHT) wn = __builtin_bitreverse32(wn);
            make(wn, prev, A[RIGHT ? v : 7 - v]);
            prev = wn;
            ++s;
        }
    }
}

// Chunks ca .. ce-1, four consecutive ones per step, with every row's shifts
// outside its bounds masked: BOTH: shifts up to m_j; otherwise the shifts past
// m_j, on the row's one-neighbour side (right for j <= half). Only a side that
// some row uses is read: the other side's words can lie outside the guards.
template <bool BOTH>
__device__ __forceinline__ void mx_edge(v4f (&acc)[2 * kBlk], const MxLane &ln, const uint8_t *__restrict__ dig, int L,
                                        int ca, int ce, int nrec)
{
    const int half = (L - 1) / 2;
    const uint32_t shr = (uint32_t)ln.r, shl = (uint32_t)(31 - ln.r);
    constexpr uint32_t kStep = BOTH ? 2 * kRecBytes : kRecBytes;
    const bool need_r = BOTH || 32 * ln.J32 <= half, need_l = BOTH || min(32 * ln.J32 + kMxTile, L) - 1 > half;
#pragma unroll 1
    for (int c4 = ca; c4 < ce; c4 += 4) {
        const int c = c4 + ln.g;
        const uint32_t cl = (uint32_t)min(c, nrec - 1);
        const uint32_t o16 = cl * kStep + 16u * (uint32_t)ln.col, o8 = cl * kStep + 256u + 8u * (uint32_t)ln.col;
        const v8i bx = mx_rec(dig, o16, o8);
        v8i ba = bx;
        if (BOTH) ba = mx_rec(dig + kRecBytes, o16, o8);
        uint32_t x[kBlk + 1], y[kBlk + 1];
#pragma unroll
        for (int i = 0; i < kBlk + 1; ++i) {
            x[i] = need_r ? ln.word(ln.J32 + c + i) : 0u;
            y[i] = need_l ? __builtin_bitreverse32(ln.word(ln.J32 - c - 1 + i)) : 0u;
        }
#pragma unroll
        for (int b = 0; b < kBlk; ++b) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int i = 2 * b + p;
                const int j = 32 * (ln.J32 + b) + 16 * p + ln.r;
                const int m = min(j, L - 1 - j);
                // the shifts 32c + t of this row: t < n (BOTH) or t >= n
                const int n = min(32, max(0, m + 1 - 32 * c));
                const uint32_t lowm = n > 0 ? 0xFFFFFFFFu >> (32 - n) : 0u;
                const uint32_t V = c >= ce ? 0u : BOTH ? lowm : ~lowm;
                if (!__any(V != 0u)) continue;
                const uint32_t R = __builtin_amdgcn_alignbit(x[b + 1], x[b], shr + 16u * p);
                const uint32_t W = __builtin_amdgcn_alignbit(y[b], y[b + 1], shl - 16u * p);
                if (BOTH) {
                    const uint32_t q = xor_and(R, W, V), q2 = q >> 2;
                    acc[i] = mx_mfma(q & kM0, q & kM1, q2 & kM0, q2 & kM1, bx, acc[i]);
                    const uint32_t t = and_signed(R, W, ln.S[i]) & V, t2 = t >> 2;
                    acc[i] = mx_mfma(t & kM0, t & kM1, t2 & kM0, t2 & kM1, ba, acc[i]);
                } else {
                    const uint32_t q = (j <= half ? R : W) & V, q2 = q >> 2;
                    acc[i] = mx_mfma(q & kM0, q & kM1, q2 & kM0, q2 & kM1, bx, acc[i]);
                }
            }
        }
    }
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx(
    const WalkDev *__restrict__ walks, const BatchEntry *__restrict__ batch, const EvalItem *__restrict__ items)
{
    const EvalItem it = items[blockIdx.x];
    if (it.walk == kMxNoWalk) return;
    const BatchEntry be = batch[it.walk];
    if (!be.lsplit || !be.ss->use) return;
    const WalkDev &w = walks[be.slot];
    const int L = (int)w.L;
    const uint32_t n_lmt = be.fixed ? be.n_lmt : w.n_lmt;
    const uint32_t start = be.fixed ? be.start : step_start(w);
    // the tile: it.tile tiles past the one of the neighbourhood's first
    // element; nothing to do when no candidate lies in it
    const int ntile = (L + kMxTile - 1) / kMxTile;
    const int j_first = (int)((start + 1u) % (uint32_t)L);
    const int J0 = kMxTile * ((j_first / kMxTile + (int)it.tile) % ntile);
    const int jt = min(J0 + kMxTile, L) - 1;
    if (!(j_first >= J0 && j_first <= jt) && (J0 - j_first + (J0 < j_first ? L : 0)) >= (int)n_lmt) return;
    const int half = (L - 1) / 2;
    const int nco = (int)split_chunks((uint32_t)L), nbo = (int)split_both_chunks((uint32_t)L);
    const int per = (nco + (int)be.lsplit - 1) / (int)be.lsplit;
    const int c_lo = (int)it.ks * per, c_hi = min(nco, c_lo + per);
    const int m0 = min(J0, L - 1 - J0), m1 = min(jt, L - 1 - jt);
    const int m_min = min(m0, m1), m_max = J0 <= half && half <= jt ? half : max(m0, m1);
    const int M_max = max(L - 1 - J0, jt);

    const int lane = (int)threadIdx.x;
    MxLane ln;
    ln.w = reinterpret_cast<const uint32_t *>(w.pivot) - kPad;
    ln.J32 = J0 >> 5;
    ln.r = lane & 15;
    ln.g = lane >> 4;
    ln.col = lane & 15;
    v4f acc[2 * kBlk];
#pragma unroll
    for (int i = 0; i < 2 * kBlk; ++i) acc[i] = v4f{0.f, 0.f, 0.f, 0.f};

    {
        // one neighbour: chunks o0 .. o1-1, those from f0 on past every m_j;
        // a tile across the middle has both sides and is all edge
        const int o0 = max(c_lo, (m_min + 1) >> 5), o1 = min(c_hi, (M_max >> 5) + 1);
        int f0 = o1, N = 0;
        if (jt <= half || J0 > half) {
            f0 = max(o0, (m_max + 32) >> 5);
            N = f0 < o1 ? (o1 - f0) / 4 : 0;
        }
        if (N > 0) {
            if (jt <= half) mx_one<true>(acc, ln, be.dig_one, f0, N);
            else            mx_one<false>(acc, ln, be.dig_one, f0, N);
            mx_edge<false>(acc, ln, be.dig_one, L, f0 + 4 * N, o1, nco);
        }
        mx_edge<false>(acc, ln, be.dig_one, L, o0, N > 0 ? f0 : o1, nco);
    }
    {
        uint32_t sw[kBlk];
#pragma unroll
        for (int b = 0; b < kBlk; ++b) sw[b] = ln.word(ln.J32 + b);
        // rows with s_j = -1 change sign (accumulator register q: row 4 g + q)
#pragma unroll
        for (int i = 0; i < 2 * kBlk; ++i) {
            const uint32_t bits = sw[i >> 1] >> (16 * (i & 1) + 4 * ln.g);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[i][q] = __uint_as_float(__float_as_uint(acc[i][q]) ^ ((bits << (31 - q)) & 0x80000000u));
            ln.S[i] = (uint32_t)-(int)((sw[i >> 1] >> (16 * (i & 1) + ln.r)) & 1u);
        }
    }
    const int b1 = min(c_hi, (m_max >> 5) + 1);
    if (c_lo < b1) {
        const int fb = min(b1, (m_min + 1) >> 5);
        const int N = fb > c_lo ? (fb - c_lo) / 4 : 0;
        if (N > 0) mx_both(acc, ln, be.dig_both, c_lo, N);
        mx_edge<true>(acc, ln, be.dig_both, L, c_lo + 4 * N, b1, nbo);
    }

    // digit column x weighs 32^x (in units of 8: the products are eighths);
    // the 16 columns of a row sit in 16 lanes: each stage adds a partner's half
    // of the values, until lane x of a group holds rows 4g .. 4g+3 of block x
    const double wcol = ldexp(8.0, 5 * ln.col);
    double v[32];
    {
        const bool up = ln.col & 8;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const double lo = (double)acc[i >> 2][i & 3] * wcol, hi = (double)acc[8 + (i >> 2)][i & 3] * wcol;
            v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, 8);
        }
    }
#pragma unroll
    for (int n = 16, d = 4; n >= 4; n >>= 1, d >>= 1) {
        const bool up = ln.col & d;
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = (up ? v[i + n] : v[i]) + __shfl_xor(up ? v[i] : v[i + n], d);
    }
    double *__restrict__ out = be.lpart + (size_t)it.ks * L;
    const int j = J0 + 16 * ln.col + 4 * ln.g;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (j + q < L) out[j + q] = v[q];
}

hipError_t launch_mx(const WalkDev *walks, const BatchEntry *batch, const EvalItem *items, uint32_t n_items,
                     hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    k_mx<<<n_items, 64, 0, s>>>(walks, batch, items);
    return hipGetLastError();
}

}  // namespace psl
