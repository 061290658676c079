// psl_split.hip -- the matrix evaluation of libpsl (gfx950).
//
// Eq. (5) summed over the neighbours of Algorithm 1, as products of 0/1
// matrices with coefficient vectors. For shift k with c = C_k and
// T(x) = T_alpha(|x|), the one-element flip of Section 3 gives
// C'_k = c + 4(x_R + x_L - 1) where both neighbours of j exist
// (k <= m_j = min(j, L-1-j)) and c + 2(2x - 1) where one does
// (m_j < k <= M_j = max(j, L-1-j)); x_R = 1 where s_j s_{j+k} = -1, x_L = 1
// where s_j s_{j-k} = -1. So
//   both: T(c) + XNOR(x_R, x_L) (T(c-4) - T(c)) + AND(x_R, x_L) (T(c+4) - T(c-4)),
//   one:  T(c-2) + x (T(c+2) - T(c-2)),
// and F_j is a sum of prefix sums of the constant parts plus three 0/1
// matrices times coefficient vectors. The matrix cores take the matrices as
// FP4 (a bit of the sequence is a nibble of 0.5 or 1.0 after one masking
// operation) and the coefficients as exact fixed-point numbers in kDig
// balanced base-32 digits, each exact in FP6: the FP32 accumulators then hold
// exact integers, and only the rounding of a coefficient to the quantum U
// enters. This file holds the per-step preparation (coefficients, digits,
// prefix sums, scale and path choice) and the matrix kernel.
#include "psl_chunks.h"
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
// byte i of out[q]; digits 14 and 15 are 0). v (below 2^68) in three 30-bit words
// of six digits; adding 16 to every 5-bit field (kBias) turns the balanced digits
// d in -16..15 into plain fields d + 16. The FP6 (E2M3) code of n/8, n = 0..16, is
// n; 0x20 is the sign. Odd shifts meet 1.0 in the FP4 matrix and v is their
// coefficient / U; even ones meet 0.5 and v is twice that. A shift's product is
// then at most 2 or 1 in size and a multiple of 1/16: sums over 699050 successive
// coefficients are exact in FP32, and no item has more (mx_splits).
constexpr int kBias = 0x21084210;

__device__ __forceinline__ uint32_t digit_codes(uint32_t v)
{
    const uint32_t neg = ~(v >> 4) & 0x01010101u;                          // d < 0
    const uint32_t mag = ((v ^ ((neg << 4) - neg)) & 0x0F0F0F0Fu) + neg;   // |d|
    return mag | (neg << 5);
}

__device__ __forceinline__ void split_digits(double v, uint32_t (&out)[4])
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
    for (int q = 0; q < 4; ++q) out[q] = digit_codes(out[q]);
}

// The step's preparation of a matrix walk, one block per segment of its shifts
// (2^shift of them, in tiles of 256), in one pass over C: the near-peak list
// (chunk_octs builds the same one), the digit records, and the prefix sums of
// T(|C_k-2|) - T(|C_k|) and T(|C_k+2|) - T(|C_k|) within the segment; their totals,
// and those of T(|C_k|), k_mx's first items turn into offsets (split_offsets). Blocks of the batch's other walks make
// the chunk sums of the table evaluation (k_chunks).
//
// A record holds one 32-shift chunk (shifts 32c .. 32c+31) of one coefficient:
// 16 columns (digits) of 32 FP6 codes, the first 12 bytes of each column, then
// the last 12 of each (kRecBytes); slot 8 r + q of a column is shift 32c + 4q + r,
// the order in which the matrix kernel's masks leave the bits of a word. The
// threads leave the codes of a tile in LDS (one word per shift and four
// columns); then one thread per (coefficient, chunk, four columns, half the
// slots) packs them. The values of a prefix have either sign, and each goes
// through about 16 roundings within a segment (split_offsets says what F's
// rounding comes to).
//
// One pass instead of three (chunk sums, coefficients, a serial scan per walk
// that took 0.94 ms of a step at L = 1048575 and 0.21 ms for 64 walks at
// L = 131071). Prefixes, 16 of the 40 bytes written per shift, are scanned and
// stored only in tiles that hold some candidate's m_j or M_j; the others' values
// stay in their threads until the next such tile. The next tile's C is loaded
// while a tile's digits are made, and the scans go through lane permutations of
// the vector units instead of LDS. Bound by vector issue, mostly the digits
// (about 75 operations per coefficient; 100 with codes of n/4 for even shifts in
// place of twice the coefficient), and by the writes: 64 walks at L = 131071,
// N_lmt = 6912, 184 -> 113 us (their 220 MB take 45 us), full neighbourhoods at
// 1024 walks 3.10 -> 2.46 ms (5.9 GB take 1.2 ms), one walk at L = 16383
// 7.2 -> 5.8 us.
constexpr int kPrepThreads = 256;
constexpr int kPrepStride = 36;         // words per chunk and four columns in LDS (32 and padding)

struct PrepLds {
    __align__(16) uint32_t codes[3][4][8 * kPrepStride];
    double tot[2][kPrepThreads / 64];   // the wavefronts' totals of a tile
    double acc[3][kPrepThreads / 64];   // and of the tiles before it without stored prefixes
};

// v plus the value that lane-permuting control CTRL brings from another lane (0
// where it brings none, or outside the rows of ROWS).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    return v + __longlong_as_double((long long)dpp_mov<CTRL, ROWS>(0, (uint64_t)__double_as_longlong(v)));
}
// Inclusive scan of v over the wavefront: within rows of 16 lanes by row shifts,
// then the rows before (row_bcast:15 into rows 1 and 3, row_bcast:31 into 2 and 3).
__device__ __forceinline__ double wave_scan(double v)
{
    v = dpp_add<0x111, 0xF>(v);
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);
    return dpp_add<0x143, 0xC>(v);
}

// Whether some element of a circular range of n elements from j0 lies in a .. b.
__device__ __forceinline__ bool range_hits(int L, int j0, int n, int a, int b)
{
    return (j0 >= a && j0 <= b) || a - j0 + (a < j0 ? L : 0) < n;
}

__device__ __forceinline__ void prep_segment(PrepLds &sh, const WalkDev &w, const BatchEntry &be,
                                             const double *__restrict__ T, uint32_t start, int n_lmt, int seg,
                                             int shift, double *segtot)
{
    const int L = (int)w.L;
    const int j0 = (int)((start + 1u) % (uint32_t)L);
    // exact: U is a power of two; twice the even shifts' coefficients (split_digits)
    const double inv = (threadIdx.x & 1 ? 1.0 : 2.0) / split_scale(T, w.psl_pivot);
    const int cut = w.psl_pivot - 8;                           // the near-peak cut
    const int nbo = (int)split_both_chunks((uint32_t)L), nco = (int)split_chunks((uint32_t)L);
    const int k_end = seg + 1 == (int)seg_count((uint32_t)L, (uint32_t)shift) ? 32 * nco : (seg + 1) << shift;
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    const int slot = (t >> 5) * kPrepStride + 8 * (t & 3) + ((t & 31) >> 2);
    double *__restrict__ pre = be.pre;
    const int32_t *__restrict__ C = w.C;
    double carry[3] = {0.0, 0.0, 0.0}, acc[3] = {0.0, 0.0, 0.0};
    bool kept = false;                                         // acc holds tiles without stored prefixes
    int next = C[min((seg << shift) + t, L - 1)];
    for (int k0 = seg << shift; k0 < k_end; k0 += kPrepThreads) {
        const int k = k0 + t;
        const bool in = k >= 1 && k < L;
        const bool both = (k0 >> 5) < nbo;                     // some chunk of the tile has both-neighbour shifts
        const int kz = min(k0 + kPrepThreads, L) - 1;
        // the tiles that the combine reads prefixes of: shifts m_j and M_j of a candidate
        const bool want = range_hits(L, j0, n_lmt, k0, kz) || range_hits(L, j0, n_lmt, L - 1 - kz, L - 1 - k0);
        const int c = in ? next : 0;
        next = C[min(k + kPrepThreads, L - 1)];
        const int a0 = c < 0 ? -c : c;
        const int a4 = c + 4 < 0 ? -(c + 4) : c + 4, m4 = c - 4 < 0 ? 4 - c : c - 4;
        const int a2 = c + 2 < 0 ? -(c + 2) : c + 2, m2 = c - 2 < 0 ? 2 - c : c - 2;
        const double t0 = T[a0], tp2 = T[a2], tm2 = T[m2], tp4 = T[a4], tm4 = T[m4];
        {
            const bool take = in && a0 >= cut;
            const uint64_t bal = __ballot(take);
            if (bal) {
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&be.near[0], (uint32_t)__popcll(bal));
                base = (uint32_t)__shfl((int)base, 0);
                const uint32_t q = base + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
                if (take && q < (uint32_t)kNearCap) be.near[1 + q] = (uint32_t)k;
            }
        }
        uint32_t d[4];
        split_digits(in ? (tp2 - tm2) * inv : 0.0, d);
#pragma unroll
        for (int q = 0; q < 4; ++q) sh.codes[2][q][slot] = d[q];
        if (both) {
            split_digits(in ? (tm4 - t0) * inv : 0.0, d);
#pragma unroll
            for (int q = 0; q < 4; ++q) sh.codes[0][q][slot] = d[q];
            split_digits(in ? (tp4 - tm4) * inv : 0.0, d);
#pragma unroll
            for (int q = 0; q < 4; ++q) sh.codes[1][q][slot] = d[q];
        }
        double v[2] = {in ? tm2 - t0 : 0.0, in ? tp2 - t0 : 0.0};
        acc[2] += in ? t0 : 0.0;
        if (!want) {
#pragma unroll
            for (int x = 0; x < 2; ++x) acc[x] += v[x];
            kept = true;
        } else {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                v[x] = wave_scan(v[x]);
                if (lane == 63) sh.tot[x][wave] = v[x];
            }
            if (kept) {
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const double a = wave_scan(acc[x]);
                    if (lane == 63) sh.acc[x][wave] = a;
                }
            }
        }
        __syncthreads();
        if (want) {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                if (kept) {
                    for (int q = 0; q < kPrepThreads / 64; ++q) carry[x] += sh.acc[x][q];
                    acc[x] = 0.0;
                }
                double off = carry[x];
                for (int q = 0; q < kPrepThreads / 64; ++q) {
                    if (q < wave) off += sh.tot[x][q];
                    carry[x] += sh.tot[x][q];
                }
                if (k < L) pre[(size_t)x * L + k] = off + v[x];
            }
            kept = false;
        }
        // task e: half e / 96 of the slots, coefficient (e / 32) % 3, chunk (e / 4) % 8, columns 4 (e % 4) .. +3
        const int h = t >= 96 ? 1 : 0, e = t - 96 * h;
        const int set = e >> 5, cc = (e >> 2) & 7, q = e & 3;
        const int ch = (k0 >> 5) + cc;
        if (t < 192 && ch < (set == 2 ? nco : nbo)) {
            const uint4 *src = reinterpret_cast<const uint4 *>(&sh.codes[set][q][cc * kPrepStride]) + 4 * h;
            uint32_t x[4][4];                              // [column][4 codes in 24 bits]
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                const uint4 u = src[y];
                // 16-bit lanes: columns 0 and 2, columns 1 and 3
                const uint32_t e01 = (u.x & 0x00FF00FFu) | ((u.y & 0x00FF00FFu) << 6);
                const uint32_t e23 = (u.z & 0x00FF00FFu) | ((u.w & 0x00FF00FFu) << 6);
                const uint32_t f01 = ((u.x >> 8) & 0x00FF00FFu) | (((u.y >> 8) & 0x00FF00FFu) << 6);
                const uint32_t f23 = ((u.z >> 8) & 0x00FF00FFu) | (((u.w >> 8) & 0x00FF00FFu) << 6);
                x[0][y] = (e01 & 0xFFFFu) | ((e23 & 0xFFFFu) << 12);
                x[1][y] = (f01 & 0xFFFFu) | ((f23 & 0xFFFFu) << 12);
                x[2][y] = (e01 >> 16) | ((e23 >> 16) << 12);
                x[3][y] = (f01 >> 16) | ((f23 >> 16) << 12);
            }
            uint8_t *rec = (set == 2 ? be.dig_one + (size_t)ch * kRecBytes
                                     : be.dig_both + ((size_t)ch * 2 + (size_t)set) * kRecBytes) +
                           kRecBytes / 2 * h;
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                uint32_t *o = reinterpret_cast<uint32_t *>(rec + 12 * (4 * q + y));
                o[0] = x[y][0] | (x[y][1] << 24);
                o[1] = (x[y][1] >> 8) | (x[y][2] << 16);
                o[2] = (x[y][2] >> 16) | (x[y][3] << 8);
            }
        }
        __syncthreads();                                   // the tile's codes and totals have been read
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) {                          // acc is 0 where the last tile took it
        const double a = wave_scan(acc[x]);
        if (lane == 63) sh.acc[x][wave] = a;
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 3; ++x)
        for (int q = 0; q < kPrepThreads / 64; ++q) carry[x] += sh.acc[x][q];
    if (t < 3) segtot[t] = t == 0 ? carry[0] : t == 1 ? carry[1] : carry[2];
}

__global__ __launch_bounds__(kPrepThreads) void k_prep(const WalkDev *walks, BatchEntry *batch, Tables tabs,
                                                       SegMap map, uint32_t *pend, uint32_t *tab, EvalCall call)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        eval_call(batch, call);
        if (pend) pend[0] = 0;          // the previous step's pending list has been consumed
        tab[0] = 0;
    }
    __shared__ union Lds {
        PrepLds prep;
        ChunkLds chunk;
        __device__ Lds() {}
    } sh;
    uint32_t b, seg;
    seg_of(map, blockIdx.x, b, seg);
    const BatchEntry be = batch[b];
    const WalkDev &w = walks[be.slot];
    if (be.lsplit)
        prep_segment(sh.prep, w, be, tabs.T[w.alpha], call.on ? call.start : be.fixed ? be.start : step_start(w),
                     (int)(be.fixed ? be.n_lmt : w.n_lmt), (int)seg, (int)map.shift, be.segoff + 3 * (size_t)seg);
    else
        chunk_segment(sh.chunk, be, w, tabs.T[w.alpha], map, seg);
}

// The segment totals of value array x of a matrix walk as the offsets of
// its segments (the sum of the segments before; in place; of x = 2 the walk's
// total), by one wavefront:
// each lane the totals of a run of segments, carried with Neumaier's
// compensation. With x = 0 also the step's scale and path choice: the matrix path is
// taken when the near-peak list holds the PSL (sparse form) and the
// quantization error, at most (L-1) U, is below 1e-14 of a lower bound of
// every neighbour's F (T(P-4) for the pivot's PSL P, and at least 1); a walk
// that does not take it is counted in *tab, which the table evaluation looks
// at first.
// FP64 rounding comes on top, of sums whose terms have both signs: with fewer than
// 64 rounded additions between a term and F_j, at most 64 x 2^-53 times the sum of
// the terms' absolute values, which is 1.7 F_j (alpha = 1) to 17 F_j (alpha = 16,
// L = 512 to 600, where 4 is most against |C_k|): 1.2e-13 of F_j at the most. Seen
// over L = 512 to 9001, random and low-PSL pivots, alpha = 1 to 16: 6.7e-16 (the
// table evaluation's F: 4.0e-15).
__device__ __forceinline__ void split_offsets(const WalkDev &w, const BatchEntry &be, const Tables &tabs, uint32_t *tab,
                                              int x, int lane)
{
    const int L = (int)w.L;
    if (lane == 0 && x == 0) {
        const double *__restrict__ T = tabs.T[w.alpha];
        const int P = w.psl_pivot;
        const double U = split_scale(T, P);
        const double flow = P > 4 ? T[P - 4] : 0.0;
        const bool exact_enough = (double)(L - 1) * U <= 1e-14 * (flow > 1.0 ? flow : 1.0);
        const bool sparse_psl = be.near[0] <= be.near_lim;
        const uint32_t use = exact_enough && sparse_psl ? 1u : 0u;
        be.ss->U = U;
        be.ss->use = use;
        if (!use) atomicAdd(tab, 1u);
    }
    const int n = (int)seg_count((uint32_t)L, be.seg_shift);
    const int per = (n + 63) / 64, lo = lane * per, hi = min(n, lo + per);
    double *__restrict__ v = be.segoff + x;
    double s = 0.0, c = 0.0;
#pragma unroll 4
    for (int i = lo; i < hi; ++i) nsum_add(s, c, v[3 * i]);
    // exclusive scan of the lanes' sums
    for (int d = 1; d < 64; d <<= 1) {
        const double os = __shfl_up(s, d), oc = __shfl_up(c, d);
        if (lane >= d) {
            nsum_add(s, c, os);
            c += oc;
        }
    }
    if (x == 2) {                       // T(|C_k|): the sum over all shifts
        if (lane == 63) be.ss->total = s + c;
        return;
    }
    double es = __shfl_up(s, 1), ec = __shfl_up(c, 1);
    if (lane == 0) es = ec = 0.0;
#pragma unroll 4
    for (int i = lo; i < hi; ++i) {
        const double a = v[3 * i];
        v[3 * i] = es + ec;
        nsum_add(es, ec, a);
    }
}

hipError_t launch_prep(const WalkDev *walks, BatchEntry *batch, uint32_t nb, const Tables &tabs,
                       const SegMap &map, int scan, uint32_t *pend, uint32_t *tab, const EvalCall &call,
                       hipStream_t s)
{
    if (map.shift < kSegShiftMin || map.shift > kSegShiftMax || map.nb != nb || !tab) return hipErrorInvalidValue;
    if (scan && (!map.tot || !map.tmax)) return hipErrorInvalidValue;
    if (nb == 0 || map.total == 0) return hipSuccess;
    SegMap m = map;
    if (!scan) m.tot = nullptr, m.tmax = nullptr;
    k_prep<<<map.total, kPrepThreads, 0, s>>>(walks, batch, tabs, m, pend, tab, call);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !scan) return e;
    return launch_seg_scan(walks, batch, m, s);
}

// ------------------------------------------------------- matrix kernel

// Items of one wavefront. A main item is (walk, tile of kMxTile = 256
// consecutive elements, k-split). The tile's elements J0 + 32 b + 16 p + r
// (b = 0..7, p = 0..1, r = 0..15) are the rows of 16 products per step of
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
// the record's slot order and digit scales match. Chunks past the range's end
// (N is rounded up) read a record of zeros.
//
// One-neighbour chunks come first, with the sequence's bits as they are (the
// matrix of a window is the same for all b + c, so it is masked once); then
// the rows with s_j = -1 change sign (their x is 1 minus the bit, and the
// combine takes T(c+2) as their constant part), and the both-neighbour chunks
// add XNOR (which s_j does not change) and AND of the bits times s_j: with the
// XNOR word masked, the AND word is one more operation. Both go into the same
// accumulators, which stay exact (split_digits). The digits and the sequence's
// words are loaded steps ahead, into rings: two wavefronts per SIMD (what the
// 64 accumulators and the windows leave) do not hide a load's latency.
//
// What bounds it: at 1024 walks of L = 131071 the matrix cores are busy 66 % of
// the time and vector issue 71 %; the 8.6e9 products alone take 76 ms (9.1 ns each
// per SIMD, measured with nothing beside them).
// 86.7 ms per step of that batch; with XOR and AND words masked one by one and
// digits loaded one step ahead 99.4 ms, as int8 digit products for the linear
// part and table lookups for the rest 228 ms. One walk at L = 1048575 6.19 ms
// per step (7.2 before), 64 walks at L = 131071 with N_lmt = 6912 419 us (464).
//
// Main items hold the chunks all of whose shifts have both neighbours, or one,
// for every row of the tile. The chunks between (those with some row's m_j,
// and in the tile across the middle all one-neighbour ones) are an edge item's,
// every row's shifts masked on either side of its m_j: the edge items of a
// tile, of 64 rows each (or one that takes them in turn, in launches that fill
// the GPU anyway), write partial sums of their own.
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v3i __attribute__((ext_vector_type(3), aligned(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr uint32_t kM0 = 0x11111111u, kM1 = 0x22222222u;
constexpr int kBlk = kMxTile / 32;       // pairs of 16-row blocks of a tile
constexpr int kPad = 256;                // words before the sequence that the word offsets start from

__device__ __forceinline__ v4f mx_mfma(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, v8i B, v4f acc)
{
    const v8i A = {(int)x0, (int)x1, (int)x2, (int)x3, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, B, acc, 4, 2, 0, 0, 0, 0);
}

// ~(a ^ b) & m, and (a ^ s) & y, one operation each: with y the former of two
// windows a and b, the latter is (a ^ s) & (b ^ s) & m
__device__ __forceinline__ uint32_t xnor_and(uint32_t a, uint32_t b, uint32_t m)
{
    return __builtin_amdgcn_bitop3_b32(a, b, m, 0x82);
}
__device__ __forceinline__ uint32_t signed_and(uint32_t a, uint32_t s, uint32_t y)
{
    return __builtin_amdgcn_bitop3_b32(a, s, y, 0x28);
}

// This lane's column of a digit record.
__device__ __forceinline__ v8i mx_rec(const uint8_t *__restrict__ base, uint32_t off)
{
    const v3i a = *(const __attribute__((address_space(1))) v3i *)(base + off);
    const v3i b = *(const __attribute__((address_space(1))) v3i *)(base + off + kRecBytes / 2);
    return v8i{a.x, a.y, a.z, b.x, b.y, b.z, 0, 0};
}

// v of the lane that mirrors this one within 2 d lanes of a row of 16 (d = 8, 4, 2,
// 1): a register move, where a butterfly's exchange goes through LDS (one walk at
// L = 16383: 10.0 us per launch, 9.2 with these in the main items; 1024 walks at
// L = 131071 no change. In the edge items as well the main items' loops came out
// 1.7 % slower).
__device__ __forceinline__ double mx_partner(double v, int d)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint64_t o = d == 8   ? dpp_mov<0x140, 0xF>(u, u)      // row_mirror
                       : d == 4 ? dpp_mov<0x141, 0xF>(u, u)      // row_half_mirror
                       : d == 2 ? dpp_mov<0x1B, 0xF>(u, u)       // quad_perm 3 2 1 0
                                : dpp_mov<0xB1, 0xF>(u, u);      // quad_perm 1 0 3 2
    return __longlong_as_double((long long)o);
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

// The both-neighbour products of chunks c0 .. c1-1, all of whose shifts are at
// most every row's m_j; record `zero` holds zeros.
__device__ __forceinline__ void mx_both(v4f (&acc)[2 * kBlk], const MxLane &ln, const uint8_t *__restrict__ dig, int c0,
                                        int c1, int zero)
{
    const int N = (c1 - c0 + 3) >> 2;
    const int cb = c0 + ln.g * N;
    const int ng = min(N, c1 - cb);                       // this lane's chunks
    const uint32_t offz = (uint32_t)zero * (2 * kRecBytes) + 12u * (uint32_t)ln.col;
    const uint32_t shr = (uint32_t)ln.r, shl = (uint32_t)(31 - ln.r);
    uint32_t R[8][2], R2[8][2], W[8][2], W2[8][2];        // right and left windows, and shifted by 2
    uint32_t rprev, lprev, rq[4], lq[4];
    v8i bx[4], ba[4];
    uint32_t off = (uint32_t)cb * (2 * kRecBytes) + 12u * (uint32_t)ln.col;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        bx[k] = mx_rec(dig, k < ng ? off : offz);
        ba[k] = mx_rec(dig + kRecBytes, k < ng ? off : offz);
        off += 2 * kRecBytes;
    }
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
    for (int s = 0; s < N;) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            if (s >= N) break;
            const uint32_t on = s + 2 < ng ? off : offz;
            bx[(v + 2) & 3] = mx_rec(dig, on);
            ba[(v + 2) & 3] = mx_rec(dig + kRecBytes, on);
            off += 2 * kRecBytes;
            const uint32_t rn = rq[v & 3], lw = lq[v & 3];
            rq[v & 3] = ln.word(ln.J32 + cb + s + 13);
            lq[v & 3] = ln.word(ln.J32 - cb - s - 6);
#pragma unroll
            for (int b = 0; b < kBlk; ++b) {
                const int u = (v + b) & 7, x = (b - v) & 7;
                uint32_t y[2][4];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    y[p][0] = xnor_and(R[u][p], W[x][p], kM0);
                    y[p][1] = xnor_and(R[u][p], W[x][p], kM1);
                    y[p][2] = xnor_and(R2[u][p], W2[x][p], kM0);
                    y[p][3] = xnor_and(R2[u][p], W2[x][p], kM1);
                    acc[2 * b + p] = mx_mfma(y[p][0], y[p][1], y[p][2], y[p][3], bx[v & 3], acc[2 * b + p]);
                }
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const uint32_t S = ln.S[2 * b + p];
                    acc[2 * b + p] =
                        mx_mfma(signed_and(R[u][p], S, y[p][0]), signed_and(R[u][p], S, y[p][1]),
                                signed_and(R2[u][p], S, y[p][2]), signed_and(R2[u][p], S, y[p][3]), ba[v & 3],
                                acc[2 * b + p]);
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

// The one-neighbour products (right or left side) of chunks c0 .. c1-1, all of
// whose shifts are past every row's m_j.
template <bool RIGHT>
__device__ __forceinline__ void mx_one(v4f (&acc)[2 * kBlk], const MxLane &ln, const uint8_t *__restrict__ dig, int c0,
                                       int c1, int zero)
{
    const int N = (c1 - c0 + 3) >> 2;
    const int cb = c0 + ln.g * N;
    const int ng = min(N, c1 - cb);
    const uint32_t offz = (uint32_t)zero * kRecBytes + 12u * (uint32_t)ln.col;
    const uint32_t sh = RIGHT ? (uint32_t)ln.r : (uint32_t)(31 - ln.r);
    uint32_t A[8][2][4];                    // the matrices of eight windows
    uint32_t prev, wq[4];
    v8i bq[8];                              // digits, loaded kAhead steps ahead
    constexpr int kAhead = 6;
    uint32_t off = (uint32_t)cb * kRecBytes + 12u * (uint32_t)ln.col;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
        bq[k] = mx_rec(dig, k < ng ? off : offz);
        off += kRecBytes;
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
    for (int s = 0; s < N;) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            if (s >= N) break;
            bq[(v + kAhead) & 7] = mx_rec(dig, s + kAhead < ng ? off : offz);
            off += kRecBytes;
            uint32_t wn = wq[v & 3];
            wq[v & 3] = ln.word(RIGHT ? ln.J32 + cb + s + 13 : ln.J32 - cb - s - 6);
#pragma unroll
            for (int b = 0; b < kBlk; ++b) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int i = 2 * b + p;
                    const uint32_t(&a)[4] = A[RIGHT ? (v + b) & 7 : (b - v) & 7][p];
                    acc[i] = mx_mfma(a[0], a[1], a[2], a[3], bq[v], acc[i]);
                }
            }
            if (!RIGHT) wn = __builtin_bitreverse32(wn);
            make(wn, prev, A[RIGHT ? v : 7 - v]);
            prev = wn;
            ++s;
        }
    }
}

// The edge of 64 rows (64 qd .. +63 of the tile): chunks ca .. ce-1, four
// consecutive ones per step; shifts up to a row's m_j go into the
// both-neighbour sums, the others into the one-neighbour sums of its side
// (right for j <= half; the sign of a row with s_j = -1 as FP4's sign bit).
// out: the tile's places.
__device__ __forceinline__ void mx_edge(const MxLane &ln, const BatchEntry &be, int L, int qd, int ca, int ce, int nco,
                                        int nbo, double *__restrict__ out)
{
    const int half = (L - 1) / 2;
    const uint32_t shr = (uint32_t)ln.r, shl = (uint32_t)(31 - ln.r);
    const int w0 = ln.J32 + 2 * qd;                       // the rows' first word
    v4f acc[4];
    uint32_t S[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
        S[i] = (uint32_t)-(int)((ln.word(w0 + (i >> 1)) >> (16 * (i & 1) + ln.r)) & 1u);
    }
#pragma unroll 1
    for (int c4 = ca; c4 < ce; c4 += 4) {
        const int c = c4 + ln.g;
        const bool both = c4 <= (half >> 5);              // some chunk of the step has both-neighbour shifts
        const uint32_t oo = (uint32_t)min(c, nco) * kRecBytes + 12u * (uint32_t)ln.col;
        const uint32_t ob = (uint32_t)min(c, nbo) * (2 * kRecBytes) + 12u * (uint32_t)ln.col;
        const v8i bo = mx_rec(be.dig_one, oo), bx = mx_rec(be.dig_both, ob), ba = mx_rec(be.dig_both + kRecBytes, ob);
        uint32_t x[3], y[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            x[i] = ln.word(w0 + c + i);
            y[i] = __builtin_bitreverse32(ln.word(w0 - c - 1 + i));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = 32 * (w0 + (i >> 1)) + 16 * (i & 1) + ln.r;
            const int n = min(32, max(0, min(j, L - 1 - j) + 1 - 32 * c));     // shifts 32c + t, t < n: both
            const uint32_t low = n > 0 ? 0xFFFFFFFFu >> (32 - n) : 0u;
            const uint32_t VB = c < ce ? low : 0u, VO = c < ce ? ~low : 0u;
            const uint32_t R = __builtin_amdgcn_alignbit(x[(i >> 1) + 1], x[i >> 1], shr + 16u * (i & 1));
            const uint32_t W = __builtin_amdgcn_alignbit(y[i >> 1], y[(i >> 1) + 1], shl - 16u * (i & 1));
            const uint32_t q = (j <= half ? R : W) & VO, q2 = q >> 2, sg = S[i] & 0x88888888u;
            acc[i] = mx_mfma((q & kM0) | sg, (q & kM1) | sg, (q2 & kM0) | sg, (q2 & kM1) | sg, bo, acc[i]);
            if (both) {
                const uint32_t e = xnor_and(R, W, VB), e2 = e >> 2;
                acc[i] = mx_mfma(e & kM0, e & kM1, e2 & kM0, e2 & kM1, bx, acc[i]);
                const uint32_t t = signed_and(R, S[i], e), t2 = t >> 2;
                acc[i] = mx_mfma(t & kM0, t & kM1, t2 & kM0, t2 & kM1, ba, acc[i]);
            }
        }
    }
    // as in k_mx, down to one value per lane: register col % 4 of block col / 4
    const double wcol = ldexp(8.0, 5 * ln.col);
    double v[8];
    {
        const bool up = ln.col & 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const double lo = (double)acc[i >> 2][i & 3] * wcol, hi = (double)acc[2 + (i >> 2)][i & 3] * wcol;
            v[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, 8);
        }
    }
#pragma unroll
    for (int n = 4, d = 4; n >= 1; n >>= 1, d >>= 1) {
        const bool up = ln.col & d;
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = (up ? v[i + n] : v[i]) + __shfl_xor(up ? v[i] : v[i + n], d);
    }
    // (stored without the test, rows past L - 1 harm nothing, but the main items'
    // loops came out 2 % slower: 1024 walks at L = 131071 86.2 -> 87.8 ms)
    const int row = 64 * qd + 16 * (ln.col >> 2) + 4 * ln.g + (ln.col & 3);
    if (32 * ln.J32 + row < L) out[row] = v[0];
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx(
    const WalkDev *__restrict__ walks, const BatchEntry *__restrict__ batch, const EvalItem *__restrict__ items,
    Tables tabs, uint32_t *tab)
{
    const EvalItem it = items[blockIdx.x];
    if (it.walk == kMxNoWalk) return;
    const BatchEntry be = batch[it.walk];
    const WalkDev &w = walks[be.slot];
    if (it.tile == kMxOffsets) {        // the walk's offsets and path choice, beside the products
        if (be.lsplit) split_offsets(w, be, tabs, tab, (int)it.ks, (int)threadIdx.x);
        else if (threadIdx.x == 0 && it.ks == 0) atomicAdd(tab, 1u);
        return;
    }
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
    const int m0 = min(J0, L - 1 - J0), m1 = min(jt, L - 1 - jt);
    const int m_min = min(m0, m1), m_max = J0 <= half && half <= jt ? half : max(m0, m1);
    const int M_max = max(L - 1 - J0, jt);
    // chunks: both neighbours [0, fb), one [f0, oe), between them the edge
    const bool one_side = jt <= half || J0 > half;
    const int fb = (m_min + 1) >> 5, oe = (M_max >> 5) + 1, f0 = one_side ? min(oe, (m_max + 32) >> 5) : oe;

    const int lane = (int)threadIdx.x;
    MxLane ln;
    ln.w = reinterpret_cast<const uint32_t *>(w.pivot) - kPad;
    ln.J32 = J0 >> 5;
    ln.r = lane & 15;
    ln.g = lane >> 4;
    ln.col = lane & 15;
    if (it.ks >= be.lsplit) {           // edge item: its part of the tile's rows
        const int part = (int)(it.ks - be.lsplit);
        double *out = be.lpart + (size_t)be.lsplit * be.lrow + (size_t)kMxTile * it.tile;
        for (int qd = it.pad ? 0 : part; qd < (it.pad ? 4 : part + 1); ++qd)
            if (J0 + 64 * qd < L) mx_edge(ln, be, L, qd, fb, f0, nco, nbo, out);
        return;
    }
    // the k-split: an equal part of the tile's work, a both-neighbour chunk
    // (two products of 26 cycles each on the vector units) counting as three
    // one-neighbour chunks
    const int total = 3 * fb + (oe - f0);
    const int per = (total + (int)be.lsplit - 1) / (int)be.lsplit;
    const int p0 = (int)it.ks * per, p1 = p0 + per;
    const int b0 = min(fb, (p0 + 2) / 3), b1 = min(fb, (p1 + 2) / 3);
    const int o0 = min(oe, f0 + max(0, p0 - 3 * fb)), o1 = min(oe, f0 + max(0, p1 - 3 * fb));
    v4f acc[2 * kBlk];
#pragma unroll
    for (int i = 0; i < 2 * kBlk; ++i) acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
    if (o0 < o1) {
        if (jt <= half) mx_one<true>(acc, ln, be.dig_one, o0, o1, nco);
        else            mx_one<false>(acc, ln, be.dig_one, o0, o1, nco);
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
    if (b0 < b1) mx_both(acc, ln, be.dig_both, b0, b1, nbo);

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
            v[i] = (up ? hi : lo) + mx_partner(up ? lo : hi, 8);
        }
    }
#pragma unroll
    for (int n = 16, d = 4; n >= 4; n >>= 1, d >>= 1) {
        const bool up = ln.col & d;
#pragma unroll
        for (int i = 0; i < n; ++i) v[i] = (up ? v[i + n] : v[i]) + mx_partner(up ? v[i] : v[i + n], d);
    }
    double *__restrict__ out = be.lpart + (size_t)it.ks * be.lrow + (size_t)kMxTile * it.tile + 16 * ln.col + 4 * ln.g;
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = v[q];          // rows past L - 1: not read
}

hipError_t launch_mx(const WalkDev *walks, const BatchEntry *batch, const EvalItem *items, uint32_t n_items,
                     const Tables &tabs, uint32_t *tab, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    k_mx<<<n_items, 64, 0, s>>>(walks, batch, items, tabs, tab);
    return hipGetLastError();
}

}  // namespace psl
