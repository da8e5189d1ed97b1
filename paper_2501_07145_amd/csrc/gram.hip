// Linear Gram of primal features, K = PhiX PhiY^T (Sec. 1: the Gram matrix of the low-rank feature map is the
// matrix of inner products of the features); the same kernels project the increments of RFSF-TRP.
//
// Arithmetic. The operands are 32-bit, and so are the products and sums, but the products run on the bfloat16
// matrix instructions, which are 16 times as fast as the 32-bit ones: a float is the sum of three bfloat16
// numbers, x = hi + mid + lo (each the rounding of what the ones before it leave over, 8 significand bits each,
// 24 in all: nothing is lost), a product of two bfloat16 numbers is exact in 32 bits, and of the nine products of
// a pair of floats the six largest are added up in the 32-bit accumulators, smallest first. The three that are
// left out (mid*lo, lo*mid, lo*lo) are together below 2^-24 of the product, as much as rounding it to 32 bits
// may cost (numbers below about 2^-114 lose their last bits, whose bfloat16 would be too small: 1e-7 of a product with 2^-116,
// 1.3e-5 with 2^-123). Measured against 64 bits, the sums are a third closer than with v_mfma_f32_32x32x2f32, which rounds
// after every product: relative error of K 1.2e-6 against 1.95e-6 on 10000 x 10000 x 5121, 1.8e-6 against 2.8e-6
// on 50000 x 5000 x 10241. The instructions round downwards, though, whatever the sign of the sum: of products with 128
// columns the error averages -1.1e-8 of their root mean square (its own 5.5e-8; v_mfma_f32_32x32x2f32: 1.8e-7, average zero).
// RFSF-TRP adds products up over time, one row each, and there such a part grows with the number of rows
// instead of its root: `FLIP`.
// Infinite operands, and finite ones that round to an infinite bfloat16, would turn into NaN in the split
// (inf - inf): entries that come out as NaN without a NaN in their rows are computed again in 32 bits (settle_nan).
//
// Large tiles of 128 columns and more take two terms of 16-bit floating point instead, x s = hi + lo with a power of two s for
// each row, and three products (lo*hi, hi*lo, hi*hi): half the matrix instructions. The two terms hold 11 significand
// bits each and the sign of the second one more; what they leave over is one unit of the last place of a float for a
// quarter of the numbers, nothing for the others, and lo*lo is left out (4e-8 of a product, root mean square). Both are less
// than what adding up loses, where half as many additions round: relative error of K against 64 bits, three terms and two, 1.63e-7
// and 1.43e-7 with 128 columns of normal numbers, 3.0e-7 and 2.3e-7 with 400, 5.3e-7 and 4.6e-7 with 1001 of features, 1.07e-6 and
// 9.8e-7 with 5121, 1.5e-6 and 1.4e-6 with 10241 (mean error -2.37e-7 and -2.31e-7 of 5121 columns). The range of these
// numbers is narrow. A row's scale brings the largest of about 48 of its numbers to 2^9 .. 2^10 (32 at its beginning, which are in LDS
// anyway, and four at each of four places spread over it): numbers down to 2^-12 of that keep both terms in full, smaller ones an
// error of 2^-25 (scaled); numbers more than 64 times as large overflow, which shows as NaN, and the tile is computed
// again with three terms, as are, from the outset, tiles with rows beyond 2^-91 .. 2^109 or with rows that are zero wherever they are
// sampled but not everywhere (a third of 7494 rows zero, 1001 columns: 267 -> 321 us for looking through them).
// Such tiles cost what both ways cost: 10000 rows with themselves, 5121 columns 2.12 ms, with three terms from the outset in every
// tile 3.63, with one number 2^20 times the others in one row 3.40, in a row of every tile 5.83 (a kernel of three terms alone 2.97;
// 1025 columns 0.47, 0.86, 0.72 and 1.17).
// The error of small numbers is no error of their products if those of the large ones are part of the same sum, and without limit if
// the large ones meet zeros. So the sum of |a b| over the sampled columns is computed for every pair of rows, and a tile in which one
// of them is below 2^15 takes three terms. What small numbers add to the error is K 2^-25 (2^10 + 2^10) at most, K / 32 units of
// 2^-24 times that sum, and 2 K units if numbers that were not sampled are up to 2^16 and all meet small ones. (Features, raw
// and normalised, of walks and of noise, and increments against normal numbers: 2^16.8 and more.)
#include "rfsf_internal.h"
#include <algorithm>
#include <type_traits>

namespace rfsf {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

// FLIP: the rows of A for which this is the sign bit enter negated, and so do the results that they give, so that rounding
// downwards comes out as rounding upwards for half of the rows: whole blocks of 32, the edge of the smallest tile, so that a
// scalar register holds the sign. Blocks are chosen by the top bit of their number times an irrational fraction of 2^32
// (the golden section), which takes half of the blocks of every stretch and of every arithmetic progression in it.
__device__ __forceinline__ uint32_t flip_of_row(int64_t row) { return ((uint32_t)(row >> 5) * 0x9e3779b1u) & 0x80000000u; }
__device__ __forceinline__ void flip(float (&x)[8], uint32_t sign)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(__float_as_uint(x[e]) ^ sign);
}

struct Split8 { bf16x8 hi, mid, lo; };
__device__ __forceinline__ uint32_t round_pair(float a, float b)          // v_cvt_pk_bf16_f32
{
    const floatx2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// The three terms of eight consecutive numbers of a row: 44 vector instructions for the 8 floats of a lane.
__device__ __forceinline__ Split8 split8(const float (&x)[8])
{
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x[2 * i], b = x[2 * i + 1];
        h[i] = round_pair(a, b);
        const float ra = a - __uint_as_float(h[i] << 16), rb = b - __uint_as_float(h[i] & 0xffff0000u);
        m[i] = round_pair(ra, rb);
        const float sa = ra - __uint_as_float(m[i] << 16), sb = rb - __uint_as_float(m[i] & 0xffff0000u);
        l[i] = round_pair(sa, sb);
    }
    return {__builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3])),
            __builtin_bit_cast(bf16x8, make_uint4(m[0], m[1], m[2], m[3])),
            __builtin_bit_cast(bf16x8, make_uint4(l[0], l[1], l[2], l[3]))};
}

__device__ __forceinline__ floatx16 mfma(const bf16x8 &a, const bf16x8 &b, const floatx16 &c)   // 32 x 32, 16 columns of K
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma(const bf16x8 &a, const bf16x8 &b, const floatx4 &c)     // 16 x 16, 32 columns of K
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// acc[v] += a * b[v] for one block row and NB block columns.
template <int NB, typename Acc>
__device__ __forceinline__ void mfma_split(const Split8 &a, const Split8 (&b)[NB], Acc (&acc)[NB])
{
#define RFSF_TERM(X, Y)                                                                                        \
    _Pragma("unroll") for (int v = 0; v < NB; ++v) acc[v] = mfma(a.X, b[v].Y, acc[v])
    RFSF_TERM(lo, hi);
    RFSF_TERM(hi, lo);
    RFSF_TERM(mid, mid);
    RFSF_TERM(mid, hi);
    RFSF_TERM(hi, mid);
    RFSF_TERM(hi, hi);
#undef RFSF_TERM
}

// Two terms: eight consecutive numbers of a row times its scale, and the three products, smallest first.
struct Half8 { uint32_t hi[4], lo[4]; };
__device__ __forceinline__ void split_pair(Half8 &f, int i, float a, float b, float scale)
{
    const floatx2 v = {a * scale, b * scale};
    const halfx2 hi = __builtin_convertvector(v, halfx2);                                                // v_cvt_pk_f16_f32
    const floatx2 rest = {fmaf(a, scale, -(float)hi[0]), fmaf(b, scale, -(float)hi[1])};                 // v_fma_mix_f32
    f.hi[i] = __builtin_bit_cast(uint32_t, hi);
    f.lo[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, halfx2));
}
// Magnitudes of eight consecutive numbers of a row times its scale, or `zero` for those of a row without any.
__device__ __forceinline__ halfx8 magnitudes(const float (&x)[8], float scale, float zero)
{
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const floatx2 pair = {fmaf(fabsf(x[2 * i]), fabsf(scale), zero), fmaf(fabsf(x[2 * i + 1]), fabsf(scale), zero)};
        v[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, halfx2));
    }
    return __builtin_bit_cast(halfx8, make_uint4(v[0], v[1], v[2], v[3]));
}
__device__ __forceinline__ floatx16 product(int k, const Half8 &a, const Half8 &b, const floatx16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, k == 0 ? a.lo : a.hi),
                                                  __builtin_bit_cast(halfx8, k == 1 ? b.lo : b.hi), c, 0, 0, 0);
}

// One operand pair of a launch: row-major, K-contiguous. Batched launches (one product per level of RFSF-TRP) add
// blockIdx.y times the steps.
struct GramArgs {
    const float *A, *B;
    float *C;
    int64_t Nx, Ny, K, lda, ldb, ldc;
    int64_t step_a, step_b, step_c;
};

// Stores four consecutive rows i .. i+3 of column j, of a block with this sign (FLIP); `mirror` also writes their mirror image, row j. `diagonal`: the
// tile meets the diagonal, and only what lies on or above it counts.
template <bool FLIP>
__device__ __forceinline__ void store_quad(const GramArgs &g, float *C, int64_t i, int64_t j, float (&v)[4], bool mirror,
                                           bool diagonal, bool vec_mirror, uint32_t sign)
{
    if (j >= g.Ny) return;
    if constexpr (FLIP) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(__float_as_uint(v[e]) ^ sign);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (i + e < g.Nx && (!diagonal || i + e <= j)) C[(i + e) * g.ldc + j] = v[e];
    }
    if (!mirror) return;
    float *dst = C + j * g.ldc + i;
    if (!diagonal && vec_mirror && i + 3 < g.Nx) {
        *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < g.Nx && (!diagonal || i + e < j)) dst[e] = v[e];
    }
}

// True if the row of K numbers holds a NaN. The whole wavefront, like the next two.
__device__ __forceinline__ bool holds_nan(const float *row, int64_t K)
{
    const int lane = threadIdx.x & 63;
    for (int64_t k0 = lane; k0 - lane < K; k0 += 256) {
        bool nan = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float x = row[min(k0 + 64 * u, K - 1)];
            nan |= x != x;
        }
        if (__ballot(nan)) return true;
    }
    return false;
}
__device__ __forceinline__ float wave_dot(const float *a, const float *b, int64_t K)
{
    float s = 0.f;
    for (int64_t k = threadIdx.x & 63; k < K; k += 64) s = fmaf(a[k], b[k], s);
#pragma unroll
    for (int o = 32; o > 0; o /= 2) s += __shfl_xor(s, o);
    return s;
}
// Goes over the ROWS x W entries from (i0, j0) on that this wavefront has stored, with NaN among them (told from the sum of
// a lane's entries: one addition each in an epilogue that is bound by its own length). An entry of a row
// that holds a NaN is one; the others owe theirs to the split and are summed up again. The rows' last columns are looked at
// first, all rows at a time, and a row's other columns only if that leaves it open. (10000 rows with themselves, 5121
// columns, one of them NaN: 2.97 ms against 2.94 without; 2500 rows, 1025 columns 78 us against 71, all NaN 95, where summing
// every such entry up again by itself, K dependent steps of a thread, took 1.3 and 5.6 ms.)
template <int W, int ROWS, bool SYM>
__device__ __forceinline__ void settle_nan(const GramArgs &g, const float *A, const float *B, float *C, int64_t i0, int64_t j0,
                                           bool diagonal)
{
    static_assert(ROWS <= 64 && W <= 64 && 64 % W == 0, "a bit for every row");
    constexpr int PER = 64 / W, LOADS = ROWS / PER < 8 ? ROWS / PER : 8;      // rows per load; loads in flight
    static_assert(ROWS % (PER * LOADS) == 0, "");
    const int lane = threadIdx.x & 63;
    const bool row_ok = lane < ROWS && i0 + lane < g.Nx, col_ok = lane < W && j0 + lane < g.Ny;
    const float last_a = row_ok ? A[(i0 + lane) * g.lda + g.K - 1] : 0.f, last_b = col_ok ? B[(j0 + lane) * g.ldb + g.K - 1] : 0.f;
    const uint64_t nan_rows = __ballot(last_a != last_a);
    uint64_t nan_cols = __ballot(last_b != last_b), known = nan_cols;
    __threadfence_block();                                   // the entries other lanes have stored
    for (int r0 = 0; r0 < ROWS; r0 += PER * LOADS) {
        float v[LOADS];
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int64_t i = i0 + r0 + PER * u + lane / W, j = j0 + lane % W;
            v[u] = i < g.Nx && j < g.Ny && (!diagonal || i <= j) ? C[i * g.ldc + j] : 0.f;
        }
#pragma unroll 1
        for (int r = r0; r < r0 + PER * LOADS; ++r) {
            bool mine = false;
#pragma unroll
            for (int u = 0; u < LOADS; ++u) mine |= u == (r - r0) / PER && v[u] != v[u];
            uint64_t open = __ballot(mine) >> (W * ((r - r0) % PER));
            if (W < 64) open &= ((uint64_t)1 << (W % 64)) - 1;
            open &= ~nan_cols;
            if (open == 0 || (nan_rows >> r & 1) != 0) continue;
            const int64_t i = i0 + r;
            const float *a = A + i * g.lda;
            if (holds_nan(a, g.K)) continue;
            while (open != 0) {
                const int c = __ffsll((unsigned long long)open) - 1;
                const uint64_t bit = (uint64_t)1 << c;
                const int64_t j = j0 + c;
                const float *b = B + j * g.ldb;
                open &= ~bit;
                if ((known & bit) == 0) {
                    known |= bit;
                    if (holds_nan(b, g.K)) nan_cols |= bit;
                }
                if ((nan_cols & bit) != 0) continue;
                const float s = wave_dot(a, b, g.K);
                if (lane == 0) {
                    C[i * g.ldc + j] = s;
                    if (SYM) C[j * g.ldc + i] = s;
                }
            }
        }
    }
}

// Consecutive workgroup ids go to the eight XCDs in turn, each with an L2 of its own: tile `id` of an order that
// keeps neighbours close, cut into eight contiguous pieces.
__device__ __forceinline__ int64_t rank_of_block(int64_t tiles)
{
    const int64_t per = (tiles + 7) / 8;
    return (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
}
unsigned xcd_grid(int64_t tiles) { return (unsigned)((tiles + 7) / 8 * 8); }

// ---------------------------------------------------------------------------------------------------------------
// Small problems: too few tiles to fill the chip with large ones, time is latency. Tile (16 NR) x (16 NR), NW
// wavefronts that share out the columns of K in steps of 32, step s to wavefront s mod NW, and work without any
// barrier: each loads its fragments from global memory straight into registers, one step ahead. The partial tiles are
// added through LDS at the end in a fixed order. 16 x 16 blocks (v_mfma_f32_16x16x32_bf16: lane l holds columns
// 8 (l / 16) .. + 7 of row l mod 16) rather than 32 x 32: a 16-byte load then touches 16 rows instead of 32, and what
// bounds the loop is one row (cache line) per cycle of the CU's address unit, 37 cycles a load with 32 rows.
// Any row stride and alignment (the loads need four bytes).
// Registers are bounded so that a CU holds two workgroups of four wavefronts or of 32 x 32 tiles (with one, 3000 rows with
// themselves, 1025 columns, take 115 us instead of 90).
struct __attribute__((packed, aligned(4))) Float4u { float x, y, z, w; };

template <int NR, int NW, bool SYM, bool FLIP>
__global__ __launch_bounds__(64 * NW, NR <= 2 ? 4 : 2) void gram_small(GramArgs g, int64_t tiles, int64_t tiles_j)
{
    constexpr int NH = NW / 2;                  // wavefronts that keep a partial tile in LDS (NR: 16-row blocks per side)
    __shared__ floatx4 red[NH * NR * NR * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quarter = lane >> 4, col = lane & 15;
    const int64_t rank = rank_of_block(tiles);
    if (rank >= tiles) return;
    int64_t bi, bj;
    if (SYM) {          // column by column of the upper triangle: column c holds rows 0 .. c
        bj = (int64_t)((sqrt(8.0 * (double)rank + 1.0) - 1.0) * 0.5);
        while (bj * (bj + 1) / 2 > rank) --bj;
        while ((bj + 1) * (bj + 2) / 2 <= rank) ++bj;
        bi = rank - bj * (bj + 1) / 2;
    } else {
        bi = rank / tiles_j;
        bj = rank - bi * tiles_j;
    }
    const float *A = g.A + blockIdx.y * g.step_a, *B = g.B + blockIdx.y * g.step_b;
    float *C = g.C + blockIdx.y * g.step_c;
    const int64_t i0 = bi * (16 * NR), j0 = bj * (16 * NR);
    // rows beyond the matrix are redirected to its last one: what they contribute is never stored
    const float *p[2 * NR];
    uint32_t sign[NR];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        sign[t] = __builtin_amdgcn_readfirstlane(flip_of_row(i0 + 16 * t));
        p[t] = A + min(i0 + 16 * t + col, g.Nx - 1) * g.lda + 8 * quarter;
        p[NR + t] = B + min(j0 + 16 * t + col, g.Ny - 1) * g.ldb + 8 * quarter;
    }
    floatx4 acc[NR][NR];
#pragma unroll
    for (int a = 0; a < NR; ++a)
#pragma unroll
        for (int b = 0; b < NR; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    float raw[2 * NR][8];
    auto fetch = [&](int64_t step) {
#pragma unroll
        for (int t = 0; t < 2 * NR; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const Float4u v = *reinterpret_cast<const Float4u *>(p[t] + 32 * step + 4 * c);
                raw[t][4 * c] = v.x;
                raw[t][4 * c + 1] = v.y;
                raw[t][4 * c + 2] = v.z;
                raw[t][4 * c + 3] = v.w;
            }
    };
    auto split_all = [&](Split8 (&a)[NR], Split8 (&b)[NR]) {
#pragma unroll
        for (int t = 0; t < NR; ++t) {
            if (FLIP) flip(raw[t], sign[t]);
            a[t] = split8(raw[t]);
            b[t] = split8(raw[NR + t]);
        }
    };
    auto multiply = [&](const Split8 (&a)[NR], const Split8 (&b)[NR]) {
#pragma unroll
        for (int t = 0; t < NR; ++t) mfma_split<NR>(a[t], b, acc[t]);
    };
    const int64_t nfull = g.K / 32;
    const int rest = (int)(g.K - 32 * nfull);
    if (wave < nfull) fetch(wave);
    for (int64_t s = wave; s < nfull; s += NW) {
        Split8 a[NR], b[NR];
        split_all(a, b);
        if (s + NW < nfull) fetch(s + NW);
        multiply(a, b);
    }
    if (rest != 0 && wave == (int)(nfull % NW)) {      // the columns left over, number by number
#pragma unroll
        for (int t = 0; t < 2 * NR; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e) raw[t][e] = 8 * quarter + e < rest ? p[t][32 * nfull + e] : 0.f;
        Split8 a[NR], b[NR];
        split_all(a, b);
        multiply(a, b);
    }
    // partial tiles: the second half of the wavefronts to the first, then all of those by everybody
    auto slot = [&](int w, int blk) { return (w * NR * NR + blk) * 64 + lane; };
    if (wave >= NH) {
#pragma unroll
        for (int b = 0; b < NR * NR; ++b) red[slot(wave - NH, b)] = acc[b / NR][b % NR];
    }
    __syncthreads();
    if (wave < NH) {
#pragma unroll
        for (int b = 0; b < NR * NR; ++b) red[slot(wave, b)] += acc[b / NR][b % NR];
    }
    __syncthreads();
    // result layout of a 16x16 block: lane l holds column l mod 16 and rows 4 (l / 16) + 0 .. 3
    const bool vec_mirror = g.ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0;
    for (int b = wave; b < NR * NR; b += NW) {
        floatx4 sum = red[slot(0, b)];
#pragma unroll
        for (int w = 1; w < NH; ++w) sum += red[slot(w, b)];
        float v[4] = {sum[0], sum[1], sum[2], sum[3]};
        const int64_t ib = i0 + (b / NR) * 16, jb = j0 + (b % NR) * 16;
        const float any = v[0] + v[1] + v[2] + v[3];
        store_quad<FLIP>(g, C, ib + 4 * quarter, jb + col, v, SYM, SYM && bi == bj, vec_mirror,
                         __builtin_amdgcn_readfirstlane(flip_of_row(ib)));
        if (__ballot(any != any)) settle_nan<16, 16, SYM>(g, A, B, C, ib, jb, SYM && bi == bj);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Up to eight rows on one side (a request against stored features): a wavefront takes two rows of the other side (four of
// kThinMany and more, against more than four) and all of the few, four columns of each per lane and step, adds up in plain 32-bit
// multiply-adds and then over its lanes; of fewer than kThinSplit rows its workgroup's wavefronts share out the columns (SPLIT). What
// bounds it is reading the long side once, and for hundreds of rows its latency; tiles leave most of the chip without work and pad the
// short side to 16 or 32.
// In tiles of 32 x 32 and more and here, us a call: 1 x 1000, 1025 columns 8.1 and 6.5, 1 x 30, 5121 columns 24 and 6.4, 3 x 40, 10241
// columns 48 and 7.2, 1 x 10000, 5121 columns 76 and 36 (5.7 TB/s), 8 x 10000 80 and 62. Errors against 64 bits, of a row's length times
// another's: 4.7e-9 and 4.5e-9 with 320 columns, 5.1e-9 and 2.7e-9 with 1025, 5.3e-9 and 2.7e-9 with 2049, but 4.5e-9 and 5.7e-9 with
// 192, hence kThinColumns.
constexpr int kFew = 8, kThinWaves = 4;
constexpr int64_t kThinColumns = 320, kThinWide = 2048, kThinSplit = 2048, kThinMany = 8192;
// Where it is the faster way: for one and two rows everywhere; for more it takes as many loads as there are rows, while a tile's cost
// hardly grows. 768 workgroups run at once, the rows of 6144 (12288 of those of four per wavefront), and up to 8192 rows tiles are of 32 x 32,
// one per CU, up to 16384 of 64 x 64. (Tiles and here, us in a graph: 8 x 2047, 513 columns 6.4 and 7.8, 901 8.4 and 8.1, 8 x 300, 513 6.3
// and 6.0; 8 x 4097, 2049 14.6 and 11.9, 5 x 5500, 4097 23.3 and 21.9, 8 x 5500, 3001 18.3 and 19.6; 8 x 7000, 2049 14.8 and 18.3, 5121 30
// and 39, 10241 69 and 103; 8 x 10000, 2049 29 and 23; 8 x 14000, 2049 30.3 and 31.2, 2561 36.3 and 35.0; 4 x 8192, 7169 38.7 and 38.4,
// and past the last-level cache 8193 45 and 47, 10241 72 and 78; 4 x 6000, 10241 52 and 41.)
bool thin_pays(int64_t few, int64_t many, int64_t ncols)
{
    if (few <= 2 || ncols < kThinColumns) return ncols >= kThinColumns;
    if (few <= 4) return many <= 6144 || many > 8192 || 4 * many * ncols <= (int64_t)256 << 20;
    if (many < kThinSplit) return ncols >= 576 + many / 7;
    if (many <= 8192) return ncols >= kThinWide && many <= (few <= 6 ? 6144 : 4096);
    return ncols >= (many > 12288 && many <= 16384 ? 2304 : kThinWide);
}
template <int FEW, int ROWS, bool SPLIT>
__global__ __launch_bounds__(64 * kThinWaves) void gram_thin(const float *__restrict__ few, const float *__restrict__ many, float *__restrict__ C,
                                                             int64_t n_few, int64_t n_many, int64_t K, int64_t ld_few, int64_t ld_many,
                                                             int64_t step_few, int64_t step_many)
{
    __shared__ float part[SPLIT ? kThinWaves : 1][ROWS * FEW];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t first = (SPLIT ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * kThinWaves + wave) * ROWS;
    if (first >= n_many) return;
    const float *a[FEW], *b[ROWS];                           // rows that do not exist are the last one, and not stored
#pragma unroll
    for (int r = 0; r < FEW; ++r) a[r] = few + min((int64_t)r, n_few - 1) * ld_few;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) b[r] = many + min(first + r, n_many - 1) * ld_many;
    float acc[ROWS][FEW];
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int j = 0; j < FEW; ++j) acc[i][j] = 0.f;
    const int64_t whole = K / 256 * 256;
#pragma unroll 2
    for (int64_t k = 4 * lane + (SPLIT ? 256 * wave : 0); k < whole; k += SPLIT ? 256 * kThinWaves : 256) {
        Float4u x[ROWS], y[FEW];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) x[i] = *reinterpret_cast<const Float4u *>(b[i] + k);
#pragma unroll
        for (int j = 0; j < FEW; ++j) y[j] = *reinterpret_cast<const Float4u *>(a[j] + k);
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
#pragma unroll
            for (int j = 0; j < FEW; ++j)
                acc[i][j] = fmaf(x[i].w, y[j].w, fmaf(x[i].z, y[j].z, fmaf(x[i].y, y[j].y, fmaf(x[i].x, y[j].x, acc[i][j]))));
    }
    // the columns left over, one per lane
    for (int64_t k = whole + lane + (SPLIT ? 64 * wave : 0); k < K; k += SPLIT ? 64 * kThinWaves : 64) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
#pragma unroll
            for (int j = 0; j < FEW; ++j) acc[i][j] = fmaf(b[i][k], a[j][k], acc[i][j]);
    }
    auto store = [&](int i, int j, float v) {
        if (j < n_few && first + i < n_many) C[j * step_few + (first + i) * step_many] = v;
    };
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int j = 0; j < FEW; ++j) {
#pragma unroll
            for (int o = 32; o > 0; o /= 2) acc[i][j] += __shfl_xor(acc[i][j], o);
            if (lane == 0) {
                if constexpr (SPLIT) part[wave][i * FEW + j] = acc[i][j];
                else store(i, j, acc[i][j]);
            }
        }
    if constexpr (SPLIT) {
        __syncthreads();
        if (wave == 0 && lane < ROWS * FEW)
            store(lane / FEW, lane % FEW, (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
    }
}
hipError_t launch_thin(const GramArgs &g, hipStream_t stream)
{
    const bool few_x = g.Nx <= g.Ny;
    const float *few = few_x ? g.A : g.B, *many = few_x ? g.B : g.A;
    const int64_t n_few = few_x ? g.Nx : g.Ny, n_many = few_x ? g.Ny : g.Nx, ld_few = few_x ? g.lda : g.ldb, ld_many = few_x ? g.ldb : g.lda;
    const int64_t step_few = few_x ? g.ldc : 1, step_many = few_x ? 1 : g.ldc;
    const bool split = n_many < kThinSplit;
    const int64_t rows = n_few > 4 && n_many >= kThinMany ? 4 : 2, per_workgroup = split ? rows : rows * kThinWaves, workgroups = (n_many + per_workgroup - 1) / per_workgroup;
    if (workgroups > 0x7fffffffLL) return hipErrorInvalidValue;
#define RFSF_THIN(FEW, ROWS, SPLIT)                                                                                                              \
    hipLaunchKernelGGL((gram_thin<FEW, ROWS, SPLIT>), dim3((unsigned)workgroups), dim3(64 * kThinWaves), 0, stream, few, many, g.C, n_few, \
                       n_many, g.K, ld_few, ld_many, step_few, step_many)
#define RFSF_THIN_ROWS(FEW, ROWS)            \
    do {                                     \
        if (split) RFSF_THIN(FEW, 2, true);  \
        else RFSF_THIN(FEW, ROWS, false);    \
    } while (0)
    if (n_few <= 1) RFSF_THIN_ROWS(1, 2);
    else if (n_few <= 2) RFSF_THIN_ROWS(2, 2);
    else if (n_few <= 4) RFSF_THIN_ROWS(4, 2);
    else if (rows == 2) RFSF_THIN_ROWS(kFew, 2);
    else RFSF_THIN_ROWS(kFew, 4);
#undef RFSF_THIN_ROWS
#undef RFSF_THIN
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Large problems: tile 256 x 128, four wavefronts 2 x 2 of 128 x 64, steps of 16 columns of K in three LDS buffers.
// The floats go from global memory straight into LDS (global_load_lds: lane i of a wavefront deposits its bytes at
// LDS base + i times their number, no register and no LDS-write instruction involved), two steps ahead, and are split
// when they are read: a wavefront splits (128 + 64) x 16 numbers for 48 matrix instructions of three terms, 5.5 vector
// instructions for each, or 24 of two terms, 6 for each. 128 x 64 also keeps the LDS reads at a
// quarter of the matrix time. Two workgroups per CU (75 KB of LDS and 256 registers each), so that one computes while
// the other waits at its barrier, starts or stores.
// Bound: power. With two terms the clock falls from 2.4 to 1.4 to 1.7 GHz on whole-chip products; a step of a CU takes 1650
// cycles with one workgroup on it where its matrix instructions take 768, 2000 to 2200 with two. Three terms and two:
// 50000 x 5000 x 10241 26.4 and 18.4 ms (58 % of the requests hit the L2), 10000 rows with themselves, 5121 columns 3.02 and 2.14,
// 5000 rows 0.97 and 0.60, 7494 rows, 1001 columns 0.420 and 0.268, 59952 x 200 x 400 77 and 54 us. Tiles of 256 x 256 with
// eight wavefronts, one workgroup per CU, take 16.6 ms for the largest but 320 us for 7494 rows and 66 for 59952 x 200 x 400: the
// start and the stores of a tile, 35000 cycles, have nothing to hide behind. v_mfma_f32_32x32x2f32 gave 38.8 and 3.90 ms.
// LDS layout of one buffer: 384 rows (256 of A, 128 of B) of 4 chunks of 16 bytes; slot p of row r holds chunk
// p ^ ((r / 4) mod 4): the XOR makes the fragment reads (16 consecutive rows, same chunk) hit 16 distinct 16-byte
// positions of the 256-byte bank row, and a direct load can produce it because each lane chooses what it fetches.
// ALIGNED: rows start on 16 bytes and are loaded 16 bytes per lane; otherwise four bytes per lane.
constexpr int kBigM = 256, kBigN = 128, kBigRows = kBigM + kBigN, kStep = 16;
constexpr int kBigBuffer = kBigRows * kStep;                  // floats
constexpr int64_t kBigMaxStride = (int64_t)1 << 21;           // offsets inside a tile are 32-bit byte offsets

struct TileCoord { int64_t bi, bj; };
constexpr int kStrip = 4;        // tile rows per strip: 4 x 8 tiles, 1024 x 1024 entries, share their panels in an L2
// A column of a strip begins one row further down than the one before it: the workgroups of an XCD go to its four shader
// engines in turn, and one of these would get all tiles of a row, which one row of the matrix can make slow ones (10000 rows with
// themselves, 5121 columns, one number that does not fit two terms 4.76 -> 3.40 ms, 1025 columns 1.00 -> 0.72; others unchanged).
template <bool SYM>
__device__ __forceinline__ TileCoord big_tile(int64_t rank, int64_t nti, int64_t ntj)
{
    if (!SYM) {
        const int64_t full = kStrip * ntj, I = rank / full, r = rank - I * full;
        const int64_t h = min(nti - kStrip * I, (int64_t)kStrip);
        return {kStrip * I + (r + r / h) % h, r / h};
    }
    // a strip starts at column tile 2 kStrip I; column c of its first 2 h ones holds rows 0 .. c / 2
    for (int64_t I = 0;; ++I) {
        const int64_t h = min(nti - kStrip * I, (int64_t)kStrip), w = ntj - 2 * kStrip * I;
        const int64_t count = h * w - h * (h - 1);
        if (rank >= count) {
            rank -= count;
            continue;
        }
        for (int64_t c = 0; c < 2 * h; ++c) {
            if (rank <= c / 2) return {kStrip * I + rank, 2 * kStrip * I + c};
            rank -= c / 2 + 1;
        }
        return {kStrip * I + (rank + rank / h) % h, 2 * kStrip * I + 2 * h + rank / h};
    }
}
int64_t big_tiles(int64_t Nx, int64_t Ny, bool sym)
{
    const int64_t nti = (Nx + kBigM - 1) / kBigM, ntj = (Ny + kBigN - 1) / kBigN;
    return sym ? nti * ntj - nti * (nti - 1) : nti * ntj;
}

// Lane i's BYTES bytes at base + off to LDS at address dst + BYTES * i. Written out so that the compiler, which cannot tell
// the buffers apart, does not wait for the loads in flight before every read of LDS; the caller waits. (m0 is a register
// that the compiler manages by itself; that it is written here has to be said, and is warned about.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int BYTES>
__device__ __forceinline__ void direct_load(const char *base, uint32_t off, uint32_t dst)
{
    const uint32_t to = __builtin_amdgcn_readfirstlane(dst);
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

template <typename T>
__device__ __forceinline__ T uniform(T x)
{
    const uint64_t bits = __builtin_bit_cast(uint64_t, x);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)bits), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(bits >> 32));
    return __builtin_bit_cast(T, hi << 32 | lo);
}
// A tile's place, the sources of its direct loads and the steps of its columns: what the kernels of large tiles share.
typedef __attribute__((address_space(3))) float LdsFloat;
template <bool ALIGNED, bool CALLED = false>
struct BigTile {
    // Direct loads: instruction j of wavefront w fills rows RI (w NL + j) .. + RI - 1 of the buffer (RI rows per
    // instruction). Rows beyond the matrix are redirected to its last one.
    static constexpr int RI = ALIGNED ? 16 : 4, NL = kBigRows / RI / 4;
    const GramArgs &g;
    float *buf;                         // three buffers in LDS
    uint32_t lds;                       // address of the first one there
    const float *A, *B;
    float *C;
    int64_t i0, j0, nfull, nsteps;
    int tid, lane, wave, half, col, wi, wj, rest, shift, fsw, frag_a, frag_b;
    uint32_t off[NL];                   // byte offset of this lane's source from the operand's tile

    __device__ __forceinline__ BigTile(const GramArgs &args, LdsFloat *buffers, int64_t i, int64_t j)
        : g(args), buf((float *)buffers), lds((uint32_t)(uintptr_t)buffers), i0(i), j0(j)
    {
        A = g.A + blockIdx.y * g.step_a;
        B = g.B + blockIdx.y * g.step_b;
        C = g.C + blockIdx.y * g.step_c;
        tid = threadIdx.x;
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        half = lane >> 5;
        col = lane & 31;
        wi = wave >> 1;
        wj = wave & 1;
        // the last, partial step comes first (buffer 0), number by number with zeros beyond K; full step s follows
        // in buffer (s + shift) mod 3
        nfull = g.K / kStep;
        rest = (int)(g.K - kStep * nfull);
        shift = rest != 0 ? 1 : 0;
        nsteps = nfull + shift;
        fsw = (col >> 2) & 3;
        frag_a = (wi * 128 + col) * kStep;
        frag_b = (kBigM + wj * 64 + col) * kStep;
        const int lrow = ALIGNED ? lane >> 2 : lane >> 4;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int row0 = RI * (wave * NL + l), row = row0 + lrow;
            const int slot = ALIGNED ? lane & 3 : (lane >> 2) & 3;
            const int column = 4 * (slot ^ ((row >> 2) & 3)) + (ALIGNED ? 0 : lane & 3);
            off[l] = (uint32_t)(row_of(row) * (row0 >= kBigM ? g.ldb : g.lda) + column) * 4u;
        }
    }
    // row of the operand that row `row` of a buffer holds, counted from the tile's first one
    __device__ __forceinline__ int64_t row_of(int row) const
    {
        const bool is_b = row >= kBigM;
        const int64_t left = is_b ? g.Ny - 1 - j0 : g.Nx - 1 - i0, r = is_b ? row - kBigM : row;
        return r < left ? r : left;
    }
    __device__ __forceinline__ const float *source(int row) const
    {
        return row >= kBigM ? B + (j0 + row_of(row)) * g.ldb : A + (i0 + row_of(row)) * g.lda;
    }
    __device__ __forceinline__ void load(float *dst, int64_t k0) const
    {
        const char *base_a = reinterpret_cast<const char *>(A + i0 * g.lda), *base_b = reinterpret_cast<const char *>(B + j0 * g.ldb);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int row0 = RI * (wave * NL + l);              // uniform
            const char *base = (row0 >= kBigM ? base_b : base_a) + 4 * k0;
            direct_load<ALIGNED ? 16 : 4>(CALLED ? uniform(base) : base, off[l], lds + 4u * (uint32_t)(dst - buf + row0 * kStep));
        }
    }
    // FEW: the first two steps only, their number being more than two; the third one is left to the caller.
    template <bool FEW>
    __device__ __forceinline__ void first_steps() const
    {
        if (rest != 0) {
            float v[kBigBuffer / 256];
#pragma unroll
            for (int u = 0; u < kBigBuffer / 256; ++u) {
                const int e = tid + 256 * u, row = e / kStep, k = e % kStep;
                v[u] = k < rest ? source(row)[kStep * nfull + k] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kBigBuffer / 256; ++u) {
                const int e = tid + 256 * u, row = e / kStep, k = e % kStep;
                buf[row * kStep + 4 * ((k >> 2) ^ ((row >> 2) & 3)) + (k & 3)] = v[u];
            }
        } else if (nsteps > 0) {
            load(buf, 0);
        }
        if (nsteps > 1) load(buf + kBigBuffer, kStep * (1 - shift));
        if (!FEW && nsteps > 2) load(buf + 2 * kBigBuffer, kStep * (2 - shift));
    }
    __device__ __forceinline__ void read8(const float *rd, int at, float (&x)[8]) const
    {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float4 v = *reinterpret_cast<const float4 *>(rd + at + 4 * ((2 * half + c) ^ fsw));
            x[4 * c] = v.x;
            x[4 * c + 1] = v.y;
            x[4 * c + 2] = v.z;
            x[4 * c + 3] = v.w;
        }
    }
    // waits for this wavefront's loads and LDS operations and then for everybody
    __device__ __forceinline__ void everybody() const
    {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    // Called by step s when it has read all of its buffer: waits for this wavefront's loads of the next step (those of the
    // step after it stay in flight) and then for everybody: the next step can be read, and this step's buffer takes the
    // loads of the step three ahead.
    __device__ __forceinline__ void next_step(int64_t s, float *rd) const
    {
        if (s + 2 < nsteps) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + 3 < nsteps) load(rd, kStep * (s + 3 - shift));
    }
};
__device__ __forceinline__ void clear(floatx16 (&acc)[4][2])
{
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
}
__device__ __forceinline__ bool any_nan(const floatx16 (&acc)[4][2])     // of the wavefront (or inf - inf)
{
    float sum = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) sum += acc[a][b][e];
    return __ballot(sum != sum) != 0;
}

// One tile with three terms, from the first load to the last entry.
template <bool ALIGNED, bool SYM, bool FLIP, bool CALLED>
__device__ __forceinline__ void three_term_tile(const GramArgs &g, LdsFloat *buffers, int64_t i0, int64_t j0)
{
    const BigTile<ALIGNED, CALLED> tile(g, buffers, i0, j0);
    float *buf = tile.buf;
    const int wi = tile.wi, wj = tile.wj, half = tile.half, col = tile.col;
    const int64_t nsteps = tile.nsteps;
    floatx16 acc[4][2];
    clear(acc);
    // Software pipeline. A step enters with the split fragments of its two blocks of B and of its first block of A; the
    // matrix instructions of one block of A run while the next one is split. Before the last block's, when
    // everything of this step has been read, the wavefront waits for its loads of the next step (those of the
    // step after it stay in flight) and then for everybody: the next step can be read, and this step's buffer takes
    // the loads of the step three ahead. The next step's first fragments are read and split under the last
    // block's matrix instructions.
    Split8 b[2], a;
    uint32_t sign[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) sign[t] = flip_of_row(i0 + wi * 128 + 32 * t);
    auto first_fragments = [&](const float *rd, Split8 (&nb)[2], Split8 &na) {
        float x[3][8];
        tile.read8(rd, tile.frag_b, x[0]);
        tile.read8(rd, tile.frag_b + 32 * kStep, x[1]);
        tile.read8(rd, tile.frag_a, x[2]);
        nb[0] = split8(x[0]);
        nb[1] = split8(x[1]);
        if (FLIP) flip(x[2], sign[0]);
        na = split8(x[2]);
    };
    auto interleave = [&](auto vector_tag) {
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                      // one matrix instruction
            __builtin_amdgcn_sched_group_barrier(0x002, decltype(vector_tag)::value, 0);    // and vector ones behind it
        }
    };
    auto step = [&](int64_t s, float *rd, const float *next) {
        float x[3][8];
#pragma unroll
        for (int t = 0; t < 3; ++t) tile.read8(rd, tile.frag_a + (t + 1) * 32 * kStep, x[t]);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            mfma_split<2>(a, b, acc[t]);
            if (FLIP) flip(x[t], sign[t + 1]);
            a = split8(x[t]);
            interleave(std::integral_constant<int, 4>{});
            __builtin_amdgcn_sched_barrier(0);
        }
        tile.next_step(s, rd);
        Split8 nb[2], na;
        first_fragments(next, nb, na);                          // (junk after the last step, not used)
        mfma_split<2>(a, b, acc[3]);
        interleave(std::integral_constant<int, 11>{});
        __builtin_amdgcn_sched_barrier(0);
        b[0] = nb[0];
        b[1] = nb[1];
        a = na;
    };
    tile.template first_steps<false>();
    if (nsteps > 0) {
        tile.everybody();
        first_fragments(buf, b, a);
        for (int64_t s = 0; s < nsteps; s += 3) {
            step(s, buf, buf + kBigBuffer);
            if (s + 1 < nsteps) step(s + 1, buf + kBigBuffer, buf + 2 * kBigBuffer);
            if (s + 2 < nsteps) step(s + 2, buf + 2 * kBigBuffer, buf);
        }
    }
    // result layout of a 32x32 block: lane holds column lane % 32 and rows 8 q + 4 (lane / 32) + 0 .. 3
    const bool vec_mirror = g.ldc % 4 == 0 && reinterpret_cast<uintptr_t>(tile.C) % 16 == 0;
    const bool diagonal = SYM && j0 < i0 + kBigM;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4] = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
                store_quad<FLIP>(g, tile.C, i0 + (wi * 4 + a) * 32 + 8 * q + 4 * half, j0 + (wj * 2 + b) * 32 + col, v, SYM,
                                 diagonal, vec_mirror, sign[a]);
            }
    if (any_nan(acc)) {
#pragma unroll 1
        for (int h = 0; h < 2; ++h) settle_nan<64, 64, SYM>(g, tile.A, tile.B, tile.C, i0 + wi * 128 + 64 * h, j0 + wj * 64, diagonal);
    }
}

// The same as a call: a kernel that ends with it keeps its registers to itself.
// (A function's arguments come in vector registers; what is the same for all lanes goes back to scalar ones.)
template <bool ALIGNED, bool SYM, bool FLIP>
__device__ __attribute__((noinline)) void three_term_tile_call(GramArgs g, LdsFloat *buf, int64_t i0, int64_t j0)
{
    three_term_tile<ALIGNED, SYM, FLIP, true>(g, buf, uniform(i0), uniform(j0));
}

template <bool SYM>
__device__ __forceinline__ bool place_of_tile(int64_t tiles, int64_t nti, int64_t ntj, int64_t &i0, int64_t &j0)
{
    const int64_t rank = rank_of_block(tiles);
    if (rank >= tiles) return false;
    const TileCoord tc = big_tile<SYM>(rank, nti, ntj);
    i0 = (int64_t)__builtin_amdgcn_readfirstlane((int)tc.bi) * kBigM;
    j0 = (int64_t)__builtin_amdgcn_readfirstlane((int)tc.bj) * kBigN;
    return true;
}

template <bool ALIGNED, bool SYM, bool FLIP>
__global__ __launch_bounds__(256, 2) void gram_big(GramArgs g, int64_t tiles, int64_t nti, int64_t ntj)
{
    __shared__ __attribute__((aligned(16))) float buf[3 * kBigBuffer];
    int64_t i0, j0;
    if (!place_of_tile<SYM>(tiles, nti, ntj, i0, j0)) return;
    three_term_tile<ALIGNED, SYM, FLIP, false>(g, (LdsFloat *)buf, i0, j0);
}

constexpr int kPartStride = 65;          // floats between the rows of a wavefront's 32 x 64 part of a result in LDS

// Two terms (top of the file). Below 128 columns the three terms' error is the smaller one, and the scales take as long as
// the products save. A tile that cannot do with two terms ends with a call of the three-term code: inlined, that code and
// what it keeps alive pushes the registers of the loop below into scratch memory (2.1 -> 5.7 ms).
constexpr int64_t kTwoTermColumns = 128;
constexpr int kSamples = 4, kLargest = 9, kMostUp = 100, kUpOfZeros = kMostUp + 1;
constexpr float kLeastSum = 0x1p15f;
template <bool ALIGNED, bool SYM, bool FLIP>
__global__ __launch_bounds__(256, 2) void gram_big_two_terms(GramArgs g, int64_t tiles, int64_t nti, int64_t ntj)
{
    __shared__ __attribute__((aligned(16))) float buf[3 * kBigBuffer];
    __shared__ __attribute__((aligned(16))) float scales[kBigRows];
    __shared__ int verdict;                     // 1: the tile takes three terms
    int64_t i0, j0;
    if (!place_of_tile<SYM>(tiles, nti, ntj, i0, j0)) return;
    const BigTile<ALIGNED> tile(g, (LdsFloat *)buf, i0, j0);
    const int tid = tile.tid, lane = tile.lane, wi = tile.wi, wj = tile.wj, half = tile.half, col = tile.col;
    floatx16 acc[4][2];
    {
        const int64_t nsteps = tile.nsteps;
        tile.template first_steps<true>();
        // Scales: from the largest of the first two steps' numbers of a row and of sixteen more spread over it, which lie where
        // the third step's will.
        constexpr int kOwn = (kBigRows + 255) / 256;             // rows of a thread
        float *samples = buf + 2 * kBigBuffer;
        Float4u sample[kOwn][kSamples];
#pragma unroll
        for (int h = 0; h < kOwn; ++h) {
            const float *src = tile.source(min(tid + 256 * h, kBigRows - 1));
#pragma unroll
            for (int k = 0; k < kSamples; ++k) sample[h][k] = *reinterpret_cast<const Float4u *>(src + (g.K - 4) * (k + 1) / kSamples);
        }
#pragma unroll
        for (int h = 0; h < kOwn; ++h) {
            const int row = min(tid + 256 * h, kBigRows - 1);
#pragma unroll
            for (int k = 0; k < kSamples; ++k)
                *reinterpret_cast<float4 *>(&samples[row * kStep + 4 * (k ^ ((row >> 2) & 3))]) =
                    make_float4(sample[h][k].x, sample[h][k].y, sample[h][k].z, sample[h][k].w);
        }
        if (tid == 0) verdict = 0;
        tile.everybody();
        bool outside = false;
#pragma unroll
        for (int h = 0; h < kOwn; ++h) {
            const int row = min(tid + 256 * h, kBigRows - 1);
            const float last = sample[h][kSamples - 1].w;
            float most = 0.f;
#pragma unroll
            for (int k = 0; k < kSamples; ++k)
                most = fmaxf(fmaxf(fmaxf(fabsf(sample[h][k].x), fabsf(sample[h][k].y)),
                                   fmaxf(fabsf(sample[h][k].z), fabsf(sample[h][k].w))), most);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float4 v = *reinterpret_cast<const float4 *>(&buf[k / 4 * kBigBuffer + row * kStep + 4 * ((k + (row >> 2)) & 3)]);
                most = fmaxf(fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))), most);
            }
            const int exponent = (int)(__float_as_uint(most) >> 23) - 127;      // of the largest; -127 for zero
            const int up = most == 0.f ? kUpOfZeros : kLargest - exponent;
            outside |= most != 0.f && (up > kMostUp || up < -kMostUp);
            // Zero wherever it is sampled: anything else in it has no scale that would fit it, so it is looked through.
            if (most == 0.f && last == last) {
                const float *src = tile.source(row);
                uint32_t bits = 0;
#pragma unroll 16
                for (int64_t k = 0; k < g.K; k += 4) {
                    const Float4u v = *reinterpret_cast<const Float4u *>(src + min(k, g.K - 4));
                    bits |= __float_as_uint(v.x) | __float_as_uint(v.y) | __float_as_uint(v.z) | __float_as_uint(v.w);
                }
                outside |= (bits & 0x7fffffffu) != 0u;
            }
            scales[row] = last != last ? last : __uint_as_float((uint32_t)(127 + up) << 23);
        }
        if (__ballot(outside) && lane == 0) verdict = 1;
        __syncthreads();
        float scale_a[4], scale_b[2];           // of this lane's rows in the blocks of A (flipped where those are) and B
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            scale_a[t] = scales[wi * 128 + 32 * t + col];
            if (FLIP) scale_a[t] = __uint_as_float(__float_as_uint(scale_a[t]) ^ flip_of_row(i0 + wi * 128 + 32 * t));
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) scale_b[t] = scales[kBigM + (wj * 2 + t) * 32 + col];
        // The sums of |a b| over the sampled columns, by the matrix units (3000 rows with 3000, 400 columns 49.2 -> 50.9 us, 10000 with
        // themselves, 5121 columns 2.03 ms with them and without).
        {
            const auto of_zeros = [](float scale) { return fabsf(scale) == __uint_as_float((uint32_t)(127 + kUpOfZeros) << 23) ? 0x1p9f : 0.f; };
            clear(acc);
#pragma unroll 1
            for (int s = 0; s < 3; ++s) {
                halfx8 of_b[2];
                float x[8];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    tile.read8(buf + s * kBigBuffer, tile.frag_b + u * 32 * kStep, x);
                    of_b[u] = magnitudes(x, scale_b[u], of_zeros(scale_b[u]));
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    tile.read8(buf + s * kBigBuffer, tile.frag_a + t * 32 * kStep, x);
                    const halfx8 of_a = magnitudes(x, scale_a[t], of_zeros(scale_a[t]));
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(of_a, of_b[u], acc[t][u], 0, 0, 0);
                }
            }
            float least = acc[0][0][0];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int e = 0; e < 16; ++e) least = fminf(least, acc[t][u][e]);
            if (__ballot(least < kLeastSum) && lane == 0) verdict = 1;
        }
        __syncthreads();
        if (verdict != 0) {
            three_term_tile_call<ALIGNED, SYM, FLIP>(g, (LdsFloat *)buf, i0, j0);
            return;
        }
        tile.load(buf + 2 * kBigBuffer, kStep * (2 - tile.shift));            // nobody reads the samples any more
        // Software pipeline. A step enters with the split fragments of its two blocks of B and of its first block of A, and
        // with the numbers of the second. A pair of floats is split behind every matrix instruction (in this order: left to
        // itself the scheduler makes lumps, and a matrix instruction hides about four others, not sixty): four instructions
        // for each of blocks 1, 2, 3 of A and, of the next step, both of B and block 0 of A, read from LDS one fragment ahead.
        Half8 b[2], nb[2], a[4];
        float x[2][8];                                          // the fragment that is being split and the next one
        auto step = [&](int64_t s, float *rd, const float *next) {
#pragma unroll
            for (int w = 0; w < 6; ++w) {
                if (w == 2) tile.next_step(s, rd);
                if (w < 2) tile.read8(rd, tile.frag_a + (w + 2) * 32 * kStep, x[(w + 1) % 2]);
                else if (w < 4) tile.read8(next, tile.frag_b + (w - 2) * 32 * kStep, x[(w + 1) % 2]);
                else tile.read8(next, tile.frag_a + (w - 4) * 32 * kStep, x[(w + 1) % 2]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int slot = 4 * w + i, t = slot / 6, u = slot % 2;
                    acc[t][u] = product(slot % 6 / 2, a[t], b[u], acc[t][u]);
                    Half8 &f = w < 3 ? a[w + 1] : w < 5 ? nb[w - 3] : a[0];
                    split_pair(f, i, x[w % 2][2 * i], x[w % 2][2 * i + 1], w < 3 ? scale_a[w + 1] : w < 5 ? scale_b[w - 3] : scale_a[0]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            b[0] = nb[0];
            b[1] = nb[1];
        };
        clear(acc);
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            tile.read8(buf, w < 2 ? tile.frag_b + w * 32 * kStep : tile.frag_a, x[0]);
#pragma unroll
            for (int i = 0; i < 4; ++i) split_pair(w < 2 ? b[w] : a[0], i, x[0][2 * i], x[0][2 * i + 1], w < 2 ? scale_b[w] : scale_a[0]);
        }
        tile.read8(buf, tile.frag_a + 32 * kStep, x[0]);
        for (int64_t s = 0; s < nsteps; s += 3) {
            step(s, buf, buf + kBigBuffer);
            if (s + 1 < nsteps) step(s + 1, buf + kBigBuffer, buf + 2 * kBigBuffer);
            if (s + 2 < nsteps) step(s + 2, buf + 2 * kBigBuffer, buf);
        }
    }
    // Entries that are NaN although neither of their rows ends in one: a row did not fit its scale, or a NaN or an infinity stands
    // somewhere else in it. (NaN in a row that ends in one needs no second look: settle_nan would leave it alone, too.)
    bool open = false;
    float of_col[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) of_col[u] = scales[kBigM + (wj * 2 + u) * 32 + col];
    if (any_nan(acc)) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float of_row = scales[wi * 128 + 32 * t + 8 * (e / 4) + 4 * half + e % 4];
#pragma unroll
                for (int u = 0; u < 2; ++u) open |= acc[t][u][e] != acc[t][u][e] && of_row == of_row && of_col[u] == of_col[u];
            }
    }
    if (__ballot(open) && lane == 0) verdict = 1;
    __syncthreads();
    if (verdict != 0) {
        three_term_tile_call<ALIGNED, SYM, FLIP>(g, (LdsFloat *)buf, i0, j0);
        return;
    }
    // Back from the scales 2^a and 2^b of its rows by one power of two, -(a + b): it rounds once and can be as large as 200, where
    // the product of two powers would overflow (times a sum of zero: NaN) or vanish although the result is an ordinary number.
    int down[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) down[u] = 2 * 127 - (int)(__float_as_uint(of_col[u]) >> 23);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int up = (int)(__float_as_uint(scales[wi * 128 + 32 * t + 8 * (e / 4) + 4 * half + e % 4]) >> 23);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float v = acc[t][u][e];
                if (FLIP) v = __uint_as_float(__float_as_uint(v) ^ flip_of_row(i0 + wi * 128 + 32 * t));
                acc[t][u][e] = __builtin_amdgcn_ldexpf(v, down[u] - up);
            }
        }
    // All results are made before the first is stored: left to itself the compiler moves each to its store (5904 rows with
    // themselves, 301 columns 89 -> 85.5 us, 10000, 1025 columns 442 -> 434; without aligned rows 96 -> 98).
    if constexpr (ALIGNED) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(acc[t][u]));
    }
    // result layout of a 32x32 block: lane holds column lane % 32 and rows 8 q + 4 (lane / 32) + 0 .. 3
    const bool vec_mirror = g.ldc % 4 == 0 && reinterpret_cast<uintptr_t>(tile.C) % 16 == 0;
    const bool diagonal = SYM && j0 < i0 + kBigM;
    float *C = tile.C;
    if (!diagonal && i0 + kBigM <= g.Nx && g.ldc <= kBigMaxStride && (!SYM || vec_mirror)) {
        // all rows exist: scalar row addresses, one offset per lane
        float *at_tile = C + (i0 + wi * 128) * g.ldc + j0 + wj * 64, *image = C + (j0 + wj * 64) * g.ldc + i0 + wi * 128;
        const uint32_t at = (uint32_t)(4 * half * g.ldc + col) * 4u, image_at = (uint32_t)(col * g.ldc + 4 * half) * 4u;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (j0 + (wj * 2 + u) * 32 + col >= g.Ny) continue;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float *row = at_tile + (32 * t + 8 * q + e) * g.ldc + 32 * u;
                        *reinterpret_cast<float *>(reinterpret_cast<char *>(row) + at) = acc[t][u][4 * q + e];
                    }
                    if (SYM) {
                        float *row = image + 32 * u * g.ldc + 32 * t + 8 * q;
                        *reinterpret_cast<float4 *>(reinterpret_cast<char *>(row) + image_at) =
                            make_float4(acc[t][u][4 * q], acc[t][u][4 * q + 1], acc[t][u][4 * q + 2], acc[t][u][4 * q + 3]);
                    }
                }
        }
    } else {
        // through LDS, 32 rows at a time, a row or a column per instruction
        float *part = buf + tile.wave * 32 * kPartStride;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) part[(8 * (e / 4) + 4 * half + e % 4) * kPartStride + 32 * u + col] = acc[t][u][e];
            const int64_t ib = i0 + wi * 128 + 32 * t, jb = j0 + wj * 64;
#pragma unroll 1
            for (int r = 0; r < 32; ++r) {
                const int64_t i = ib + r, j = jb + lane;
                if (i < g.Nx && j < g.Ny && (!diagonal || i <= j)) C[i * g.ldc + j] = part[r * kPartStride + lane];
            }
            if (SYM) {
#pragma unroll 1
                for (int c = 0; c < 64; c += 2) {
                    const int64_t i = ib + col, j = jb + c + half;
                    if (i < g.Nx && j < g.Ny && (!diagonal || i < j)) C[j * g.ldc + i] = part[col * kPartStride + c + half];
                }
            }
        }
    }
}

template <int NR, int NW>
hipError_t launch_small(const GramArgs &g, bool sym, bool flip, int batch, hipStream_t stream)
{
    const int64_t ti = (g.Nx + 16 * NR - 1) / (16 * NR), tj = (g.Ny + 16 * NR - 1) / (16 * NR);
    const int64_t tiles = sym ? ti * (ti + 1) / 2 : ti * tj;
    if (tiles > 0x7fffffffLL - 8) return hipErrorInvalidValue;
    const dim3 grid(xcd_grid(tiles), (unsigned)batch);
#define RFSF_SMALL(SY, FL) hipLaunchKernelGGL((gram_small<NR, NW, SY, FL>), grid, dim3(64 * NW), 0, stream, g, tiles, tj)
    if (flip) RFSF_SMALL(false, true);
    else if (sym) RFSF_SMALL(true, false);
    else RFSF_SMALL(false, false);
#undef RFSF_SMALL
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gram(const float *PhiX, int64_t Nx, int64_t ldx, const float *PhiY, int64_t Ny,
                       int64_t ldy, int64_t ncols, float *K, int64_t ldk, hipStream_t stream, bool rows_add_up, int batch,
                       int64_t step_x, int64_t step_y, int64_t step_k, int64_t points)
{
    if (Nx == 0 || Ny == 0) return hipSuccess;
    const GramArgs g = {PhiX, PhiY, K, Nx, Ny, ncols, ldx, ldy, ldk, step_x, step_y, step_k};
    // K = PhiX PhiX^T: only what lies on or above the diagonal is computed, and written twice
    const bool sym = PhiX == PhiY && Nx == Ny && ldx == ldy && !rows_add_up;
    const auto count = [&](int64_t edge, int64_t rows) {
        const int64_t ti = (rows + edge - 1) / edge, tj = (Ny + edge - 1) / edge;
        return (sym ? ti * (ti + 1) / 2 : ti * tj) * batch;
    };
    const auto rounds_of = [&](int64_t rows) { return (big_tiles(rows, Ny, sym) * batch + 255) / 256; };
    const int64_t few = std::min(Nx, Ny), many = std::max(Nx, Ny);
    if (!rows_add_up && batch == 1 && few <= kFew && thin_pays(few, many, ncols)) return launch_thin(g, stream);
    // Large tiles run one per CU at a time or, faster together, two; with `rounds` = their number over 256, rounded up,
    // three terms take as long as about 1340 tiles of 64 x 64 per round do. Two terms: 64 x 64 tiles take about
    // 0.57 (105 + columns) / 10000 us each and 12 more, large ones 20 us and 0.76 (200 + columns) / 17.5 us a round, fitted
    // to both kinds at 201, 401, 1025 and 5121 columns (rows with themselves, 64 x 64 against large: 3500 rows 42, 56, 113,
    // 496 us against 42, 52, 80, 269; 2500 rows 26, 35, 67, 279 against 41, 50, 75, 235; 4000 rows, two rounds, 48, 68, 137,
    // 606 against 56, 70, 118, 464). Two terms are for calls that three would run in large tiles as well: the small ones add up in four
    // or eight sums, and their error is half that of a large tile's single one (5121 columns 5.0e-7 and 9.4e-7), which
    // 2500, 3000 and 4000 rows, faster as they would be, are not to lose.
    // RFSF-TRP's products: large tiles are slower up to 800 tiles of 64 x 64 per round and faster from about 1000 on (features of sequences of two
    // points, five levels, 200 projections, 200 frequencies, 64 x 64 and large: 2400 sequences 48.8 and 53.7 us, 3200 55.4 and 55.4, 4400 71.8 and
    // 57.5; 16 frequencies 24.4 and 25.8, 27.8 and 27.9, 34.4 and 30.5; 500 73 and 85, 89 and 87, 121 and 94), but their error is 1.1 (32 columns) to
    // 1.4 times (400 and 1000) that of the small ones. So only calls of which a row for every point, which these products once
    // had, would be above the line of the others take them, and of these not those that the rows that there are leave below 800.
    const bool two = ncols >= kTwoTermColumns;
    const auto above_line = [&](int64_t rows) {
        const int64_t small = count(64, rows), rounds = rounds_of(rows);
        return small > 1340 * rounds && (!two || small * (105 + ncols) > 140000 + rounds * (150000 + 760 * ncols));
    };
    const int64_t tiles = big_tiles(Nx, Ny, sym);
    const bool large = points ? above_line(points) && count(64, Nx) > 800 * rounds_of(Nx) : above_line(Nx);
    if (large && ldx <= kBigMaxStride && ldy <= kBigMaxStride) {
        if (tiles > 0x7fffffffLL - 8) return hipErrorInvalidValue;
        const bool aligned = ldx % 4 == 0 && ldy % 4 == 0 && step_x % 4 == 0 && step_y % 4 == 0 &&
                             reinterpret_cast<uintptr_t>(PhiX) % 16 == 0 && reinterpret_cast<uintptr_t>(PhiY) % 16 == 0;
        const int64_t nti = (Nx + kBigM - 1) / kBigM, ntj = (Ny + kBigN - 1) / kBigN;
        const dim3 grid(xcd_grid(tiles), (unsigned)batch);
#define RFSF_BIG(AL, SY, FL) hipLaunchKernelGGL((two ? gram_big_two_terms<AL, SY, FL> : gram_big<AL, SY, FL>), grid, dim3(256), 0, stream, g, tiles, nti, ntj)
        if (aligned) {
            if (rows_add_up) RFSF_BIG(true, false, true);
            else if (sym) RFSF_BIG(true, true, false);
            else RFSF_BIG(true, false, false);
        } else {
            if (rows_add_up) RFSF_BIG(false, false, true);
            else if (sym) RFSF_BIG(false, true, false);
            else RFSF_BIG(false, false, false);
        }
#undef RFSF_BIG
        return hipGetLastError();
    }
    // 32 x 32 tiles while 64 x 64 ones would not give every CU one (700 rows with themselves, 121 tiles of 64 x 64:
    // 16 us against 22 with 1025 columns, 65 against 74 with 5121; 1500 rows, 300 tiles: 158 against 131 with 5121)
    // ... and between 150 and 256 of them 64 x 64 tiles with eight wavefronts, which leave the rows' panels to half as many
    // readers (1000 x 1000, 501 columns 15.7 -> 12.6 us; 300 x 2000, 1501 columns, 160 tiles 36.3 -> 29.1; 1400 rows with
    // themselves, 1025 columns, 253 tiles 29.8 -> 23.5; 1000 rows, 136 tiles 22.1 and 21.8; 700 rows, 66 tiles 10.8 and 20.1)
    // ... and 16 x 16 while every CU gets at most one: what bounds a workgroup alone on its CU is how much it has to read (14 bytes a
    // clock; sixteen wavefronts or two steps ahead change nothing), here half of what a tile of 32 x 32 does (100 x 100 rows, 5121 columns 41 ->
    // 20 us, 200 x 200, 8191 60 -> 31, 16 x 1000, 5121 33 -> 20, 300 x 300, 361 tiles, 2049 columns and more about the same, 400 x 400, 625 tiles,
    // 18 and 24 with 2049)
    if (count(16, Nx) <= 256) return launch_small<1, 8>(g, sym, rows_add_up, batch, stream);
    if (count(64, Nx) <= 150) return launch_small<2, 8>(g, sym, rows_add_up, batch, stream);
    if (count(64, Nx) <= 256) return launch_small<4, 8>(g, sym, rows_add_up, batch, stream);
    return launch_small<4, 4>(g, sym, rows_add_up, batch, stream);
}

}  // namespace rfsf
