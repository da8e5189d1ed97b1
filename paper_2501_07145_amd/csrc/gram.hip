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
#include "rfsf_internal.h"
#include <type_traits>

namespace rfsf {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

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

// One operand pair of a launch: row-major, K-contiguous. Batched launches (one product per level of RFSF-TRP) add
// blockIdx.y times the steps.
struct GramArgs {
    const float *A, *B;
    float *C;
    int64_t Nx, Ny, K, lda, ldb, ldc;
    int64_t step_a, step_b, step_c;
};

// Stores four consecutive rows i .. i+3 of column j; `mirror` also writes their mirror image, row j. `diagonal`: the
// tile meets the diagonal, and only what lies on or above it counts.
template <bool FLIP>
__device__ __forceinline__ void store_quad(const GramArgs &g, float *C, int64_t i, int64_t j, float (&v)[4], bool mirror,
                                           bool diagonal, bool vec_mirror)
{
    if (j >= g.Ny) return;
    if constexpr (FLIP) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(__float_as_uint(v[e]) ^ flip_of_row(i + e));
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
// Small problems: too few tiles to fill the chip with large ones, time is latency. Tile (32 T) x (32 T), NW
// wavefronts that share out the columns of K in steps of 32, step s to wavefront s mod NW, and work without any
// barrier: each loads its fragments from global memory straight into registers, one step ahead. The partial tiles are
// added through LDS at the end in a fixed order. 16 x 16 blocks (v_mfma_f32_16x16x32_bf16: lane l holds columns
// 8 (l / 16) .. + 7 of row l mod 16) rather than 32 x 32: a 16-byte load then touches 16 rows instead of 32, and what
// bounds the loop is one row (cache line) per cycle of the CU's address unit, 37 cycles a load with 32 rows.
// Any row stride and alignment (the loads need four bytes).
// Registers are bounded so that a CU holds two workgroups of four wavefronts or of 32 x 32 tiles (with one, 3000 rows with
// themselves, 1025 columns, take 115 us instead of 90).
struct __attribute__((packed, aligned(4))) Float4u { float x, y, z, w; };

template <int T, int NW, bool SYM, bool FLIP>
__global__ __launch_bounds__(64 * NW, T == 1 ? 4 : 2) void gram_small(GramArgs g, int64_t tiles, int64_t tiles_j)
{
    constexpr int NR = 2 * T, NH = NW / 2;      // 16-row blocks per side; wavefronts that keep a partial tile in LDS
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
    const int64_t i0 = bi * (32 * T), j0 = bj * (32 * T);
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
        store_quad<FLIP>(g, C, ib + 4 * quarter, jb + col, v, SYM, SYM && bi == bj, vec_mirror);
        if (__ballot(any != any)) settle_nan<16, 16, SYM>(g, A, B, C, ib, jb, SYM && bi == bj);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Large problems: tile 256 x 128, four wavefronts 2 x 2 of 128 x 64, steps of 16 columns of K in three LDS buffers.
// The floats go from global memory straight into LDS (global_load_lds: lane i of a wavefront deposits its bytes at
// LDS base + i times their number, no register and no LDS-write instruction involved), two steps ahead, and are split
// when they are read: a wavefront splits (128 + 64) x 16 numbers for 48 matrix instructions, 5.5 vector
// instructions for each, which issue in the 32 cycles that it takes (measured: up to six are free, with
// eight the rate falls by a fifth; 64 x 64 per wavefront would need 7.3). 128 x 64 also keeps the LDS reads at a
// quarter of the matrix time. Two workgroups per CU (74 KB of LDS and 256 registers each), so that one computes while
// the other waits at its barrier.
// Bound: power. On 50000 x 5000 x 10241 the matrix pipes are busy 66 % of the cycles and the clock falls from 2.4 to
// 1.7 GHz: 26.0 ms, 1.18 PFLOP/s of bfloat16 products (the library's bfloat16 product of two 8192 x 8192 matrices
// reaches 1.25 to 1.30 here), 197 TFLOP/s of the product asked for. v_mfma_f32_32x32x2f32 gave 38.8 ms, 132 TFLOP/s, 0.84 of
// its peak. 10000 rows with themselves, 5121 columns: 2.97 ms against 3.90.
// LDS layout of one buffer: 384 rows (256 of A, 128 of B) of 4 chunks of 16 bytes; slot p of row r holds chunk
// p ^ ((r / 4) mod 4): the XOR makes the fragment reads (16 consecutive rows, same chunk) hit 16 distinct 16-byte
// positions of the 256-byte bank row, and a direct load can produce it because each lane chooses what it fetches.
// ALIGNED: rows start on 16 bytes and are loaded 16 bytes per lane; otherwise four bytes per lane.
constexpr int kBigM = 256, kBigN = 128, kBigRows = kBigM + kBigN, kStep = 16;
constexpr int kBigBuffer = kBigRows * kStep;                  // floats
constexpr int64_t kBigMaxStride = (int64_t)1 << 21;           // offsets inside a tile are 32-bit byte offsets

struct TileCoord { int64_t bi, bj; };
constexpr int kStrip = 4;        // tile rows per strip: 4 x 8 tiles, 1024 x 1024 entries, share their panels in an L2
template <bool SYM>
__device__ __forceinline__ TileCoord big_tile(int64_t rank, int64_t nti, int64_t ntj)
{
    if (!SYM) {
        const int64_t full = kStrip * ntj, I = rank / full, r = rank - I * full;
        const int64_t h = min(nti - kStrip * I, (int64_t)kStrip);
        return {kStrip * I + r % h, r / h};
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
        return {kStrip * I + rank % h, 2 * kStrip * I + 2 * h + rank / h};
    }
}
int64_t big_tiles(int64_t Nx, int64_t Ny, bool sym)
{
    const int64_t nti = (Nx + kBigM - 1) / kBigM, ntj = (Ny + kBigN - 1) / kBigN;
    return sym ? nti * ntj - nti * (nti - 1) : nti * ntj;
}

// Lane i's BYTES bytes at base + off to LDS at dst + BYTES * i. Written out so that the compiler, which cannot tell
// the buffers apart, does not wait for the loads in flight before every read of LDS; the caller waits. (m0 is a register
// that the compiler manages by itself; that it is written here has to be said, and is warned about.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int BYTES>
__device__ __forceinline__ void direct_load(const char *base, uint32_t off, float *dst)
{
    const uint32_t to = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)dst);
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

template <bool ALIGNED, bool SYM, bool FLIP>
__global__ __launch_bounds__(256, 2) void gram_big(GramArgs g, int64_t tiles, int64_t nti, int64_t ntj)
{
    __shared__ __attribute__((aligned(16))) float buf[3][kBigBuffer];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int wi = wave >> 1, wj = wave & 1;
    const int64_t rank = rank_of_block(tiles);
    if (rank >= tiles) return;
    const TileCoord tc = big_tile<SYM>(rank, nti, ntj);
    const int64_t i0 = (int64_t)__builtin_amdgcn_readfirstlane((int)tc.bi) * kBigM;
    const int64_t j0 = (int64_t)__builtin_amdgcn_readfirstlane((int)tc.bj) * kBigN;
    const float *A = g.A + blockIdx.y * g.step_a, *B = g.B + blockIdx.y * g.step_b;
    float *C = g.C + blockIdx.y * g.step_c;

    floatx16 acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    // Direct loads: instruction j of wavefront w fills rows RI (w NL + j) .. + RI - 1 of the buffer (RI rows per
    // instruction). Rows beyond the matrix are redirected to its last one.
    constexpr int RI = ALIGNED ? 16 : 4, NL = kBigRows / RI / 4;
    const int lrow = ALIGNED ? lane >> 2 : lane >> 4;
    uint32_t off[NL];                   // byte offset of this lane's source from the operand's tile
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int row0 = RI * (wave * NL + j), row = row0 + lrow;
        const int slot = ALIGNED ? lane & 3 : (lane >> 2) & 3;
        const int column = 4 * (slot ^ ((row >> 2) & 3)) + (ALIGNED ? 0 : lane & 3);
        const bool is_b = row0 >= kBigM;
        const int64_t left = is_b ? g.Ny - 1 - j0 : g.Nx - 1 - i0, r = is_b ? row - kBigM : row;
        off[j] = (uint32_t)((r < left ? r : left) * (is_b ? g.ldb : g.lda) + column) * 4u;
    }
    const char *base_a = reinterpret_cast<const char *>(A + i0 * g.lda);
    const char *base_b = reinterpret_cast<const char *>(B + j0 * g.ldb);
    auto load = [&](float *dst, int64_t k0) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int row0 = RI * (wave * NL + j);              // uniform
            direct_load<ALIGNED ? 16 : 4>((row0 >= kBigM ? base_b : base_a) + 4 * k0, off[j], dst + row0 * kStep);
        }
    };
    const int64_t nfull = g.K / kStep;
    const int rest = (int)(g.K - kStep * nfull);
    // the last, partial step comes first (buffer 0), number by number with zeros beyond K; full step s follows
    // in buffer (s + shift) mod 3
    const int shift = rest != 0 ? 1 : 0;
    const int64_t nsteps = nfull + shift;
    if (rest != 0) {
        float v[kBigBuffer / 256];
#pragma unroll
        for (int u = 0; u < kBigBuffer / 256; ++u) {
            const int e = tid + 256 * u, row = e / kStep, k = e % kStep;
            const bool is_b = row >= kBigM;
            const int64_t left = is_b ? g.Ny - 1 - j0 : g.Nx - 1 - i0, r = is_b ? row - kBigM : row;
            const float *src = is_b ? B + j0 * g.ldb : A + i0 * g.lda;
            v[u] = k < rest ? src[(r < left ? r : left) * (is_b ? g.ldb : g.lda) + kStep * nfull + k] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kBigBuffer / 256; ++u) {
            const int e = tid + 256 * u, row = e / kStep, k = e % kStep;
            buf[0][row * kStep + 4 * ((k >> 2) ^ ((row >> 2) & 3)) + (k & 3)] = v[u];
        }
    }
    const int fsw = (col >> 2) & 3;
    const int frag_a = (wi * 128 + col) * kStep, frag_b = (kBigM + wj * 64 + col) * kStep;
    auto read8 = [&](const float *rd, int at, float (&x)[8]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float4 v = *reinterpret_cast<const float4 *>(rd + at + 4 * ((2 * half + c) ^ fsw));
            x[4 * c] = v.x;
            x[4 * c + 1] = v.y;
            x[4 * c + 2] = v.z;
            x[4 * c + 3] = v.w;
        }
    };
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
        read8(rd, frag_b, x[0]);
        read8(rd, frag_b + 32 * kStep, x[1]);
        read8(rd, frag_a, x[2]);
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
        for (int t = 0; t < 3; ++t) read8(rd, frag_a + (t + 1) * 32 * kStep, x[t]);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            mfma_split<2>(a, b, acc[t]);
            if (FLIP) flip(x[t], sign[t + 1]);
            a = split8(x[t]);
            interleave(std::integral_constant<int, 4>{});
            __builtin_amdgcn_sched_barrier(0);
        }
        if (s + 2 < nsteps) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + 3 < nsteps) load(rd, kStep * (s + 3 - shift));
        Split8 nb[2], na;
        first_fragments(next, nb, na);                          // (junk after the last step, not used)
        mfma_split<2>(a, b, acc[3]);
        interleave(std::integral_constant<int, 11>{});
        __builtin_amdgcn_sched_barrier(0);
        b[0] = nb[0];
        b[1] = nb[1];
        a = na;
    };
    if (nsteps > 0) {
        if (shift == 0) load(buf[0], 0);
        if (nsteps > 1) load(buf[1], kStep * (1 - shift));
        if (nsteps > 2) load(buf[2], kStep * (2 - shift));
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        first_fragments(buf[0], b, a);
        for (int64_t s = 0; s < nsteps; s += 3) {
            step(s, buf[0], buf[1]);
            if (s + 1 < nsteps) step(s + 1, buf[1], buf[2]);
            if (s + 2 < nsteps) step(s + 2, buf[2], buf[0]);
        }
    }
    // result layout of a 32x32 block: lane holds column lane % 32 and rows 8 q + 4 (lane / 32) + 0 .. 3
    const bool vec_mirror = g.ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0;
    const bool diagonal = SYM && tc.bj < 2 * tc.bi + 2;
    float any = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) any += acc[a][b][e];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4] = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
                store_quad<FLIP>(g, C, i0 + (wi * 4 + a) * 32 + 8 * q + 4 * half, j0 + (wj * 2 + b) * 32 + col, v, SYM,
                                 diagonal, vec_mirror);
            }
    if (__ballot(any != any)) {
#pragma unroll 1
        for (int h = 0; h < 2; ++h) settle_nan<64, 64, SYM>(g, A, B, C, i0 + wi * 128 + 64 * h, j0 + wj * 64, diagonal);
    }
}

template <int T, int NW>
hipError_t launch_small(const GramArgs &g, bool sym, bool flip, int batch, hipStream_t stream)
{
    const int64_t ti = (g.Nx + 32 * T - 1) / (32 * T), tj = (g.Ny + 32 * T - 1) / (32 * T);
    const int64_t tiles = sym ? ti * (ti + 1) / 2 : ti * tj;
    if (tiles > 0x7fffffffLL - 8) return hipErrorInvalidValue;
    const dim3 grid(xcd_grid(tiles), (unsigned)batch);
#define RFSF_SMALL(SY, FL) hipLaunchKernelGGL((gram_small<T, NW, SY, FL>), grid, dim3(64 * NW), 0, stream, g, tiles, tj)
    if (flip) RFSF_SMALL(false, true);
    else if (sym) RFSF_SMALL(true, false);
    else RFSF_SMALL(false, false);
#undef RFSF_SMALL
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gram(const float *PhiX, int64_t Nx, int64_t ldx, const float *PhiY, int64_t Ny,
                       int64_t ldy, int64_t ncols, float *K, int64_t ldk, hipStream_t stream, bool rows_add_up, int batch,
                       int64_t step_x, int64_t step_y, int64_t step_k)
{
    if (Nx == 0 || Ny == 0) return hipSuccess;
    const GramArgs g = {PhiX, PhiY, K, Nx, Ny, ncols, ldx, ldy, ldk, step_x, step_y, step_k};
    // K = PhiX PhiX^T: only what lies on or above the diagonal is computed, and written twice
    const bool sym = PhiX == PhiY && Nx == Ny && ldx == ldy && !rows_add_up;
    const auto count = [&](int64_t edge) {
        const int64_t ti = (Nx + edge - 1) / edge, tj = (Ny + edge - 1) / edge;
        return (sym ? ti * (ti + 1) / 2 : ti * tj) * batch;
    };
    // Large tiles run one per CU at a time or, faster together, two; with `rounds` = their number over 256, rounded up,
    // they take as long as about 1340 tiles of 64 x 64 per round do (measured for 201, 1025 and 5121 columns, both kinds,
    // symmetric and not: 2500 x 2500, 200 large or 1600 small tiles, 32 / 98 / 411 us against 36 / 108 / 477;
    // 4000 rows with themselves, 272 or 2016 tiles, 57 / 169 / 725 against 47 / 135 / 576).
    const int64_t tiles = big_tiles(Nx, Ny, sym), rounds = (tiles * batch + 255) / 256;
    if (count(64) > 1340 * rounds && ldx <= kBigMaxStride && ldy <= kBigMaxStride) {
        if (tiles > 0x7fffffffLL - 8) return hipErrorInvalidValue;
        const bool aligned = ldx % 4 == 0 && ldy % 4 == 0 && step_x % 4 == 0 && step_y % 4 == 0 &&
                             reinterpret_cast<uintptr_t>(PhiX) % 16 == 0 && reinterpret_cast<uintptr_t>(PhiY) % 16 == 0;
        const int64_t nti = (Nx + kBigM - 1) / kBigM, ntj = (Ny + kBigN - 1) / kBigN;
        const dim3 grid(xcd_grid(tiles), (unsigned)batch);
#define RFSF_BIG(AL, SY, FL) hipLaunchKernelGGL((gram_big<AL, SY, FL>), grid, dim3(256), 0, stream, g, tiles, nti, ntj)
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
    if (count(64) <= 150) return launch_small<1, 8>(g, sym, rows_add_up, batch, stream);
    if (count(64) <= 256) return launch_small<2, 8>(g, sym, rows_add_up, batch, stream);
    return launch_small<2, 4>(g, sym, rows_add_up, batch, stream);
}

}  // namespace rfsf
