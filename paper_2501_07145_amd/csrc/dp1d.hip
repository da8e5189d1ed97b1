// RFSF-DP-1D features (Sec. 3.3, eq. (dp1d)): F independent size-1 copies of the one-dimensional
// random Fourier signature feature map (static map of Sec. 3.1, eq. (rff_1d), scale of the appendix
// class RandomFourierFeatures1D; recursion of Sec. 3.2, eq. (rfsf_rec), p = 1):
//     phi_m(x)[i] = sqrt(2) cos((x . W_m[:, i]) / lengthscale + bias_m[i])
//     A_m[i] <- A_m[i] + A_{m-1}[i](before the step) * (phi_m(x_k)[i] - phi_m(x_{k-1})[i]),  A_0 = 1
//     out[n, 1 + (m-1) F + i] = A_m[i] / sqrt(F),  out[n, 0] = 1.
// One fused kernel, nothing but X, W and bias is read: components never interact, so no sketch and
// no FFT are needed and the increments never leave the chip.
#include "rfsf_internal.h"

#include <type_traits>

namespace rfsf {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kRows = 32;          // time points per tile
constexpr int kRawBufferWord3 = 0x00020000;   // buffer descriptor, last word: untyped 32-bit data
constexpr int kTileStride = 36;    // floats per component in the transposition tile: 16-byte accesses of 16
                                   // consecutive components then fall on 16 distinct groups of four banks

// sqrt(2) cos(pi x) to 1.5e-7 absolute (and what the rounding of x costs) for |x| < 2^22: x = k + r with |r| <= 1/2, k
// from adding 1.5 * 2^23, whose lowest mantissa bit is then the parity of k, and r exact; a degree-5 polynomial in
// r^2 (Chebyshev interpolant of sqrt(2) cos(pi sqrt(u)) on [0, 1/4]) and the sign (-1)^k, added to the sign bit.
// Half-turns rather than radians: the reduction takes no multiplication and rounds nothing. `rest` is what rounding the
// phase to half-turns has left of it. Eleven vector instructions against twelve, and vector instructions are what bounds
// the kernel (three wavefronts per SIMD; running a wavefront's matrix instructions under its own cosines changed nothing).
__device__ __forceinline__ float sqrt2_cospi(float x, float rest)
{
    const float t = x + 12582912.0f;
    const float r = (x - (t - 12582912.0f)) + rest;
    const float u = r * r;
    float p = fmaf(u, -0.0345010571f, 0.332251191f);
    p = fmaf(u, p, -1.88827479f);
    p = fmaf(u, p, 5.73988152f);
    p = fmaf(u, p, -6.97886419f);
    p = fmaf(u, p, 1.41421354f);
    return __uint_as_float((__float_as_uint(t) << 31) + __float_as_uint(p));
}

// orders the LDS accesses of one wavefront (the hardware runs them in program order; this keeps the
// compiler from moving them) without waiting for the global loads in flight
__device__ __forceinline__ void lds_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// The recurrence of one level down the rows of a tile for this lane's component. c: the component's
// sqrt(2) cos values in the transposition tile; E[r] holds, on entry, the previous level's accumulator
// before row r and, on exit, this level's.
template <bool FIRST_LEVEL, bool FULL>
__device__ __forceinline__ void run_rows(const float *c, bool first_tile, float (&E)[kRows], float &a, float &pc, int nrow)
{
#pragma unroll
    for (int g = 0; g < kRows / 4; ++g) {
        const floatx4 v = *reinterpret_cast<const floatx4 *>(c + 4 * g);
        if (g == 0) pc = first_tile ? v[0] : pc;           // first point of the sequence: no increment
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 4 * g + j;
            float u = v[j] - pc;
            if (FULL) {
                pc = v[j];
            } else {
                u = r < nrow ? u : 0.f;
                pc = r < nrow ? v[j] : pc;
            }
            const float e_old = FIRST_LEVEL ? 1.0f : E[r];
            E[r] = a;
            a = fmaf(e_old, u, a);
        }
    }
}

// Workgroup = (sequence, slab of 256 components), four wavefronts of 64 components each. Per tile of
// 32 time points and per level: theta = X_tile * W_m on the matrix cores (two 32x32 blocks per
// wavefront), sqrt(2) cos, transposed through a wavefront-private LDS tile so that lane c then owns
// component c for all 32 rows and runs the recurrence down the rows. E[r] carries, from one level
// to the next, the value of the previous level's accumulator before row r. The W columns of the next
// level are fetched right after the matrix instructions of the current one and land under its cosines.
template <int KSTEPS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KSTEPS <= 4 ? 4 : KSTEPS <= 16 ? 3 : 2, 4)))
void dp1d_features_kernel(
    const float *__restrict__ X, const float *__restrict__ W, const float *__restrict__ bias,
    float scale_turns, int64_t L, int d, int M, int F, float *__restrict__ out, int64_t ld_out)
{
    constexpr int KP = 2 * KSTEPS, XS = KP | 1;
    __shared__ float xs[2 * kRows * XS];
    __shared__ __attribute__((aligned(16))) float tile[4][64 * kTileStride];
    extern __shared__ float level_state[];             // [2][M][256]: accumulators, then last cosines
    float (*acc_state)[256] = reinterpret_cast<float (*)[256]>(level_state);
    float (*cos_state)[256] = reinterpret_cast<float (*)[256]>(level_state + (size_t)M * 256);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, col = lane & 31;
    const int64_t n = blockIdx.x;
    const int comp0 = blockIdx.y * 256 + wave * 64;
    const int my_comp = comp0 + lane;
    const float *xseq = X + n * L * d;
    for (int m = 0; m < M; ++m) acc_state[m][tid] = 0.f, cos_state[m][tid] = 0.f;

    constexpr int NX = (kRows * KP + 255) / 256;
    float xr[NX];
    auto fetch_tile = [&](int64_t t0) {
        const int nrow = (int)min((int64_t)kRows, L - t0);
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const int i = tid + 256 * u;
            const int r = i / KP, c = i - r * KP;
            xr[u] = (i < kRows * KP && r < nrow && c < d) ? xseq[(t0 + r) * d + c] : 0.f;
        }
    };
    auto put_tile = [&](float *buf) {
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const int i = tid + 256 * u;
            const int r = i / KP, c = i - r * KP;
            if (i < kRows * KP) buf[r * XS + c] = xr[u];
        }
    };
    // B fragments: this lane's W entries of one level for its two blocks of 32 components, fetched with
    // buffer loads: one descriptor per pair of rows (scalar registers only) whose extent ends with the
    // level's d rows, so that rows beyond d read as zero, and one constant lane offset per block.
    float w[2][KSTEPS], bm[2];
    const int fcol[2] = {min(comp0 + col, F - 1), min(comp0 + 32 + col, F - 1)};
    const int w_lane_offset[2] = {4 * (half * F + fcol[0]), 4 * (half * F + fcol[1])};
    auto fetch_w = [&](const float *wm, int m, int cb) {
        // the descriptors advance by two rows per step from values the compiler cannot hoist out of the
        // level loop (kept there, 3 K scalar registers would be spilled)
        int pair_bytes = 2 * F * 4, left = d * F * 4;
        asm volatile("" : "+s"(pair_bytes), "+s"(left));
        const char *base = reinterpret_cast<const char *>(wm);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(base), (short)0, left, kRawBufferWord3);
            w[cb][kk] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows, w_lane_offset[cb], 0, 0));
            const int adv = min(pair_bytes, left);
            base += adv;
            left -= adv;
        }
        bm[cb] = bias[(int64_t)m * F + fcol[cb]];
    };
    fetch_w(W, 0, 0);
    fetch_w(W, 0, 1);
    fetch_tile(0);
    put_tile(xs);
    __syncthreads();
    float *my_tile = tile[wave];
    int cur = 0;
    for (int64_t t0 = 0; t0 < L; t0 += kRows, cur ^= 1) {
        const int nrow = (int)min((int64_t)kRows, L - t0);
        const bool more = t0 + kRows < L;
        if (more) fetch_tile(t0 + kRows);
        const float *xt = xs + cur * (kRows * XS) + col * XS + half;
        float xa[KSTEPS];                                  // the tile's A fragments, for all levels
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) xa[kk] = xt[2 * kk];
        float E[kRows];
        for (int m = 0; m < M; ++m) {
            const int mn = m + 1 == M ? 0 : m + 1;
            const float *wn = W + (int64_t)mn * d * F;
            // per block of 32 components: projection, then the next level's W columns are requested, then the
            // cosines; lane (half, col) holds rows 8 g + 4 half + (0..3) of component col: one 16-byte store each
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KSTEPS; ++kk)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[kk], w[cb][kk], acc, 0, 0, 0);
                const float b = bm[cb] * 0.318309886183790672f;          // phase in half-turns, and what its rounding left
                const float rest = fmaf(bm[cb], 0.318309886183790672f, -b) + bm[cb] * 1.2841276486e-8f;
                fetch_w(wn, mn, cb);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    floatx4 v;
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = sqrt2_cospi(fmaf(acc[4 * g + j], scale_turns, b), rest);
                    *reinterpret_cast<floatx4 *>(my_tile + (32 * cb + col) * kTileStride + 8 * g + 4 * half) = v;
                    __builtin_amdgcn_sched_barrier(0);        // four cosines at a time: bounds their temporaries
                }
            }
            lds_order();
            // recurrence down the rows for this lane's component
            float a = acc_state[m][tid];
            float pc = cos_state[m][tid];
            const float *c = my_tile + lane * kTileStride;
            if (nrow == kRows) {
                if (m == 0) run_rows<true, true>(c, t0 == 0, E, a, pc, nrow);
                else run_rows<false, true>(c, t0 == 0, E, a, pc, nrow);
            } else {
                if (m == 0) run_rows<true, false>(c, t0 == 0, E, a, pc, nrow);
                else run_rows<false, false>(c, t0 == 0, E, a, pc, nrow);
            }
            acc_state[m][tid] = a;
            cos_state[m][tid] = pc;
            lds_order();
        }
        if (more) put_tile(xs + (cur ^ 1) * (kRows * XS));
        __syncthreads();
    }
    float *row = out + n * ld_out;
    if (blockIdx.y == 0 && tid == 0) row[0] = 1.0f;
    const float scale = 1.0f / sqrtf((float)F);
    if (my_comp < F)
        for (int m = 0; m < M; ++m) row[1 + (int64_t)m * F + my_comp] = acc_state[m][tid] * scale;
}

// Many sequences: the frequencies of 64 S components, split for the 16-bit matrix instructions, stay in LDS while a workgroup's
// wavefronts (twelve, eight from 19 channels on) go through sequences of their own, without meeting.
// A float is the sum of three bfloat16 numbers and six of the nine products are added up, smallest first (as in gram.hip; the three
// left out are below 2^-24 of the product): 8 instructions of 32 cycles for a tile of 32 points and 32 components of 17 channels
// where v_mfma_f32_32x32x2f32 takes 9 of 64, with less error (angles of 10 radians, 17 channels: root mean square 7.7e-7 in 32 bits).
// Two terms of half precision and three products would take 4, but err by 9.3e-7 there, 2.2e-7 instead of 1.0e-7 with 2 channels.
// Splitting the frequencies again for every tile would cost what they spare.
// The last term is 2^-16 of a number, and bfloat16 loses bits below 2^-126 as 32-bit numbers do: points of a tile that are all below
// 2^-63 are multiplied by kRaise before they are split, and the angle's factor is divided by it. (Points of 2^-120 with a lengthscale
// of 2^-120: root mean square error 1.5e-4 without, 2.9e-7 with it; a raised number meets the largest of 32 bits without overflow. The
// same for the frequencies of a workgroup would take 0.2 to 0.4 us of calls of 4 to 7 us.)
// Finite numbers from 0x1.ffp127 on are rounded to an infinite first term, whose rest is NaN: a tile with points of 2^127 and more is
// halved, and the first terms of frequencies end at the largest bfloat16 number (an infinity still leaves NaN: its last term is).
// Channels 2 k + half go to the lane's half of the products' columns, so that a lane splits the channels that it loads, in pairs p of
// k = 2 p and 2 p + 1. What a pair multiplies with what is laid out in tuples of four registers (an operand): of four pairs
// their hi, mid and lo; of a single one hi, mid, lo, hi; of two hi, hi, mid, mid and lo, lo, hi, hi.
// The lane that holds rows 8 g + 4 half + (0 .. 3) of a component gets the other four from the other half of the wavefront (v_permlane32_swap
// of the two blocks of 32 components): a transposition through LDS would take the room of the frequencies.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
// Wavefronts of a workgroup, one per CU: as many as hold the points' operands in registers.
__host__ __device__ constexpr int resident_waves(int KSTEPS) { return KSTEPS <= 9 ? 12 : 8; }
constexpr float kSmall = 0x1p-63f, kHuge = 0x1p127f, kRaise = 0x1p48f, kLargestTerm = 0x1.fep127f;
struct Terms { uint32_t hi, mid, lo; };
__device__ __forceinline__ uint32_t round_pair(float a, float b)
{
    const floatx2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
template <bool ANY_SIZE = false>
__device__ __forceinline__ Terms split_pair(float a, float b)
{
    Terms t;
    if constexpr (ANY_SIZE)
        t.hi = round_pair(__builtin_amdgcn_fmed3f(a, -kLargestTerm, kLargestTerm), __builtin_amdgcn_fmed3f(b, -kLargestTerm, kLargestTerm));
    else
        t.hi = round_pair(a, b);
    const float ra = a - __uint_as_float(t.hi << 16), rb = b - __uint_as_float(t.hi & 0xffff0000u);
    t.mid = round_pair(ra, rb);
    t.lo = round_pair(ra - __uint_as_float(t.mid << 16), rb - __uint_as_float(t.mid & 0xffff0000u));
    return t;
}
__host__ __device__ constexpr int pairs_of(int KSTEPS) { return (KSTEPS + 1) / 2; }
__host__ __device__ constexpr int right_tuples(int pairs) { return pairs / 4 * 3 + pairs % 4; }
__host__ __device__ constexpr int left_tuples(int pairs) { return pairs / 4 * 3 + (pairs % 4 == 0 ? 0 : pairs % 4 == 1 ? 2 : pairs % 4 == 2 ? 3 : 5); }
template <int PAIRS>
__device__ __forceinline__ void tuples_of_frequencies(const Terms (&w)[PAIRS], uint4 (&t)[right_tuples(PAIRS)])
{
    constexpr int Q = PAIRS / 4;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const Terms &a = w[4 * q], &b = w[4 * q + 1], &c = w[4 * q + 2], &d = w[4 * q + 3];
        t[3 * q] = make_uint4(a.hi, b.hi, c.hi, d.hi);
        t[3 * q + 1] = make_uint4(a.mid, b.mid, c.mid, d.mid);
        t[3 * q + 2] = make_uint4(a.lo, b.lo, c.lo, d.lo);
    }
    if constexpr (PAIRS % 4 >= 2) {
        const Terms &a = w[4 * Q], &b = w[4 * Q + 1];
        t[3 * Q] = make_uint4(a.hi, b.hi, a.mid, b.mid);
        t[3 * Q + 1] = make_uint4(a.lo, b.lo, a.hi, b.hi);
    }
    if constexpr (PAIRS % 2 == 1) {
        const Terms &a = w[PAIRS - 1];
        t[right_tuples(PAIRS) - 1] = make_uint4(a.hi, a.mid, a.lo, a.hi);
    }
}
template <int PAIRS>
__device__ __forceinline__ void tuples_of_points(const Terms (&x)[PAIRS], uint4 (&t)[left_tuples(PAIRS)])
{
    constexpr int Q = PAIRS / 4;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const Terms &a = x[4 * q], &b = x[4 * q + 1], &c = x[4 * q + 2], &d = x[4 * q + 3];
        t[3 * q] = make_uint4(a.hi, b.hi, c.hi, d.hi);
        t[3 * q + 1] = make_uint4(a.mid, b.mid, c.mid, d.mid);
        t[3 * q + 2] = make_uint4(a.lo, b.lo, c.lo, d.lo);
    }
    if constexpr (PAIRS % 4 >= 2) {
        const Terms &a = x[4 * Q], &b = x[4 * Q + 1];
        t[3 * Q] = make_uint4(a.lo, b.lo, a.mid, b.mid);
        t[3 * Q + 1] = make_uint4(a.hi, b.hi, a.hi, b.hi);
        t[3 * Q + 2] = make_uint4(a.hi, b.hi, a.mid, b.mid);
    }
    if constexpr (PAIRS % 2 == 1) {
        const Terms &a = x[PAIRS - 1];
        t[left_tuples(PAIRS) - 2] = make_uint4(a.lo, a.mid, 0u, 0u);
        t[left_tuples(PAIRS) - 1] = make_uint4(a.hi, a.hi, a.hi, a.mid);
    }
}
// Products of 32 points with 32 components; right: the lane's tuples of frequencies in LDS, 64 apart.
template <int PAIRS>
__device__ __forceinline__ floatx16 multiply(const uint4 (&x)[left_tuples(PAIRS)], const uint4 *right)
{
    constexpr int Q = PAIRS / 4;
    floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto product = [&](const uint4 &a, const uint4 &b) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint4 hi = right[64 * (3 * q)], mid = right[64 * (3 * q + 1)], lo = right[64 * (3 * q + 2)];
        product(x[3 * q + 2], hi);
        product(x[3 * q], lo);
        product(x[3 * q + 1], mid);
        product(x[3 * q + 1], hi);
        product(x[3 * q], mid);
        product(x[3 * q], hi);
    }
    if constexpr (PAIRS % 4 >= 2) {
        const uint4 a = right[64 * (3 * Q)], b = right[64 * (3 * Q + 1)];
        product(x[3 * Q], a);
        product(x[3 * Q + 2], b);
        product(x[3 * Q + 1], a);
    }
    if constexpr (PAIRS % 2 == 1) {
        const uint4 a = right[64 * (right_tuples(PAIRS) - 1)];
        product(x[left_tuples(PAIRS) - 2], a);
        product(x[left_tuples(PAIRS) - 1], a);
    }
    return acc;
}
// LDS of a resident workgroup: frequencies and phases of S blocks of 64 components, accumulators and last cosines of the wavefronts.
__host__ __device__ constexpr size_t resident_lds(int KSTEPS, int M, int S)
{
    return (size_t)M * S * (2 * right_tuples(pairs_of(KSTEPS)) * 64 * sizeof(uint4) + 64 * sizeof(float)) +
           (size_t)resident_waves(KSTEPS) * M * 2 * 64 * sizeof(float);
}
template <int KSTEPS>
__global__ __launch_bounds__(64 * resident_waves(KSTEPS)) __attribute__((amdgpu_waves_per_eu(resident_waves(KSTEPS) / 4, resident_waves(KSTEPS) / 4))) void dp1d_resident_kernel(
    const float *__restrict__ X, const float *__restrict__ W, const float *__restrict__ bias, float scale_turns, int64_t N,
    int64_t L, int d, int M, int F, int S, float *__restrict__ out, int64_t ld_out)
{
    constexpr int PAIRS = pairs_of(KSTEPS), RT = right_tuples(PAIRS), WAVES = resident_waves(KSTEPS);
    extern __shared__ __attribute__((aligned(16))) char resident[];
    uint4 *freq = reinterpret_cast<uint4 *>(resident);                              // [M][S][2][RT][64]
    float *phase = reinterpret_cast<float *>(freq + (size_t)M * S * 2 * RT * 64);   // [M][S][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *state = phase + (size_t)M * S * 64 + (size_t)wave * M * 128;             // [M][2][64]
    const int half = lane >> 5, col = lane & 31;
    const int comp0 = blockIdx.y * (64 * S);
    for (int i = tid; i < M * S * 128; i += 64 * WAVES) {
        const int l = i & 63, cb = (i >> 6) & 1, ms = i >> 7, m = ms / S, s = ms - m * S;
        const int comp = min(comp0 + 64 * s + 32 * cb + (l & 31), F - 1);
        const float *src = W + (int64_t)m * d * F + comp;
        Terms w[PAIRS];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const int c0 = 4 * p + (l >> 5), c1 = c0 + 2;
            w[p] = split_pair<true>(c0 < d ? src[(int64_t)c0 * F] : 0.f, c1 < d ? src[(int64_t)c1 * F] : 0.f);
        }
        uint4 t[RT];
        tuples_of_frequencies<PAIRS>(w, t);
#pragma unroll
        for (int r = 0; r < RT; ++r) freq[((size_t)(ms * 2 + cb) * RT + r) * 64 + l] = t[r];
    }
    for (int i = tid; i < M * S * 64; i += 64 * WAVES) {
        const int m = i / (64 * S), comp = comp0 + i - m * (64 * S);
        phase[i] = bias[(int64_t)m * F + min(comp, F - 1)];
    }
    __syncthreads();
    const int sub = wave % S, my_comp = comp0 + 64 * sub + lane;
    if (comp0 + 64 * sub >= F) return;                       // (no block of components for this wavefront)
    const int64_t at_once = (int64_t)gridDim.x * (WAVES / S);
    const float out_scale = 1.0f / sqrtf((float)F);
    float raw[2 * PAIRS];
    auto fetch = [&](int64_t n, int64_t t0) {                // rows beyond the sequence are its last one, channels beyond d meet zeros
        const float *src = X + (n * L + min(t0 + col, L - 1)) * d;
#pragma unroll
        for (int k = 0; k < 2 * PAIRS; ++k) raw[k] = src[min(2 * k + half, d - 1)];
    };
    int64_t n = (int64_t)(wave / S) * gridDim.x + blockIdx.x;      // (what does not fill a round is spread over the CUs)
    if (n < N) fetch(n, 0);
    for (; n < N; n += at_once) {
        for (int m = 0; m < M; ++m) state[m * 128 + lane] = 0.f;
        for (int64_t t0 = 0; t0 < L; t0 += kRows) {
            const int nrow = (int)min((int64_t)kRows, L - t0);
            float most = 0.f;                                // the largest point, a NaN aside
#pragma unroll
            for (int k = 0; k < 2 * PAIRS; k += 2) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(raw[k]), "v"(raw[k + 1]));
            float turns = scale_turns;
            if (__ballot(!(most < kSmall)) == 0) {
                turns *= 1.0f / kRaise;
#pragma unroll
                for (int k = 0; k < 2 * PAIRS; ++k) raw[k] *= kRaise;
            } else if (__ballot(most >= kHuge) != 0) {
                turns *= 2.0f;
#pragma unroll
                for (int k = 0; k < 2 * PAIRS; ++k) raw[k] *= 0.5f;
            }
            Terms xt[PAIRS];
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) xt[p] = split_pair(raw[2 * p], raw[2 * p + 1]);
            uint4 x[left_tuples(PAIRS)];
            tuples_of_points<PAIRS>(xt, x);
            const bool more = t0 + kRows < L;                // the next tile, or the first one of the next sequence
            fetch(more ? n : min(n + at_once, N - 1), more ? t0 + kRows : 0);
            float E[kRows];                                  // the level below before each row; level 0 is 1
#pragma unroll
            for (int r = 0; r < kRows; ++r) E[r] = 1.0f;
            for (int m = 0; m < M; ++m) {
                const uint4 *right = freq + (size_t)((m * S + sub) * 2) * RT * 64 + lane;
                const floatx16 acc[2] = {multiply<PAIRS>(x, right), multiply<PAIRS>(x, right + RT * 64)};
                const float bm = phase[(m * S + sub) * 64 + lane];
                const float b = bm * 0.318309886183790672f;          // phase in half-turns, and what its rounding left
                const float rest = fmaf(bm, 0.318309886183790672f, -b) + bm * 1.2841276486e-8f;
                float a = state[m * 128 + lane], pc = state[m * 128 + 64 + lane];
                auto rows = [&](auto full_tag) {
                    constexpr bool FULL = decltype(full_tag)::value;
#pragma unroll
                    for (int g = 0; g < kRows / 8; ++g) {
                        if (!FULL && 8 * g >= nrow) break;
                        float c[8];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[0][4 * g + j]), __float_as_uint(acc[1][4 * g + j]), false, false);
                            c[j] = sqrt2_cospi(fmaf(__uint_as_float(both[0]), turns, b), rest);
                            c[4 + j] = sqrt2_cospi(fmaf(__uint_as_float(both[1]), turns, b), rest);
                        }
                        if (g == 0) pc = t0 == 0 ? c[0] : pc;        // first point of the sequence: no increment
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int r = 8 * g + j;
                            const float u = FULL || r < nrow ? c[j] - pc : 0.f, below = E[r];
                            pc = FULL || r < nrow ? c[j] : pc;
                            E[r] = a;
                            a = fmaf(below, u, a);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                if (nrow == kRows) rows(std::integral_constant<bool, true>{});
                else rows(std::integral_constant<bool, false>{});
                state[m * 128 + lane] = a;
                state[m * 128 + 64 + lane] = pc;
            }
        }
        if (my_comp < F) {
            float *row = out + n * ld_out;
            if (my_comp == 0) row[0] = 1.0f;
            for (int m = 0; m < M; ++m) row[1 + (int64_t)m * F + my_comp] = state[m * 128 + lane] * out_scale;
        }
    }
}

// Few long sequences: workgroup = (sequence, 64 components), eight wavefronts that share out the time points, a stretch
// of 31 or more steps each (whole tiles; a stretch starts with the last point of the one before). A wavefront runs the recurrence for
// every first level at once, A^{(a..l)} for all a <= l (E[a][r]: the sum of the level below before row r), and the
// first wavefront joins the eight stretches from left to right through LDS. Registers hold it all up to five levels
// (four with more than 32 channels);
// one workgroup per CU. Nothing but LDS is needed beyond what the whole-sequence kernel takes.
constexpr int kStretches = 8;
constexpr int kMaxSplitLevels = 5;
constexpr int64_t kSplitPoints = 65, kSplitWorkgroups = 128;
template <int KSTEPS, int M>
__global__ __launch_bounds__(64 * kStretches) __attribute__((amdgpu_waves_per_eu(2, 2))) void dp1d_stretches_kernel(
    const float *__restrict__ X, const float *__restrict__ W, const float *__restrict__ bias,
    float scale_turns, int64_t L, int64_t steps, int d, int F, float *__restrict__ out, int64_t ld_out)
{
    constexpr int KP = 2 * KSTEPS, XS = KP | 1, NA = M * (M + 1) / 2;
    static_assert(NA * 64 <= 64 * kTileStride, "the sums of a stretch fit its tile");
    __shared__ __attribute__((aligned(16))) float tile[kStretches][64 * kTileStride];
    __shared__ float xs[kStretches][kRows * XS];
    constexpr auto at = [](int a, int l) { return a * M - a * (a - 1) / 2 + l - a; };
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int64_t n = blockIdx.x;
    const int comp0 = blockIdx.y * 64;
    const float *xseq = X + n * L * d;
    float *my_tile = tile[wave], *my_x = xs[wave];
    const int fcol[2] = {min(comp0 + col, F - 1), min(comp0 + 32 + col, F - 1)};
    const int64_t begin = wave * steps, end = min(begin + steps, L - 1);       // first and last point of the stretch

    float A[NA], pc[M], E[M][kRows];
#pragma unroll
    for (int i = 0; i < NA; ++i) A[i] = 0.f;
#pragma unroll
    for (int m = 0; m < M; ++m) pc[m] = 0.f;
    float w[2][KSTEPS], bm[2];
    const int w_lane_offset[2] = {4 * (half * F + fcol[0]), 4 * (half * F + fcol[1])};
    auto fetch = [&](const float *Wp, const float *bp, int m, int cb) {        // as in the whole-sequence kernel
        int pair_bytes = 2 * F * 4, left = d * F * 4;
        const char *base = reinterpret_cast<const char *>(Wp + (int64_t)m * d * F);
        asm volatile("" : "+s"(pair_bytes), "+s"(left));
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(base), (short)0, left, kRawBufferWord3);
            w[cb][kk] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows, w_lane_offset[cb], 0, 0));
            const int adv = min(pair_bytes, left);
            base += adv;
            left -= adv;
        }
        bm[cb] = bp[(int64_t)m * F + fcol[cb]];
    };
    fetch(W, bias, 0, 0);
    fetch(W, bias, 0, 1);
    for (int64_t t0 = begin; begin < L - 1 && t0 <= end; t0 += kRows) {
        const int nrow = (int)min((int64_t)kRows, end + 1 - t0);
        for (int i = lane; i < kRows * KP; i += 64) {
            const int r = i / KP, c = i - r * KP;
            my_x[r * XS + c] = r < nrow && c < d ? xseq[(t0 + r) * d + c] : 0.f;
        }
        lds_order();
        // (otherwise the compiler keeps the columns of all levels in registers, and spills them)
        const float *wt = W, *bt = bias;
        asm volatile("" : "+s"(wt), "+s"(bt));
#pragma unroll
        for (int m = 0; m < M; ++m) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KSTEPS; ++kk)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(my_x[col * XS + half + 2 * kk], w[cb][kk], acc, 0, 0, 0);
                const float b = bm[cb] * 0.318309886183790672f;
                const float rest = fmaf(bm[cb], 0.318309886183790672f, -b) + bm[cb] * 1.2841276486e-8f;
                fetch(wt, bt, m + 1 < M ? m + 1 : 0, cb);              // the block's columns of the next level
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    floatx4 v;
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = sqrt2_cospi(fmaf(acc[4 * g + j], scale_turns, b), rest);
                    *reinterpret_cast<floatx4 *>(my_tile + (32 * cb + col) * kTileStride + 8 * g + 4 * half) = v;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            lds_order();
#pragma unroll
            for (int g = 0; g < kRows / 4; ++g) {
                const floatx4 v = *reinterpret_cast<const floatx4 *>(my_tile + lane * kTileStride + 4 * g);
                if (g == 0) pc[m] = t0 == begin ? v[0] : pc[m];       // first point of the stretch: no increment
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 4 * g + j;
                    const float u = r < nrow ? v[j] - pc[m] : 0.f;
                    pc[m] = r < nrow ? v[j] : pc[m];
#pragma unroll
                    for (int a = 0; a <= m; ++a) {
                        const float below = a < m ? E[a][r] : 1.0f, old = A[at(a, m)];
                        E[a][r] = old;
                        A[at(a, m)] = fmaf(below, u, old);
                    }
                }
            }
            lds_order();
        }
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) my_tile[64 * i + lane] = A[i];
    __syncthreads();
    if (wave != 0) return;
    for (int s = 1; s < kStretches; ++s) {                            // A^{(1..l)} of what is joined so far
        float B[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) B[i] = tile[s][64 * i + lane];
#pragma unroll
        for (int l = M - 1; l >= 0; --l) {                            // descending: the lower levels are still the old ones
            float acc = A[l] + B[l];
#pragma unroll
            for (int j = 1; j <= l; ++j) acc = fmaf(A[j - 1], B[at(j, l)], acc);
            A[l] = acc;
        }
    }
    float *row = out + n * ld_out;
    if (blockIdx.y == 0 && lane == 0) row[0] = 1.0f;
    const float scale = 1.0f / sqrtf((float)F);
    if (comp0 + lane < F) {
#pragma unroll
        for (int m = 0; m < M; ++m) row[1 + (int64_t)m * F + comp0 + lane] = A[m] * scale;
    }
}

template <int KSTEPS>
hipError_t launch_stretches(const float *X, const float *W, const float *bias, float scale_turns, int64_t N,
                            int64_t L, int d, int M, int F, float *out, int64_t ld_out, hipStream_t stream)
{
    // steps of a stretch: whole tiles with the point that it shares with the one before
    const int64_t each = (L - 1 + kStretches - 1) / kStretches, steps = (each + 1 + kRows - 1) / kRows * kRows - 1;
    const dim3 grid((unsigned)N, (unsigned)((F + 63) / 64));
    switch (M) {
#define RFSF_STRETCHES_CASE(LEVELS)                                                                           \
    case LEVELS:                                                                                              \
        hipLaunchKernelGGL((dp1d_stretches_kernel<KSTEPS, LEVELS>), grid, dim3(64 * kStretches), 0, stream, X, W, bias, \
                           scale_turns, L, steps, d, F, out, ld_out);                                     \
        break
        RFSF_STRETCHES_CASE(1);
        RFSF_STRETCHES_CASE(2);
        RFSF_STRETCHES_CASE(3);
        RFSF_STRETCHES_CASE(4);
    case 5:
        if constexpr (KSTEPS <= 16) {
            hipLaunchKernelGGL((dp1d_stretches_kernel<KSTEPS, 5>), grid, dim3(64 * kStretches), 0, stream, X, W, bias,
                               scale_turns, L, steps, d, F, out, ld_out);
            break;
        }
        return hipErrorInvalidValue;
#undef RFSF_STRETCHES_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Blocks of 64 components that a workgroup of the resident kernel holds: those of 1, 2, 3, 4 that keep most of the wavefronts of the chip
// at work in every round of sequences; 0 where even one does not fit the LDS, or where the kernel above is the faster one: up to
// six channels, whose 32-bit products cost little, unless it has more to do for its slabs of 256 components and whole last tiles.
// Kernel above and this one, us: 4999 x 257 points, 1000 components, five levels, d = 4 2470 and 2535, 8 2805 and 2690, 12 3375 and 2900,
// 17 3840 and 3235 (3250 to 3530 from box to box), 32 5735 and 3775, 64 9010 and 5805; 1500 x 256, 256 components, d = 2, 4, 6, 8 164, 174,
// 189, 203 and 191, 190, 195, 195; 1500 x 100, 128 components, d = 2 84 and 44; 130 x 257, 256 components, d = 17 81 and 61; 20000 x 2,
// 64 components, d = 3 310 and 45.
// Of few levels the loads and the split of a tile's points are more of its cost, and batches that leave each workgroup of the kernel
// above a CU or half of one have less to gain: with one level 7 x 22 points, six channels, 97 components 4.1 and 4.6 us, 36 x 53, 50,
// 1461 10.9 and 14.6, 30 x 23, 5, 419 4.2 and 4.7, 864 x 151, 5, 1719 105 and 121, 364 x 55, 56, 507 24 and 34, but 407 x 55, 34, 354 26
// and 17; two levels 4916 x 262, 6, 2047 2100 and 2285, 97 x 18, 60, 492 10.1 and 11.8; small batches of more levels
// gain as large ones do (24 x 3, 39, 1010, three levels 11.3 and 8.2, 80 x 237, 49, 935, five 204 and 116). Of 4300 drawn shapes, 2000 of one
// level, 1500 of two and three with F just below multiples of 256, 24 are slower by these lines by more than 4 % and 0.3 us, one by 21 %; on
// average they take 0.74 of the time of the kernel above.
constexpr int64_t kCUs = 256;
// What a whole tile of 64 components costs, where one of the kernel above costs 1 (0: less, whatever that has to do for its slabs).
template <int KSTEPS>
double dearer_tile(int M, bool few)
{
    if (KSTEPS <= 3) return (KSTEPS == 1 ? 1.08 : KSTEPS == 2 ? 1.0 : 0.95) + 0.43 / (double)(M < 5 ? M : 5);
    if (M == 1 && (few || KSTEPS > 24)) return 1.4;
    if (M <= 2 && KSTEPS == 4) return 1.1;
    return M <= 3 && few && KSTEPS > 24 ? 1.25 : 0.0;
}
struct Resident { int blocks; int64_t per_slab; };
template <int KSTEPS>
Resident resident_plan(int64_t N, int64_t L, int M, int F)
{
    Resident best = {0, 0};
    const int64_t blocks = (F + 63) / 64, rest = L % kRows;
    const int64_t others = N * ((F + 255) / 256);            // workgroups of the kernel above
    const double tiles = (double)(L / kRows) + (rest == 0 ? 0.0 : 0.3 + 0.175 * (double)((rest + 7) / 8));
    if (dearer_tile<KSTEPS>(M, others <= 2 * kCUs) * tiles * (double)blocks > (double)((L + kRows - 1) / kRows * ((F + 255) / 256 * 4))) return best;
    if (M == 1 && others <= (KSTEPS <= 3 && L <= kRows ? 2 : 1) * kCUs && (L > 8 || KSTEPS > 16) && L <= (KSTEPS <= 3 ? 2 : 1) * kRows) return best;
    double most = 0.0;
    for (int S = 1; S <= 4; ++S) {
        if (resident_lds(KSTEPS, M, S) > kLdsPerCu) break;
        const int64_t slabs = (blocks + S - 1) / S;
        if (resident_waves(KSTEPS) % S != 0 || slabs > 65535) continue;
        const int64_t per_slab = slabs < kCUs ? kCUs / slabs : 1, at_once = per_slab * (resident_waves(KSTEPS) / S);
        const int64_t rounds = (N + at_once - 1) / at_once;
        // wavefronts with a sequence, of those of whole rounds of workgroups on all CUs
        const double busy = (double)(blocks * N) / (double)(rounds * resident_waves(KSTEPS) * kCUs * ((slabs * per_slab + kCUs - 1) / kCUs));
        if (busy > most) most = busy, best = {S, per_slab};
    }
    return best;
}
template <int KSTEPS>
hipError_t launch_resident(const Resident &plan, const float *X, const float *W, const float *bias, float scale_turns, int64_t N,
                           int64_t L, int d, int M, int F, float *out, int64_t ld_out, hipStream_t stream)
{
    const size_t lds = resident_lds(KSTEPS, M, plan.blocks);
    static LdsLimit limit;
    const hipError_t e = allow_lds(limit, reinterpret_cast<const void *>(dp1d_resident_kernel<KSTEPS>), lds);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(N < plan.per_slab ? N : plan.per_slab), (unsigned)((F + 64 * plan.blocks - 1) / (64 * plan.blocks)));
    hipLaunchKernelGGL(dp1d_resident_kernel<KSTEPS>, grid, dim3(64 * resident_waves(KSTEPS)), lds, stream, X, W, bias, scale_turns, N, L, d, M, F,
                       plan.blocks, out, ld_out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dp1d(const float *X, const float *W, const float *bias, float scale_turns, int64_t N,
                       int64_t L, int d, int M, int F, float *out, int64_t ld_out, hipStream_t stream)
{
    if (N == 0) return hipSuccess;
    // Workgroups of the whole-sequence kernel, three of which a CU holds, against half the CUs
    if (M <= (d <= 32 ? kMaxSplitLevels : kMaxSplitLevels - 1) && L >= kSplitPoints && N * ((F + 255) / 256) <= kSplitWorkgroups && (F + 63) / 64 <= 65535) {
        if (d <= 4) return launch_stretches<2>(X, W, bias, scale_turns, N, L, d, M, F, out, ld_out, stream);
        if (d <= 8) return launch_stretches<4>(X, W, bias, scale_turns, N, L, d, M, F, out, ld_out, stream);
        if (d <= 18) return launch_stretches<9>(X, W, bias, scale_turns, N, L, d, M, F, out, ld_out, stream);
        if (d <= 32) return launch_stretches<16>(X, W, bias, scale_turns, N, L, d, M, F, out, ld_out, stream);
        return launch_stretches<32>(X, W, bias, scale_turns, N, L, d, M, F, out, ld_out, stream);
    }
    dim3 grid((unsigned)N, (unsigned)((F + 255) / 256));
    const size_t dyn = sizeof(float) * 2 * (size_t)M * 256;
    // static LDS of the kernel (X double buffer + transposition tiles) plus the per-level state can pass
    // 64 KB for many levels on a wide state
#define RFSF_LAUNCH_DP1D(KS)                                                                                  \
    do {                                                                                                      \
        const Resident plan = resident_plan<KS>(N, L, M, F);                                                  \
        if (plan.blocks > 0) return launch_resident<KS>(plan, X, W, bias, scale_turns, N, L, d, M, F, out, ld_out, stream); \
        constexpr size_t kStatic = sizeof(float) * (2 * kRows * ((2 * KS) | 1) + 4 * 64 * kTileStride);             \
        static LdsLimit limit;                                                                                \
        const hipError_t e = allow_lds(limit, reinterpret_cast<const void *>(dp1d_features_kernel<KS>), dyn, kStatic); \
        if (e != hipSuccess) return e;                                                                        \
        hipLaunchKernelGGL(dp1d_features_kernel<KS>, grid, dim3(256), dyn, stream, X, W, bias,                \
                           scale_turns, L, d, M, F, out, ld_out);                                         \
    } while (0)
    // Matrix instructions and loads of W for padding channels cost as much as for others, 0.26 ms per pair of them in 4999 x 257
    // points, 1000 components, five levels: with pairs 2, 4, 9, 16 and 32 alone, d = 6 2.75 -> 2.52 ms, 12 3.79 -> 3.36, 24 5.71 ->
    // 4.43, 40 9.73 -> 6.89, 48 9.74 -> 7.46, and 64 9.76 -> 8.90 with the points' fragments kept in registers.
    if (d <= 2) RFSF_LAUNCH_DP1D(1);
    else if (d <= 4) RFSF_LAUNCH_DP1D(2);
    else if (d <= 6) RFSF_LAUNCH_DP1D(3);
    else if (d <= 8) RFSF_LAUNCH_DP1D(4);
    else if (d <= 12) RFSF_LAUNCH_DP1D(6);
    else if (d <= 18) RFSF_LAUNCH_DP1D(9);
    else if (d <= 24) RFSF_LAUNCH_DP1D(12);
    else if (d <= 32) RFSF_LAUNCH_DP1D(16);
    else if (d <= 40) RFSF_LAUNCH_DP1D(20);
    else if (d <= 48) RFSF_LAUNCH_DP1D(24);
    else RFSF_LAUNCH_DP1D(32);
#undef RFSF_LAUNCH_DP1D
    return hipGetLastError();
}

}  // namespace rfsf
