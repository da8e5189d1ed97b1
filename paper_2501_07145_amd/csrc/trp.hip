// RFSF-TRP (Sec. 3.4, eqs. (trp_def), (trp), (trp_rec); appendix class TensorizedRandomProjection):
// the increments of the random Fourier features are projected per level by an independent Gaussian
// matrix Z_m [Q x 2F] (one GEMM per level on the matrix cores, the same kernel as the feature Gram)
// and combined over time by Hadamard products,
//     A_m <- A_m + A_{m-1}(before the step) (.) (Z_m delta_m[k]),  A_0 = 1,  Phi_m = A_m / sqrt(Q).
// This file holds the second stage: the recurrence over time, one thread per sequence and one or four
// components, or per piece of a sequence and component.
#include "rfsf_internal.h"

#include <cmath>

namespace rfsf {
namespace {


typedef float floatv4 __attribute__((ext_vector_type(4)));

template <int V> struct Vec;
template <> struct Vec<1> { typedef float type; };
template <> struct Vec<4> { typedef floatv4 type; };
__device__ __forceinline__ float lane_of(float v, int) { return v; }
__device__ __forceinline__ float lane_of(floatv4 v, int i) { return v[i]; }

// P[(n*rows + k)*M*Q + m*Q + q] = Z_m . (delta_m[k] / 2)  (the projection kernel writes halved increments;
// the factor 2 is restored here). A thread owns V consecutive components of one sequence (V = 4: 16-byte
// loads; the threads of a sequence then read whole rows of P, and consecutive levels and time steps
// continue the same stream); B time steps are loaded per batch so that B*M loads are in flight per
// thread. The last, partial batch loads clamped rows and skips their updates.
template <int kMaxLevels, int B, int V>
__global__ __launch_bounds__(256) void trp_scan_kernel(const float *__restrict__ P, int64_t n_seq, int64_t L, int64_t rows, int M,
                                                       int Q, float *__restrict__ out, int64_t ld_out, float scale)
{
    typedef typename Vec<V>::type vec;
    const int QV = (Q + V - 1) / V;
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t n = g / QV;
    if (n >= n_seq) return;
    const int q = (int)(g - n * QV) * V;
    float *row = out + n * ld_out;
    if (q == 0) row[0] = 1.0f;
    float A[kMaxLevels][V];
#pragma unroll
    for (int m = 0; m < kMaxLevels; ++m)
#pragma unroll
        for (int i = 0; i < V; ++i) A[m][i] = 0.f;
    const int64_t T = L - 1, MQ = (int64_t)M * Q;
    const float *p = P + n * rows * MQ + q;
    for (int64_t k = 0; k < T; k += B) {
        vec v[B][kMaxLevels];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int64_t kj = min(k + j, T - 1);
#pragma unroll
            for (int m = 0; m < kMaxLevels; ++m)
                v[j][m] = *reinterpret_cast<const vec *>(p + kj * MQ + (int64_t)min(m, M - 1) * Q);
        }
#pragma unroll
        for (int j = 0; j < B; ++j)
            if (k + j < T) {
#pragma unroll
                for (int m = kMaxLevels - 1; m >= 0; --m)         // descending: A[m-1] is still the old value
                    if (m < M) {
#pragma unroll
                        for (int i = 0; i < V; ++i)
                            A[m][i] = fmaf(m ? A[m - 1][i] : 1.0f, 2.0f * lane_of(v[j][m], i), A[m][i]);
                    }
            }
    }
#pragma unroll
    for (int m = 0; m < kMaxLevels; ++m)
        if (m < M) {
#pragma unroll
            for (int i = 0; i < V; ++i) row[1 + (int64_t)m * Q + q + i] = A[m][i] * scale;
        }
}

// Few long sequences: a sequence is cut into pieces of `steps` time steps, one thread per component of a piece, which
// runs the recurrence for every first level at once (A^{(a..l)}, all a <= l) and leaves the sums in its own column of
// the rows it has read: the piece's part of P, seen as [steps * M][Q], takes M(M+1)/2 of them per component.
template <int M, int B>
__global__ __launch_bounds__(256) void trp_pieces_kernel(float *P, int64_t n_seq, int64_t L, int64_t rows, int Q, int pieces, int64_t steps)
{
    constexpr int NA = M * (M + 1) / 2;
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x, v = g / Q, n = v / pieces;
    if (n >= n_seq) return;
    const int64_t T = L - 1, k0 = (v - n * pieces) * steps, k1 = min(k0 + steps, T);
    constexpr auto at = [](int a, int l) { return a * M - a * (a - 1) / 2 + l - a; };
    const int64_t MQ = (int64_t)M * Q;
    float *p = P + n * rows * MQ + (g - v * Q);
    float A[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) A[i] = 0.f;
    for (int64_t k = k0; k < k1; k += B) {
        float u[B][M];
#pragma unroll
        for (int j = 0; j < B; ++j)
#pragma unroll
            for (int m = 0; m < M; ++m) u[j][m] = p[min(k + j, k1 - 1) * MQ + (int64_t)m * Q];
#pragma unroll
        for (int j = 0; j < B; ++j)
            if (k + j < k1) {
#pragma unroll
                for (int l = M - 1; l >= 0; --l)                    // descending: the lower levels are still the old ones
#pragma unroll
                    for (int a = 0; a <= l; ++a)
                        A[at(a, l)] = fmaf(l > a ? A[at(a, l > a ? l - 1 : l)] : 1.0f, 2.0f * u[j][l], A[at(a, l)]);
            }
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) p[k0 * MQ + (int64_t)i * Q] = A[i];
}

// The pieces of a sequence from left to right (A^{(1..l)}(xy) = A^{(1..l)}(x) + A^{(1..l)}(y) + sum over j of
// A^{(1..j)}(x) A^{(j+1..l)}(y)), one thread per component; the numbers of the next kAhead pieces are in flight.
template <int M>
__global__ __launch_bounds__(64) void trp_join_kernel(const float *__restrict__ P, int64_t n_seq, int64_t rows, int Q, int pieces,
                                                      int64_t steps, float *__restrict__ out, int64_t ld_out, float scale)
{
    constexpr int NA = M * (M + 1) / 2, kAhead = 4;
    const int64_t g = (int64_t)blockIdx.x * 64 + threadIdx.x, n = g / Q;
    if (n >= n_seq) return;
    const int q = (int)(g - n * Q);
    constexpr auto at = [](int a, int l) { return a * M - a * (a - 1) / 2 + l - a; };
    const int64_t MQ = (int64_t)M * Q, stride = steps * MQ;
    const float *p = P + n * rows * MQ + q;
    float A[M], B[kAhead][NA];
#pragma unroll
    for (int m = 0; m < M; ++m) A[m] = p[(int64_t)m * Q];
    auto fetch = [&](int slot, int s) {
#pragma unroll
        for (int i = 0; i < NA; ++i) B[slot][i] = p[s * stride + (int64_t)i * Q];
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
        if (1 + i < pieces) fetch(i, 1 + i);
    for (int s0 = 1; s0 < pieces; s0 += kAhead) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (s0 + i < pieces) {
#pragma unroll
                for (int l = M - 1; l >= 0; --l) {
                    float acc = A[l] + B[i][at(0, l)];
#pragma unroll
                    for (int j = 1; j <= l; ++j) acc = fmaf(A[j - 1], B[i][at(j, l)], acc);
                    A[l] = acc;
                }
                if (s0 + i + kAhead < pieces) fetch(i, s0 + i + kAhead);
            }
        }
    }
    float *row = out + n * ld_out;
    if (q == 0) row[0] = 1.0f;
#pragma unroll
    for (int m = 0; m < M; ++m) row[1 + (int64_t)m * Q + q] = A[m] * scale;
}

// Pieces per sequence (1: whole). A batch of four steps takes a thread about 1.5 us whatever the number of threads, a
// piece of the join 0.25 us, so a sequence of T steps is best cut into about sqrt(1.5 T) pieces; no more than
// fill the chip with four wavefronts per SIMD, at least 32 steps each, and no cut where the whole sequences have a thread
// for every lane of one wavefront per SIMD. A function of the batch, N sequences, however many of them a launch takes: the
// workspace does not decide in which order a sequence is summed up.
constexpr int64_t kLanes = 256 * 4 * 64;
struct TrpCut { int pieces; int64_t steps; };
TrpCut trp_cut(int64_t N, int64_t L, int M, int Q)
{
    const int64_t T = L - 1, threads = (N < kLanes ? N : kLanes) * Q;
    if (M > 8 || threads >= kLanes) return {1, T};
    int64_t want = (int64_t)sqrt(1.5 * (double)T);
    if (want > 4 * kLanes / threads) want = 4 * kLanes / threads;
    if (want > T / 32) want = T / 32;
    for (; want >= 4; --want) {                      // (three passes over fewer pieces gain nothing)
        const int64_t steps = (T + want - 1) / want, pieces = (T + steps - 1) / steps;
        // the last piece, too, has to hold its sums, (M+1)/2 rows of P
        if (2 * (T - (pieces - 1) * steps) >= M + 1) return {(int)pieces, steps};
    }
    return {1, T};
}

}  // namespace

hipError_t launch_trp_scan(float *P, int64_t N, int64_t n_seq, int64_t L, int64_t rows, int M, int Q, float *out, int64_t ld_out,
                           hipStream_t stream)
{
    if (n_seq == 0) return hipSuccess;
    const float scale = 1.0f / sqrtf((float)Q);
    const TrpCut cut = trp_cut(N, L, M, Q);
    if (cut.pieces > 1) {
        const int64_t piece_blocks = (n_seq * cut.pieces * Q + 255) / 256, join_blocks = (n_seq * Q + 63) / 64;
        if (piece_blocks > 2147483647 || join_blocks > 2147483647) return hipErrorInvalidValue;
        switch (M) {
#define RFSF_TRP_PIECES_CASE(LEVELS)                                                                          \
    case LEVELS:                                                                                              \
        hipLaunchKernelGGL((trp_pieces_kernel<LEVELS, (64 / LEVELS > 16 ? 16 : 64 / LEVELS)>), dim3((unsigned)piece_blocks), \
                           dim3(256), 0, stream, P, n_seq, L, rows, Q, cut.pieces, cut.steps);                \
        hipLaunchKernelGGL(trp_join_kernel<LEVELS>, dim3((unsigned)join_blocks), dim3(64), 0, stream, P, n_seq, rows, Q, \
                           cut.pieces, cut.steps, out, ld_out, scale);                                        \
        break
            RFSF_TRP_PIECES_CASE(1);
            RFSF_TRP_PIECES_CASE(2);
            RFSF_TRP_PIECES_CASE(3);
            RFSF_TRP_PIECES_CASE(4);
            RFSF_TRP_PIECES_CASE(5);
            RFSF_TRP_PIECES_CASE(6);
            RFSF_TRP_PIECES_CASE(7);
            RFSF_TRP_PIECES_CASE(8);
#undef RFSF_TRP_PIECES_CASE
        }
        return hipGetLastError();
    }
    // 16-byte loads need whole groups of four components and rows of P that start on 16 bytes
    const bool wide = Q % 4 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0;
    const int64_t threads = n_seq * (wide ? Q / 4 : Q);
    const int64_t blocks = (threads + 255) / 256;
    if (blocks > 2147483647) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
#define RFSF_LAUNCH_TRP_SCAN(LEVELS, STEPS, WIDTH)                                                            \
    hipLaunchKernelGGL((trp_scan_kernel<LEVELS, STEPS, WIDTH>), grid, dim3(256), 0, stream, P, n_seq, L, rows, M, Q, out,   \
                       ld_out, scale)
    // up to eight levels have kernels of their own (no loads for levels that do not exist); the batch length
    // keeps about 24 loads of 16 bytes, or 64 of 4 bytes, in flight per thread
#define RFSF_TRP_SCAN_CASE(LEVELS)                                                                            \
    case LEVELS:                                                                                              \
        if (wide) RFSF_LAUNCH_TRP_SCAN(LEVELS, (24 / LEVELS > 8 ? 8 : 24 / LEVELS), 4);                       \
        else RFSF_LAUNCH_TRP_SCAN(LEVELS, (64 / LEVELS > 16 ? 16 : 64 / LEVELS), 1);                          \
        break
    switch (M) {
        RFSF_TRP_SCAN_CASE(1);
        RFSF_TRP_SCAN_CASE(2);
        RFSF_TRP_SCAN_CASE(3);
        RFSF_TRP_SCAN_CASE(4);
        RFSF_TRP_SCAN_CASE(5);
        RFSF_TRP_SCAN_CASE(6);
        RFSF_TRP_SCAN_CASE(7);
        RFSF_TRP_SCAN_CASE(8);
    default:
        if (wide) RFSF_LAUNCH_TRP_SCAN(16, 1, 4);
        else RFSF_LAUNCH_TRP_SCAN(16, 4, 1);
    }
#undef RFSF_TRP_SCAN_CASE
#undef RFSF_LAUNCH_TRP_SCAN
    return hipGetLastError();
}

}  // namespace rfsf
