// Internal declarations shared by the translation units of librfsf_ts (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace rfsf {

constexpr size_t kLdsPerCu = 160 * 1024;
constexpr int kMaxDevices = 64;
// More LDS than 64 KB has to be allowed for every kernel, on each device that runs it. It is allowed to all that a CU has, once, so
// that neither calls of other sizes nor other threads take it back. One LdsLimit per kernel; `fixed`: its LDS that is not dynamic.
struct LdsLimit { std::atomic<bool> raised[kMaxDevices]; };
inline hipError_t allow_lds(LdsLimit &limit, const void *kernel, size_t dynamic, size_t fixed = 0)
{
    if (dynamic + fixed <= 64 * 1024) return hipSuccess;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    const bool known = device >= 0 && device < kMaxDevices;
    if (known && limit.raised[device].load(std::memory_order_relaxed)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsPerCu - fixed));
    if (e == hipSuccess && known) limit.raised[device].store(true, std::memory_order_relaxed);
    return e;
}

// A launch of the tuned sketch kernels may cut every sequence into `pieces` pieces of `pairs` pairs of time
// steps each (workgroup v then owns piece v % pieces of sequence v / pieces). `mode` 1: instead of the features, the
// accumulators of the recurrence (sets of bins 0 .. D/2 of the transform, complex) of piece p of sequence n are
// written at spectra + n * seq_stride + p * piece_stride (float2); `mode` 2: no time step is run, accumulators are
// read from there and turned into features (the final transforms).
// Transforms up to 2048 points: the sets are those of all M(M+1)/2 ranges of tensor positions (a <= l, ordered by a),
// mode 2 joins `join` pieces per sequence, and a null `spectra` stands for the increments' own place.
// Transforms of 4096 and 8192 points: the sets are the levels of the launch, which may be the last ones of increment
// rows that hold `row_levels` levels (the pointers to the increments and the tables are then advanced to the first
// level to run); mode 2 reads joined accumulators.
// `points`: see Points.
struct Points {
    const float *X = nullptr, *W = nullptr, *sign = nullptr;      // [n_seq, L, d], [M, d, F], [M, 2F]
    int d = 0;
    float quarters = 0.f, quarters_rest = 0.f;                    // quarter-turns of angle per unit of X . W, in two terms
};
struct TimeCut {
    int pieces, row_levels;
    int64_t pairs;
    float2 *spectra;
    int mode, join;
    int64_t seq_stride, piece_stride;
    bool solo = false;           // mode 1: the kernel whose wavefronts work by themselves (sketch_fft_scan_solo.h)
    Points points = {};          // ... and which, with X set, computes the increments itself: none are in memory
    static TimeCut whole(int64_t L, int M) { return {1, M, (L + 1) / 2, nullptr, 0, 1, 0, 0}; }
};
constexpr int kMaxCutLevels = 8;                       // the tuned kernels run at most eight levels
struct PieceRows { const float2 *rows[kMaxCutLevels]; };

// Increment workspace: row g = n * L + t holds, for every level m, the 2F numbers
// phi_m(x_{t+1}) - phi_m(x_t) of sequence n; rows with t = L-1 exist but are never read.
// Element (g, m, a) sits at ((g * M + m) * 2F + a).

// Steps 1-2: random Fourier features of every time point and their time increments
// for `n_seq` sequences starting at X (already offset to the chunk), halved.
// sign == nullptr: row layout, element (g, m, a) of row g = n * L + t at ((g * M + m) * 2F + a), no signs.
// sign != nullptr ([M, 2F], the CountSketch signs): pair layout with the signs applied. With Lp = L rounded up
// to even, increment k = n * Lp + t of coordinate a sits at ((((k / 2) * M + m) * 2F + p) * 2 + k % 2), p = 2a for a
// cosine (a < F) and 2(a - F) + 1 for a sine: the two increments of a pair of consecutive time steps are one float2.
// n_seq * Lp * M * 2F floats in all.
// `lengths` (may be null, pair layout): each sequence's own number of points; increments beyond them may be left out.
// `tables` (may be null): the sketch tables are built as well, by workgroups of the same launch where that pays.
// `compact` (row layout): the rows with t = L-1 do not exist and row n * (L - 1) + t follows row n * (L - 1) + t - 1.
struct TableJob;
hipError_t launch_rff_increments(const float *X, const float *W, const float *sign, float inv_lengthscale,
                                 int64_t n_seq, int64_t L, int d, int M, int F, bool bf16,
                                 float *dphi, hipStream_t stream, const TableJob *tables, const int64_t *lengths, bool compact = false);

// Steps 3-4: CountSketch, FFT-domain level recursion over time, inverse transform; writes
// (D is the transform length, a power of two; Dout <= D the number of buckets per level: equal to D,
// or smaller when the buckets are no power of two and the convolutions are linear, folded at the end)
// columns 0 .. M*D of `n_seq` rows of out (already offset to the chunk).
// `lengths` (may be null: all L) holds each sequence's own number of points, X being padded to L.
// `state` is scratch for the generic kernel: sketch_fft_scan_state_bytes (accumulators, and the work buffers
// when they do not fit in LDS).
// `table` (sketch_fft_scan_table_bytes, built once per call) feeds the tuned kernel.
// `cut` (tuned kernels only): how the launch cuts the sequences in time and which levels of the increment rows
// it runs; TimeCut::whole(L, M) for the plain case.
hipError_t launch_sketch_fft_scan(const float *dphi, const int32_t *hash, const float *sign,
                                  const uint32_t *table, int64_t n_seq, int64_t L, const int64_t *lengths, int M, int F,
                                  int D, int Dout, int order, float *out, int64_t ld_out, float *state,
                                  hipStream_t stream, TimeCut cut);
// Joins the pieces of a launch series that cut the sequences in time (csrc/join_pieces.hip).
// pieces_of_start.rows[a]: accumulators written by the launch that ran levels a+1 .. M (row = sequence *
// pieces + piece, M-a levels of `bins` complex numbers each). Writes M levels of `bins` numbers per sequence
// to `joined`.
hipError_t launch_join_pieces(const PieceRows &pieces_of_start, int64_t n_seq, int pieces, int M, int bins,
                              float2 *joined, hipStream_t stream);
// Joins the pieces of every sequence (all M(M+1)/2 ranges of tensor positions, layout of TimeCut) and leaves the M
// levels of the whole sequence in the place of the first piece's.
hipError_t launch_join_chain(float2 *spectra, int64_t n_seq, int pieces, int M, int bins, int64_t seq_stride,
                             int64_t piece_stride, hipStream_t stream);
// The job of building the tables of a shape (csrc/sketch_tables.h); false if its kernel needs none.
bool sketch_table_job(const int32_t *hash, int M, int F, int D, int Dout, uint32_t *table, TableJob *job);
hipError_t launch_build_tables(const TableJob &job, int M, hipStream_t stream);
bool sketch_fft_scan_is_tuned(int M, int F, int D);
// The tuned kernel of the shape can hold the accumulators of all ranges of tensor positions (transforms up to 2048).
bool sketch_fft_scan_joint(int M, int F, int D);
int sketch_fft_scan_joint_per_cu(int M, int D);            // its workgroups that a CU holds, by registers
int sketch_fft_scan_joint_fit(int M, int F, int D, int order);      // ... and by LDS
bool sketch_fft_scan_joint_splits(int M, int D, int order);        // splitting whole sequences can gain
constexpr int kSoloWaves = 4;      // wavefronts of a workgroup of the kernel whose wavefronts work by themselves
// Pieces of this shape run in the kernel whose wavefronts work by themselves; its tables hold no lists. The pairs of steps that
// a workgroup of it transforms at a time, or 0; its workgroups that a CU holds.
int sketch_fft_scan_solo_pairs(int M, int F, int D, int order, int d, bool bf16);
int sketch_fft_scan_solo_per_cu(int M, int F, int D);
bool sketch_fft_scan_solo_fused(int F, int d, int D);             // it can compute the increments itself
uint32_t sketch_fft_scan_solo_zero(int F, int D);          // TableJob::zero_off of its tables
int sketch_fft_scan_wavefronts(int M, int D);                      // of a workgroup for whole sequences
int sketch_fft_scan_pairs_per_iteration(int D);            // pairs of steps a wavefront transforms at a time
bool sketch_fft_scan_fits(int M, int F, int D, int order);  // false: neither kernel can run it (LDS need above a CU's)
size_t sketch_fft_scan_table_bytes(int M, int F, int D);   // 0 when the generic kernel runs
size_t sketch_fft_scan_lds_bytes(int M, int F, int D);
size_t sketch_fft_scan_state_bytes(int64_t n_seq, int M, int D, int order);

// Level-0 column and zero blocks for sequences without increments (L == 1).
hipError_t launch_fill_trivial(float *out, int64_t n_seq, int64_t ld_out, int64_t ncols, hipStream_t stream);

// K[Nx, Ny] = PhiX PhiY^T. `rows_add_up`: the caller sums over rows of K, so that their rounding errors must not
// share a sign. `batch` > 1: that many products in one launch, the pointers advanced by the steps (floats) from one to
// the next. `points` > 0 (RFSF-TRP): the points that the rows of PhiX, increments, lie between.
hipError_t launch_gram(const float *PhiX, int64_t Nx, int64_t ldx, const float *PhiY, int64_t Ny,
                       int64_t ldy, int64_t ncols, float *K, int64_t ldk, hipStream_t stream, bool rows_add_up = false,
                       int batch = 1, int64_t step_x = 0, int64_t step_y = 0, int64_t step_k = 0, int64_t points = 0);

// RFSF-DP-1D features, one fused kernel; d <= 64 and M <= 16 (checked by the API layer). scale_turns: angles in
// half-turns per unit of X . W, 1 / (pi lengthscale).
hipError_t launch_dp1d(const float *X, const float *W, const float *bias, float scale_turns, int64_t N,
                       int64_t L, int d, int M, int F, float *out, int64_t ld_out, hipStream_t stream);

// RFSF-TRP second stage: recurrence over time on the projected increments P[n_seq*rows][M][Q], which it may overwrite, of n_seq
// sequences of a batch of N, the first L - 1 of a sequence's rows (L - 1 or L); M <= 16.
hipError_t launch_trp_scan(float *P, int64_t N, int64_t n_seq, int64_t L, int64_t rows, int M, int Q, float *out, int64_t ld_out,
                           hipStream_t stream);

hipError_t launch_normalize(float *Phi, int64_t N, int64_t ld, int M, int D, hipStream_t stream);

// Benchmark helper (csrc/probe.hip): read, write, non-temporal write, copy GB/s over `scratch`, fp32 matrix and
// fp32 vector TFLOP/s of issue loops, in this order; waits for the stream.
hipError_t probe_peaks(void *scratch, size_t bytes, double out[6], hipStream_t stream);
hipError_t launch_validate_tables(const int32_t *hash, const float *sign, int64_t count, int D,
                                  int *flag, hipStream_t stream);


// Per-kernel event timing (see rfsf_ts_profile_enable). A Scope records a start event when
// constructed and a stop event when destroyed, if profiling is on.
enum KernelClass { kRffIncrements = 0, kSketchFftScan = 1, kGram = 2, kNormalize = 3, kDp1d = 4, kTrpProject = 5, kTrpScan = 6, kNumKernelClasses = 7 };
struct ProfileScope {
    ProfileScope(KernelClass k, hipStream_t stream, bool allowed = true);
    ~ProfileScope();
    int slot;
    hipStream_t stream;
};

}  // namespace rfsf
