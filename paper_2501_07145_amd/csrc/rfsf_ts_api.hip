// C ABI of librfsf_ts: argument checks, chunking over sequences, kernel launches.
#include "../../include/rfsf_ts.h"
#include "rfsf_internal.h"
#include "sketch_tables.h"

#include <cmath>
#include <vector>

namespace rfsf {
namespace {
struct TimedLaunch { hipEvent_t start, stop; KernelClass k; };
bool g_profile_on = false;
std::vector<TimedLaunch> g_launches;
}  // namespace

ProfileScope::ProfileScope(KernelClass k, hipStream_t s, bool allowed) : slot(-1), stream(s)
{
    if (!g_profile_on || !allowed) return;
    TimedLaunch t{nullptr, nullptr, k};
    if (hipEventCreate(&t.start) != hipSuccess) return;
    if (hipEventCreate(&t.stop) != hipSuccess) { (void)hipEventDestroy(t.start); return; }
    (void)hipEventRecord(t.start, stream);
    g_launches.push_back(t);
    slot = (int)g_launches.size() - 1;
}
ProfileScope::~ProfileScope()
{
    if (slot >= 0) (void)hipEventRecord(g_launches[slot].stop, stream);
}
}  // namespace rfsf

namespace {

constexpr size_t kAlign = 256;
// Increments held per launch, at most. Measured on the N = 10000, L = 200, M = 5, F = 512 batch (41 GB of
// increments): one launch 22.9 ms, two 23.5, four 24.6, sixteen 26.5, 64 launches of 0.64 GB 45 ms; a chunk
// small enough for the last-level cache (64 sequences) cannot fill the chip, since the consumer runs one
// workgroup per sequence. Hence: as few launches as a 48 GiB scratch allows.
constexpr size_t kChunkBytesTarget = (size_t)48 << 30;
constexpr size_t kIncrementTail = 4096;   // the kernels for 4096 and 8192 points may read up to 1023 floats past the last row

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

bool is_pow2_in_range(int32_t D) { return D >= 2 && D <= 4096 && (D & (D - 1)) == 0; }

// Length of the FFTs. The convolutions are circular modulo D; a transform of P points gives them exactly when
// D divides P (the result, circular modulo P, is folded modulo D at the end) or when P holds the linear
// convolution of M sketches of length D without wrap-around, M*(D-1)+1 numbers. Candidates, in this order: D
// itself when it is a power of two in [2, 4096] or one of 100, 200, 500, 1000 (the bucket counts of the paper's
// own experiments, which have transforms of their own with radices 10, 5, 2); then the powers of two from 64 on
// that are multiples of D or hold the linear convolution. The first one whose shape fits a tuned kernel is
// taken (a small D with many random features, for instance, does not fit at its own length: its wavefronts
// would carry 16 staging areas each); if none does, the first candidate at all, for the generic kernel.
// 0 if there is no candidate up to 8192 points.
int transform_length(int32_t M, int32_t F, int32_t D)
{
    if (D < 1 || D > 4096) return 0;
    const bool pow2 = is_pow2_in_range(D);
    const bool own = pow2 || D == 100 || D == 200 || D == 500 || D == 1000;
    if (own && rfsf::sketch_fft_scan_is_tuned(M, F, D)) return D;
    const int64_t need = (int64_t)M * (D - 1) + 1;
    int first = pow2 ? D : 0;
    for (int64_t P = 2; P <= 8192; P *= 2) {
        if (!(pow2 ? P >= D : P >= need)) continue;
        if (first == 0) first = (int)P;
        if (P >= 64 && rfsf::sketch_fft_scan_is_tuned(M, F, (int)P)) return (int)P;
    }
    return first;
}

int check_shape(const rfsf_ts_shape *s)
{
    if (!s) return RFSF_E_NULLPTR;
    if (s->N < 0 || s->L < 1 || s->d < 1 || s->M < 1 || s->F < 1) return RFSF_E_BAD_SHAPE;
    if (s->N > ((int64_t)1 << 40) || s->L > ((int64_t)1 << 40) || s->d > (1 << 20) || s->M > (1 << 10) ||
        s->F > (1 << 24))
        return RFSF_E_BAD_SHAPE;
    if (transform_length(s->M, s->F, s->D) == 0) return RFSF_E_D_NOT_POW2;
    if (s->order < 0) return RFSF_E_BAD_SHAPE;
    if (s->ld_out < 1 + (int64_t)s->M * s->D) return RFSF_E_BAD_STRIDE;
    return RFSF_OK;
}

// Few long sequences (the shape of the paper's sequence-length runs, Sec. 4: N = 10, L up to 1e5) would keep one
// workgroup per sequence busy and the rest of the chip idle. They are cut in time instead: `pieces` pieces of
// `pairs` pairs of steps per sequence, joined afterwards (csrc/join_pieces.hip). A function of the shape alone, so that
// every entry point and every workspace size computes the same sums in the same order. The tuned kernels only
// (any signature order they have: a step's truncated exponential is a factor of the product over steps either way).
// The rule comes from pieces that cost (M+1)/2 times the transforms (one launch per first tensor position, as transforms
// of 4096 and 8192 points still take; M = 5; D = 100, 256, 1024; L = 1e3, 1e4): up to 64 sequences every cut
// into about 1024 / N pieces of at least 32 pairs wins (1.3x at N = 64 .. 30x at N = 1); no cut unless it brings at
// least M + 1 pieces; at most 128 pieces (they are joined one after the other). What it leaves whole, sketch_cut may split.
struct TimeCutPlan { int pieces; int64_t pairs; };
TimeCutPlan time_cut_plan(const rfsf_ts_shape *s)
{
    const int64_t all_pairs = s->L / 2;                     // L - 1 steps
    const TimeCutPlan whole = {1, (s->L + 1) / 2};
    const int P = transform_length(s->M, s->F, s->D);
    if (s->order > 3 || s->M < 2 || s->M > rfsf::kMaxCutLevels || s->N < 1 || s->N > 64 ||
        !rfsf::sketch_fft_scan_is_tuned(s->M, s->F, P))
        return whole;
    int64_t want = 1024 / s->N;                             // about four workgroups per CU
    if (want > all_pairs / 32) want = all_pairs / 32;
    if (want > 128) want = 128;
    if (want < s->M + 1) return whole;
    for (int levels = 1; levels < s->M; ++levels)           // every launch of the series runs a tuned kernel
        if (!rfsf::sketch_fft_scan_is_tuned(levels, s->F, P)) return whole;
    const int64_t pairs = (all_pairs + want - 1) / want;
    return {(int)((all_pairs + pairs - 1) / pairs), pairs};
}

// The cut that a launch makes. Shapes that time_cut_plan leaves whole but whose batch does not fill the chip with
// one workgroup per sequence -- more than 64 sequences, or sequences too short for M + 1 pieces of 32 pairs -- are
// split as well where one launch produces all ranges of positions (sketch_fft_scan_joint): the transforms are then
// not repeated, so a few iterations of a workgroup per piece are enough to gain. The pieces' accumulators take the place of
// their increments, so these splits need no workspace of their own; a piece has to be long enough for that.
// A function of the shape alone, like the plan.
// Two pieces of each of 150 sequences of 500 points (512 buckets, two workgroups per CU): 443 -> 354 us; of 200 sequences
// where a CU holds one workgroup (500 buckets, five levels): 463 -> 491, hence as many pieces as CUs hold.
constexpr int64_t kSplitSequences = 256, kCUs = 256;
// An iteration of a workgroup alone on its CU takes about 3 us, a piece in the join 0.3: with p pairs in all and pieces of
// i iterations, 3 i + 0.3 p / (i * pairs per iteration) is least at i^2 = p / (10 * pairs per iteration).
constexpr int64_t kSplitPieces = 64, kJoinsPerIteration = 10;
// More pieces than most_joined_in_place are joined by a kernel of its own, a wavefront per 64 bins that keeps several pieces in
// flight, fewer by the kernel of the final transforms, where a thread takes its bins one after the other: one or two of them
// up to 512 points, three to five from 1024 on. (A single sequence, joined there and by its own kernel: 1024 buckets, five levels,
// 5 pieces 49 and 46 us, 10 pieces 63 and 49; three levels, 10 pieces 43 and 40; 2048 buckets, four levels, 5 pieces 63 and 58, 10 pieces 72
// and 59. 40 sequences in 6 pieces: 83 and 79, 99 and 94, three levels 57 both; 1024 buckets, two levels, 8 pieces 31 and 33. 256 buckets,
// four levels, 13 pieces: 30.4 and 31.4.)
constexpr int kJoinInPlace = 16;
int most_joined_in_place(int M, int P, bool solo)
{
    if (solo || P <= 512) return kJoinInPlace;
    return M > 3 ? 4 : 9;
}
// A single level only adds its increments up, a pair costs a thread a fortieth of that: whole sequences of fewer than this
// many loads per thread are not split (60 points: 22 us whole, 25 split with 32 frequencies, 23 and 30 with 128; 150 points 33
// and 32, 300 points 48 and 38, 512 frequencies, 60 points 64 and 52, all of 60 sequences in 256 buckets).
constexpr int64_t kSumLoads = 128;
// Order of the recurrence that a launch runs: a single level is the same in all of them.
int kernel_order(const rfsf_ts_shape *s) { return s->order < 2 || s->M == 1 ? 1 : s->order; }
struct SketchCut { int pieces; int64_t pairs; bool joint, in_place, solo; };
// The cut for the kernel whose wavefronts work by themselves (csrc/sketch_fft_scan_solo.h), which takes whole sequences and
// pieces alike and `step` pairs of steps per iteration of a workgroup. Time is counted in iterations of a CU that holds as many
// workgroups as it can: with n of them an iteration takes (2 + n) / (2 + that many) (D = 100, five levels, 2 to 4 on a CU 6.1,
// 7.9 and 9.6 us); the beginning and the end of a workgroup take 0.4 of one, the join 0.05 per piece and 18 MB of accumulators. What is
// left over when all CUs have been filled a whole number of times is spread over them, so that pieces are chosen to leave a little
// over or nearly nothing. Pieces end at a multiple of the pairs that a wavefront takes per iteration (step / 4); each of its wavefronts takes a
// quarter, rounded up to such a multiple, and the last ones up to three times that less, or nothing: where one of them has an iteration more
// than others, that counts 0.6.
// (100 x 1000 points, D = 100, five levels: 8, 9, 10, 11 pieces, 800 to 1100 workgroups on 256 CUs that hold four, 106, 97, 93, 117 us;
// 300 x 300 points 2, 3, 4: 102, 88, 95; 1280 x 257 1, 2, 3: 258, 236, 253; 59 x 172, D = 64, five levels 4, 6, 8: 31, 32, 28. Over 726 shapes
// of 12 to 3000 sequences whose numbers of pieces were all timed, the one chosen is 1.8 % slower than the best on average, by 7 % or more for
// one in ten.)
// Batches that leave CUs without a workgroup are left to the other kernels, whose wavefronts share out a piece's levels
// (a single sequence of 100 points 27.8 us, 30.7 here; ten of 1000 49 and 56); from 7 pairs per CU on, 15 with five levels or
// more and few frequencies, the number of pieces is one that leaves none (59 x 172, D = 64, five levels, in the other kernels 39 us, 28 here; 39 x 179,
// D = 100, six, 59 frequencies 42 and 36; 60 x 200 points, D = 100, four levels: elsewhere, for want of workgroups, 43 us, 35 here; 40 x
// 200, D = 256 50.5 and 47.7; 50 x 120, D = 128, three levels 29.8 and 26.1; but 25 x 120, D = 256 34.7 and 39.6, 50 x 120, D = 100, five
// levels 35.4 and 37.8). Left to them as well are sequences that fill less than half
// of an iteration (3000 x 14 points, 64 buckets, three levels 51 and 54) or, from 128 points per transform on, less than four
// (1000 x 30 points, 256 buckets, four levels 64 and 70).
// With three and four levels the other kernels' workgroups fill a CU, and less is gained. Pieces of less than one and a
// half iterations are left to them where there is nothing else to gain either: where the increments come from memory (whole
// sequences; 1186 x 31 points, 20 channels, 56 frequencies, 64 buckets, three levels 54 and 66 us, 5816 x 66, 3, 73, 100 365 and 420;
// of 38 such calls 29 were slower by more than 5 %, one faster), or where they are so few that projecting them costs less than
// doing it on idle lanes, fewer than four frequencies per channel (774 x 43, 8, 13, 100, three levels 33 and 43; 23 and 5 of 37); longer
// sequences are then cut in fewer pieces (90 x 165, 6 channels, 18 frequencies, 128 buckets, four levels 30, elsewhere 36; 318 x 56, 8, 24, 100 41 and 36).
bool solo_fused(const rfsf_ts_shape *s, int P) { return s->rff_bf16 == 0 && rfsf::sketch_fft_scan_solo_fused(s->F, s->d, P); }
SketchCut solo_cut(const rfsf_ts_shape *s, int P, int step)
{
    const SketchCut none = {0, 0, false, false, false};
    const int64_t slots = (s->L + 1) / 2, all_pairs = s->L / 2, floats_per_pair = (int64_t)s->M * 4 * s->F;
    const int64_t needed = (int64_t)s->M * (s->M + 1) * (P / 2 + 1);                   // floats of a piece's accumulators
    const int64_t per_cu = rfsf::sketch_fft_scan_solo_per_cu(s->M, s->F, P), own = step / rfsf::kSoloWaves;    // pairs of a wavefront
    if (2 * all_pairs < step || (P >= 128 && all_pairs < 4 * step)) return none;
    const bool fused = solo_fused(s, P), little = (s->M == 3 || s->M == 4) && (!fused || s->F < 4 * s->d);
    const int64_t fewest = s->N * all_pairs > kCUs * (s->M > 4 && s->F < 48 ? 15 : 7) ? kCUs : 0;
    SketchCut best = none;
    double least = 0.0;
    for (int64_t want = 1; want <= kSplitPieces && want * step <= all_pairs + step; ++want) {
        const int64_t pairs = ((all_pairs + want - 1) / want + own - 1) / own * own, pieces = (all_pairs + pairs - 1) / pairs;
        // every piece, the last one too, has to hold its accumulators
        if (little && fused && all_pairs >= 3 * step && 2 * all_pairs < 3 * step * pieces) continue;
        if (pieces > kJoinInPlace || s->N * pieces <= fewest || (pieces < 2 ? slots : pairs) * floats_per_pair < needed ||
            (slots - (pieces - 1) * pairs) * floats_per_pair < needed)
            continue;
        const int64_t workgroups = s->N * pieces, full = workgroups / (kCUs * per_cu), rest = workgroups - full * kCUs * per_cu;
        // iterations of a workgroup: between those of its longest wavefront and the mean
        const double its = 0.4 * (double)pairs / (double)step + 0.6 * (double)((pairs + step - 1) / step);
        const double of_rest = (2.0 + (double)((rest + kCUs - 1) / kCUs)) / (2.0 + (double)per_cu);
        const double cost = (double)full * (its + 0.4) + (rest > 0 ? its * of_rest + 0.4 : 0.0) + 0.05 * (double)pieces +
                            (double)workgroups * (double)needed * 4.0 / 18e6;
        if (best.pieces == 0 || cost < least) {
            least = cost;
            best = {(int)pieces, pieces < 2 ? slots : pairs, true, true, true};
        }
    }
    if (little && 2 * all_pairs < 3 * step * best.pieces && (fused || best.pieces == 1)) return none;
    return s->N * best.pieces > kCUs ? best : none;
}
// The same for sequences that time_cut_plan cuts, hundreds of iterations each: the other kernels are the faster ones with 100 buckets
// and increments from memory up to four levels (6 x 30072 points, 77 frequencies, three levels 280 and 341 us; of 48 such calls 17
// slower by more than 5 %, 6 faster), and with 128, four levels and few frequencies per channel (22 x 12271 points, 8 channels, 22
// frequencies 207 and 259; 6 of 8, none faster).
bool solo_pieces(const rfsf_ts_shape *s, int P)
{
    if (!solo_fused(s, P)) return P != 100 || s->M > 4;
    return P != 128 || s->M < 4 || s->F >= 6 * s->d;
}
SketchCut sketch_cut(const rfsf_ts_shape *s)
{
    const TimeCutPlan plan = time_cut_plan(s);
    const int P = transform_length(s->M, s->F, s->D);
    const bool joint = rfsf::sketch_fft_scan_joint(s->M, s->F, P);
    const int step = joint && s->L > 1 ? rfsf::sketch_fft_scan_solo_pairs(s->M, s->F, P, kernel_order(s), s->d, s->rff_bf16 != 0) : 0;
    if (plan.pieces > 1) return {plan.pieces, plan.pairs, joint, false, step > 0 && s->N * plan.pieces > kCUs && solo_pieces(s, P)};
    if (step > 0 && s->N > 0) {
        const SketchCut cut = solo_cut(s, P, step);
        if (cut.pieces > 0) return cut;
    }
    const int64_t slots = (s->L + 1) / 2, all_pairs = s->L / 2;
    const int64_t floats_per_pair = (int64_t)s->M * 4 * s->F;
    const int64_t needed = (int64_t)s->M * (s->M + 1) * (P / 2 + 1);                   // floats of a piece's accumulators
    const SketchCut whole = {1, plan.pairs, false, false, false};
    if (!joint || s->N < 1 || s->N > kSplitSequences || s->L < 3) return whole;
    const int fpw = rfsf::sketch_fft_scan_pairs_per_iteration(P);
    const int64_t per_cu = rfsf::sketch_fft_scan_joint_per_cu(s->M, P), fit = rfsf::sketch_fft_scan_joint_fit(s->M, s->F, P, kernel_order(s));
    const int64_t at_once = kCUs * (fit < per_cu ? fit : per_cu);
    int64_t most = kCUs * per_cu / s->N;           // pieces that fill the chip
    if (most > kSplitPieces) most = kSplitPieces;
    if (!rfsf::sketch_fft_scan_joint_splits(s->M, P, kernel_order(s))) return whole;
    const int threads = 64 * rfsf::sketch_fft_scan_wavefronts(s->M, P);
    if (s->M == 1 && all_pairs * ((s->F + threads - 1) / threads) < kSumLoads) return whole;
    // iterations of the kernel per piece: the fewest that keep to `most`, and no fewer than balance the join
    int64_t its = (all_pairs + most * fpw - 1) / (most > 0 ? most * fpw : 1);
    while (its * its * kJoinsPerIteration * fpw < all_pairs) ++its;
    for (; most >= 2; ++its) {
        const int64_t pairs = its * fpw, pieces = (all_pairs + pairs - 1) / pairs;
        if (pieces < 2) break;
        // Many frequencies leave a CU fewer workgroups than its registers do. Pieces then take several rounds, and gain only
        // if there are more than twice as many of them: alone on its CU, the kernel that advances all ranges of positions
        // takes 1.2 to 1.7 times as long per step. (500 points, four levels, 1000 frequencies, 512 buckets, sketch kernel: 200
        // sequences in two pieces, two rounds, 1928 us, whole 1200; 150 in three, two rounds, 1369, whole 1058; 128 in four,
        // two rounds, 1224, in two and one 1138. 300 points, 700 frequencies, 256 buckets: 100 in five pieces, two rounds, 393.)
        const int64_t rounds = (s->N * pieces + at_once - 1) / at_once;
        if (rounds > 1 && 2 * rounds >= pieces) continue;
        // every piece, the last one too, has to hold its accumulators
        if (pairs * floats_per_pair >= needed && (slots - (pieces - 1) * pairs) * floats_per_pair >= needed)
            return {(int)pieces, pairs, true, true, false};
    }
    return whole;
}
// floats of one sequence's pieces: per piece and first position a the accumulators of levels a+1 .. M (bins
// 0 .. P/2 of the transform, complex), plus the joined accumulators of the sequence
size_t piece_floats(const rfsf_ts_shape *s, int pieces)
{
    const size_t bins = (size_t)transform_length(s->M, s->F, s->D) / 2 + 1;
    size_t per_piece = 0;
    for (int a = 0; a < s->M; ++a) per_piece += (size_t)(s->M - a) * bins * 2;
    return per_piece * (size_t)pieces + (size_t)s->M * bins * 2;
}

// Bytes of workspace one sequence needs: its increment rows plus its state (the generic kernel's
// accumulators; the rows of its pieces when the sequences are cut in time).
void per_sequence_bytes(const rfsf_ts_shape *s, size_t *incr, size_t *state)
{
    // rows of increments per sequence: L in the row layout, L rounded up to even in the pair layout
    *incr = (size_t)((s->L + 1) & ~(int64_t)1) * (size_t)s->M * 2u * (size_t)s->F * sizeof(float);
    *state = rfsf::sketch_fft_scan_state_bytes(1, s->M, transform_length(s->M, s->F, s->D), s->order == 2 ? 2 : 1);
    const TimeCutPlan plan = time_cut_plan(s);
    if (plan.pieces > 1) *state += sizeof(float) * piece_floats(s, plan.pieces);
}

// Fixed part: packed hash/sign table plus room for aligning the three sections.
size_t fixed_bytes(const rfsf_ts_shape *s)
{
    return align_up(rfsf::sketch_fft_scan_table_bytes(s->M, s->F, transform_length(s->M, s->F, s->D))) + kIncrementTail +
           3 * kAlign;
}

int64_t chunk_for(const rfsf_ts_shape *s, size_t bytes)
{
    size_t incr, state;
    per_sequence_bytes(s, &incr, &state);
    const size_t fixed = fixed_bytes(s);
    if (bytes < fixed) return 0;
    return (int64_t)((bytes - fixed) / (incr + state));
}

}  // namespace

extern "C" const char *rfsf_ts_strerror(int code)
{
    switch (code) {
        case RFSF_OK: return "success";
        case RFSF_E_NULLPTR: return "a required pointer is NULL";
        case RFSF_E_BAD_SHAPE: return "bad shape: need N >= 0, L >= 1, d >= 1, M >= 1, F >= 1 within limits";
        case RFSF_E_D_NOT_POW2: return "D must be a power of two in [2, 4096], or satisfy M*(D-1)+1 <= 8192";
        case RFSF_E_BAD_STRIDE: return "leading dimension smaller than the row length";
        case RFSF_E_BAD_LENGTHSCALE: return "lengthscale must be finite and > 0";
        case RFSF_E_WORKSPACE_TOO_SMALL: return "workspace smaller than rfsf_ts_workspace_bytes' minimum";
        case RFSF_E_HIP: return "HIP runtime error";
        case RFSF_E_BAD_TABLE: return "hash outside [0, D) or sign not +-1";
        case RFSF_E_UNSUPPORTED: return "configuration not supported by this build";
        case RFSF_E_STATIC_SCRATCH_TOO_SMALL:
            return "one sequence needs more than the 64 MiB built-in scratch: use rfsf_ts_features with a workspace";
        default: return "unknown rfsf_ts error code";
    }
}

extern "C" int rfsf_ts_workspace_bytes(const rfsf_ts_shape *shape, size_t *recommended_bytes,
                                       size_t *minimum_bytes)
{
    const int rc = check_shape(shape);
    if (rc != RFSF_OK) return rc;
    size_t incr, state;
    per_sequence_bytes(shape, &incr, &state);
    const size_t per = incr + state;
    int64_t chunk = (int64_t)(kChunkBytesTarget / per);
    if (chunk < 1) chunk = 1;
    if (chunk > shape->N) chunk = shape->N > 0 ? shape->N : 1;
    // equal-sized chunks: no small trailing launch
    if (shape->N > 0) {
        const int64_t nchunks = (shape->N + chunk - 1) / chunk;
        chunk = (shape->N + nchunks - 1) / nchunks;
    }
    if (recommended_bytes) *recommended_bytes = (size_t)chunk * per + fixed_bytes(shape);
    if (minimum_bytes) *minimum_bytes = per + fixed_bytes(shape);
    return RFSF_OK;
}

extern "C" int rfsf_ts_time_cut(const rfsf_ts_shape *shape, int32_t *pieces, int64_t *pairs_per_piece)
{
    const int rc = check_shape(shape);
    if (rc != RFSF_OK) return rc;
    const TimeCutPlan plan = time_cut_plan(shape);
    if (pieces) *pieces = plan.pieces;
    if (pairs_per_piece) *pairs_per_piece = plan.pairs;
    return RFSF_OK;
}

namespace {
// Body of rfsf_ts_features. `may_create` = false keeps the call free of anything that creates runtime
// objects: no profiling events are recorded.
int features_impl(const rfsf_ts_shape *shape, const float *X, const int64_t *lengths, const float *W,
                  const int32_t *hash, const float *sign, float lengthscale, float *out, void *workspace,
                  size_t workspace_bytes, void *hip_stream, bool may_create)
{
    int rc = check_shape(shape);
    if (rc != RFSF_OK) return rc;
    if (!(lengthscale > 0.0f) || !std::isfinite(lengthscale)) return RFSF_E_BAD_LENGTHSCALE;
    if (shape->N == 0) return RFSF_OK;
    if (!X || !W || !hash || !sign || !out) return RFSF_E_NULLPTR;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int64_t ncols = 1 + (int64_t)shape->M * shape->D;

    if (shape->L == 1) {      // no increments: empty sums
        return rfsf::launch_fill_trivial(out, shape->N, shape->ld_out, ncols, stream) == hipSuccess
                   ? RFSF_OK : RFSF_E_HIP;
    }
    if ((int64_t)shape->M * ((shape->F + 127) / 128) > 65535) return RFSF_E_UNSUPPORTED;   // grid limits
    if (shape->rff_bf16 != 0 && shape->d > 128) return RFSF_E_UNSUPPORTED;
    if (shape->order > 3) return RFSF_E_UNSUPPORTED;
    if ((int64_t)shape->M * 2 * shape->F > ((int64_t)1 << 26)) return RFSF_E_UNSUPPORTED;   // 32-bit row offsets
    if (!rfsf::sketch_fft_scan_fits(shape->M, shape->F, transform_length(shape->M, shape->F, shape->D), shape->order < 2 ? 1 : shape->order))
        return RFSF_E_UNSUPPORTED;        // order 3 outside the tuned kernel's shapes
    if (!workspace) return RFSF_E_NULLPTR;
    int64_t chunk = chunk_for(shape, workspace_bytes);
    if (chunk < 1) return RFSF_E_WORKSPACE_TOO_SMALL;
    if (chunk > shape->N) chunk = shape->N;

    size_t incr, state_b;
    per_sequence_bytes(shape, &incr, &state_b);
    char *base = static_cast<char *>(workspace);
    const size_t mis = (size_t)(reinterpret_cast<uintptr_t>(base) % kAlign);
    char *p_table = base + (mis ? kAlign - mis : 0);
    const int P = transform_length(shape->M, shape->F, shape->D);
    char *p_incr = p_table + align_up(rfsf::sketch_fft_scan_table_bytes(shape->M, shape->F, P));
    char *p_state = p_incr + align_up((size_t)chunk * incr + kIncrementTail);
    float *dphi = reinterpret_cast<float *>(p_incr);
    float *state = reinterpret_cast<float *>(p_state);
    uint32_t *table = reinterpret_cast<uint32_t *>(p_table);
    rfsf::TableJob tables;                  // built with the first chunk's increments
    const bool has_tables = rfsf::sketch_table_job(hash, shape->M, shape->F, P, shape->D, table, &tables);
    const float inv_ls = 1.0f / lengthscale;
    const SketchCut plan = sketch_cut(shape);
    if (plan.solo) {                                      // no lists, and slots of its own
        tables.groups = 0;
        tables.zero_off = rfsf::sketch_fft_scan_solo_zero(shape->F, P);
    }
    // ... whose increments it computes itself where it can
    const bool fused = plan.solo && solo_fused(shape, P);
    // the tuned consumer takes the increments in the pair layout with the signs applied, the generic one in
    // the row layout without
    const float *producer_sign = rfsf::sketch_fft_scan_is_tuned(shape->M, shape->F, P) ? sign : nullptr;
    for (int64_t n0 = 0; n0 < shape->N; n0 += chunk) {
        const int64_t cnt = shape->N - n0 < chunk ? shape->N - n0 : chunk;
        if (fused) {
            if (n0 == 0) {                                // (no increments are launched: the tables belong to the sketch kernel)
                rfsf::ProfileScope scope(rfsf::kSketchFftScan, stream, may_create);
                if (rfsf::launch_build_tables(tables, shape->M, stream) != hipSuccess) return RFSF_E_HIP;
            }
        } else {
            rfsf::ProfileScope scope(rfsf::kRffIncrements, stream, may_create);
            if (rfsf::launch_rff_increments(X + n0 * shape->L * shape->d, W, producer_sign, inv_ls, cnt, shape->L, shape->d,
                                            shape->M, shape->F, shape->rff_bf16 != 0, dphi, stream,
                                            n0 == 0 && has_tables ? &tables : nullptr,
                                            producer_sign && lengths ? lengths + n0 : nullptr) != hipSuccess)
                return RFSF_E_HIP;
        }
        const int64_t *chunk_lengths = lengths ? lengths + n0 : nullptr;
        if (plan.pieces == 1 && !plan.solo) {
            rfsf::ProfileScope scope(rfsf::kSketchFftScan, stream, may_create);
            if (rfsf::launch_sketch_fft_scan(dphi, hash, sign, table, cnt, shape->L, chunk_lengths,
                                             shape->M, shape->F, P, shape->D, kernel_order(shape),
                                             out + n0 * shape->ld_out, shape->ld_out, state, stream,
                                             rfsf::TimeCut::whole(shape->L, shape->M)) != hipSuccess)
                return RFSF_E_HIP;
        } else if (plan.joint) {
            // sequences cut in time: the accumulators of all ranges of tensor positions of every piece, the join (of many
            // pieces by a launch of its own) and the final transforms (timed as one launch of the sketch kernel class)
            rfsf::ProfileScope scope(rfsf::kSketchFftScan, stream, may_create);
            const int order = kernel_order(shape), bins = P / 2 + 1;
            rfsf::TimeCut cut = {plan.pieces, shape->M, plan.pairs, nullptr, 1, plan.pieces, 0, 0, plan.solo};
            if (fused) {
                const double quarters = 0.63661977236758134308 / (double)lengthscale;
                cut.points = {X + n0 * shape->L * shape->d, W, sign, shape->d, (float)quarters, (float)(quarters - (double)(float)quarters)};
            }
            if (plan.in_place) {
                cut.piece_stride = plan.pairs * (int64_t)shape->M * 2 * shape->F;          // float2 per pair: M * 2F
                cut.seq_stride = (shape->L + 1) / 2 * (int64_t)shape->M * 2 * shape->F;
            } else {
                cut.spectra = reinterpret_cast<float2 *>(state);
                cut.piece_stride = (int64_t)shape->M * (shape->M + 1) / 2 * bins;
                cut.seq_stride = plan.pieces * cut.piece_stride;
            }
            if (rfsf::launch_sketch_fft_scan(dphi, hash, sign, table, cnt, shape->L, chunk_lengths, shape->M, shape->F, P,
                                             shape->D, order, out + n0 * shape->ld_out, shape->ld_out, nullptr, stream,
                                             cut) != hipSuccess)
                return RFSF_E_HIP;
            if (plan.pieces > most_joined_in_place(shape->M, P, plan.solo)) {
                if (rfsf::launch_join_chain(cut.spectra ? cut.spectra : reinterpret_cast<float2 *>(dphi), cnt, plan.pieces,
                                            shape->M, bins, cut.seq_stride, cut.piece_stride, stream) != hipSuccess)
                    return RFSF_E_HIP;
                cut.join = 1;
            }
            cut.pieces = 1;
            cut.mode = 2;
            if (rfsf::launch_sketch_fft_scan(dphi, hash, sign, table, cnt, shape->L, chunk_lengths, shape->M, shape->F, P,
                                             shape->D, order, out + n0 * shape->ld_out, shape->ld_out, nullptr, stream,
                                             cut) != hipSuccess)
                return RFSF_E_HIP;
        } else {
            // the same with one launch per first position: the accumulators of levels a+1 .. M of every piece for
            // a = 0 .. M-1, the join, and the final transforms of the joined accumulators (timed as one launch of the sketch kernel class)
            rfsf::ProfileScope scope(rfsf::kSketchFftScan, stream, may_create);
            rfsf::PieceRows rows = {};
            const int order = kernel_order(shape);
            float2 *next = reinterpret_cast<float2 *>(state);
            const size_t bins = (size_t)P / 2 + 1;
            const size_t level_words = rfsf::sketch_fft_scan_table_bytes(shape->M, shape->F, P) / sizeof(uint32_t) / (size_t)shape->M;
            for (int a = 0; a < shape->M; ++a) {
                const int levels = shape->M - a;
                rows.rows[a] = next;
                if (rfsf::launch_sketch_fft_scan(dphi + (size_t)a * 4 * shape->F, hash, sign, table + (size_t)a * level_words,
                                                 cnt, shape->L, chunk_lengths, levels, shape->F, P, shape->D, order,
                                                 out + n0 * shape->ld_out, shape->ld_out, nullptr, stream,
                                                 rfsf::TimeCut{plan.pieces, shape->M, plan.pairs, next, 1, 1,
                                                               (int64_t)plan.pieces * levels * (int64_t)bins, levels * (int64_t)bins}) != hipSuccess)
                    return RFSF_E_HIP;
                next += (size_t)cnt * plan.pieces * levels * bins;
            }
            if (rfsf::launch_join_pieces(rows, cnt, plan.pieces, shape->M, (int)bins, next, stream) != hipSuccess)
                return RFSF_E_HIP;
            if (rfsf::launch_sketch_fft_scan(dphi, hash, sign, table, cnt, shape->L, chunk_lengths, shape->M, shape->F, P,
                                             shape->D, order, out + n0 * shape->ld_out, shape->ld_out, nullptr, stream,
                                             rfsf::TimeCut{1, shape->M, (shape->L + 1) / 2, next, 2, 1, shape->M * (int64_t)bins, 0}) != hipSuccess)
                return RFSF_E_HIP;
        }
    }
    return RFSF_OK;
}

// Scratch of the entry point that allocates nothing: one array per GPU, part of the library's code object.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
// Device address of `scratch` on the current device, resolved once per device (each GPU holds its own copy
// at its own address); nullptr if the lookup fails.
void *static_scratch_address()
{
    static void *address[rfsf::kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= rfsf::kMaxDevices) return nullptr;
    if (!address[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        address[dev] = ptr;
    }
    return address[dev];
}
}  // namespace

extern "C" int rfsf_ts_features(const rfsf_ts_shape *shape, const float *X, const float *W,
                                const int32_t *hash, const float *sign, float lengthscale, float *out,
                                void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return features_impl(shape, X, nullptr, W, hash, sign, lengthscale, out, workspace, workspace_bytes, hip_stream,
                         true);
}

extern "C" int rfsf_ts_features_ragged(const rfsf_ts_shape *shape, const float *X, const int64_t *lengths,
                                       const float *W, const int32_t *hash, const float *sign, float lengthscale,
                                       float *out, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return features_impl(shape, X, lengths, W, hash, sign, lengthscale, out, workspace, workspace_bytes, hip_stream,
                         true);
}

extern "C" int rfsf_ts_features_static(const rfsf_ts_shape *shape, const float *X, const float *W,
                                       const int32_t *hash, const float *sign, float lengthscale, float *out,
                                       void *hip_stream)
{
    const int rc = check_shape(shape);
    if (rc != RFSF_OK) return rc;
    if (shape->N > 0 && shape->L > 1) {      // one sequence (increments + state) plus the tables must fit
        size_t incr, state;
        per_sequence_bytes(shape, &incr, &state);
        if (incr + state > kStaticScratchBytes || fixed_bytes(shape) > kStaticScratchBytes - (incr + state))
            return RFSF_E_STATIC_SCRATCH_TOO_SMALL;
    }
    void *ptr = static_scratch_address();
    if (!ptr) return RFSF_E_HIP;
    return features_impl(shape, X, nullptr, W, hash, sign, lengthscale, out, ptr, kStaticScratchBytes, hip_stream,
                         false);
}

extern "C" int rfsf_ts_validate_tables(const int32_t *hash, const float *sign, int32_t M, int32_t F,
                                       int32_t D, void *hip_stream)
{
    if (!hash || !sign) return RFSF_E_NULLPTR;
    if (M < 1 || F < 1) return RFSF_E_BAD_SHAPE;
    if (D < 1 || D > 4096) return RFSF_E_D_NOT_POW2;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    int *flag = nullptr;
    if (hipMalloc(&flag, sizeof(int)) != hipSuccess) return RFSF_E_HIP;
    int host = 0;
    int rc = RFSF_OK;
    if (hipMemcpyAsync(flag, &host, sizeof(int), hipMemcpyHostToDevice, stream) != hipSuccess ||
        rfsf::launch_validate_tables(hash, sign, (int64_t)M * 2 * F, D, flag, stream) != hipSuccess ||
        hipMemcpyAsync(&host, flag, sizeof(int), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        rc = RFSF_E_HIP;
    (void)hipFree(flag);
    if (rc != RFSF_OK) return rc;
    return host ? RFSF_E_BAD_TABLE : RFSF_OK;
}

extern "C" int rfsf_ts_gram(const float *PhiX, int64_t Nx, int64_t ldx, const float *PhiY, int64_t Ny,
                            int64_t ldy, int64_t ncols, float *K, int64_t ldk, void *hip_stream)
{
    if (Nx < 0 || Ny < 0 || ncols < 0) return RFSF_E_BAD_SHAPE;
    if (ldx < ncols || ldy < ncols || ldk < Ny) return RFSF_E_BAD_STRIDE;
    if (Nx == 0 || Ny == 0) return RFSF_OK;
    if (!PhiX || !PhiY || !K) return RFSF_E_NULLPTR;
    if ((Nx + 63) / 64 > 65535 || (Ny + 63) / 64 > 2147483647) return RFSF_E_UNSUPPORTED;     // (stated limits; tiles are counted in grid.x)
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    rfsf::ProfileScope scope(rfsf::kGram, stream);
    return rfsf::launch_gram(PhiX, Nx, ldx, PhiY, Ny, ldy, ncols, K, ldk, stream) == hipSuccess
               ? RFSF_OK : RFSF_E_HIP;
}

extern "C" int rfsf_ts_normalize_features(float *Phi, int64_t N, int64_t ld, int32_t M, int32_t D,
                                          void *hip_stream)
{
    if (N < 0 || M < 1 || D < 1 || N > 0x7fffffffLL) return RFSF_E_BAD_SHAPE;
    if (ld < 1 + (int64_t)M * D) return RFSF_E_BAD_STRIDE;
    if (N == 0) return RFSF_OK;
    if (!Phi) return RFSF_E_NULLPTR;
    rfsf::ProfileScope scope(rfsf::kNormalize, static_cast<hipStream_t>(hip_stream));
    return rfsf::launch_normalize(Phi, N, ld, M, D, static_cast<hipStream_t>(hip_stream)) == hipSuccess
               ? RFSF_OK : RFSF_E_HIP;
}

extern "C" int rfsf_dp1d_features(int64_t N, int64_t L, int32_t d, int32_t M, int32_t F, const float *X,
                                  const float *W, const float *bias, float lengthscale, float *out,
                                  int64_t ld_out, void *hip_stream)
{
    if (N < 0 || L < 1 || d < 1 || M < 1 || F < 1 || N > 0x7fffffffLL || L > ((int64_t)1 << 40) || F > (1 << 24))
        return RFSF_E_BAD_SHAPE;
    if (ld_out < 1 + (int64_t)M * F) return RFSF_E_BAD_STRIDE;
    if (!(lengthscale > 0.0f) || !std::isfinite(lengthscale)) return RFSF_E_BAD_LENGTHSCALE;
    if (d > 64 || M > 16 || (F + 255) / 256 > 65535) return RFSF_E_UNSUPPORTED;
    if ((int64_t)d * F * 4 > 0x7fffffffLL) return RFSF_E_UNSUPPORTED;     // a level of W is addressed with 32-bit byte offsets
    if (N == 0) return RFSF_OK;
    if (!X || !W || !bias || !out) return RFSF_E_NULLPTR;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    rfsf::ProfileScope scope(rfsf::kDp1d, stream);
    const float scale_turns = (float)(0.31830988618379067154 / (double)lengthscale);
    return rfsf::launch_dp1d(X, W, bias, scale_turns, N, L, d, M, F, out, ld_out, stream) == hipSuccess
               ? RFSF_OK : RFSF_E_HIP;
}

namespace {
int check_trp_shape(const rfsf_ts_shape *s)
{
    if (!s) return RFSF_E_NULLPTR;
    if (s->N < 0 || s->L < 1 || s->d < 1 || s->M < 1 || s->F < 1 || s->D < 1) return RFSF_E_BAD_SHAPE;
    if (s->N > ((int64_t)1 << 40) || s->L >= ((int64_t)1 << 31) || s->d > (1 << 20) || s->F > (1 << 24) ||
        s->D > (1 << 24))
        return RFSF_E_BAD_SHAPE;
    if (s->ld_out < 1 + (int64_t)s->M * s->D) return RFSF_E_BAD_STRIDE;
    if (s->M > 16 || (int64_t)s->M * 2 * s->F > ((int64_t)1 << 26) || (int64_t)s->M * s->D > ((int64_t)1 << 26) ||
        (int64_t)s->M * ((s->F + 127) / 128) > 65535 || (s->rff_bf16 != 0 && s->d > 128))
        return RFSF_E_UNSUPPORTED;
    return RFSF_OK;
}
void trp_per_sequence_bytes(const rfsf_ts_shape *s, size_t *incr, size_t *proj)
{
    *incr = (size_t)s->L * (size_t)s->M * 2u * (size_t)s->F * sizeof(float);
    *proj = (size_t)s->L * (size_t)s->M * (size_t)s->D * sizeof(float);
}
constexpr size_t kTrpFixed = 3 * kAlign;
// Sequences of up to this many points leave out the row of their last point, which is no increment: one row in L of the projection, the
// products and the scan, for counting the places of the rows in the projection; with up to 8 channels (16 as bf16 operands), whose projection leaves
// room for both ways, all do. (With rows left out and kept, features, us: 7500 x 8 points, 2 channels, 200 frequencies and projections 413 and 464,
// 2 x 129, 3, 16, 32768 69 and 78, 312 x 64, 18, 228, 400 232 and 233, 200 x 100 244 and 241, 100 x 200 235 and 229.)
constexpr int64_t kCloseUpPoints = 64;
// Sequences per launch of the TRP kernels: at most 65535, and 65535 * 64 rows. The kernels count their tiles and threads
// in grid.x and would take more; the recommended workspace, and what is refused, follow from these numbers.
int64_t trp_chunk_cap(const rfsf_ts_shape *s)
{
    const int64_t by_rows = (int64_t)65535 * 64 / s->L;
    return by_rows < 65535 ? by_rows : 65535;
}
}  // namespace

extern "C" int rfsf_trp_workspace_bytes(const rfsf_ts_shape *shape, size_t *recommended_bytes,
                                        size_t *minimum_bytes)
{
    const int rc = check_trp_shape(shape);
    if (rc != RFSF_OK) return rc;
    size_t incr, proj;
    trp_per_sequence_bytes(shape, &incr, &proj);
    const size_t per = incr + proj;
    if (trp_chunk_cap(shape) < 1) return RFSF_E_UNSUPPORTED;     // one sequence alone is beyond the limit
    int64_t chunk = (int64_t)(kChunkBytesTarget / per);
    if (chunk > trp_chunk_cap(shape)) chunk = trp_chunk_cap(shape);
    if (chunk < 1) chunk = 1;
    if (chunk > shape->N) chunk = shape->N > 0 ? shape->N : 1;
    if (shape->N > 0) {
        const int64_t nchunks = (shape->N + chunk - 1) / chunk;
        chunk = (shape->N + nchunks - 1) / nchunks;
    }
    if (recommended_bytes) *recommended_bytes = (size_t)chunk * per + kTrpFixed;
    if (minimum_bytes) *minimum_bytes = per + kTrpFixed;
    return RFSF_OK;
}

extern "C" int rfsf_trp_features(const rfsf_ts_shape *shape, const float *X, const float *W, const float *Z,
                                 float lengthscale, float *out, void *workspace, size_t workspace_bytes,
                                 void *hip_stream)
{
    int rc = check_trp_shape(shape);
    if (rc != RFSF_OK) return rc;
    if (!(lengthscale > 0.0f) || !std::isfinite(lengthscale)) return RFSF_E_BAD_LENGTHSCALE;
    if (shape->N == 0) return RFSF_OK;
    if (!X || !W || !Z || !out) return RFSF_E_NULLPTR;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int Q = shape->D;
    if (shape->L == 1)
        return rfsf::launch_fill_trivial(out, shape->N, shape->ld_out, 1 + (int64_t)shape->M * Q, stream) == hipSuccess
                   ? RFSF_OK : RFSF_E_HIP;
    if (trp_chunk_cap(shape) < 1) return RFSF_E_UNSUPPORTED;
    if (!workspace) return RFSF_E_NULLPTR;
    size_t incr, proj;
    trp_per_sequence_bytes(shape, &incr, &proj);
    if (workspace_bytes < incr + proj + kTrpFixed) return RFSF_E_WORKSPACE_TOO_SMALL;
    int64_t chunk = (int64_t)((workspace_bytes - kTrpFixed) / (incr + proj));
    if (chunk > shape->N) chunk = shape->N;
    if (chunk > trp_chunk_cap(shape)) chunk = trp_chunk_cap(shape);
    char *base = static_cast<char *>(workspace);
    const size_t mis = (size_t)(reinterpret_cast<uintptr_t>(base) % kAlign);
    float *dphi = reinterpret_cast<float *>(base + (mis ? kAlign - mis : 0));
    float *P = reinterpret_cast<float *>(reinterpret_cast<char *>(dphi) + align_up((size_t)chunk * incr));
    const int twoF = 2 * shape->F;
    const int64_t rf = (int64_t)shape->M * twoF, MQ = (int64_t)shape->M * Q;
    const float inv_ls = 1.0f / lengthscale;
    const bool close_up = shape->L <= kCloseUpPoints || shape->d <= (shape->rff_bf16 != 0 ? 16 : 8);
    for (int64_t n0 = 0; n0 < shape->N; n0 += chunk) {
        const int64_t cnt = shape->N - n0 < chunk ? shape->N - n0 : chunk;
        {
            rfsf::ProfileScope scope(rfsf::kRffIncrements, stream);
            if (rfsf::launch_rff_increments(X + n0 * shape->L * shape->d, W, nullptr, inv_ls, cnt, shape->L, shape->d,
                                            shape->M, shape->F, shape->rff_bf16 != 0, dphi, stream, nullptr, nullptr, close_up) != hipSuccess)
                return RFSF_E_HIP;
        }
        {   // P[:, m, :] = dphi[:, m, :] Z_m^T, the levels' products in one launch
            rfsf::ProfileScope scope(rfsf::kTrpProject, stream);
            const int64_t points = cnt * shape->L - 1;       // (the last one has no increment)
            if (rfsf::launch_gram(dphi, close_up ? points - cnt + 1 : points, rf, Z, Q, twoF, twoF, P, MQ, stream, true, shape->M,
                                  twoF, (int64_t)Q * twoF, Q, points) != hipSuccess)
                return RFSF_E_HIP;
        }
        {
            rfsf::ProfileScope scope(rfsf::kTrpScan, stream);
            if (rfsf::launch_trp_scan(P, shape->N, cnt, shape->L, close_up ? shape->L - 1 : shape->L, shape->M, Q, out + n0 * shape->ld_out, shape->ld_out,
                                      stream) != hipSuccess)
                return RFSF_E_HIP;
        }
    }
    return RFSF_OK;
}

extern "C" int rfsf_ts_probe_peaks(void *scratch, size_t scratch_bytes, rfsf_ts_peaks *out, void *hip_stream)
{
    if (!scratch || !out) return RFSF_E_NULLPTR;
    if (scratch_bytes < 64) return RFSF_E_WORKSPACE_TOO_SMALL;
    double v[6];
    if (rfsf::probe_peaks(scratch, scratch_bytes, v, static_cast<hipStream_t>(hip_stream)) != hipSuccess) return RFSF_E_HIP;
    *out = rfsf_ts_peaks{v[0], v[1], v[2], v[3], v[4], v[5]};
    return RFSF_OK;
}

extern "C" int rfsf_ts_profile_enable(int on)
{
    rfsf::g_profile_on = on != 0;
    return RFSF_OK;
}

extern "C" int rfsf_ts_profile_read(rfsf_ts_profile *out, int reset)
{
    if (!out) return RFSF_E_NULLPTR;
    *out = rfsf_ts_profile{0.0, 0, 0.0, 0, 0.0, 0, 0.0, 0, 0.0, 0, 0.0, 0, 0.0, 0};
    int rc = RFSF_OK;
    for (const rfsf::TimedLaunch &t : rfsf::g_launches) {
        float ms = 0.f;
        if (hipEventSynchronize(t.stop) != hipSuccess || hipEventElapsedTime(&ms, t.start, t.stop) != hipSuccess) {
            rc = RFSF_E_HIP;
            continue;
        }
        switch (t.k) {
            case rfsf::kRffIncrements: out->ms_rff_increments += ms; ++out->launches_rff_increments; break;
            case rfsf::kSketchFftScan: out->ms_sketch_fft_scan += ms; ++out->launches_sketch_fft_scan; break;
            case rfsf::kGram: out->ms_gram += ms; ++out->launches_gram; break;
            case rfsf::kNormalize: out->ms_normalize += ms; ++out->launches_normalize; break;
            case rfsf::kDp1d: out->ms_dp1d += ms; ++out->launches_dp1d; break;
            case rfsf::kTrpProject: out->ms_trp_project += ms; ++out->launches_trp_project; break;
            default: out->ms_trp_scan += ms; ++out->launches_trp_scan; break;
        }
    }
    if (reset) {
        for (const rfsf::TimedLaunch &t : rfsf::g_launches) {
            (void)hipEventDestroy(t.start);
            (void)hipEventDestroy(t.stop);
        }
        rfsf::g_launches.clear();
    }
    return rc;
}
