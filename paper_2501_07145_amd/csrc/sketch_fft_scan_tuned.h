// Tuned kernel for steps 3-4 (CountSketch, Fourier-domain level recursion over time, inverse
// transform; Sec. 3.5, eqs. (cs), (ts_def), (ts_rec) with p = 1).
//
// Work decomposition (one workgroup per sequence, M wavefronts, wavefront m owns level m; a transform always
// lives in one wavefront: 16 points per lane up to D = 1024, 32 for D = 2048, 20 for 100, 200, 500 and 1000):
//   per iteration every wavefront handles FPW pairs of consecutive time steps of its level:
//     1. CountSketch as a gather. The signed increments of the 2*FPW time steps arrive in LDS in
//        their natural order (step 2k -> real part, step 2k+1 -> imaginary part of the float2 of
//        coordinate a, one staging area per pair): the producing kernel stores them in exactly this
//        form, signs applied, and they are loaded from global memory straight into LDS
//        (global_load_lds_dwordx4: 16 bytes per lane at LDS base + 16 * lane), without passing
//        through registers and without LDS-write instructions. A table built once per call lists,
//        for every bucket, the first two coordinates that hash to it; the few coordinates that
//        are third or later in their bucket are first folded into the bucket's first coordinate
//        by conflict-free read-add-write rounds (one round per rank, so no two lanes of a round
//        touch the same float2). Then each FFT lane reads the (at most two) sources of each of
//        its R buckets straight into its FFT registers. No LDS atomics (a full-wavefront
//        ds_add_f32 costs ~190 cycles on this chip), no clearing, and the summation order is
//        fixed, so results are bit-reproducible.
//     2. FPW complex FFTs of length D held in the wavefront's LDS slots, G = D/R lanes per
//        transform with R points per lane in registers (passes of butterflies in registers with an LDS exchange
//        between them, which the middle pass of 512 to 2048 points spares: WaveFft; no workgroup barrier
//        inside the transform),
//   then, after one barrier, every thread owns a few frequency bins, separates the two real
//   transforms of each slot, and advances the accumulators A_1..A_M of its bins by the two
//   time steps (A_m += A_{m-1}(before the step) * C_m, A_0 = 1; with signature order 2 also
//   + 1/2 A_{m-2}(before the step) * C_{m-1} * C_m, with order 3 also + 1/6 A_{m-3} C_{m-2} C_{m-1} C_m:
//   Sec. 3.5 eq. (ts_rec), the terms q = 2, 3).
//   After the last time step, wavefront m transforms A_m back and writes block m of the row.
//   (Fetching the next iteration's rows ahead of time was tried in several placements and was never
//   faster: the pace is set by the instruction streams of the resident workgroups, not by the load
//   latency of one of them. What did pay off every time was more resident wavefronts.)
//
// The increments arrive pre-multiplied by 1/2 and by their CountSketch sign (done by the producing
// kernel); 1/2 is the factor of the two-for-one separation  C0 = (Z[f] + conj Z[D-f]) / 2,  C1 = (Z[f] - conj Z[D-f]) / 2i.
#pragma once

#include "rfsf_internal.h"

#include <type_traits>

namespace rfsf {
namespace tuned {

// LDS index padding: one float2 of padding after every 16, so that the strided exchange of the
// Stockham passes and the contiguous accesses are both free of bank conflicts.
__host__ __device__ constexpr int pad(int e) { return e + (e >> 4); }

// Twiddles of a butterfly of r points behind the first pass (twiddle_entry).
__host__ __device__ constexpr int twiddles(int r) { return (r & (r - 1)) == 0 ? r / 2 : r - 1; }

template <int LOG2D_, int LOG2R_ = 4, bool ROWED = (LOG2D_ >= 9 && LOG2D_ <= 11)>
struct Plan {
    static constexpr int LOG2D = LOG2D_;
    static constexpr int D = 1 << LOG2D;
    static constexpr int LOG2R = LOG2R_;
    static constexpr int kMinWaves = LOG2R_ > 4 ? 2 : 4;   // wavefronts per SIMD the register budget is set for
    static constexpr int R = 1 << LOG2R;        // points per lane
    static constexpr int G = D / R;             // lanes per transform
    static_assert(G <= 64, "a transform lives in one wavefront");
    static constexpr int FPW = 64 / G;          // transforms per wavefront
    static constexpr int GF = G;                // entries per fold round
    // Lanes of a transform in rows of 16 (ROWS of them): the middle pass meets in registers (WaveFft::run_rows)
    static constexpr bool kRowed = ROWED, kTwoPass = false;
    static constexpr int ROWS = G / 16, MID = kRowed ? ROWS * (R / 16) : 1;
    static constexpr int kMidTwiddles = kRowed ? 16 * (MID / 2) : 0;     // float2: 16 / ROWS butterflies of a lane, ROWS rows
    static constexpr int PD = D + D / 16;       // padded transform length in float2
    static constexpr int NP = LOG2D <= 4 ? 1 : (LOG2D <= 8 ? 2 : 3);
    static constexpr int radix(int p)
    {
        switch (LOG2D) {
            case 4: return 16;
            case 5: return p == 0 ? 16 : 2;
            case 6: return p == 0 ? 16 : 4;
            case 7: return p == 0 ? 16 : 8;
            case 8: return 16;
            case 9: return p == 1 ? 2 : 16;
            // three passes: the small radix goes in the middle, where its inputs lie in as many rows of lanes and meet
            // without an exchange (kRowed). D = 512 takes 16 points per lane and a radix-2 middle pass rather than 32 points
            // per lane and two passes: half the registers and half the LDS per workgroup doubles the resident
            // workgroups (20 % faster even when the middle pass had an exchange of its own)
            case 10: return p == 1 ? 4 : 16;
            default: return p == 1 ? 8 : 16;    // 11 (32 points per lane)
        }
    }
    static constexpr int Ns(int p) { return p == 0 ? 1 : Ns(p - 1) * radix(p - 1); }
    // butterflies of pass p with distinct twiddles: butterfly u of a lane has k = (lg + G*u) mod Ns,
    // the same for every u when Ns divides G
    static constexpr int tw_sets(int p) { return G % Ns(p) == 0 ? 1 : R / radix(p); }
    // The twiddles of a radix-16 pass (8 per set) would cost 16 registers per set; they live in an
    // LDS table shared by the workgroup instead. Smaller last passes (64 and 128 points) keep theirs in registers; those of
    // the middle pass differ from butterfly to butterfly and row to row and follow in the table (kMidTwiddles).
    static constexpr bool tw_in_lds(int p) { return p > 0 && radix(p) >= 16; }
    static constexpr int tw_regs(int p) { return (p == 0 || tw_in_lds(p) || kRowed) ? 0 : tw_sets(p) * twiddles(radix(p)); }
    static constexpr int tw_lds(int p) { return tw_in_lds(p) ? tw_sets(p) * twiddles(radix(p)) * G : 0; }   // float2 entries
    static constexpr int kBoundTwiddles = tw_in_lds(NP - 1) ? tw_sets(NP - 1) * (radix(NP - 1) - 1) * G : 0;   // see tuned_lds_bound
    // array offsets of pass p: register twiddles (complex), LDS twiddles (float2) and write bases
    static constexpr int tw_off(int p) { return p <= 1 ? 0 : tw_off(p - 1) + tw_regs(p - 1); }
    static constexpr int twl_off(int p) { return p <= 1 ? 0 : twl_off(p - 1) + tw_lds(p - 1); }
    static constexpr int NTWL = twl_off(NP) + kMidTwiddles;
    static constexpr int wb_off(int p) { return p == 0 ? 0 : wb_off(p - 1) + R / radix(p - 1); }
    static constexpr int NTW = tw_off(NP) == 0 ? 1 : tw_off(NP);
    static constexpr int NWB = wb_off(NP);
    static constexpr int roff(int q) { return G >= 16 ? q * (G + G / 16) : tuned::pad(G * q); }
    static constexpr int pad(int e) { return tuned::pad(e); }     // position in a slot of element e
};

// Transform lengths 2^a 5^b that the paper's own experiments use as bucket counts (100, 200, 500, 1000): exact
// transforms of that length instead of a linear convolution in the next power of two above M (D - 1) + 1.
// 20 points per lane, D / 20 lanes per transform (the remaining lanes of a wavefront repeat the work of the
// first ones, see the kernel). Selected as Plan<D>.
//
// 100, 200 and 500 points as 20 x G, G lanes: a lane transforms the 20 points it holds, which needs no twiddles, then the 20 butterflies of
// G points are dealt to the lanes: four, two or one each (with 500 points the last five lanes repeat others). One exchange; passes of radix 10, 10 and
// 5, 2 or none took one more from 200 points on, and twiddles behind each. Features (with the
// projection kernel where they have one), three passes and two, us: 2000 x 200 points, two levels, 100 buckets 132 -> 112, 200 200 -> 180, 500
// 986 -> 793, five levels 287 -> 286, 665 -> 609, 2569 -> 2327; 1500 x 333, 500 buckets, order 2, four levels 1632 -> 1543, five 2999 -> 3020. (With 100
// points most of it is LDS that slots without padding leave to a fourth workgroup of single wavefronts.)
template <int DD>
struct TwoPassPlan {
    static constexpr int LOG2D = DD;
    static constexpr int D = DD;
    static constexpr int R = 20;
    static constexpr int G = D / R;
    static constexpr int FPW = 64 / G;
    static constexpr int GF = G;
    static constexpr bool kRowed = false, kTwoPass = true;
    static constexpr int PD = D;
    static constexpr int NB = G > R ? 1 : R / G;        // butterflies of a lane in the second pass
    static constexpr int kButterflyLanes = R / NB;      // lanes with butterflies of their own
    static constexpr int NTWL = NB * twiddles(G) * kButterflyLanes;
    static constexpr int kBoundTwiddles = D == 100 ? 90 : D == 200 ? 190 : 850;      // of three passes, see tuned_lds_bound
    static constexpr int NTW = 1, NWB = 1;
    static constexpr int roff(int q) { return G * q; }
    __host__ __device__ static constexpr int pad(int e) { return e; }
    static constexpr int kMinWaves = 4;
    static_assert(D == R * G && G * FPW <= 64 && R == NB * kButterflyLanes, "");
};
template <> struct Plan<100> : TwoPassPlan<100> {};
template <> struct Plan<200> : TwoPassPlan<200> {};
template <> struct Plan<500> : TwoPassPlan<500> {};
// 1000 points: three passes of radix 10; slots are padded so that the positions of a pass are a base plus constants and the writes of a
// transform take 140 bank rows instead of 180; the twiddles of all passes after the first live in the LDS table.
template <int DD>
struct ThreePassPlan {
    static constexpr int LOG2D = DD;
    static constexpr int D = DD;
    static constexpr int R = 20;
    static constexpr int G = D / R;
    static constexpr int FPW = 64 / G;
    static constexpr int GF = G;
    static constexpr bool kRowed = false, kTwoPass = false;
    static constexpr int kPad = 50;             // one float2 of padding after every kPad of a slot
    static constexpr int PD = D + (D - 1) / kPad;
    static constexpr int NP = 3;
    static constexpr int radix(int) { return 10; }
    static constexpr int Ns(int p) { return p == 0 ? 1 : Ns(p - 1) * radix(p - 1); }
    static constexpr int tw_sets(int p) { return G % Ns(p) == 0 ? 1 : R / radix(p); }
    static constexpr bool tw_in_lds(int p) { return p > 0; }
    static constexpr int tw_regs(int) { return 0; }
    static constexpr int tw_lds(int p) { return tw_in_lds(p) ? tw_sets(p) * twiddles(radix(p)) * G : 0; }
    static constexpr int tw_off(int) { return 0; }
    static constexpr int twl_off(int p) { return p <= 1 ? 0 : twl_off(p - 1) + tw_lds(p - 1); }
    static constexpr int NTWL = twl_off(NP);
    static constexpr int kBoundTwiddles = NTWL;
    static constexpr int wb_off(int p) { return p == 0 ? 0 : wb_off(p - 1) + R / radix(p - 1); }
    static constexpr int NTW = 1;
    static constexpr int NWB = wb_off(NP);
    static constexpr int roff(int q) { return G * q + G * q / kPad; }
    __host__ __device__ static constexpr int pad(int e) { return e + e / kPad; }
    static constexpr int kMinWaves = 4;
};
template <> struct Plan<1000> : ThreePassPlan<1000> {};
// 2048 points in one wavefront: 32 points per lane (twice the registers, half the resident wavefronts, no barrier
// inside the transform). Selected as Plan<2048>.
template <> struct Plan<2048> : Plan<11, 5> {};
// Kernels that keep the exchange of the middle pass. Rows that meet in registers are faster in most, 0.94 of the time over all lengths, levels and
// orders, and spill less; but what the compiler makes of them leaves these slower (features, six shapes each, 60 and 250 frequencies: 3 x 400, 30 x
// 1000 and 100 x 200 points cut in time, 300 x 60, 700 x 40 and 2500 x 30 whole; geometric mean and largest against the exchange): 512 points cut, two
// levels 1.03, 1.06; 1024 cut, orders 2 and 3, four levels 1.03 and 1.05, 1.12, five 1.06 and 1.04, 1.07, six 1.05 and 1.03, 1.07; 1024 whole, seven,
// orders 2 and 3 1.03 and 1.05, 1.11; 2048 whole, seven, order 3 1.26, 1.40; 4096, order 3, four and six 1.07 and 1.19, 1.43, order 1, eight
// 1.07, 1.09. (Left in rows: 1024 cut, three, orders 2 and 3 1.01, 0.96 to 1.12, five, order 1 1.02; 512 whole, two, 1.00, 0.93 to 1.06; 4096, order
// 3, five 1.02, 0.96 to 1.17.)
constexpr bool exchanges(int LOG2D, int M, int ORDER, bool JOINT)
{
    switch (LOG2D) {
        case 9: return JOINT && M == 2;
        case 10: return ORDER > 1 && (JOINT ? M >= 4 && M <= 6 : M == 7);
        case 2048: return !JOINT && M == 7 && ORDER == 3;
        case 12: return ORDER == 3 ? M == 4 || M == 6 : ORDER == 1 && M == 8;
        default: return false;
    }
}
template <int LOG2D, bool EXCHANGES> struct PlanBy : Plan<LOG2D> {};
template <> struct PlanBy<9, true> : Plan<9, 4, false> {};
template <> struct PlanBy<10, true> : Plan<10, 4, false> {};
template <> struct PlanBy<2048, true> : Plan<11, 5, false> {};
template <int LOG2D, int M, int ORDER, bool JOINT> using KernelPlan = PlanBy<LOG2D, exchanges(LOG2D, M, ORDER, JOINT)>;

// Geometry of one LDS slot (float2 units): [0, ZS) data -- the staging area uses [0, 2F), the transform [0, PD) --,
// [ZS] a float2 that is always zero (source of buckets without a first or second coordinate). A direct load deposits
// 128 coordinates; of the last one of a pair the lanes beyond 2F stay out. (With all 64, F = 32 staged twice what it
// has: 1000 x 100 points, four levels, D = 64 and F = 32 59 us against 45, D = 128 and F = 70 94 against 68, five
// levels, D = 256 and F = 70 206 against 190.)
__host__ __device__ constexpr int staged(int twoF) { return (twoF + 127) & ~127; }      // by whole direct loads
__host__ __device__ constexpr int zero_slot(int PD, int twoF) { return PD > twoF ? PD : twoF; }
__host__ __device__ constexpr int slot_stride(int PD, int twoF) { return (zero_slot(PD, twoF) + 2) & ~1; }

// Per-level table built once per call (uint32 words):
//   [0]                 NG, number of fold rounds (0 if the level has lists)
//   [1]                 number of list rows (0 if the level has fold rounds)
//   [2, 2 + R)          list rows of bucket group q (the buckets lg + G q)
//   [64, 64 + D)        gather words: low 16 bits byte offset of the bucket's first coordinate in the
//                       staging area, high 16 bits of its second one (zero float2 if there is none)
//   [.., + 2F*G)        fold entries, G per round: low 16 bits byte offset of the coordinate to fold,
//                       high 16 bits byte offset of the first coordinate of its bucket (0xffff: padding)
//                       or list rows, G words each, group after group, a multiple of four per group: word lg holds
//                       two more coordinates of bucket lg + G q, in the form of the gather words
struct TableLayout {
    int gather, fold, words;
};
__host__ __device__ inline TableLayout table_layout(int D, int G, int twoF)
{
    TableLayout t;
    t.gather = 64;
    t.fold = t.gather + D;
    t.words = (t.fold + twoF * G + 63) & ~63;
    return t;
}
constexpr uint32_t kFoldPad = 0xffffu;
constexpr int kFoldInRegs = 4;      // fold rounds whose entries are fetched with the other tables; later rounds load
                                    // theirs on the spot (4 measured best of 2, 4, 6, 8)

constexpr int bitrev(int x, int bits)
{
    int r = 0;
    for (int i = 0; i < bits; ++i) r |= ((x >> i) & 1) << (bits - 1 - i);
    return r;
}
constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }

// Butterflies with the twiddle inside: w = c (1 + i t) is kept as (c, t), w b = c (b.x - t b.y, b.y + t b.x) takes two
// multiply-adds and a +- w b four more. Multiplying by w first and adding afterwards takes eight instructions and rounds
// three times; this rounds twice. What bounds these transforms is the number of vector instructions and of LDS
// accesses (1024 points: 436 instead of 508 vector instructions and 8 instead of 15 twiddles read per lane; the sketch kernel of
// 2000 x 200 points, D = 512, four levels 817 -> 772 us, 3000 x 200, D = 256, six levels 1140 -> 1010, 1000 x 100, D = 2048 1323 ->
// 1281, 500 x 100, D = 2000 in 8192 points 2748 -> 2501; D = 1024 is bound by its exchanges: 2097 and 2095). Errors of the features
// against 64 bits over fifteen shapes of all lengths: 4.4e-7 -> 4.1e-7 (geometric mean), none larger by more than a hundredth.
// Behind a first pass, input t of an r-point butterfly carries w^t: the butterfly is the polynomial of its inputs at the
// points w exp(-2 pi i q / r), even and odd powers apart, which needs the powers w^(r/2), ..., w^2, w alone, times roots.
// A right angle has c = 0: 2^-40 stands for it, whose square is lost beside 1.
__device__ __forceinline__ float2 twiddle_form(float c, float s)
{
    return c == 0.f ? make_float2(0x1p-40f, s * 0x1p40f) : make_float2(c, s / c);
}
__device__ __forceinline__ void butterfly(float2 &a, float2 &b, float2 w)               // a + w b, a - w b
{
    const float u = fmaf(-w.y, b.y, b.x), v = fmaf(w.y, b.x, b.y), x = a.x, y = a.y;
    a = make_float2(fmaf(w.x, u, x), fmaf(w.x, v, y));
    b = make_float2(fmaf(-w.x, u, x), fmaf(-w.x, v, y));
}
__device__ __forceinline__ void butterfly_i(float2 &a, float2 &b, float2 w)             // a - i w b, a + i w b
{
    const float u = fmaf(-w.y, b.y, b.x), v = fmaf(w.y, b.x, b.y), x = a.x, y = a.y;
    a = make_float2(fmaf(w.x, v, x), fmaf(-w.x, u, y));
    b = make_float2(fmaf(-w.x, v, x), fmaf(w.x, u, y));
}
__device__ __forceinline__ void butterfly_one(float2 &a, float2 &b)                      // a + b, a - b
{
    const float2 x = a, y = b;
    a = make_float2(x.x + y.x, x.y + y.y);
    b = make_float2(x.x - y.x, x.y - y.y);
}
__device__ __forceinline__ void butterfly_one_i(float2 &a, float2 &b)                    // a - i b, a + i b
{
    const float2 x = a, y = b;
    a = make_float2(x.x + y.y, x.y - y.x);
    b = make_float2(x.x - y.y, x.y + y.x);
}
// Entry e of the twiddles of an r-point butterfly whose inputs carry powers of exp(-2 pi i k / (Ns r)). Powers of two: entry 0
// belongs to the stage that combines single inputs, entries H/2 + j, j < H/2, to the one that combines H and H of
// them, at its roots j (roots j + H/2 are -i times these). Ten points: entries 0 to 3 the even powers 2, 4, 6, 8, as real
// and imaginary part, then those of the stage that combines five and five. Five points: the powers 1 to 4, likewise. 25 points: the powers
// 5, 10, 15, 20, then, for inputs b = 1 .. 4 modulo 5 and q = 0 .. 4, power b times the 25th root of unity to the b q.
template <int r>
__device__ __forceinline__ float2 twiddle_entry(int e, int k, int Ns)
{
    float s, c;
    if constexpr ((r & (r - 1)) == 0) {
        const int H = e == 0 ? 1 : 2 << (31 - __clz(e)), j = e == 0 ? 0 : e - H / 2;
        sincospif(-(float)(k + j * Ns) / (float)(H * Ns), &s, &c);
        return twiddle_form(c, s);
    } else if (r == 10 && e >= 4) {
        sincospif(-2.0f * (float)(k + (e - 4) * Ns) / (float)(10 * Ns), &s, &c);
        return twiddle_form(c, s);
    } else {
        const int power = r == 25 && e >= 4 ? ((e - 4) / 5 + 1) * (k + (e - 4) % 5 * Ns) : k * (e + 1) * (r == 10 ? 2 : r == 25 ? 5 : 1);
        sincospif(-2.0f * (float)power / (float)(Ns * r), &s, &c);
        return make_float2(c, s);
    }
}
// Transform of the N inputs from B on (bit-reversed order in, natural order out), half after half, so that work can start with
// the first inputs that arrive. tw[e]: twiddle_entry e.
template <int B, int N, int r>
__device__ __forceinline__ void dft_halves(float2 (&x)[r], const float2 (&tw)[twiddles(r)])
{
    if constexpr (N > 1) {
        constexpr int H = N / 2;
        dft_halves<B, H>(x, tw);
        dft_halves<B + H, H>(x, tw);
#pragma unroll
        for (int j = 0; j < (H > 1 ? H / 2 : 1); ++j) {
            const float2 w = tw[H > 1 ? H / 2 + j : 0];
            butterfly(x[B + j], x[B + j + H], w);
            if (H > 1) butterfly_i(x[B + j + H / 2], x[B + j + H / 2 + H], w);
        }
    }
}
// The same without twiddles (w = 1): their constants, and the trivial ones cost nothing. Z > 1: only the first r / Z inputs (of natural
// order) are not zero, so that stages of up to Z points copy them.
template <int B, int N, int Z, int r>
__device__ __forceinline__ void dft_halves_plain(float2 (&x)[r])
{
    static_assert(r <= 16, "");
    if constexpr (N == Z) {
#pragma unroll
        for (int j = 1; j < N; ++j) x[B + j] = x[B];
    } else if constexpr (N > 1) {
        constexpr float c[4] = {1.0f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f};      // of j pi / 8
        constexpr float t[4] = {0.0f, -0.41421356237309505f, -1.0f, -2.4142135623730950f};                    // minus tangent
        constexpr int H = N / 2;
        dft_halves_plain<B, H, Z>(x);
        dft_halves_plain<B + H, H, Z>(x);
#pragma unroll
        for (int j = 0; j < (H > 1 ? H / 2 : 1); ++j) {
            const int e = j * (8 / H);
            if (j == 0) butterfly_one(x[B], x[B + H]);
            else butterfly(x[B + j], x[B + j + H], make_float2(c[e], t[e]));
            if (H > 1) {
                if (j == 0) butterfly_one_i(x[B + H / 2], x[B + H / 2 + H]);
                else butterfly_i(x[B + j + H / 2], x[B + j + H / 2 + H], make_float2(c[e], t[e]));
            }
        }
    }
}

__device__ __forceinline__ float2 cmulf(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 cfmaf(float2 a, float2 b, float2 c)   // a * b + c
{
    return make_float2(fmaf(a.x, b.x, fmaf(-a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(a.y, b.x, c.y)));
}

// In-register forward DFT of 5 points at x[B], x[B + ST], ..., natural order in and out.
template <int B, int ST, int TOTAL>
__device__ __forceinline__ void dft5(float2 (&x)[TOTAL])
{
    constexpr float c1 = 0.30901699437494742f, c2 = -0.80901699437494742f;    // cos(2 pi / 5), cos(4 pi / 5)
    constexpr float s1 = 0.95105651629515357f, s2 = 0.58778525229247313f;     // sin(2 pi / 5), sin(4 pi / 5)
    const float2 x0 = x[B], x1 = x[B + ST], x2 = x[B + 2 * ST], x3 = x[B + 3 * ST], x4 = x[B + 4 * ST];
    const float2 t1 = make_float2(x1.x + x4.x, x1.y + x4.y), t2 = make_float2(x2.x + x3.x, x2.y + x3.y);
    const float2 t3 = make_float2(x1.x - x4.x, x1.y - x4.y), t4 = make_float2(x2.x - x3.x, x2.y - x3.y);
    x[B] = make_float2(x0.x + t1.x + t2.x, x0.y + t1.y + t2.y);
    const float2 a1 = make_float2(fmaf(c1, t1.x, fmaf(c2, t2.x, x0.x)), fmaf(c1, t1.y, fmaf(c2, t2.y, x0.y)));
    const float2 a2 = make_float2(fmaf(c2, t1.x, fmaf(c1, t2.x, x0.x)), fmaf(c2, t1.y, fmaf(c1, t2.y, x0.y)));
    const float2 b1 = make_float2(fmaf(s1, t3.x, s2 * t4.x), fmaf(s1, t3.y, s2 * t4.y));
    const float2 b2 = make_float2(fmaf(s2, t3.x, -s1 * t4.x), fmaf(s2, t3.y, -s1 * t4.y));
    // X1 = a1 - i b1, X4 = a1 + i b1, X2 = a2 - i b2, X3 = a2 + i b2
    x[B + ST] = make_float2(a1.x + b1.y, a1.y - b1.x);
    x[B + 4 * ST] = make_float2(a1.x - b1.y, a1.y + b1.x);
    x[B + 2 * ST] = make_float2(a2.x + b2.y, a2.y - b2.x);
    x[B + 3 * ST] = make_float2(a2.x - b2.y, a2.y + b2.x);
}

// In-register forward DFTs of 10 and 20 points, natural order in and out. 5 has no factor in common with 2 and 4, so that points numbered
// by both remainders fall into transforms of five and of two or four points with no twiddles between them.
__device__ __forceinline__ void dft10_plain(float2 (&x)[10])
{
    float2 y[10];
#pragma unroll
    for (int n = 0; n < 10; ++n) y[n] = x[(n / 5 * 5 + n % 5 * 2) % 10];
    dft5<0, 1, 10>(y);
    dft5<5, 1, 10>(y);
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        butterfly_one(y[q], y[5 + q]);
        x[6 * q % 10] = y[q];
        x[(5 + 6 * q) % 10] = y[5 + q];
    }
}
__device__ __forceinline__ void dft20_plain(float2 (&x)[20])
{
    float2 y[20];
#pragma unroll
    for (int n = 0; n < 20; ++n) y[n] = x[(n / 5 * 5 + n % 5 * 4) % 20];
    dft5<0, 1, 20>(y);
    dft5<5, 1, 20>(y);
    dft5<10, 1, 20>(y);
    dft5<15, 1, 20>(y);
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        butterfly_one(y[q], y[10 + q]);
        butterfly_one(y[5 + q], y[15 + q]);
        butterfly_one(y[q], y[5 + q]);
        butterfly_one_i(y[10 + q], y[15 + q]);
        x[16 * q % 20] = y[q];
        x[(5 + 16 * q) % 20] = y[10 + q];
        x[(10 + 16 * q) % 20] = y[5 + q];
        x[(15 + 16 * q) % 20] = y[15 + q];
    }
}
template <typename Twiddle>
__device__ __forceinline__ void dft10(float2 (&x)[10], Twiddle tw)
{
#pragma unroll
    for (int u = 1; u < 5; ++u) {
        const float2 w = tw(u - 1);
        x[2 * u] = cmulf(x[2 * u], w);
        x[2 * u + 1] = cmulf(x[2 * u + 1], w);
    }
    dft5<0, 2, 10>(x);
    dft5<1, 2, 10>(x);
    float2 y[10];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        y[q] = x[2 * q];
        y[q + 5] = x[2 * q + 1];
        butterfly(y[q], y[q + 5], tw(4 + q));
    }
#pragma unroll
    for (int q = 0; q < 10; ++q) x[q] = y[q];
}
template <int Q, typename Twiddle>
__device__ __forceinline__ void dft25_row(float2 (&x)[25], Twiddle tw)
{
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 1; b < 5; ++b) x[5 * Q + b] = cmulf(x[5 * Q + b], tw(4 + 5 * (b - 1) + Q));
    dft5<5 * Q, 1, 25>(x);
}
// 25 points as 5 x 5; the twiddles of the inputs b modulo 5 wait until the transforms over those inputs are done (twiddle_entry).
template <typename Twiddle>
__device__ __forceinline__ void dft25(float2 (&x)[25], Twiddle tw)
{
#pragma unroll
    for (int a = 1; a < 5; ++a) {
        const float2 w = tw(a - 1);
#pragma unroll
        for (int b = 0; b < 5; ++b) x[5 * a + b] = cmulf(x[5 * a + b], w);
    }
    dft5<0, 5, 25>(x);
    dft5<1, 5, 25>(x);
    dft5<2, 5, 25>(x);
    dft5<3, 5, 25>(x);
    dft5<4, 5, 25>(x);
    // (no twiddles of transforms to come: registers)
    dft25_row<0>(x, tw);
    dft25_row<1>(x, tw);
    dft25_row<2>(x, tw);
    dft25_row<3>(x, tw);
    dft25_row<4>(x, tw);
    float2 y[25];
#pragma unroll
    for (int n = 0; n < 25; ++n) y[n / 5 + 5 * (n % 5)] = x[n];
#pragma unroll
    for (int n = 0; n < 25; ++n) x[n] = y[n];
}

// Forward DFT of r points, natural order in and out; input t times the t-th power of the twiddle that tw stands for.
// (AHEAD: the nine twiddles of a ten-point butterfly are read before it starts, which is faster by 1 to 2 per cent where the registers
// hold them.)
template <bool AHEAD, int r, typename Twiddle>
__device__ __forceinline__ void dft(float2 (&x)[r], Twiddle tw)
{
    if constexpr (r == 10 && !AHEAD) {
        dft10(x, tw);
    } else if constexpr (r == 10) {
        float2 w[9];
#pragma unroll
        for (int e = 0; e < 9; ++e) w[e] = tw(e);
        dft10(x, [&](int e) { return w[e]; });
    } else if constexpr (r == 25) {
        dft25(x, tw);
    } else if constexpr (r == 5) {
#pragma unroll
        for (int t = 1; t < 5; ++t) x[t] = cmulf(x[t], tw(t - 1));
        dft5<0, 1, 5>(x);
    } else {
        float2 w[twiddles(r)], y[r];
#pragma unroll
        for (int e = 0; e < twiddles(r); ++e) w[e] = tw(e);
#pragma unroll
        for (int t = 0; t < r; ++t) y[bitrev(t, ilog2(r))] = x[t];
        dft_halves<0, r>(y, w);
#pragma unroll
        for (int t = 0; t < r; ++t) x[t] = y[t];
    }
}
template <int Z = 1, int r>
__device__ __forceinline__ void dft_plain(float2 (&x)[r])
{
    static_assert(Z == 1 || r == 16, "");
    if constexpr (r == 10) {
        dft10_plain(x);
    } else if constexpr (r == 20) {
        dft20_plain(x);
    } else {
        float2 y[r];
#pragma unroll
        for (int t = 0; t < r; ++t) y[bitrev(t, ilog2(r))] = x[t];
        dft_halves_plain<0, r, Z>(y);
#pragma unroll
        for (int t = 0; t < r; ++t) x[t] = y[t];
    }
}
// Order in which a pass reads a lane's R points: butterfly after butterfly, each in the order in which it can start (that of memory
// with ten and five points, where it made no difference).
template <int R, int r>
__device__ constexpr int read_order(int i)
{
    constexpr int NB = R / r;
    const int u = i / r, t = i % r;
    return (r & (r - 1)) == 0 ? u + NB * bitrev(t, ilog2(r)) : i;
}

// The same for a thread whose float2 are not complex numbers but two independent reals (pk; bins 0 and D/2
// of a real sequence's transform, which one thread carries in the two halves of its values): the products
// become componentwise. With pk false these are cmulf and cfmaf, operation for operation.
// (pk: true or false, or, in a vector register, all bits set or none, which a logic instruction chooses by in 2.7 cycles of a SIMD: a
// select takes 4.5, from vcc up to 16. In the kernel of a workgroup per sequence, where one wavefront in eight has such a thread, it gains
// nothing and costs registers: 20 x 4000 points, 512 buckets, four levels 305 -> 323 us.)
__device__ __forceinline__ float choose(bool pk, float x, float y) { return pk ? x : y; }
__device__ __forceinline__ float choose(uint32_t pk, float x, float y)
{
    return __uint_as_float(__builtin_amdgcn_bitop3_b32(pk, __float_as_uint(x), __float_as_uint(y), 0xca));
}
template <typename Packed>
__device__ __forceinline__ float2 cmulf_pk(float2 a, float2 b, Packed pk)
{
    const float s = choose(pk, 0.f, b.y), r = choose(pk, b.y, b.x);
    return make_float2(fmaf(a.x, b.x, -a.y * s), fmaf(a.x, s, a.y * r));
}
template <typename Packed>
__device__ __forceinline__ float2 cfmaf_pk(float2 a, float2 b, float2 c, Packed pk)
{
    const float s = choose(pk, 0.f, b.y), r = choose(pk, b.y, b.x);
    return make_float2(fmaf(a.x, b.x, fmaf(-a.y, s, c.x)), fmaf(a.x, s, fmaf(a.y, r, c.y)));
}

// Exchanges the odd halves (BY = 32) or rows of 16 lanes (BY = 16) of a with the even ones of b.
template <int BY>
__device__ __forceinline__ void swap_rows(float &a, float &b)
{
    const unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    if constexpr (BY == 32) {
        const auto s = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        a = __uint_as_float(s[0]);
        b = __uint_as_float(s[1]);
    } else {
        const auto s = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        a = __uint_as_float(s[0]);
        b = __uint_as_float(s[1]);
    }
}
template <int BY>
__device__ __forceinline__ void swap_rows(float2 &a, float2 &b)
{
    swap_rows<BY>(a.x, b.x);
    swap_rows<BY>(a.y, b.y);
}

// Orders the LDS traffic of one wavefront: its LDS instructions execute in order, so only the
// compiler has to be kept from moving accesses across this point.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exchange point inside a transform, which lives in one wavefront: a compiler-level ordering.
template <typename P>
__device__ __forceinline__ void transform_fence()
{
    wave_lds_fence();
}

// Per-lane constants of the wavefront-local FFT.
template <typename P>
struct WaveFft {
    float2 tw[P::NTW];
    int wbase[P::NWB];
    int rbase, second, rows_in, rows_out;      // second: this lane's first butterfly of the second of two passes
    const float2 *mid;      // rows: this lane's twiddles of the middle pass
    const float2 *twl;      // LDS twiddle table of the passes whose twiddles are there, entry ((set * twiddles(r) + e) * G + lg)

    // `roots`: D float2 of LDS that are free until the caller's next use of them. Short transforms pick their register
    // twiddles out of a table of the D-th roots of unity: computed where they are needed, D = 64 and 128 have 12 and 14
    // inlined sine-cosine codes per lane, fetched and run once by every workgroup. Long ones have few, and run long. Ends
    // with a workgroup barrier.
    static constexpr bool has_roots()
    {
        if constexpr (P::kTwoPass) return false;
        else return P::tw_off(P::NP) > 0 && P::D <= 256;
    }
    static constexpr bool kRoots = has_roots();
    __device__ __forceinline__ void init(int lg, float2 *twl_table, float2 *roots)
    {
        rbase = P::pad(lg);
        twl = twl_table + lg;
        if constexpr (kRoots) {
            for (int i = threadIdx.x; i < P::D; i += blockDim.x) {
                float s, c;
                sincospif(-2.0f * (float)i / (float)P::D, &s, &c);
                roots[i] = twiddle_form(c, s);
            }
        }
        if constexpr (P::kRowed) {
            // the last pass's, then the middle one's: [row][butterfly g][entry], k1 = ROWS g + row (one loop for both: a second
            // inlined sine-cosine is a function call)
            constexpr int LAST = P::tw_lds(P::NP - 1), TW = P::MID / 2, BF = 16 / P::ROWS;
            for (int i = threadIdx.x; i < P::NTWL; i += blockDim.x) {
                const int m = i - LAST, l = i % P::G, ue = i / P::G;
                const bool last = m < 0;
                const int e = last ? ue % 8 : m % TW, k = last ? l + P::G * (ue / 8) : P::ROWS * (m / TW % BF) + m / (TW * BF);
                twl_table[i] = twiddle_entry<16>(e, k, last ? P::D / 16 : 16);
            }
            mid = twl_table + LAST + (lg >> 4) * (TW * BF);
            rows_in = lg * 17;
            rows_out = (lg >> 4) * 17 + (lg & 15);
        } else if constexpr (P::kTwoPass) {
            // [butterfly of a lane][entry][lane]
            constexpr int TW = twiddles(P::G), LANES = P::kButterflyLanes;
            for (int i = threadIdx.x; i < P::NTWL; i += blockDim.x)
                twl_table[i] = twiddle_entry<P::G>(i / LANES % TW, i % LANES + P::G * (i / (LANES * TW)), P::R);
            second = lg % LANES;
            twl = twl_table + second;
        } else {
            fill_table<1>(twl_table);
        }
        __syncthreads();
        if constexpr (P::kRowed) init_pass<P::NP - 1>(lg, roots);        // (where the last pass writes)
        else if constexpr (!P::kTwoPass) init_pass<0>(lg, roots);
        if constexpr (kRoots) __syncthreads();
    }

    // Workgroup-cooperative fill of the LDS twiddle table; the caller synchronises afterwards.
    template <int PI>
    __device__ __forceinline__ void fill_table(float2 *twl_table)
    {
        if constexpr (PI < P::NP) {
            if constexpr (P::tw_in_lds(PI)) {
                constexpr int r = P::radix(PI), Ns = P::Ns(PI), TW = twiddles(r);
                for (int i = threadIdx.x; i < P::tw_lds(PI); i += blockDim.x) {
                    const int l = i % P::G, ue = i / P::G, e = ue % TW, u = ue / TW;
                    twl_table[P::twl_off(PI) + i] = twiddle_entry<r>(e, (l + P::G * u) % Ns, Ns);
                }
            }
            fill_table<PI + 1>(twl_table);
        }
    }

    template <int PI>
    __device__ __forceinline__ void init_pass(int lg, const float2 *roots)
    {
        if constexpr (PI < P::NP) {
            constexpr int r = P::radix(PI), Ns = P::Ns(PI), NB = P::R / r;
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int j = lg + P::G * u;
                const int k = j % Ns;
                wbase[P::wb_off(PI) + u] = P::pad((j - k) * r + k);
            }
            if constexpr (PI > 0 && !P::tw_in_lds(PI)) {
                constexpr int NSETS = P::tw_sets(PI);
#pragma unroll
                for (int u = 0; u < NSETS; ++u) {
                    const int k = (lg + P::G * u) % Ns;
#pragma unroll
                    for (int e = 0; e < twiddles(r); ++e) {
                        float2 &w = tw[P::tw_off(PI) + u * twiddles(r) + e];
                        if constexpr (kRoots) {
                            const int H = e == 0 ? 1 : 2 << ilog2(e), j = e == 0 ? 0 : e - H / 2;
                            w = roots[(k + j * Ns) * (P::D / (2 * H * Ns))];
                        } else {
                            w = twiddle_entry<r>(e, k, Ns);
                        }
                    }
                }
            }
            init_pass<PI + 1>(lg, roots);
        }
    }

    // Forward transform of the slot at `slot` (float2 LDS pointer, padded, natural order in and out).
    __device__ __forceinline__ void run(float2 *slot) const
    {
        float2 v[P::R];
#pragma unroll
        for (int q = 0; q < P::R; ++q) v[q] = slot[rbase + P::roff(q)];
        run_from_registers(slot, v);
    }
    // The same with the input already in registers: v[q] is point lg + G*q of the lane's transform.
    // FEW (where few is set): only the first R / FEW of them are not zero.
    template <bool AHEAD = true, int FEW = 1>
    __device__ __forceinline__ void run_from_registers(float2 *slot, float2 (&v)[P::R], [[maybe_unused]] bool few = false) const
    {
        if constexpr (P::kRowed) run_rows<FEW>(slot, v, few);
        else if constexpr (P::kTwoPass) run_two<AHEAD>(slot, v);
        else run_pass<0, AHEAD, FEW>(slot, v, few);
    }
    // 100, 200 and 500 points. Result t of lane l lies at G t + l in between, which the lanes write next to each other and read G apart: 25 and
    // 5 share no factor with the number of banks, 10 shares two, and the ten lanes of such a transform (200 points) still fall on ten different
    // ones.
    template <bool AHEAD>
    __device__ __forceinline__ void run_two(float2 *slot, float2 (&v)[P::R]) const
    {
        constexpr int G = P::G, NB = P::NB, TW = twiddles(G);
        dft_plain(v);
        transform_fence<P>();                                // every lane has its inputs in registers
#pragma unroll
        for (int t = 0; t < P::R; ++t) slot[rbase + G * t] = v[t];
        transform_fence<P>();
        float2 x[NB][G];
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int t = 0; t < G; ++t) x[u][t] = slot[G * second + G * G * u + t];
        transform_fence<P>();
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            dft<AHEAD>(x[u], [&](int e) { return twl[(u * TW + e) * P::kButterflyLanes]; });
#pragma unroll
            for (int t = 0; t < G; ++t) slot[second + G * u + P::R * t] = x[u][t];
        }
        transform_fence<P>();
    }

    // 512, 1024 and 2048 points as 16 x MID x 16. Point l + G q, l = l0 + 16 l1, is in lane l. The first pass, over q, leaves k1 = 0 .. 15 in
    // a lane's registers; the middle one runs over l1, which is the row of 16 lanes (and, with 2048 points, one of the lane's two
    // halves). Rows meet by v_permlane32_swap and v_permlane16_swap, which exchange halves of two registers: afterwards row r holds, of
    // every row, the k1 that are r modulo ROWS, and the butterflies are a lane's own. That spares one of two exchanges through LDS,
    // whose 16 writes hold a SIMD for 18 cycles each and take 7 of the CU's LDS, for 32 swaps of 8 cycles of a SIMD. (Meeting by
    // swaps of copies, which leave both partners' values in both lanes, took 64 and 100 other instructions and was slower than the
    // exchange.) Sketch kernel, 10000 x 200 points, 1024 buckets, five levels 10.6 -> 10.0 ms, 2000 x 2000, 512, four 7.6 -> 7.2,
    // 50000 x 64, 2048, five 46 -> 45.4: most of what it spares is hidden behind the wait for the increments.
    __device__ __forceinline__ static void meet_rows(float2 (&y)[16])
    {
        if constexpr (P::ROWS == 4) {
#pragma unroll
            for (int a = 0; a < 16; ++a)
                if (!(a & 2)) swap_rows<32>(y[a], y[a | 2]);
        }
#pragma unroll
        for (int a = 0; a < 16; a += 2) swap_rows<16>(y[a], y[a | 1]);
    }
    template <int FEW>
    __device__ __forceinline__ void run_rows(float2 *slot, float2 (&v)[P::R], [[maybe_unused]] bool few) const
    {
        constexpr int NB = P::R / 16, ROWS = P::ROWS, MID = P::MID;
        float2 y[NB][16];
        int in = rows_in, out = rows_out;
        if constexpr (NB > 1) asm volatile("" : "+v"(in), "+v"(out));
#pragma unroll
        for (int u = 0; u < NB; ++u) {
#pragma unroll
            for (int t = 0; t < 16; ++t) y[u][t] = v[u + t * NB];
            if (FEW > 1 && few) dft_plain<FEW>(y[u]);
            else dft_plain(y[u]);
            meet_rows(y[u]);
            if constexpr (NB > 1) __builtin_amdgcn_sched_barrier(0);
        }
        transform_fence<P>();                                // every lane has its inputs in registers
#pragma unroll
        for (int g = 0; g < 16 / ROWS; ++g) {
            float2 x[MID];
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int i = 0; i < ROWS; ++i) x[i + ROWS * u] = y[u][ROWS * g + i];
            dft<true>(x, [&](int e) { return mid[g * (MID / 2) + e]; });
            float2 *dst = slot + out + 17 * ROWS * g;
#pragma unroll
            for (int k2 = 0; k2 < MID; ++k2) dst[17 * 16 * k2] = x[k2];
            if constexpr (NB > 1) __builtin_amdgcn_sched_barrier(0);     // (no twiddles of butterflies to come: registers)
        }
        transform_fence<P>();
#pragma unroll
        for (int u = 0; u < NB; ++u) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int t = bitrev(i, 4);                  // (in the order in which the butterfly can start)
                v[16 * u + t] = slot[in + 17 * P::G * u + t];
            }
        }
        transform_fence<P>();
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            float2 x[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) x[t] = v[16 * u + t];
            constexpr int set = P::tw_sets(P::NP - 1) == 1 ? 0 : 1;
            dft<true>(x, [&](int e) { return twl[P::twl_off(P::NP - 1) + (set * u * 8 + e) * P::G]; });
            float2 *dst = slot + wbase[P::wb_off(P::NP - 1) + u];
#pragma unroll
            for (int t = 0; t < 16; ++t) dst[P::pad(t * (P::D / 16))] = x[t];
            if constexpr (NB > 1) __builtin_amdgcn_sched_barrier(0);
        }
        transform_fence<P>();
    }

    template <int PI, bool AHEAD = true, int FEW = 1>
    __device__ __forceinline__ void run_pass(float2 *slot, float2 (&v)[P::R], [[maybe_unused]] bool few = false) const
    {
        if constexpr (PI < P::NP) {
            constexpr int r = P::radix(PI), Ns = P::Ns(PI), NB = P::R / r;
            transform_fence<P>();                    // every lane has its inputs in registers
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                float2 x[r];
#pragma unroll
                for (int t = 0; t < r; ++t) x[t] = v[u + t * NB];
                if constexpr (PI == 0) {
                    if (FEW > 1 && few) dft_plain<FEW>(x);
                    else dft_plain(x);
                } else {
                    constexpr int TW = twiddles(r), set = P::tw_sets(PI) == 1 ? 0 : 1;    // multiplier of u below
                    dft<AHEAD>(x, [&](int e) {
                        if constexpr (P::tw_in_lds(PI)) return twl[P::twl_off(PI) + (set * u * TW + e) * P::G];
                        else return tw[P::tw_off(PI) + set * u * TW + e];
                    });
                }
                float2 *dst = slot + wbase[P::wb_off(PI) + u];
#pragma unroll
                for (int t = 0; t < r; ++t) dst[P::pad(t * Ns)] = x[t];
            }
            transform_fence<P>();
            if constexpr (PI + 1 < P::NP) {
#pragma unroll
                for (int i = 0; i < P::R; ++i) {
                    const int q = read_order<P::R, P::radix(PI + 1)>(i);
                    v[q] = slot[rbase + P::roff(q)];
                }
                run_pass<PI + 1, AHEAD>(slot, v);
            }
        }
    }
};

// Number of transforms a workgroup has in flight per iteration (= its wavefronts when a transform lives in one
// wavefront). Normally one per level. With 5 or 6 levels that makes workgroups of 5 or 6 wavefronts, and the
// hardware then keeps far fewer of them resident than registers and LDS allow (measured with an empty kernel
// of the same footprint, ~116 registers and 51 KB: 1.7 workgroups = 8.6 wavefronts per CU for 5 wavefronts per
// workgroup, 15.6 wavefronts for 4 or 8 per workgroup: the dispatcher reserves registers for
// ceil(wavefronts / 4) wavefronts on every SIMD). For D = 1024 those level counts therefore run 8 wavefronts
// that take the (pair, level) transforms of the sequence in order, 8 at a time, whatever level they belong to. The
// same helps where one wavefront per level gives a CU too few wavefronts for other reasons: D = 1024 and 1000
// with up to three levels, and D = 2048, whose slots let one workgroup per CU be resident whatever its size.
// (Features, order 1, how much longer a wavefront per level takes, 1500 x 333 and 400 x 100 points: D = 1024 25 and 7 % with 5 levels, 18
// and 4 with 6, with 1 to 3 -2 and 24, -1 and 51, 10 and 20, with 4 -2 and 9, with 7 3 and -9; D = 1000 16 and 9 with 5, 26 and 3 with 6, 3 and
// 16, 28 and 54, 6 and 21 with 1 to 3; D = 500 16 and 4 with 5, 10 and -2 with 6; D = 512 20 and 4 with 5. D = 2048, 600 x 200 points, 0, -4, 18, 6, 16,
// 11 and 5 with 1 to 7. Below 256 points, where a wavefront carries four or more transforms, dealt items lose: D = 200 2.2 to 3.0 times as
// long, D = 256 40 %. Left with a wavefront per level though dealt items are ahead at places: D = 512 with 6 levels, 9 and -1, and
// D = 500 with 3, 4 and 23, 3000 x 60 -3.)
__host__ __device__ constexpr int transforms_in_flight(int M, int LOG2D) {
    return ((LOG2D == 10 || LOG2D == 1000) && (M <= 3 || M == 5 || M == 6)) || (LOG2D == 2048 && M <= 7) ||
                   (LOG2D == 500 && (M == 5 || M == 6)) || (LOG2D == 9 && M == 5)
               ? 8 : M;
}

// The kernel for whole sequences of orders 2 and 3 carries values from pair to pair, dealt items one set for every pair of a wavefront: with 500
// and 512 points (two pairs) that costs it 15 to 46 spills, a wavefront per level 0 to 13. (Features, dealt and per level, us, 1500 x 333 and
// 400 x 100 points, 7 channels, order 2: 500 points, five levels, 250 frequencies 3613 and 3358, 318 and 256, six 4400 and 3657, 405 and
// 293; 512, five, 256 2670 and 2628, 249 and 217; order 3 4035 and 3366, 361 and 256, 5025 and 4116, 472 and 331, 3381 and 2668, 319 and
// 223. With one pair, 1000 and 1024 points, dealt items stay ahead: 1024, five levels, order 2 4543 and 5467, 437 and 442, order 3 5331 and
// 5505, 501 and 449.)
__host__ __device__ constexpr int whole_transforms_in_flight(int M, int LOG2D, int order)
{
    return order > 1 && (LOG2D == 500 || LOG2D == 9) ? M : transforms_in_flight(M, LOG2D);
}

typedef const __attribute__((address_space(1))) uint32_t *GlobalWords;   // table words, known to be in global memory

// LDS of a workgroup with NTR transforms in flight: their slots and the twiddle table of the plan.
__host__ __device__ constexpr size_t tuned_lds_bytes(int NTR, int FPW, int PD, int NTWL, int F)
{
    return sizeof(float2) * ((size_t)NTR * FPW * slot_stride(PD, 2 * F) + NTWL);
}
// ... and with slots that hold whole direct loads, and a twiddle for every input but the first of a butterfly
// (kBoundTwiddles): what decides at which transform length a shape runs (as it did when slots and tables were that large,
// so that routes and workspace sizes stay what they were).
__host__ __device__ constexpr size_t tuned_lds_bound(int NTR, int FPW, int PD, int NTWL, int F)
{
    return tuned_lds_bytes(NTR, FPW, PD, NTWL, staged(2 * F) / 2);
}

template <int LL>
struct LevelTag {
    static constexpr int value = LL;
};
// Calls f(LevelTag<l>) for a wavefront-uniform runtime level l in [0, M).
template <int M, int LL = 0, typename Fn>
__device__ __forceinline__ void with_level(int l, Fn &&f)
{
    if constexpr (LL + 1 < M) {
        if (l == LL) f(LevelTag<LL>{});
        else with_level<M, LL + 1>(l, f);
    } else {
        f(LevelTag<LL>{});
    }
}

// What level l of one pair hands to level l+1 of the same pair in the recurrence: the values of A_l before
// each of the two steps (p), with order >= 2 also those of A_{l-1} (q) and the transforms of level l (cp),
// with order 3 also those of A_{l-2} (r) and the transforms of level l-1 (cpp).
template <int ORDER>
struct LevelCarry {
    float2 p0, p1;
    float2 q0, q1, c0p, c1p;        // used with order >= 2
    float2 r0, r1, c0pp, c1pp;      // used with order 3
    __device__ __forceinline__ void reset()
    {
        p0 = p1 = make_float2(1.f, 0.f);
        q0 = q1 = c0p = c1p = r0 = r1 = c0pp = c1pp = make_float2(0.f, 0.f);
    }
};

// Items J = 0..NTR-1 of an iteration whose first item has level L0: calls f(LevelTag<level of item J>, LevelTag<J>,
// number of pair groups item J lies behind item 0).
template <int L0, int M, int NTR, int J = 0, typename Fn>
__device__ __forceinline__ void item_loop(Fn &&f)
{
    if constexpr (J < NTR) {
        f(LevelTag<(L0 + J) % M>{}, LevelTag<J>{}, (L0 + J) / M);
        item_loop<L0, M, NTR, J + 1>(f);
    }
}

// Calls f(LevelTag<0>), ..., f(LevelTag<M-1>).
template <int M, int LL = 0, typename Fn>
__device__ __forceinline__ void level_loop(Fn &&f)
{
    if constexpr (LL < M) {
        f(LevelTag<LL>{});
        level_loop<M, LL + 1>(f);
    }
}

// One level of one pair of time steps at one bin (Sec. 3.5 eq. (ts_rec)): z and zc are the transform of the
// level's slot at the bin and at its mirror image; separates the two real transforms and advances the bin's
// accumulator a = A_LL by both steps, c carrying what level LL - 1 of the same pair left. PK: the thread may be
// the packed one (pk), whose float2 hold bins 0 and D/2 and whose z, zc are Z[0], Z[D/2]. ADDS: level 0, whose A_0 is 1, takes two
// additions instead of four multiply-adds with one and zero (the kernel of whole sequences is no faster for it: 10000 x 200 points,
// D = 1024, five levels 10.58 and 10.85 ms).
// second_step: whether the second step exists, or all bits set if it does and none if not, in a vector register.
__device__ __forceinline__ float2 if_step(bool exists, float2 C) { return exists ? C : make_float2(0.f, 0.f); }
__device__ __forceinline__ float2 if_step(uint32_t exists, float2 C)
{
    return make_float2(__uint_as_float(__float_as_uint(C.x) & exists), __uint_as_float(__float_as_uint(C.y) & exists));
}
template <int ORDER, int LL, bool PK, bool ADDS = false, typename Packed, typename Second>
__device__ __forceinline__ void level_step(float2 z, float2 zc, Packed pk, Second second_step, float2 &a, LevelCarry<ORDER> &c)
{
    auto mul = [&](float2 x, float2 y) { return PK ? cmulf_pk(x, y, pk) : cmulf(x, y); };
    auto fma = [&](float2 x, float2 y, float2 w) { return PK ? cfmaf_pk(x, y, w, pk) : cfmaf(x, y, w); };
    if constexpr (LL == 0) {
        c.reset();
        if constexpr (PK) {                                             // A_0 = 1 in both bins of the packed thread
            if constexpr (!std::is_same_v<Packed, bool>) c.p0.y = c.p1.y = choose(pk, 1.f, 0.f);
            else if (pk) c.p0.y = c.p1.y = 1.f;
        }
    }
    // separation of the two real transforms; for the packed thread C = (2 Re z, 2 Re zc), (2 Im z, 2 Im zc):
    // the values the general formulas give at f = 0 and f = D/2
    float2 C0 = make_float2(z.x + zc.x, z.y - zc.y);
    // a second step that does not exist (odd number of increments) must contribute
    // exactly nothing; the separation alone would leave rounding noise of the first
    float2 C1 = make_float2(z.y + zc.y, zc.x - z.x);
    if constexpr (PK && !std::is_same_v<Packed, bool>) {
        C0 = make_float2(choose(pk, z.x + z.x, C0.x), choose(pk, zc.x + zc.x, C0.y));
        C1 = make_float2(choose(pk, z.y + z.y, C1.x), choose(pk, zc.y + zc.y, C1.y));
    } else if constexpr (PK) {
        if (pk) {
            C0 = make_float2(z.x + z.x, zc.x + zc.x);
            C1 = make_float2(z.y + z.y, zc.y + zc.y);
        }
    }
    C1 = if_step(second_step, C1);
    const float2 a_old = a;
    float2 a_mid = ADDS && LL == 0 ? make_float2(a_old.x + C0.x, a_old.y + C0.y) : fma(c.p0, C0, a_old);
    // order >= 2 (a time step may be used up to `order` times in a row, q equal indices weighted
    // 1/q!): also the values of levels l-2 (and l-3) before each step and the transforms of
    // levels l-1 (and l-2) at both steps
    float2 h0 = make_float2(0.f, 0.f), h1 = h0;
    if constexpr (ORDER >= 2 && LL > 0) {
        h0 = mul(c.c0p, C0);
        a_mid = fma(make_float2(0.5f * c.q0.x, 0.5f * c.q0.y), h0, a_mid);
    }
    if constexpr (ORDER >= 3 && LL > 1) {
        const float2 g = mul(c.c0pp, h0);
        a_mid = fma(make_float2(c.r0.x * (1.0f / 6.0f), c.r0.y * (1.0f / 6.0f)), g, a_mid);
    }
    float2 a_new = ADDS && LL == 0 ? make_float2(a_mid.x + C1.x, a_mid.y + C1.y) : fma(c.p1, C1, a_mid);
    if constexpr (ORDER >= 2 && LL > 0) {
        h1 = mul(c.c1p, C1);
        a_new = fma(make_float2(0.5f * c.q1.x, 0.5f * c.q1.y), h1, a_new);
    }
    if constexpr (ORDER >= 3 && LL > 1) {
        const float2 g = mul(c.c1pp, h1);
        a_new = fma(make_float2(c.r1.x * (1.0f / 6.0f), c.r1.y * (1.0f / 6.0f)), g, a_new);
    }
    if constexpr (ORDER >= 3) {
        c.r0 = c.q0;
        c.r1 = c.q1;
        c.c0pp = c.c0p;
        c.c1pp = c.c1p;
    }
    if constexpr (ORDER >= 2) {
        c.q0 = c.p0;
        c.q1 = c.p1;
        c.c0p = C0;
        c.c1p = C1;
    }
    a = a_new;
    c.p0 = a_old;
    c.p1 = a_mid;
}

// Wavefronts per SIMD the register budget of the kernel is set for: the plan's, except that workgroups of 5 or 6
// wavefronts with 6 to 12 transforms per wavefront (D = 100, 128, 200) get 96 registers: their workgroups then
// find room on a CU more often (see transforms_in_flight; measured +8-15 %). Not the kernel for sequences cut in time,
// where they cost it 13 to 78 spills (features of 100 x 1000 points, 50 frequencies, 96 against 128 registers: D = 100 138
// and 128 us with five levels, 190 and 147 with six, D = 200 182 and 173, 241 and 200, D = 128 159 and 118, 231 and 152).
//
// The kernel for sequences cut in time (JOINT) holds M(M+1)/2 accumulators per bin instead of M. Four wavefronts per
// SIMD (128 registers) cost it a few dozen spills of accumulators, which are touched once per iteration; from
// kJointRegs registers of accumulators on, or with values carried from iteration to iteration, it gets the budget of two.
constexpr int kJointRegs = 44;
// Whether one thread carries both real bins (0 and D/2) where that saves a bin per thread. Not in the kernel for sequences
// cut in time with transforms of a whole wavefront: the second copy of phase 3 that the packed thread needs pushes its
// accumulators into spills (D = 1024, four levels, order 2: 101 spills packed, none unpacked and twice as fast; eight levels 1.4
// times; D = 2048, four levels, order 2, 1.7 times; shorter transforms lose up to a tenth unpacked).
constexpr bool packs(bool JOINT, bool stream, int FPW) { return !JOINT || stream || FPW > 1; }
constexpr int accumulators(int M, bool JOINT) { return JOINT ? M * (M + 1) / 2 : M; }
template <int LOG2D, int M, int NTR, bool JOINT>
constexpr int kernel_min_waves()
{
    using P = Plan<LOG2D>;
    constexpr int BPT = (P::D / 2 + !packs(JOINT, NTR != M, P::FPW) + 64 * NTR - 1) / (64 * NTR);
    if (JOINT && (P::kMinWaves <= 2 || NTR != M || 2 * BPT * accumulators(M, JOINT) > kJointRegs)) return 2;
    return P::FPW > 4 && P::FPW < 16 && (M == 5 || M == 6) && !JOINT ? 5 : P::kMinWaves;
}
// Workgroups of the JOINT kernel that a CU holds: one where eight wavefronts, or five and more of the budget of two
// wavefronts per SIMD, make up the workgroup; two otherwise (by LDS).
constexpr int joint_workgroups_per_cu(int M, int D)
{
    const bool dealt = D == 1000 || D == 1024 || D == 500 || D == 512;
    return D == 2048 || M >= 7 || (dealt && M >= 5) || ((D == 1000 || D == 1024) && M <= 3) ? 1 : 2;
}
// JOINT: transforms in flight as above where the values carried from one iteration to the next (one set per first
// position, larger for higher orders) fit the registers.
constexpr int joint_transforms_in_flight(int M, int LOG2D, int order)
{
    return (order == 1 && (LOG2D != 2048 || M <= 4)) || M <= 2 ? transforms_in_flight(M, LOG2D) : M;
}
// Whether the accumulators of the JOINT kernel fit its registers. Where they do not (D = 2048 with seven and eight levels,
// 200 to 400 spills) it takes 3 to 5 times as long per step as the kernel for whole sequences, and splitting those gains
// nothing: 120 sequences of 100 points in two pieces were 0.6 and 0.5 times as fast as whole, 60 in four 0.95 and 0.8, nine of
// 401 points in 25 (eight levels, order 2) 0.92.
constexpr bool joint_fits(int M, int D, int LOG2D, int order)
{
    const int ntr = joint_transforms_in_flight(M, LOG2D, order), bpt = (D / 2 + 64 * ntr) / (64 * ntr);
    return 2 * bpt * accumulators(M, true) < 160;
}

// Short transforms: a wavefront carries FPW = 4 .. 16 pairs of steps per iteration, while their D/2 + 1 bins occupy
// a fraction of the workgroup's threads, which would take the pairs one after the other (D = 100, five levels: 51 of 320
// threads, 12 pairs). The kernel for sequences cut in time therefore cuts its piece once more, into as many groups as
// bins fit the threads: FPW / groups transforms of an iteration belong to each, and each has its own threads and
// accumulators in phase 3. The groups are joined in LDS at the end (which has to hold all but the first's).
constexpr int joint_groups(int M, int D, int FPW, int PD)
{
    const int NB = D / 2 + 1, Q = M * (M + 1) / 2;
    for (int g = FPW; g > 1; --g)
        if (FPW % g == 0 && g * NB <= 64 * M && (g - 1) * Q * NB <= M * FPW * slot_stride(PD, 2)) return g;
    return 1;
}
// ... and from three groups on that is also the faster way for a whole sequence, for all that it advances
// M(M+1)/2 accumulators instead of M (sketch kernel, one wavefront after the other against grouped, 3000 sequences of 200
// points: D = 64, 32 frequencies, 218 -> 149 us with three levels, 597 -> 388 with six; D = 100, 50 frequencies, 382 -> 352
// with four, 768 -> 639 with six; D = 128, 64 frequencies, 731 -> 551 with five, 942 -> 677 with six). From seven levels on
// these accumulators let a CU hold one workgroup where it would hold two of the others; where the slots let it hold only
// one of those too, or with eight groups, it still gains (eight levels: D = 64, 32 frequencies, 609 -> 612; 64 buckets in
// 128 points, 96 frequencies, 1557 -> 1358; but D = 100, 50 frequencies, 843 -> 1002, D = 128, 64, 751 -> 1048).
enum class Grouped { kNever, kOneWorkgroup, kAlways };
constexpr Grouped grouped(int M, int D, int FPW, int PD)
{
    if (D > 128 || joint_groups(M, D, FPW, PD) < 3) return Grouped::kNever;
    return M <= 6 || joint_groups(M, D, FPW, PD) >= 8 ? Grouped::kAlways : Grouped::kOneWorkgroup;
}

// Index of the accumulator of tensor positions a+1 .. l+1 (0-based a <= l) among those of a bin; a = 0 first.
__host__ __device__ constexpr int acc_index(int M, int a, int l) { return a * M - a * (a - 1) / 2 + l - a; }

// Sequences of their own lengths: workgroups start in the order of their numbers, and a long sequence that starts late keeps
// its CU busy while the others are done. So they take the sequences by length, the longest first, in 64 classes (in any order
// within a class, the same for all workgroups). Every workgroup finds the sequence whose turn it is by itself, so that no
// memory has to hold an order: the classes of all sequences are read into registers, the class whose turn it is is found by halving.
// Lengths between half and whole, in order of numbers and of lengths, sketch kernel: 1501 x 333 points, 500 buckets, four levels, order 2
// 1286 and 1018 us, 1000 x 200, 1024 buckets, five levels 934 and 789; lengths from 1 on 992 and 702, 806 and 544. More sequences than fit
// the registers are left in their order: with many rounds of workgroups there is little to gain (10000 x 200, 500 buckets, sorted
// before the call 4007 -> 3880). The kernel whose wavefronts work by themselves is short and keeps its order (1000 x 100, 256 buckets 168
// and 180, 4000 x 40, 100 buckets 166 and 187, 300 x 500 128 and 122).
constexpr int kTurnRows = 32, kLengthClasses = 64;           // sequences of a lane; classes
// (From 2048 points on it is not compiled, though it would pay there, 600 x 300 points, four levels, lengths from half 1467 -> 1300 us: these
// kernels take the longest to compile.)
template <int M, int D> constexpr bool kTurns = M > 1 && D < 2048;
constexpr int64_t kTurnWork = 65536;
// Where that pays, in a kernel of its own (for batches whose sequences have one length the search would only cost registers: 600 x 200
// points, 512 buckets, five levels 430 and 441 us): more whole sequences than CUs, and enough work on each for the few microseconds of the
// search, counted in points of its transforms times the workgroups on its CU, of which `held` fit, and against the number of
// sequences that it goes through. (Sketch kernels and projection, lengths
// from half, from one and all the same, us in order of numbers and of length: 600 x 50 points, 512 buckets, five levels 105 and 96, 87 and 75,
// 121 and 123; 1500 x 50, 1000, three 267 and 246, 219 and 186, 303 and 310; 600 x 300, 1024, five 824 and 760, 608 and 489, 950 and
// 955; below the lines 320 x 10, 1024, three 29.4 and 32.4 with lengths from half, 2707 x 11, 1024, six 168 and 191, 2663 x 34, 1024, two, order
// 2 169 and 187; sequences in pieces 61 x 1134, 512, four, order 2 189 and 221, 45 x 572, 512, five 170 and 180. Of 681 drawn shapes of more
// sequences than CUs, lengths from half, 485 lie above: 0.946 of the time on average, 8 slower by more than 3 %; the others took
// 1.003. Sequences in pieces: 563 shapes, 26 slower by more than 3 %, 6 faster.)
inline bool turns_pay(int M, int D, int waves, int64_t held, int64_t sequences, int64_t pieces, int64_t pairs, int64_t L)
{
    constexpr int64_t kCUs = 256, kWorkPerSequence = 24;
    const int64_t at_once = sequences < held * kCUs ? sequences : held * kCUs;
    const double work = (double)(M * pairs * D);
    return pieces == 1 && sequences > kCUs && work * (double)at_once >= (double)(kTurnWork * kCUs) && work >= (double)(kWorkPerSequence * sequences) &&
           sequences <= 64 * kTurnRows * waves && L <= 0x7fffffffLL;
}
template <int WAVES>
__device__ __forceinline__ int sequence_in_turn(const int64_t *__restrict__ lengths, int64_t L, int count, int turn, int *scratch /* [3 * WAVES + 1] */)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int *found = scratch + 3 * WAVES;
    if (tid == 0) *found = turn;
    const float classes_per_point = (float)kLengthClasses / (float)L;
    int cls[kTurnRows];
    // rows that there are, in groups of four
    auto each_row = [&](auto body) {
#pragma unroll
        for (int g = 0; g < kTurnRows; g += 4) {
            if (64 * WAVES * g >= count) break;
#pragma unroll
            for (int r = g; r < g + 4; ++r) body(r);
        }
    };
    each_row([&](int r) {
        const int i = 64 * (r * WAVES + wave) + lane;
        const int64_t given = lengths[i < count ? i : 0], points = given < 1 ? 1 : (given > L ? L : given);
        const int c = (int)((float)(int)(L - points) * classes_per_point);
        cls[r] = i < count ? (c < kLengthClasses ? c : kLengthClasses - 1) : kLengthClasses;
    });
    // all in one class: in order of their numbers, which this finds at half the cost
    {
        const int64_t given = lengths[0], points = given < 1 ? 1 : (given > L ? L : given);
        const int c = (int)((float)(int)(L - points) * classes_per_point), one = c < kLengthClasses ? c : kLengthClasses - 1;
        int others = 0;
        each_row([&](int r) { others |= cls[r] != one && cls[r] != kLengthClasses ? 1 : 0; });
        const int any = __ballot(others) != 0 ? 1 : 0;
        if (lane == 0) scratch[2 * WAVES + wave] = any;
        __syncthreads();
        int sum = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum += scratch[2 * WAVES + w];
        if (sum == 0) {
            __syncthreads();
            return turn;
        }
    }
    int mine = 0, left = turn, buffer = 0;                   // class whose turn it is, sequences of it that come first
#pragma unroll 1
    for (int bit = kLengthClasses / 2; bit > 0; bit >>= 1) {
        int here = 0, before = 0;
        each_row([&](int r) { here += __popcll(__ballot(cls[r] < mine + bit)); });
        if (lane == 0) scratch[buffer + wave] = here;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) before += scratch[buffer + w];
        buffer = WAVES - buffer;
        if (before <= turn) {
            mine += bit;
            left = turn - before;
        }
    }
    int here = 0;
    each_row([&](int r) { here += __popcll(__ballot(cls[r] == mine)); });
    if (lane == 0) scratch[2 * WAVES + wave] = here;
    __syncthreads();
    for (int w = 0; w < wave; ++w) left -= scratch[2 * WAVES + w];
    if (left >= 0 && left < here)
        each_row([&](int r) {
            const uint64_t hits = __ballot(cls[r] == mine);
            const int first = __builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0));
            if (cls[r] == mine && first == left) *found = 64 * (r * WAVES + wave) + lane;
            left -= __popcll(hits);
        });
    __syncthreads();
    const int n = __builtin_amdgcn_readfirstlane(*found);
    __syncthreads();
    return n;
}

// JOINT: the workgroup owns one piece of a sequence cut in time (TimeCut::mode 1) and runs the recurrence for
// every first tensor position at once: per bin A^{(a..l)} += A^{(a..l-1)}(before the step) C_l for all a <= l. The
// transforms, which are most of the work, are thus done once per step and level however many first positions
// need them (one launch per first position did (M+1)/2 times as many: 10 x 1e5 steps, D = 100, five levels 2.68 ms, with
// groups 1.00). In mode 2 the same kernel joins a sequence's pieces and runs the final
// transforms.
template <int LOG2D, int M, int ORDER, int NTR, bool JOINT, bool BY_LENGTH>
__global__ __launch_bounds__(64 * NTR)
    __attribute__((amdgpu_waves_per_eu(kernel_min_waves<LOG2D, M, NTR, JOINT>(),
                                       kernel_min_waves<LOG2D, M, NTR, JOINT>() > 4 ? 8 : 4))) void sketch_fft_scan_kernel(
    const float *__restrict__ dphi, const uint32_t *__restrict__ table, int64_t L,
    const int64_t *__restrict__ lengths, int F, int Dout, float *__restrict__ out, int64_t ld_out, TimeCut cut)
{
    using P = KernelPlan<LOG2D, M, ORDER, JOINT>;
    // kStream: the workgroup's NTR transforms of an iteration are the next NTR (pair group, level) items of the
    // sequence in that order, so a wavefront changes level from iteration to iteration and an iteration
    // may end in the middle of a pair; otherwise transform w of the workgroup is always level w.
    constexpr bool kStream = NTR != M;
    static_assert(!kStream || NTR > M, "streaming needs a slot per level");
    // Bins of phase 3: f = 0 .. D/2, thread t owning f = t, t + NT, ... The transforms of real sequences are real
    // at f = 0 and f = D/2. Where that saves a bin per thread (NT divides D/2), thread 0 carries both in one
    // float2 (bin 0 in .x, bin D/2 in .y; kPack, see packs) and the bins are f = 0 .. D/2 - 1.
    constexpr int D = P::D, NT = 64 * NTR;
    constexpr bool kPack = (D / 2) % NT == 0 && packs(JOINT, NTR != M, P::FPW);
    constexpr int NB = kPack ? D / 2 : D / 2 + 1, BPT = (NB + NT - 1) / NT;
    constexpr int GR = JOINT && !kStream ? joint_groups(M, D, P::FPW, P::PD) : 1, SPG = P::FPW / GR;   // groups; transforms of each
    static_assert(GR == 1 || (BPT == 1 && !kPack), "a thread of a group owns one bin");
    // Phase 3 is compiled separately for iterations in which every item exists and has both time steps (no
    // per-item conditions and selects) when a wavefront has at most two transforms per iteration; with more the
    // extra copy costs registers.
    constexpr bool kSplitFull = P::FPW <= 2 && !JOINT;
    constexpr int kAcc = accumulators(M, JOINT), kStarts = JOINT ? M : 1;
    extern __shared__ float2 lds[];                    // [NTR][FPW][PS] slots, then the twiddle table
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wv = wave;                                     // transform of the workgroup
    // lanes beyond the G * FPW that the wavefront's transforms occupy (lengths that are no power of two) repeat the
    // work of the first ones: same addresses, same values
    constexpr int kLanesUsed = P::G * P::FPW;
    const int lane_t = kLanesUsed < 64 && lane >= kLanesUsed ? lane - kLanesUsed : lane;
    const int slot_id = lane_t / P::G;
    const int lg = lane_t % P::G;                            // lane within the transform
    const int twoF = 2 * F;
    const int ZS = zero_slot(P::PD, twoF), PS = slot_stride(P::PD, twoF);
    float2 *twl_table = lds + (size_t)NTR * P::FPW * PS;        // behind the slots
    float2 *wave_lds = lds + (size_t)wv * P::FPW * PS;
    float2 *my_slot = wave_lds + slot_id * PS;
    char *my_slot_bytes = reinterpret_cast<char *>(my_slot);
    // the workgroup's row of out, its sequence and its piece of that sequence (one piece: the whole sequence)
    int64_t row_id = blockIdx.x;
    if constexpr (BY_LENGTH) {
        const unsigned pieces = (unsigned)cut.pieces, turn = blockIdx.x / pieces;
        row_id = (unsigned)sequence_in_turn<NTR>(lengths, L, (int)(gridDim.x / pieces), (int)turn, reinterpret_cast<int *>(lds)) * pieces + (blockIdx.x - turn * pieces);
    }
    const int64_t n = JOINT ? (unsigned)row_id / (unsigned)cut.pieces : row_id, piece = row_id - n * cut.pieces;
    // this sequence's own number of points (variable-length batch: X is padded to L points, the steps beyond a
    // sequence's length do not exist); out-of-range entries are clamped, they are never used as addresses
    const int64_t Ln = lengths ? (lengths[n] < 1 ? 1 : (lengths[n] > L ? L : lengths[n])) : L;
    // the piece's own steps: 2 * cut.pairs of them from its first one on, fewer (or none) at the sequence's end
    const int64_t steps_left = JOINT ? Ln - 1 - 2 * piece * cut.pairs : 0;
    const int64_t T_all = !JOINT ? Ln - 1
                          : cut.mode == 2 || steps_left < 0 ? 0 : (steps_left < 2 * cut.pairs ? steps_left : 2 * cut.pairs);
    // One level: its block is the sum over time of the sketches, which is the sketch of the sum of the increments. They
    // are added up as they are read, and one iteration follows, on the sum as its only step.
    constexpr bool kSumFirst = M == 1;
    const int64_t T = kSumFirst && T_all > 1 ? 1 : T_all;
    const int64_t all_pairs = (T + 1) / 2;
    // pairs of a group (of the first ones; the last may have fewer or none): what the iterations run over
    const int64_t pairs = GR > 1 ? (all_pairs + GR - 1) / GR : all_pairs;
    int last_grp = 0;                                        // the group that holds the last pair
#pragma unroll
    for (int g = 1; g < GR; ++g) last_grp += all_pairs > g * pairs;
    const int64_t last_in_grp = all_pairs - 1 - last_grp * pairs;
    // this thread's group in phase 3, its bin (f = tid + NT * b where there is one group) and its group's steps
    const int grp = GR > 1 ? tid / NB : 0, bin = GR > 1 ? tid - grp * NB : tid;
    const int64_t T_left = GR > 1 ? T - 2 * grp * pairs : T;
    const int64_t T_grp = GR > 1 ? (grp >= GR || T_left < 0 ? 0 : (T_left < 2 * pairs ? T_left : 2 * pairs)) : T;
    // pair p of level l: 2F float2 at seq + l * 2 * twoF + p * pf (pair layout of the producing kernel, Lp / 2
    // pair slots per sequence with Lp = L rounded up to even)
    const int64_t pf = (int64_t)M * 2 * twoF;
    const float *seq = dphi + (n * ((L + 1) / 2) + (JOINT ? piece * cut.pairs : 0)) * pf;
    const TableLayout tl = table_layout(D, P::GF, twoF);
    const int nload = twoF / 128, last_load = twoF % 128;    // direct loads per pair, 128 coordinates each, and the rest
    // one level per wavefront for good: its increments, table and number of fold rounds
    const float *seq_fixed = seq + (int64_t)wv * 2 * twoF;
    const uint32_t *tab_fixed = table + (int64_t)wv * tl.words;
    const int NG_fixed = kStream ? 0 : (int)tab_fixed[0];
    const int rows_fixed = kStream ? 0 : (int)tab_fixed[1];

    WaveFft<P> fft;
    fft.init(lg, twl_table, lds);
    if (lg == 0) my_slot[ZS] = make_float2(0.f, 0.f);
    __syncthreads();

    float2 A[BPT][kAcc];
#pragma unroll
    for (int b = 0; b < BPT; ++b)
#pragma unroll
        for (int l = 0; l < kAcc; ++l) A[b][l] = make_float2(0.f, 0.f);
    // accumulators of a piece outside the kernel: kAcc times bins 0 .. D/2. Without a buffer of their own they take
    // the place of the piece's increments (which the host has checked to be large enough, and which this workgroup
    // alone reads: what other workgroups' direct loads pick up beyond their last coordinate is never used).
    float2 *spectra_row = JOINT ? (cut.spectra ? cut.spectra : reinterpret_cast<float2 *>(const_cast<float *>(dphi))) +
                                      n * cut.seq_stride + piece * cut.piece_stride
                                : nullptr;
    if constexpr (JOINT) {
        if (cut.mode == 2) {                                 // join the pieces of the sequence, left to right
            for (int b = 0; b < BPT; ++b) {
                const int f = tid + NT * b;
                if (f >= NB) continue;
                const bool pk = kPack && f == 0;
                float2 J[M], B[kAcc], next[kAcc];            // the next piece's numbers are in flight while one is folded in
#pragma unroll
                for (int l = 0; l < M; ++l) {
                    J[l] = spectra_row[l * (D / 2 + 1) + f];
                    if (pk) J[l].y = spectra_row[l * (D / 2 + 1) + D / 2].x;
                }
                auto fetch = [&](int s) {
                    const float2 *sp = spectra_row + s * cut.piece_stride + f;
#pragma unroll
                    for (int q = 0; q < kAcc; ++q) {
                        next[q] = sp[q * (D / 2 + 1)];
                        if (pk) next[q].y = sp[q * (D / 2 + 1) + D / 2].x;
                    }
                };
                if (cut.join > 1) fetch(1);
                for (int s = 1; s < cut.join; ++s) {
#pragma unroll
                    for (int q = 0; q < kAcc; ++q) B[q] = next[q];
                    if (s + 1 < cut.join) fetch(s + 1);
#pragma unroll
                    for (int l = M - 1; l >= 0; --l) {       // descending: the lower levels are still the old ones
                        float2 acc = make_float2(J[l].x + B[acc_index(M, 0, l)].x, J[l].y + B[acc_index(M, 0, l)].y);
#pragma unroll
                        for (int j = 1; j <= l; ++j) acc = cfmaf_pk(J[j - 1], B[acc_index(M, j, l)], acc, pk);
                        J[l] = acc;
                    }
                }
#pragma unroll
                for (int bb = 0; bb < BPT; ++bb)             // (no run-time index into the register array)
                    if (bb == b) {
#pragma unroll
                        for (int l = 0; l < M; ++l) A[bb][l] = J[l];
                    }
            }
        }
    }

    // Staging: pair pair0 + s of level lvl goes to slot s of the wavefront, 128 coordinates (1 KB) per
    // instruction, lane i supplying coordinates 2i and 2i+1. Pairs beyond the last one (final group only) are redirected
    // to the last pair and ignored later.
    auto stage_direct = [&](int lvl, int64_t pair0) {
#pragma unroll
        for (int s = 0; s < P::FPW; ++s) {
            int64_t p = GR > 1 ? (s / SPG) * pairs + pair0 + s % SPG : pair0 + s;
            if (p >= all_pairs) p = all_pairs - 1;
            const float *src = (kStream ? seq + (int64_t)lvl * 2 * twoF : seq_fixed) + p * pf + 4 * lane;
            float2 *dst = wave_lds + s * PS;
            for (int j = 0; j < nload; ++j)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + 256 * j),
                                                 (__attribute__((address_space(3))) void *)(dst + 128 * j), 16, 0, 0);
            if (2 * lane < last_load)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + 256 * nload),
                                                 (__attribute__((address_space(3))) void *)(dst + 128 * nload), 16, 0, 0);
        }
    };

    // Early staging: when the transforms of one iteration fit a thread's registers (ZREGS float2), phase 3 first
    // copies them out of LDS, the slots are released by the second barrier at once, and the next iteration's
    // direct loads are issued before the recurrence arithmetic, which then runs under their latency.
    // (Measured: 3-4 % on D = 1024 and 2048 with five levels; with 32 float2 -- D = 512, four levels -- it no
    // longer pays, and loading the next iteration's table words early as well costs more registers than it hides.) JOINT:
    // where they fit beside its accumulators.
    constexpr int ZREGS = P::FPW * BPT * NTR * 2;
    constexpr bool kEarly = GR == 1 && ZREGS <= (P::kMinWaves <= 2 ? 64 : 24)    // (a plan with twice the registers per wavefront affords more)
                            && (!JOINT || 2 * (ZREGS + BPT * kAcc) <= 200);
    uint32_t gw[P::R], fw[kFoldInRegs];
    // Fewer buckets than points (the linear route takes M D - M + 1 points at least): groups of G buckets, R of D points, that are not
    // all empty. Where they are half or a quarter of all at most (as many as the linear route's with M levels can be), the reads of the others
    // and the stages of the first pass that would only copy are left out. Features of 1000 x 151 points, projection included, us: 300 buckets in
    // 1024 points, three levels, 190 frequencies 503 -> 490, 150 in 512, four 538 -> 499, 150 in 1024, five 667 -> 632; as many buckets as
    // points 829 and 829, 1366 and 1363.
    // Sequences cut in time, 512 points with four to six levels, 2048 with five and six and with four in order 2: without it, whose branch costs
    // kernels that spill up to another 18 registers (with and without, us, 200 frequencies: 512 points, 100 x 200 points, five levels, order 2 183 and
    // 155, 101 buckets 177 and 169, six 219 and 202, order 3 310 and 281, 85 buckets 277 and 263; 600 frequencies: 2048 points, 60 x 200, five, order 1
    // 351 and 294, 400 buckets 401 and 364, six 405 and 320, 300 buckets 463 and 402, four, order 2 253 and 229, 320 buckets 208 and 212. But 512
    // points, three levels, 160 buckets 69.8 and 72.6, eight, 63 204 and 214; 2048 points, three, 600 buckets 151 and 155, four, order 1 206 and 205,
    // 320 buckets 285 and 312, order 3 263 and 257, 320 buckets 304 and 316, seven, 280 979 and 1038, eight, 240 1103 and 1157.)
    constexpr bool kSpills = JOINT && ((LOG2D == 9 && M >= 4 && M <= 6) || (LOG2D == 2048 && (M == 5 || M == 6 || (M == 4 && ORDER == 2))));
    constexpr bool kRows = P::kRowed || exchanges(LOG2D, M, ORDER, JOINT);       // 512 to 2048 points
    constexpr int kFew = !kRows || M < 2 || kSpills ? 1 : M < 4 ? 2 : 4;
    const int groups = (Dout + P::G - 1) / P::G;
    const bool few = kFew > 1 && groups <= P::R / kFew;

    // The item of this wavefront: level and first pair of its transform in the current iteration (a transform
    // carries FPW consecutive pairs of one level, a pair group). Streaming: the items of the sequence are counted
    // (group, level) with the level running fastest, and this wavefront has number iteration * NTR + wv.
    int lvl = kStream ? wv % M : wv;
    int64_t pair0 = kStream ? (wv / M) * P::FPW : 0;
    auto advance = [&](int &l, int64_t &p0) {                // the same wavefront's item one iteration later
        if constexpr (kStream) {
            l += NTR % M;
            p0 += (NTR / M) * P::FPW;
            if (l >= M) {
                l -= M;
                p0 += P::FPW;
            }
        } else {
            p0 += SPG;
        }
    };
    // first item of the iteration (the one of wavefront 0; streaming only)
    int lvl_first = 0;
    int64_t pair0_first = 0;
    LevelCarry<ORDER> carry[kStream ? P::FPW : 1][kStream ? BPT : 1][kStarts];

    if constexpr (kSumFirst) {
        // a thread adds up two coordinates at a time over all pairs, eight pairs' loads in flight; the sums go where the
        // first slot's pair would be staged. The two steps of a pair are added to each other and then to one running
        // sum: it telescopes, phi(x_k) - phi(x_0), and stays as small as the features are. (Sums of the even and the odd
        // steps apart from each other grow without bound on rough paths, and their difference is what is left: 300
        // sequences of 20001 points of white noise 2.4e-4, of 20001 alternating ones 1.8e-1.)
        const int64_t pairs_all = (T_all + 1) / 2, whole = T_all / 2;
        if (pairs_all > 0) {
            float4 *sums = reinterpret_cast<float4 *>(lds);
            for (int i = tid; i < F; i += NT) {
                const float4 *src = reinterpret_cast<const float4 *>(seq) + i;
                float sum0 = 0.f, sum1 = 0.f;
#pragma unroll 8
                for (int64_t p = 0; p < whole; ++p) {
                    const float4 x = src[p * F];
                    sum0 += x.x + x.y;
                    sum1 += x.z + x.w;
                }
                if (whole < pairs_all) {                     // the last pair has no second step
                    const float4 x = src[whole * F];
                    sum0 += x.x;
                    sum1 += x.z;
                }
                sums[i] = make_float4(sum0, 0.f, sum1, 0.f);
            }
            __syncthreads();
        }
    }
    __builtin_amdgcn_s_setprio(1);
    if (kEarly && !kSumFirst && pair0 < pairs) stage_direct(lvl, pair0);
    // an iteration exists while its first item does
    while ((kStream ? pair0_first : pair0) < pairs) {
        if (!kStream || pair0 < pairs) {                      // streaming: the last iteration may have fewer items
            // Tables of this level. They are the same whenever the level comes up and stay in L1/L2; the
            // pointer is laundered so that the compiler reloads them every iteration instead of keeping ~90
            // loop-invariant registers (table words and everything derived from them) alive across the transform.
            const uint32_t *tabl = kStream ? table + (int64_t)lvl * tl.words : tab_fixed;
            asm volatile("" : "+s"(tabl));
            // (the laundered pointer would be a generic one: loads through it would count as LDS operations too)
            const GlobalWords tabi = (GlobalWords)tabl;
            const int NG = kStream ? (int)tabi[0] : NG_fixed;
#pragma unroll
            for (int q = 0; q < P::R; ++q) gw[q] = tabi[tl.gather + lg + P::G * q];
#pragma unroll
            for (int g = 0; g < kFoldInRegs; ++g) fw[g] = g < NG ? tabi[tl.fold + g * P::GF + (lg % P::GF)] : kFoldPad << 16;

            // 1a. staging
            if (!kEarly && !kSumFirst) stage_direct(lvl, pair0);
            __builtin_amdgcn_s_waitcnt(0x0f70);                 // vmcnt(0): the direct loads have landed
            // odd number of increments, last pair: its second step does not exist; what the producer left in
            // its place (the increment across the sequence boundary) is cleared so that it cannot touch the result
            const int64_t last = last_in_grp - pair0;
            if ((T & 1) && last >= 0 && last < SPG) {
                float2 *st = wave_lds + (last_grp * SPG + (int)last) * PS;
                for (int a = lane; a < twoF; a += 64) st[a].y = 0.f;
            }
            transform_fence<P>();
            // 1b. unless the level has lists: fold the third and later coordinates of a bucket into its first one, one rank per round
            auto fold = [&](uint32_t w) {
                const uint32_t own = w & 0xffffu, tgt = w >> 16;
                if (tgt != kFoldPad) {
                    const float2 x = *reinterpret_cast<const float2 *>(my_slot_bytes + own);
                    const float2 y = *reinterpret_cast<const float2 *>(my_slot_bytes + tgt);
                    *reinterpret_cast<float2 *>(my_slot_bytes + tgt) = make_float2(x.x + y.x, x.y + y.y);
                }
                wave_lds_fence();
            };
#pragma unroll
            for (int g = 0; g < kFoldInRegs; ++g)
                if (g < NG) fold(fw[g]);
            for (int g = kFoldInRegs; g < NG; ++g) fold(tabi[tl.fold + g * P::GF + (lg % P::GF)]);
            // 1c. gather: first and second coordinate of each of this lane's buckets
            float2 v[P::R];
#pragma unroll
            for (int q = 0; q < P::R; ++q) {
                const float2 x0 = *reinterpret_cast<const float2 *>(my_slot_bytes + (gw[q] & 0xffffu));
                const float2 x1 = *reinterpret_cast<const float2 *>(my_slot_bytes + (gw[q] >> 16));
                v[q] = make_float2(x0.x + x1.x, x0.y + x1.y);
                // keep the scheduler from issuing all 2R reads at once (it would need 4R registers)
                if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                if (kFew > 1 && q + 1 == P::R / kFew && few) {
#pragma unroll
                    for (int z = P::R / kFew; z < P::R; ++z) v[z] = make_float2(0.f, 0.f);
                    break;
                }
            }
            // 1d. lists: the third and later coordinates of a bucket straight from the staging area, two per row and
            // bucket. Against folding, whose rounds each wait for an LDS round trip, they cost a table word per row:
            // the table builder chooses (many coordinates per bucket: lists).
            // Four rows at a time (each group has a multiple of four): eight reads in flight, the next four words under
            // them; two beside the accumulators of JOINT, which four push into spills (D = 100, five levels: 15 -> 36).
            if (const int rows = kStream ? (int)tabi[1] : rows_fixed) {
                constexpr int kRows = JOINT ? 2 : 4;
                const GlobalWords words = tabi + tl.fold + lg;
                uint32_t w[kRows];
#pragma unroll
                for (int i = 0; i < kRows; ++i) w[i] = words[i * P::G];
                int next = kRows;
#pragma unroll
                for (int q = 0; q < P::R; ++q) {
                    for (int x = (int)tabi[2 + q]; x > 0; x -= kRows) {
                        float2 c[2 * kRows];
#pragma unroll
                        for (int i = 0; i < kRows; ++i) {
                            c[2 * i] = *reinterpret_cast<const float2 *>(my_slot_bytes + (w[i] & 0xffffu));
                            c[2 * i + 1] = *reinterpret_cast<const float2 *>(my_slot_bytes + (w[i] >> 16));
                        }
                        const GlobalWords ahead = words + (next < rows ? next : 0) * P::G;
#pragma unroll
                        for (int i = 0; i < kRows; ++i) w[i] = ahead[i * P::G];
                        next += kRows;
#pragma unroll
                        for (int i = 0; i < 2 * kRows; ++i) v[q] = make_float2(v[q].x + c[i].x, v[q].y + c[i].y);
                    }
                }
            }
            // 2. FPW transforms per wavefront, in place in the slots. The transform is the one long stretch of
            // arithmetic of an iteration; everything else is short pieces of work between waits (loads, LDS round
            // trips, barriers). A wavefront in those phases runs at a raised priority, so that it gets its few
            // instructions issued at once and goes back to waiting instead of queueing behind other wavefronts'
            // transforms (measured: 3-7 % on every workload; the other way round, 2-3 % slower).
            __builtin_amdgcn_s_setprio(0);
            fft.template run_from_registers<true, kFew>(my_slot, v, few);
            __builtin_amdgcn_s_setprio(1);
        }
        __syncthreads();
        // 3. per-bin separation and recurrence, two time steps per slot, items in order (levels ascending
        // within a pair).
        // For D = 1024 (128-register budget, one pair per wavefront) the thread index is laundered so that
        // the LDS addresses of the bins are recomputed here (a few adds) instead of being kept across the
        // whole iteration as loop invariants, where they were spilled to scratch (measured: 8 % faster
        // there, slower for the other transform lengths).
        int tid_here = tid;
        if constexpr (LOG2D == 10 || LOG2D == 1000) asm volatile("" : "+v"(tid_here));
        float2 zreg[kEarly ? P::FPW : 1][kEarly ? BPT : 1][kEarly ? NTR : 1][2];
        if constexpr (kEarly) {
#pragma unroll
            for (int s = 0; s < P::FPW; ++s)
#pragma unroll
                for (int b = 0; b < BPT; ++b) {
                    const int f = tid_here + NT * b;
                    const int fi = P::pad(f < NB ? f : 0);
                    const int fc = kPack ? P::pad(f > 0 && f < NB ? D - f : D / 2) : P::pad(f > 0 && f < NB ? D - f : 0);
#pragma unroll
                    for (int j = 0; j < NTR; ++j) {
                        const float2 *Z = lds + ((size_t)j * P::FPW + s) * PS;
                        zreg[s][b][j][0] = Z[fi];
                        zreg[s][b][j][1] = Z[fc];
                    }
                }
            __syncthreads();                                        // the slots are free again
        }
        const int64_t pair0_now = pair0;
        advance(lvl, pair0);
        if (kEarly && pair0 < pairs) stage_direct(lvl, pair0);

        // one (pair, level) of one bin: separation of the two steps and A_LL += ... for both
        auto update_bin = [&](auto level_tag, auto packed_tag, auto full_tag, int s, int b, int j, int64_t pair0_j,
                              LevelCarry<ORDER> (&c)[kStarts]) {
            constexpr int LL = decltype(level_tag)::value;
            constexpr bool PK = kPack && decltype(packed_tag)::value != 0;   // this wavefront holds the thread of bins 0 and D/2
            constexpr bool FULL = decltype(full_tag)::value != 0;      // every item of the iteration has both steps
            const int f = tid_here + NT * b;                            // a bin that exists (the caller checks)
            const bool pk = PK && b == 0 && f == 0;
            const bool second_step = FULL || 2 * (pair0_j + s) + 1 < T;    // wavefront-uniform
            float2 z, zc;
            if constexpr (kEarly) {
                z = zreg[s][b][j][0];
                zc = zreg[s][b][j][1];
            } else {
                const float2 *Z = lds + ((size_t)j * P::FPW + s) * PS;
                z = Z[P::pad(f)];
                zc = Z[kPack ? P::pad(f > 0 ? D - f : D / 2) : P::pad(f > 0 ? D - f : 0)];
            }
            // every first tensor position up to this level (JOINT; the whole sequence needs the first one only)
            level_loop<JOINT ? LL + 1 : 1>([&](auto start_tag) {
                constexpr int a = decltype(start_tag)::value;
                level_step<ORDER, LL - a, PK>(z, zc, pk, second_step, A[b][acc_index(M, a, LL)], c[a]);
            });
        };
        // The whole of phase 3, compiled four times: for the wavefront of the packed thread and for the others,
        // and for iterations whose items all exist and have both time steps (all but the last one or two of a
        // sequence: no per-item conditions, no selects) and for the rest.
        auto phase3 = [&](auto packed_tag, auto full_tag) {
            constexpr bool FULL = decltype(full_tag)::value != 0;
            if constexpr (kStream) {
                // one branch on the level of the iteration's first item; inside it every item's level is static
                with_level<M>(lvl_first, [&](auto first_tag) {
                    constexpr int L0 = decltype(first_tag)::value;
                    item_loop<L0, M, NTR>([&](auto level_tag, auto item_tag, int group_offset) {
                        constexpr int j = decltype(item_tag)::value;
                        const int64_t pair0_j = pair0_first + group_offset * P::FPW;
                        if (FULL || pair0_j < pairs) {
#pragma unroll
                            for (int s = 0; s < P::FPW; ++s) {
                                if (!FULL && pair0_j + s >= pairs) continue;   // slot without a pair (last group only)
#pragma unroll
                                for (int b = 0; b < BPT; ++b)
                                    if (NT * BPT == NB || tid_here + NT * b < NB)
                                        update_bin(level_tag, packed_tag, full_tag, s, b, j, pair0_j, carry[s][b]);
                            }
                        }
                    });
                });
            } else {
                // with more than four transforms per wavefront and three or more levels the loop over the pairs
                // stays a loop: unrolled it needs 50-150 spilled registers (measured rolled: D = 64 ... 200 with
                // 4-8 levels 1.4-3 times faster; with one or two levels up to 45 % slower, hence the condition)
                constexpr bool kRolled = P::FPW > 4 && M >= 3;
                auto one_pair = [&](auto both_tag, int s) {
#pragma unroll
                    for (int b = 0; b < BPT; ++b) {
                        if (NT * BPT == NB || tid_here + NT * b < NB) {
                            LevelCarry<ORDER> c[kStarts];
                            level_loop<M>([&](auto level_tag) {
                                update_bin(level_tag, packed_tag, both_tag, s, b, decltype(level_tag)::value, pair0_now, c);
                            });
                        }
                    }
                };
                if constexpr (kRolled) {
                    // the pairs with both steps, then the one with the first step only, if this iteration has it: no selects
                    // in the loop, whose chain of levels the other wavefronts wait for (3000 x 200 points, D = 100, 50
                    // frequencies, eight levels 844 -> 825 us, D = 128 748 -> 710, D = 200, six levels 1168 -> 1133)
                    const int64_t left = T / 2 - pair0_now;
                    const int both = left < P::FPW ? (int)left : P::FPW;
#pragma unroll 1
                    for (int s = 0; s < both; ++s) one_pair(LevelTag<1>{}, s);
                    if (both < P::FPW && pair0_now + both < pairs) one_pair(LevelTag<0>{}, both);
                } else {
#pragma unroll
                    for (int s = 0; s < P::FPW; ++s)
                        if (FULL || pair0_now + s < pairs) one_pair(full_tag, s);     // (slots without a pair: last iteration only)
                }
            }
        };
        // groups: every thread advances its bin by its group's pairs (existence of pairs and steps is per lane)
        auto phase3_groups = [&]() {
#pragma unroll 1
            for (int i = 0; i < SPG; ++i) {
                const int64_t p = pair0_now + i;
                if (2 * p >= T_grp) break;
                const float2 *Z = lds + (size_t)(grp * SPG + i) * PS;
                const int fi = P::pad(bin), fc = P::pad(bin > 0 ? D - bin : 0);
                LevelCarry<ORDER> c[kStarts];
                level_loop<M>([&](auto level_tag) {
                    constexpr int LL = decltype(level_tag)::value;
                    const float2 z = Z[(size_t)LL * P::FPW * PS + fi], zc = Z[(size_t)LL * P::FPW * PS + fc];
                    level_loop<JOINT ? LL + 1 : 1>([&](auto start_tag) {
                        constexpr int a = decltype(start_tag)::value;
                        level_step<ORDER, LL - a, false>(z, zc, false, 2 * p + 1 < T_grp, A[0][acc_index(M, a, LL)], c[a]);
                    });
                });
            }
        };
        // full: the last pair of the last pair group that this iteration touches has a second step
        const int64_t last_pair0 = kStream ? pair0_first + ((lvl_first + NTR - 1) / M) * P::FPW : pair0_now;
        const bool full = 2 * (last_pair0 + P::FPW) - 1 < T;
        if constexpr (GR > 1) {
            if (grp < GR) phase3_groups();
        } else if (kPack && wave == 0) {
            if (kSplitFull && full) phase3(LevelTag<1>{}, LevelTag<1>{});
            else phase3(LevelTag<1>{}, LevelTag<0>{});
        } else {
            if (kSplitFull && full) phase3(LevelTag<0>{}, LevelTag<1>{});
            else phase3(LevelTag<0>{}, LevelTag<0>{});
        }
        if constexpr (kStream) advance(lvl_first, pair0_first);
        if (!kEarly) __syncthreads();
    }
    if (kEarly) __syncthreads();

    if constexpr (GR > 1) {                                  // join the groups, left to right, in the threads of the first
        if (cut.mode != 2) {
            if (grp > 0 && grp < GR) {
                float2 *dst = lds + (size_t)(grp - 1) * kAcc * NB + bin;
#pragma unroll
                for (int q = 0; q < kAcc; ++q) dst[q * NB] = A[0][q];
            }
            __syncthreads();
            if (grp == 0) {
#pragma unroll 1
                for (int g = 1; g < GR; ++g) {
                    const float2 *src = lds + (size_t)(g - 1) * kAcc * NB + bin;
                    float2 B[kAcc];
#pragma unroll
                    for (int q = 0; q < kAcc; ++q) B[q] = src[q * NB];
#pragma unroll
                    for (int a = 0; a < M; ++a) {
                        if (a > 0 && cut.mode == 0) break;   // the whole sequence: only ranges from position 1 on
#pragma unroll
                        for (int l = M - 1; l >= a; --l) {
                            const float2 x = A[0][acc_index(M, a, l)], y = B[acc_index(M, a, l)];
                            float2 acc = make_float2(x.x + y.x, x.y + y.y);
#pragma unroll
                            for (int j = a; j < l; ++j) acc = cfmaf(A[0][acc_index(M, a, j)], B[acc_index(M, j + 1, l)], acc);
                            A[0][acc_index(M, a, l)] = acc;
                        }
                    }
                }
            }
            __syncthreads();
        }
    }

    if (JOINT && cut.mode == 1) {                            // a piece of a sequence: its accumulators are the result
#pragma unroll
        for (int b = 0; b < BPT; ++b) {
            const int f = tid + NT * b;
            if (f < NB) {
#pragma unroll
                for (int l = 0; l < kAcc; ++l) {
                    float2 *sp = spectra_row + l * (D / 2 + 1);
                    const float2 y = A[b][l];
                    if (kPack && f == 0) {                   // bins 0 and D/2, both real
                        sp[0] = make_float2(y.x, 0.f);
                        sp[D / 2] = make_float2(y.y, 0.f);
                    } else {
                        sp[f] = y;
                    }
                }
            }
        }
        return;
    }

    // Phi_m = Re(FFT(conj Y_m)) / D with Y_m the Hermitian extension of A_m; slot 0 of transform m of the workgroup.
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
        const int f = tid + NT * b;
        if (f < NB) {
#pragma unroll
            for (int l = 0; l < M; ++l) {
                float2 *Y = lds + (size_t)l * P::FPW * PS;
                const float2 y = A[b][l];
                if (kPack && f == 0) {                       // bins 0 and D/2, both real
                    Y[P::pad(0)] = make_float2(y.x, 0.f);
                    Y[P::pad(D / 2)] = make_float2(y.y, 0.f);
                } else {
                    Y[P::pad(f)] = make_float2(y.x, -y.y);
                    if (f > 0 && f < D / 2) Y[P::pad(D - f)] = y;
                }
            }
        }
    }
    __syncthreads();
    if (wv < M) {                                            // (always, unless streaming)
        fft.run(my_slot);
        transform_fence<P>();
        float *row = out + row_id * ld_out;
        if (tid == 0) row[0] = 1.0f;
        const float invD = 1.0f / (float)D;
        // Dout buckets per level. Dout == D: the transform was circular in D already. Dout < D (a bucket
        // count that is no power of two): D was chosen so large that the M-fold convolution never wrapped,
        // and the linear result is folded modulo Dout here.
        for (int j = lane; j < Dout; j += 64) {
            float acc = 0.f;
            for (int e = j; e < D; e += Dout) acc += wave_lds[P::pad(e)].x;
            row[1 + (int64_t)wv * Dout + j] = acc * invD;
        }
    }
}

}  // namespace tuned
}  // namespace rfsf
