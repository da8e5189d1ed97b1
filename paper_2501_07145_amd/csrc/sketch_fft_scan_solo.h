// Steps 1-4 or 3-4 for short transforms, whole sequences and pieces of sequences cut in time (TimeCut::mode 1): a wavefront
// works by itself.
//
// The kernel with a wavefront per level (sketch_fft_scan_tuned.h) meets at two barriers per iteration, and with five levels its
// workgroups of five wavefronts leave a CU half empty (6.5 to 7.8 resident wavefronts where 16 would fit: see
// transforms_in_flight). Short transforms come several to a wavefront, so that one wavefront has room for the transforms of
// all levels of a pair of steps: slot s holds level s / SP of pair s mod SP, SP pairs at a time, and the bins of a pair
// fit its lanes. It advances its own stretch of the sequence (of the piece) without meeting anybody; the four stretches of a
// workgroup are joined in LDS at the end, left to right, which takes the accumulators of all ranges of tensor positions.
//
// What bounded the other kernel was waiting (vector instructions 0.3 of the time, LDS 0.35), and so this one has room for the
// projection: it computes the increments that it needs (Points) instead of reading them from where the projection
// kernel has written them, which costs a wavefront 800 vector instructions per iteration on top of 1000 (D = 100, five levels,
// five channels) and spares the other kernel, its traffic and the wait for it. Features, one wavefront per level, by itself with
// increments from memory, by itself with its own, us: 10 x 1e5 points, 50 frequencies, D = 100, five levels 1486, 1167, 712; 100 x
// 1000 126, 124, 105; 3000 x 200 830, 690, 441; D = 64, 32 frequencies 491, 409, 295; three levels, D = 128, 64 frequencies 438,
// 494, 265; D = 200, 120 frequencies 900, 891, 552; 2000 x 1000 points, 8 channels, four levels, D = 256, 128 frequencies 3270,
// 3600, 2250. Bound now: vector instructions (about 0.7 of the time with 13 of 16 wavefronts resident).
#pragma once

#include "sincos.h"
#include "sketch_fft_scan_tuned.h"

#include <type_traits>

namespace rfsf {
namespace tuned {

// Bank conflicts. 16 lanes at a time write float2, over 32 banks, at least 6.4 cycles for a wavefront, 32 lanes read, over 64 banks, at
// least 3.5. The lanes of a transform that write next to each other are few here (4, 5 and 8 for 64, 100 and 128 points), so
// that several transforms' meet in a bank unless the slots are the right distance apart: solo_stride. Cycles of a transform's exchanges, gather
// and separation by that count, before and after: 64 points 598 -> 526, 128 567 -> 499 (256: 517, at best 502). SQ_LDS_BANK_CONFLICT of a
// launch: 1500 x 200 points, five levels, 32 frequencies, 64 points 1.71e7 -> 1.03e7; 1500 x 200, four, 64, 128 2.54e7 -> 1.04e7: some are
// left, and not worth more: distances that count a quarter less for the exchanges of 100 points, and a sixth less for those of 256, gained nothing.
// Pairs of steps of a wavefront's iteration; 0: the levels do not fit a wavefront.
__host__ __device__ constexpr int solo_pairs(int M, int FPW) { return FPW / M; }
__host__ __device__ constexpr size_t solo_lds_with(int M, int FPW, int stride, int NTWL)
{
    return sizeof(float2) * ((size_t)kSoloWaves * solo_pairs(M, FPW) * M * stride + NTWL);
}
// From slot to slot: 4 float2 beyond a multiple of 8 with 64 points, 8 beyond one of 16 with 100 and 128, unless a CU would hold
// fewer workgroups for it.
__host__ __device__ constexpr int solo_stride(int D, int M, int FPW, int PD, int NTWL, int F)
{
    const int least = slot_stride(PD, 2 * F), grain = D == 64 ? 8 : D <= 128 ? 16 : 1;
    const int apart = (least + grain / 2 - 1) / grain * grain + grain / 2;
    const size_t held = kLdsPerCu / solo_lds_with(M, FPW, least, NTWL);       // (no more than four by their registers)
    return grain == 1 || kLdsPerCu / solo_lds_with(M, FPW, apart, NTWL) < (held < 4 ? held : 4) ? least : apart;
}
__host__ __device__ constexpr size_t solo_lds_bytes(int D, int M, int FPW, int PD, int NTWL, int F)
{
    return solo_lds_with(M, FPW, solo_stride(D, M, FPW, PD, NTWL, F), NTWL);
}

// Where the accumulators of a lane fit the registers (solo_waves_per_simd) and the levels fill the wavefront's
// transforms: largest number of levels for which that holds. Five levels at D = 200 spill 4 registers, at D = 64 one or two, the others none. What is left out: orders 2
// and 3, whose carried values do not fit; four levels at D = 200, four of six transforms used (in the other kernels and here, us: 1000 x
// 100 points, 5 channels, 50 frequencies 103 and 144, 8, 100 176 and 176, 10 x 20000, 8, 100 373 and 404, but 100 x 1000, 8, 100 192 and 157,
// 3000 x 200, 1, 128 1088 and 745); five at D = 128, which has 6 to 8 spills since W is read by 32-bit offsets (25 before, and split batches
// took 147 for 142) and would be faster here by now (50 frequencies, 5 channels, 3000 x 200 782 and 464, 100 x 1000 111 and 95).
__host__ __device__ constexpr bool solo_fits(int M, int D, int order)
{
    if (order != 1 || M < 2) return false;
    return (D == 64 && M <= 5) || (D == 100 && M <= 6) || (D == 128 && M <= 4) || (D == 200 && (M <= 3 || M == 5)) || (D == 256 && M <= 4);
}
// Wavefronts per SIMD that the registers are bounded for. (D = 256, four levels, 5000 x 100 points 639 us with three, 888 with
// four and 48 spills; three levels, 1000 x 100, 149 and 123. D = 128, four levels, takes 123 registers.)
__host__ __device__ constexpr int solo_waves_per_simd(int M, int D) { return (D >= 200 && M >= 4) ? 3 : 4; }
// Ten-point butterflies (D = 200) read their twiddles ahead where a lane's accumulators leave the registers for it: two and three levels (12 and
// 24 registers of accumulators), not five (60; 31 spills instead of 4). 3000 x 200 points, 100 frequencies, 3 and 8 channels, ahead and on the spot,
// us: two 248 and 251, 263 and 266, three 358 and 363, 381 and 385, five 952 and 822, 1059 and 928.
__host__ __device__ constexpr bool solo_reads_ahead(int M, int D) { return (D / 2 + 64) / 64 * M * (M + 1) < 40; }
constexpr int kSoloChannels = 8;
constexpr int kRawBufferWord3 = 0x00020000;   // buffer descriptor, last word: untyped 32-bit data
__host__ __device__ constexpr int solo_columns(int D) { return D <= 128 ? 1 : 2; }     // frequencies of a lane
typedef const __attribute__((address_space(1))) float *GlobalFloats;
typedef const __attribute__((address_space(4))) float *ConstantFloats;      // scalar loads where the address is uniform
// d > 0: the increments are not in memory, the wavefront computes them from points of d channels (Points), a frequency per
// lane: angles by multiply-adds of the points' channels with the lane's column of W. The channels are the same for all lanes, but
// a multiply-add with a scalar register takes 4.35 cycles of a SIMD instead of 2.6: they are in vector registers where there is room.
template <int LOG2D, int M, int ORDER, int d>
__global__ __launch_bounds__(64 * kSoloWaves) __attribute__((amdgpu_waves_per_eu(solo_waves_per_simd(M, Plan<LOG2D>::D), 4))) void sketch_fft_scan_solo_kernel(
    const float *__restrict__ dphi, const uint32_t *__restrict__ table, int64_t L, const int64_t *__restrict__ lengths, int F,
    TimeCut cut)
{
    using P = Plan<LOG2D>;
    constexpr int D = P::D, SP = solo_pairs(M, P::FPW), SLOTS = SP * M, Q = M * (M + 1) / 2;
    constexpr bool kPack = (D / 2) % 64 == 0;                // lane 0 carries the two real bins, 0 and D/2
    constexpr int NB = kPack ? D / 2 : D / 2 + 1, BPT = (NB + 63) / 64;
    extern __shared__ float2 lds[];                          // [wavefronts][SLOTS][PS] slots, then the twiddle table
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // lanes beyond those of the transforms repeat the work of the first ones: same addresses, same values
    constexpr int kLanesUsed = P::G * SLOTS;
    const int lane_t = lane % kLanesUsed, slot_id = lane_t / P::G, lg = lane_t % P::G;
    const int twoF = 2 * F, ZS = zero_slot(P::PD, twoF), PS = solo_stride(D, M, P::FPW, P::PD, P::NTWL, F);
    float2 *wave_lds = lds + (size_t)wave * SLOTS * PS, *my_slot = wave_lds + slot_id * PS;
    char *my_slot_bytes = reinterpret_cast<char *>(my_slot);
    // Workgroups go to the XCDs and their shader engines in turn, so that with an even number of pieces some would get only the last
    // ones of all sequences, which are short or empty where sequences have lengths of their own: those start with any piece. (Lengths from
    // half, us: 2150 x 698 points, 64 buckets, five levels 559 -> 481, 1800 x 1500, 64, three 606 -> 509, 1500 x 800, 128, four 554 -> 494; the
    // first piece turned every eight sequences instead 554, 604, 548. Over 500 drawn shapes 0.997 of that on average.)
    const unsigned n_pieces = (unsigned)cut.pieces, sequence = blockIdx.x / n_pieces, place = blockIdx.x - sequence * n_pieces;
    const int64_t n = sequence, piece = lengths ? (place + (sequence * 2654435769u >> 16)) % n_pieces : place;
    const int64_t Ln = lengths ? (lengths[n] < 1 ? 1 : (lengths[n] > L ? L : lengths[n])) : L;
    const int64_t steps_left = Ln - 1 - 2 * piece * cut.pairs;
    const int64_t T_piece = steps_left < 0 ? 0 : (steps_left < 2 * cut.pairs ? steps_left : 2 * cut.pairs);
    // this wavefront's stretch: `stretch` pairs from pair `first` of the piece on, T steps of them
    const int64_t stretch = ((T_piece + 1) / 2 + kSoloWaves * SP - 1) / (kSoloWaves * SP) * SP, first = wave * stretch;
    const int64_t T_left = T_piece - 2 * first, T = T_left < 0 ? 0 : (T_left < 2 * stretch ? T_left : 2 * stretch);
    const int64_t pairs = (T + 1) / 2;
    const int64_t pf = (int64_t)M * 2 * twoF;
    const int64_t t_first = 2 * (piece * cut.pairs + first);
    const float *seq = dphi + (n * ((L + 1) / 2) + piece * cut.pairs + first) * pf + 4 * lane;
    const TableLayout tl = table_layout(D, P::GF, twoF);
    const int nload = twoF / 128, last_load = twoF % 128;
    const GlobalWords tabi = (GlobalWords)table + (int64_t)(slot_id / SP) * tl.words;       // of this lane's level
    const int NG = (int)tabi[0];
    int rounds = 0;
#pragma unroll
    for (int l = 0; l < M; ++l) {
        const int of_level = __builtin_amdgcn_readfirstlane((int)((GlobalWords)table)[(int64_t)l * tl.words]);
        rounds = of_level > rounds ? of_level : rounds;
    }

    WaveFft<P> fft;
    fft.init(lg, lds + (size_t)kSoloWaves * SLOTS * PS, lds);
    if (lg == 0) my_slot[ZS] = make_float2(0.f, 0.f);
    wave_lds_fence();
    float2 A[BPT][Q];
#pragma unroll
    for (int b = 0; b < BPT; ++b)
#pragma unroll
        for (int q = 0; q < Q; ++q) A[b][q] = make_float2(0.f, 0.f);

    // Features of the points, for d > 0. Points beyond the sequence's last one are that one: their increments are zero.
    constexpr int kChannels = d > 0 ? d : 1;
    constexpr bool kVectorPoints = 2 * SP * d <= 24;         // registers for an iteration's points
    typedef std::conditional_t<kVectorPoints, GlobalFloats, ConstantFloats> PointFloats;
    const PointFloats points = (PointFloats)(cut.points.X + n * L * d);
    const float scale = 0.5f / sqrtf((float)F);
    auto point = [&](int64_t t, float (&x)[kChannels]) {
        const PointFloats src = points + (t < Ln ? t : Ln - 1) * d;
        if constexpr (kVectorPoints) {                       // vector loads of what is the same for all lanes: a uniform base and a lane's offset
            uint32_t here = 0;
            asm volatile("" : "+v"(here));
            const GlobalFloats at = (GlobalFloats)((const __attribute__((address_space(1))) char *)src + here);
#pragma unroll
            for (int c = 0; c < d; ++c) x[c] = at[c];
        } else {
#pragma unroll
            for (int c = 0; c < d; ++c) x[c] = src[c];
        }
    };
    auto signed_by = [&](uint32_t flip) { return __uint_as_float(__float_as_uint(scale) ^ (flip & 0x80000000u)); };
    auto column = [&](int l, int col, float (&w)[kChannels], float &scale_c, float &scale_s) {
        uint32_t frequency = 4u * (uint32_t)(lane + 64 * col < F ? lane + 64 * col : F - 1);
        // A scalar base and offset and a lane's own: as 64-bit addresses they are sums of 4.6 cycles of a SIMD each, 70 per iteration with five
        // channels and levels. (With signs by logic, below, and the masks of the recurrence, features, us: 100 x 1000 points, five channels, five
        // levels, D = 100 91.3 -> 88.6, 10 x 1e5 653 -> 628, 1000 x 100, eight, four, D = 256 157 -> 149, 2000 x 200, six, three, D = 128 183 ->
        // 168, three, five, D = 64 190 -> 184, five, three, D = 200 266 -> 253.)
        const auto rows = __builtin_amdgcn_make_buffer_rsrc((void *)(cut.points.W + (int64_t)l * d * F), 0, 4 * d * F, kRawBufferWord3);
        const auto flips = __builtin_amdgcn_make_buffer_rsrc((void *)(cut.points.sign + (int64_t)l * twoF), 0, 4 * twoF, kRawBufferWord3);
        asm volatile("" : "+v"(frequency));                  // (read again in every iteration, not kept in registers)
#pragma unroll
        for (int c = 0; c < d; ++c) w[c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, frequency, 4 * c * F, 0));
        scale_c = signed_by(__builtin_amdgcn_raw_buffer_load_b32(flips, frequency, 0, 0));
        scale_s = signed_by(__builtin_amdgcn_raw_buffer_load_b32(flips, frequency, 4 * F, 0));
    };
    auto features = [&](const float (&x)[kChannels], const float (&w)[kChannels], const Quarters &turn, float &s, float &c) {
        float t = x[0] * w[0];
#pragma unroll
        for (int i = 1; i < d; ++i) t = fmaf(x[i], w[i], t);
        sincos_quarters(t, turn, s, c);
    };
    constexpr int COLS = solo_columns(D);
    [[maybe_unused]] float before_s[M * COLS], before_c[M * COLS];       // of the point before the pair, per level
    if constexpr (d > 0) {
        float x[kChannels];
        point(t_first, x);
        const Quarters turn(cut.points.quarters, cut.points.quarters_rest);
#pragma unroll
        for (int j = 0; j < M * COLS; ++j) {
            if (64 * (j % COLS) >= F) continue;
            float w[kChannels], scale_c, scale_s;
            column(j / COLS, j % COLS, w, scale_c, scale_s);
            features(x, w, turn, before_s[j], before_c[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    uint32_t packed = lane == 0 ? 0xffffffffu : 0u;          // the lane of both real bins
    if constexpr (kPack) asm volatile("" : "+v"(packed));
    __builtin_amdgcn_s_setprio(1);
    for (int64_t pair0 = 0; pair0 < pairs; pair0 += SP) {
        if constexpr (d > 0) {
            const int64_t t0 = t_first + 2 * pair0;
            float x[2 * SP][kChannels];
#pragma unroll
            for (int i = 0; i < 2 * SP; ++i) point(t0 + 1 + i, x[i]);
            const Quarters turn(cut.points.quarters, cut.points.quarters_rest);
#pragma unroll
            for (int j = 0; j < M * COLS; ++j) {
                const int l = j / COLS, col = j % COLS;
                if (64 * col >= F) continue;
                float w[kChannels], scale_c, scale_s;
                column(l, col, w, scale_c, scale_s);
#pragma unroll
                for (int i = 0; i < SP; ++i) {
                    float s1, c1, s2, c2;
                    features(x[2 * i], w, turn, s1, c1);
                    features(x[2 * i + 1], w, turn, s2, c2);
                    if (lane + 64 * col < F)
                        *reinterpret_cast<float4 *>(wave_lds + (l * SP + i) * PS + 2 * (lane + 64 * col)) =
                            make_float4((c1 - before_c[j]) * scale_c, (c2 - c1) * scale_c, (s1 - before_s[j]) * scale_s, (s2 - s1) * scale_s);
                    before_s[j] = s2;
                    before_c[j] = c2;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // staging: pairs beyond the last one are the last one, and ignored later
#pragma unroll
        for (int s = 0; s < (d > 0 ? 0 : SLOTS); ++s) {
            int64_t p = pair0 + s % SP;
            if (p >= pairs) p = pairs - 1;
            const float *src = seq + s / SP * 2 * twoF + p * pf;
            float2 *dst = wave_lds + s * PS;
            for (int j = 0; j < nload; ++j)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + 256 * j),
                                                 (__attribute__((address_space(3))) void *)(dst + 128 * j), 16, 0, 0);
            if (2 * lane < last_load)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + 256 * nload),
                                                 (__attribute__((address_space(3))) void *)(dst + 128 * nload), 16, 0, 0);
        }
        GlobalWords words = tabi;
        asm volatile("" : "+v"(words));                      // (the table words are loaded again, not kept across the transform)
        uint32_t gw[P::R];
#pragma unroll
        for (int q = 0; q < P::R; ++q) gw[q] = words[tl.gather + lg + P::G * q];
        uint32_t fw[kFoldInRegs];
#pragma unroll
        for (int g = 0; g < kFoldInRegs; ++g) fw[g] = g < NG ? words[tl.fold + g * P::GF + lg] : kFoldPad << 16;
        __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0): the direct loads have landed
        // the second step of the last pair does not exist if their number is odd
        const int64_t last = pairs - 1 - pair0;
        if (d == 0 && (T & 1) && last < SP) {
#pragma unroll
            for (int l = 0; l < M; ++l) {
                float2 *st = wave_lds + (l * SP + (int)last) * PS;
                for (int a = lane; a < twoF; a += 64) st[a].y = 0.f;
            }
        }
        wave_lds_fence();
        auto fold = [&](uint32_t w) {                        // third and later coordinates of a bucket into its first one
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
            if (g < rounds) fold(fw[g]);
        for (int g = kFoldInRegs; g < rounds; ++g) fold(g < NG ? words[tl.fold + g * P::GF + lg] : kFoldPad << 16);
        float2 v[P::R];
#pragma unroll
        for (int q = 0; q < P::R; ++q) {
            const float2 x0 = *reinterpret_cast<const float2 *>(my_slot_bytes + (gw[q] & 0xffffu));
            const float2 x1 = *reinterpret_cast<const float2 *>(my_slot_bytes + (gw[q] >> 16));
            v[q] = make_float2(x0.x + x1.x, x0.y + x1.y);
            if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        fft.template run_from_registers<solo_reads_ahead(M, D)>(my_slot, v);
        __builtin_amdgcn_s_setprio(1);
        wave_lds_fence();
        // separation and recurrence, a bin per lane, pair after pair. (A second step that does not exist is taken out by a mask: selects take
        // 4.5 cycles of a SIMD, from vcc up to 16, and code of its own for such a pair costs registers, six levels at D = 100 23 spills.)
#pragma unroll 1
        for (int i = 0; i < SP; ++i) {
            const int64_t p = pair0 + i;
            if (p >= pairs) break;
            uint32_t both = 2 * p + 1 < T ? 0xffffffffu : 0u;
            asm volatile("" : "+v"(both));
#pragma unroll
            for (int b = 0; b < BPT; ++b) {
                const int f = lane + 64 * b;
                if (NB % 64 != 0 && f >= NB) continue;
                const uint32_t pk = kPack && b == 0 ? packed : 0u;
                const float2 *Z = wave_lds + i * PS;
                const int fi = P::pad(f), fc = P::pad(f > 0 ? D - f : kPack ? D / 2 : 0);
                LevelCarry<ORDER> c[M];
                level_loop<M>([&](auto level_tag) {
                    constexpr int LL = decltype(level_tag)::value;
                    const float2 z = Z[(size_t)LL * SP * PS + fi], zc = Z[(size_t)LL * SP * PS + fc];
                    level_loop<LL + 1>([&](auto start_tag) {
                        constexpr int a = decltype(start_tag)::value;
                        level_step<ORDER, LL - a, kPack, true>(z, zc, pk, both, A[b][acc_index(M, a, LL)], c[a]);
                    });
                });
            }
        }
        wave_lds_fence();
    }

    // join the stretches, left to right, in the first wavefront; one at a time through LDS
    for (int w = 1; w < kSoloWaves; ++w) {
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int b = 0; b < BPT; ++b)
                if (lane + 64 * b < NB) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) lds[q * NB + lane + 64 * b] = A[b][q];
                }
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int b = 0; b < BPT; ++b) {
                if (lane + 64 * b >= NB) continue;
                const bool pk = kPack && lane + 64 * b == 0;
                const float2 *B = lds + lane + 64 * b;
#pragma unroll
                for (int a = 0; a < M; ++a) {
#pragma unroll
                    for (int l = M - 1; l >= a; --l) {
                        const float2 x = A[b][acc_index(M, a, l)], y = B[acc_index(M, a, l) * NB];
                        float2 acc = make_float2(x.x + y.x, x.y + y.y);
#pragma unroll
                        for (int j = a; j < l; ++j) acc = cfmaf_pk(A[b][acc_index(M, a, j)], B[acc_index(M, j + 1, l) * NB], acc, pk);
                        A[b][acc_index(M, a, l)] = acc;
                    }
                }
            }
        }
    }
    if (wave != 0) return;
    float2 *spectra_row = (cut.spectra ? cut.spectra : reinterpret_cast<float2 *>(const_cast<float *>(dphi))) +
                          n * cut.seq_stride + piece * cut.piece_stride;
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
        const int f = lane + 64 * b;
        if (f >= NB) continue;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float2 *sp = spectra_row + q * (D / 2 + 1);
            if (kPack && f == 0) {
                sp[0] = make_float2(A[b][q].x, 0.f);
                sp[D / 2] = make_float2(A[b][q].y, 0.f);
            } else {
                sp[f] = A[b][q];
            }
        }
    }
}

}  // namespace tuned
}  // namespace rfsf
