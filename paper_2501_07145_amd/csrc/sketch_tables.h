// The tables of the tuned sketch kernels (layout: tuned::TableLayout), built once per call, one workgroup per level.
#pragma once

#include "rfsf_internal.h"

namespace rfsf {

// What a launch needs to build the tables. `words` per level at `table`; `coord_base`, `zero_off`: byte offsets
// within a slot of position 0 and of the float2 that is always zero.
struct TableJob {
    const int32_t *hash;
    uint32_t *table;
    int F, D, Dout, G, words, gather, fold;
    uint32_t coord_base, zero_off;
    int groups;                    // bucket groups of G buckets (points per lane) that may have lists; 0: folding only
};
// Lists are chosen over folding when they take no more than this many rows per fold round. (1000 sequences of 100 points,
// four levels, sketch kernel, with at most 1, 2, 4 rows per round: 900 frequencies in 256 buckets 1842, 943, 946 us, 1000 in
// 512 1744, 1162, 1163, 300 in 256 397, 398, 442, 200 in 128 284, 287, 305; folding alone 1757, 1715, 379, 283.)
constexpr int kListRowsPerRound = 2, kMaxGroups = 32;
constexpr int kTableThreads = 256;
// LDS of a building workgroup: bucket ends, class sizes, bucket of every coordinate, coordinates by bucket
__host__ __device__ constexpr size_t table_lds_bytes(int F, int Dout)
{
    return sizeof(int) * ((size_t)Dout + 2 * F + 1 + 2 * kMaxGroups + 2) + sizeof(uint16_t) * 4 * (size_t)F;
}

// Position in a pair's row of coordinate a: cosine and sine of a frequency are neighbours (16 bytes per pair of
// steps, so that the projection kernel writes whole lines), the cosine coordinates are 0 .. F-1, the sines F .. 2F-1.
__device__ __forceinline__ uint32_t coordinate_position(int a, int F) { return a < F ? 2u * a : 2u * (a - F) + 1u; }

// rank(a) = number of earlier coordinates of the level in the same bucket; ranks 0 and 1 go to the gather words, ranks
// >= 2 become fold entries, ordered by rank and padded so that a round of G entries never mixes two ranks (hence never
// repeats a bucket), or go to lists of their buckets, two per row, where those take no more than kListRowsPerRound rows
// per round. Coordinates are sorted into their buckets (histogram, prefix sum, placement), whose few
// members are then compared with each other: linear in 2F, where counting equal earlier buckets coordinate by coordinate
// was quadratic. Placement and the order within a rank depend on the order of LDS atomics; what is computed from the
// tables does not: the ranks are exact, and the entries of one rank touch different buckets.
// Called by all kTableThreads threads of the workgroup; `lds` holds table_lds_bytes.
__device__ __forceinline__ void build_level_table(const TableJob &job, int m, int *lds)
{
    const int tid = threadIdx.x, F = job.F, twoF = 2 * F, Dout = job.Dout;
    int *end = lds, *cls = end + Dout;                                  // [Dout], [2F + 1]
    int *rows = cls + twoF + 1, *row0 = rows + kMaxGroups, *chosen = row0 + kMaxGroups;       // list rows of a group, its first
    uint16_t *bucket = reinterpret_cast<uint16_t *>(chosen + 2), *item = bucket + twoF;
    const int32_t *hash = job.hash + (int64_t)m * twoF;
    uint32_t *tab = job.table + (int64_t)m * job.words;

    for (int e = tid; e < Dout; e += kTableThreads) end[e] = 0;
    for (int r = tid; r <= twoF; r += kTableThreads) cls[r] = 0;
    if (tid < kMaxGroups) rows[tid] = 0;
    __syncthreads();
    for (int a = tid; a < twoF; a += kTableThreads) {
        const int b = ((hash[a] % Dout) + Dout) % Dout;
        bucket[a] = (uint16_t)b;
        atomicAdd(&end[b], 1);
    }
    __syncthreads();
    if (tid < 64) {                                                     // exclusive prefix sum by one wavefront
        int carry = 0;
        for (int e0 = 0; e0 < Dout; e0 += 64) {
            const int e = e0 + tid, own = e < Dout ? end[e] : 0;
            int sum = own;
#pragma unroll
            for (int o = 1; o < 64; o *= 2) {
                const int v = __shfl_up(sum, o);
                if (tid >= o) sum += v;
            }
            if (e < Dout) end[e] = carry + sum - own;
            carry += __shfl(sum, 63);
        }
    }
    __syncthreads();
    for (int a = tid; a < twoF; a += kTableThreads) item[atomicAdd(&end[bucket[a]], 1)] = (uint16_t)a;
    __syncthreads();                                                    // end[b] is now the end of bucket b
    auto rank_of = [&](int a, int &first) {
        const int b = bucket[a];
        int r = 0;
        first = a;
        for (int i = b ? end[b - 1] : 0; i < end[b]; ++i) {
            const int o = item[i];
            r += o < a;
            first = o < first ? o : first;
        }
        return r;
    };
    for (int a = tid; a < twoF; a += kTableThreads) {
        int first;
        const int r = rank_of(a, first);
        if (r >= 2) {
            atomicAdd(&cls[r], 1);
            if (job.groups) atomicMax(&rows[bucket[a] / job.G], r / 2);         // row r / 2 - 1 of the bucket's list
        }
    }
    __syncthreads();
    if (tid == 0) {                       // class sizes -> start offsets, each class padded to G; ranks have no gaps
        int off = 0;
        for (int r = 2; r <= twoF && cls[r] > 0; ++r) {
            const int c = cls[r];
            cls[r] = off;
            off += (c + job.G - 1) / job.G * job.G;
        }
        int n = 0;
        for (int q = 0; q < job.groups; ++q) {
            row0[q] = n;
            rows[q] = (rows[q] + 3) & ~3;
            n += rows[q];
        }
        const int rounds = off / job.G;
        chosen[0] = job.groups && n > 0 && n <= kListRowsPerRound * rounds && n <= twoF;     // (the room for them)
        chosen[1] = chosen[0] ? n : rounds;
        tab[0] = chosen[0] ? 0u : (uint32_t)rounds;
        tab[1] = chosen[0] ? (uint32_t)n : 0u;
    }
    __syncthreads();
    const bool lists = chosen[0] != 0;
    if (tid < job.groups) tab[2 + tid] = lists ? (uint32_t)rows[tid] : 0u;
    for (int i = tid; i < chosen[1] * job.G; i += kTableThreads)
        tab[job.fold + i] = job.zero_off | ((lists ? job.zero_off : 0xffffu) << 16);
    for (int e = tid; e < job.D; e += kTableThreads) {
        int s0 = twoF, s1 = twoF;         // the two smallest coordinates of the bucket
        if (e < Dout)
            for (int i = e ? end[e - 1] : 0; i < end[e]; ++i) {
                const int o = item[i];
                if (o < s0) { s1 = s0; s0 = o; }
                else if (o < s1) s1 = o;
            }
        const uint32_t w0 = s0 < twoF ? job.coord_base + 8u * coordinate_position(s0, F) : job.zero_off;
        const uint32_t w1 = s1 < twoF ? job.coord_base + 8u * coordinate_position(s1, F) : job.zero_off;
        tab[job.gather + e] = w0 | (w1 << 16);
    }
    __threadfence_block();
    __syncthreads();                      // padding entries are in place before the real ones land
    for (int a = tid; a < twoF; a += kTableThreads) {
        int first;
        const int r = rank_of(a, first);
        if (r < 2) continue;
        if (lists) {                      // half (r mod 2) of word lg of row r / 2 - 1 of its bucket's list
            const int q = bucket[a] / job.G, lg = bucket[a] - q * job.G;
            uint16_t *word = reinterpret_cast<uint16_t *>(tab + job.fold + (row0[q] + r / 2 - 1) * job.G + lg);
            word[r & 1] = (uint16_t)(job.coord_base + 8u * coordinate_position(a, F));
            continue;
        }
        tab[job.fold + atomicAdd(&cls[r], 1)] =
            (job.coord_base + 8u * coordinate_position(a, F)) | ((job.coord_base + 8u * coordinate_position(first, F)) << 16);
    }
}

}  // namespace rfsf
