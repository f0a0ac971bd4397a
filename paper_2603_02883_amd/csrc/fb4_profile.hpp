// SeDA sub-formatbook construction (Sec. 3.4, "Constructing an 8-Dialect
// Sub-Formatbook"): count how often each dialect was selected on the anchor
// tokens of each group, then keep, per dynamic-range bucket (largest magnitude
// 8..15), the most frequently selected dialect of that bucket.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fb4_tables.hpp"

namespace fb4 {

constexpr int kProfileThreads = 256;

__global__ __launch_bounds__(kProfileThreads) void profile_clear_kernel(uint32_t* counts, uint32_t n)
{
    const uint32_t i = blockIdx.x * kProfileThreads + threadIdx.x;
    if (i < n) counts[i] = 0;
}

// One wavefront per row: a 32-bin histogram of the row's DIDs in LDS, then at most 32 global atomics.
__global__ __launch_bounds__(kProfileThreads) void profile_count_kernel(const uint16_t* meta, long long rows,
                                                                        long long nb, const int32_t* anchor_group,
                                                                        int n_groups, uint32_t* counts, uint32_t n_workgroups)
{
    __shared__ uint32_t hist[kProfileThreads / 64][32];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long stride = (long long)n_workgroups * (kProfileThreads / 64);
    for (long long r = (long long)blockIdx.x * (kProfileThreads / 64) + wave; r < rows; r += stride) {
        const int g = anchor_group[r];                    // wave-uniform
        if (g < 0 || g >= n_groups) continue;
        if (lane < 32) hist[wave][lane] = 0;
        __builtin_amdgcn_wave_barrier();
        const uint16_t* row = meta + r * nb;
        for (long long b = lane; b < nb; b += 64) {
            const uint32_t did = row[b] & 0xFFu;
            if (did < 32u) atomicAdd(&hist[wave][did], 1u);
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < 32) {
            const uint32_t c = hist[wave][lane];
            if (c) atomicAdd(counts + (long long)g * 32 + lane, c);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// One thread per (group, range bucket): the most frequent dialect of the bucket, lowest DID on ties (and when
// none was selected); 255 when the formatbook has no dialect of that range.
__global__ __launch_bounds__(kProfileThreads) void profile_select_kernel(const uint32_t* counts, int n_groups,
                                                                         const uint8_t* blob, uint8_t* sub)
{
    const uint32_t i = blockIdx.x * kProfileThreads + threadIdx.x;
    if (i >= (uint32_t)n_groups * 8u) return;
    const uint32_t g = i >> 3, k = i & 7u;
    const int n = *reinterpret_cast<const int32_t*>(blob + kOffCount);
    uint32_t best = 255u;
    long long best_count = -1;
    for (int d = 0; d < n; ++d) {
        const long long c = counts[(size_t)g * 32 + d];
        if (blob[kOffTop + d] == 8u + k && c > best_count) {
            best = (uint32_t)d;
            best_count = c;
        }
    }
    sub[i] = (uint8_t)best;
}

// The same in one launch: a workgroup per group looks through all rows for its anchors (a list in LDS), counts their
// dialects into 64 histograms, one per lane of a wavefront, so that neither many equal dialects nor many rows of one group
// meet in one address, and picks the group's dialects.
// kWords: metadata words per load, which divide the blocks of a row.
// us, three launches / this (rows x blocks, groups, share of anchors; graph, inputs changing): 16384 x 96, 64, 1/16 9.05 / 3.8, the
// same with all rows anchors 12.8 / 5.8, with a tenth of the rows anchors of one group 26.7 / 14.4; 1000 x 36, 64, 1/16 7.9 / 3.55; 30000 x
// 96, 200, 1/16 9.9 / 5.5.  Bound by its chain of dependent steps, most of it instructions of one workgroup: so a thread's anchors are
// found as bits and the sums and maxima exchanged inside the vector ALU (against a ballot, a place in the list and a branch per load
// and ten LDS round trips 0.82 of the time over 250 shapes of up to 512 groups, 0.855 over 400 with dense anchors).  Every workgroup
// looks through all rows (65536 x 96, 512 groups, 1/16 11.9 / 11.9).  One that gets every row as an anchor takes 0.0025 a word and
// 0.031 a load of the time that the atomics of three launches take for a row; the line below, 0.005 and 0.0175, was drawn where a tenth
// of the rows are anchors.  It keeps that worst input below 1 with loads of eight words (32768 x 136, one group 379 / 324), and at the
// longest rows that it takes with four, two and one up to 1.06, 1.27 and 1.47 (32768 x 43 378 / 557).
constexpr int64_t kProfileGroupMaxRows = 32768;
// (profile_group_kernel puts a count of words and a DID into 32 bits; the rule's rows have at most 400 * 8 / 23 words)
static_assert(((kProfileGroupMaxRows * (400 * 8 / (2 * 8 + 7)) + 1) << 5 | 31) <= 0xFFFFFFFFll, "a group's words and a DID in 32 bits");
inline bool profile_by_group(int64_t rows, int64_t blocks_per_row, int64_t n_groups, int words)
{
    return n_groups <= 512 && rows <= kProfileGroupMaxRows && rows * n_groups <= (1 << 23) && blocks_per_row * (2 * words + 7) <= 400 * words;
}
constexpr int kProfileGroupThreads = 1024;
// Lane 31 of each half-wavefront gets the half's values put together (exchanges inside the vector ALU: no LDS round trips).
template <typename Op>
__device__ __forceinline__ uint32_t half_wave(uint32_t v, Op op, uint32_t neutral)
{
    auto moved = [neutral](uint32_t x, auto ctrl) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)neutral, (int)x, decltype(ctrl)::value, 0xF, 0xF, false);
    };
    v = op(v, moved(v, std::integral_constant<int, 0xB1>{}));     // quad_perm [1,0,3,2]
    v = op(v, moved(v, std::integral_constant<int, 0x4E>{}));     // quad_perm [2,3,0,1]
    v = op(v, moved(v, std::integral_constant<int, 0x141>{}));    // row_half_mirror
    v = op(v, moved(v, std::integral_constant<int, 0x140>{}));    // row_mirror
    return op(v, moved(v, std::integral_constant<int, 0x142>{})); // row_bcast:15, the row before this one
}
constexpr uint32_t kProfileGroupRows = 16384;   // per look

template <int kWords>
__global__ __launch_bounds__(kProfileGroupThreads) void profile_group_kernel(const uint16_t* meta, uint32_t rows, uint32_t nb,
                                                                             const int32_t* anchor_group, const uint8_t* blob,
                                                                             uint32_t* counts, uint8_t* sub)
{
    __shared__ uint32_t hist[32][64];
    __shared__ uint16_t list[kProfileGroupRows];
    __shared__ uint32_t n_list, total[32];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, g = blockIdx.x;
    const uint32_t d = tid & 31u;
    const int n_dialects = *reinterpret_cast<const int32_t*>(blob + kOffCount);
    const uint32_t top = blob[kOffTop + d];
    for (uint32_t i = tid; i < 32 * 64; i += kProfileGroupThreads) hist[0][i] = 0;
    auto add = [&](uint32_t word) {
        const uint32_t did = word & 0xFFu;
        if (did < 32u) atomicAdd(&hist[did][lane], 1u);
    };
    for (uint32_t row0 = 0; row0 < rows; row0 += kProfileGroupRows) {
        constexpr uint32_t kRead = kProfileGroupRows / kProfileGroupThreads;
        int32_t group[kRead];
#pragma unroll
        for (uint32_t k = 0; k < kRead; ++k) group[k] = anchor_group[min(row0 + tid + k * kProfileGroupThreads, rows - 1u)];
        if (tid == 0) n_list = 0;
        __syncthreads();
        // this thread's anchors as bits, then one place in the list for all of them
        uint32_t mine = 0;
#pragma unroll
        for (uint32_t k = 0; k < kRead; ++k) mine |= (uint32_t)group[k] == g ? 1u << k : 0u;   // (g < 2^31: a negative entry is none)
        const uint32_t n = rows - row0;
        mine &= n < kProfileGroupRows ? (1u << ((n + kProfileGroupThreads - 1u - min(tid, n)) / kProfileGroupThreads)) - 1u : 0xFFFFu;
        // Many anchors (wave-uniform): the wavefront's places at once, in the order of the rows, so that neighbours in the list are
        // neighbours in memory.  That takes a step per row of a thread; an atomic per thread takes one per thread with an anchor, and is
        // the shorter one up to two threads per row of a thread (2.75: the same).  400 shapes, 50 to 32768 rows, 1 to 64 groups, a tenth
        // to all of the rows anchors, against a ballot and an atomic for every row of a thread: 0.855 of the time on average, none
        // slower; with the line at 32 threads of which one has three anchors 0.925, up to 1.49 (1471 x 96, one group, all rows
        // anchors, us: 12.1, 14.7 with that line, 11.5 with this).
        const uint32_t n_read = min(kRead, (n + kProfileGroupThreads - 1u) / kProfileGroupThreads);
        if ((uint32_t)__builtin_popcountll(__ballot(mine != 0u)) > 2u * n_read) {
            uint32_t anchors = 0;
#pragma unroll 1
            for (uint32_t k = 0; k < n_read; ++k) anchors += (uint32_t)__builtin_popcountll(__ballot((mine >> k) & 1u));
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&n_list, anchors);
            at = __builtin_amdgcn_readfirstlane(at);
            uint32_t row = tid;
#pragma unroll 1
            for (uint32_t k = 0; k < n_read; ++k) {
                const bool is = mine & 1u;
                const unsigned long long m = __ballot(is);
                if (is) list[at + __builtin_popcountll(m & ((1ull << lane) - 1ull))] = (uint16_t)row;
                at += (uint32_t)__builtin_popcountll(m);
                row += kProfileGroupThreads;
                mine >>= 1;
            }
        } else if (mine) {
            uint32_t at = atomicAdd(&n_list, (uint32_t)__builtin_popcount(mine));
            do {
                list[at++] = (uint16_t)(tid + (uint32_t)__builtin_ctz(mine) * kProfileGroupThreads);
                mine &= mine - 1u;
            } while (mine);
        }
        __syncthreads();
        const uint32_t per_row = nb / kWords, items = n_list * per_row;   // (the launcher bounds rows * nb)
#pragma unroll 2
        for (uint32_t i = tid; i < items; i += kProfileGroupThreads) {
            const uint32_t r = i / per_row;
            const uint16_t* at = meta + ((size_t)row0 + list[r]) * nb + (size_t)(i - r * per_row) * kWords;
            if constexpr (kWords == 1) {
                add(*at);
            } else {
                typedef uint32_t words __attribute__((ext_vector_type(kWords / 2)));
                const words v = *reinterpret_cast<const words*>(at);
#pragma unroll
                for (int j = 0; j < kWords / 2; ++j) { add(v[j]); add(v[j] >> 16); }
            }
        }
        __syncthreads();
    }
    {
        uint32_t c = hist[tid >> 5][d] + hist[tid >> 5][d + 32u];
        c = half_wave(c, [](uint32_t a, uint32_t b) { return a + b; }, 0u);
        if (d == 31) {
            total[tid >> 5] = c;
            counts[(size_t)g * 32 + (tid >> 5)] = c;
        }
    }
    __syncthreads();
    if (tid < 256) {   // 32 lanes per range bucket: the most frequent dialect, lowest DID on ties
        const bool in = (int)d < n_dialects && top == 8u + (tid >> 5);
        uint32_t key = in ? ((total[d] + 1u) << 5) | (31u - d) : 0u;   // (fits: see profile_by_group)
        key = half_wave(key, [](uint32_t a, uint32_t b) { return max(a, b); }, 0u);
        if (d == 31) sub[(size_t)g * 8 + (tid >> 5)] = key ? (uint8_t)(31u - (key & 31u)) : 255u;
    }
}

}  // namespace fb4
