// SeDA sub-formatbook construction (Sec. 3.4, "Constructing an 8-Dialect
// Sub-Formatbook"): count how often each dialect was selected on the anchor
// tokens of each group, then keep, per dynamic-range bucket (largest magnitude
// 8..15), the most frequently selected dialect of that bucket.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

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
                                                                        int n_groups, uint32_t* counts)
{
    __shared__ uint32_t hist[kProfileThreads / 64][32];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long stride = (long long)gridDim.x * (kProfileThreads / 64);
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

// All of it in one launch, a workgroup per group: looks through all rows for the group's anchors, counts theirs in LDS
// and picks the group's dialects.  No counter has to be cleared by a launch of its own and nothing is added up across
// workgroups; the price is that every workgroup reads anchor_group, and that one workgroup counts all of a group's
// rows.  Where 6 % of the rows are anchors (us, three launches against this one): 16384 rows x 96 blocks, 64 groups
// 9.0 and 7.3, 200 groups 9.4 and 7.1; 32768 rows, 64 groups 10.0 and 9.7, 256 groups 10.0 and 9.1; 1000 rows, 20 groups
// 7.8 and 5.7; 65536 rows x 36, 64 groups 11.2 and 12.8; half of 16384 rows in 8 groups 26.9 and 26.2, all of them in
// one group 193 and 241.  Behind the launch that writes anchor_group (cold caches) 12.8 and 12.1.  So: a few groups at least, and limits on the rows and on what is read in all.
constexpr int kProfileGroupThreads = 1024;
inline bool profile_in_one_launch(long long rows, long long nb, int n_groups)
{
    return n_groups >= 8 && rows <= 32768 && rows * n_groups <= (1ll << 23) && rows * nb <= (1ll << 22);
}

__global__ __launch_bounds__(kProfileGroupThreads) void profile_group_kernel(const uint16_t* meta, long long rows, long long nb,
                                                                             const int32_t* anchor_group, const uint8_t* blob,
                                                                             uint32_t* counts, uint8_t* sub)
{
    constexpr int kRead = 8;   // rows per thread and round, all in flight
    constexpr int kWaves = kProfileGroupThreads / 64;
    __shared__ uint32_t hist[kWaves][32];   // one histogram per wavefront
    __shared__ uint32_t total[32], top[33];   // top[32]: number of dialects
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quarter = lane >> 4;
    const int g = blockIdx.x;
    uint32_t tv = 0;
    if (threadIdx.x < 32) tv = blob[kOffTop + threadIdx.x];
    else if (threadIdx.x == 32) tv = *reinterpret_cast<const uint32_t*>(blob + kOffCount);
    if (lane < 32) hist[wave][lane] = 0;
    __builtin_amdgcn_wave_barrier();
    for (long long r0 = 0; r0 < rows; r0 += (long long)kProfileGroupThreads * kRead) {
        int32_t at[kRead];
#pragma unroll
        for (int j = 0; j < kRead; ++j) {
            const long long r = r0 + (long long)j * kProfileGroupThreads + threadIdx.x;
            at[j] = anchor_group[r < rows ? r : rows - 1];
            if (r >= rows) at[j] = -1;
        }
#pragma unroll
        for (int j = 0; j < kRead; ++j) {
            unsigned long long found = __ballot(at[j] == g);   // the wavefront's anchors among 64 rows
            const long long first = r0 + (long long)j * kProfileGroupThreads + (threadIdx.x - lane);
            while (found) {
                if ((found & (found - 1)) == 0) {   // one row, the usual case: all lanes
                    const uint16_t* row = meta + (first + __builtin_ctzll(found)) * nb;
                    found = 0;
                    for (long long b = lane; b < nb; b += 64) {
                        const uint32_t did = row[b] & 0xFFu;
                        if (did < 32u) atomicAdd(&hist[wave][did], 1u);
                    }
                    continue;
                }
                int mine = -1;   // several: four at a time, 16 lanes each
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    if (found && quarter == k) mine = (int)__builtin_ctzll(found);
                    found &= found - 1;   // (zero stays zero)
                }
                if (mine >= 0) {
                    const uint16_t* row = meta + (first + mine) * nb;
                    for (long long b0 = lane & 15u; b0 < nb; b0 += 16 * 8) {
                        uint32_t did[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) did[i] = row[b0 + 16 * i < nb ? b0 + 16 * i : nb - 1] & 0xFFu;
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (b0 + 16 * i < nb && did[i] < 32u) atomicAdd(&hist[wave][did[i]], 1u);
                    }
                }
            }
        }
    }
    if (threadIdx.x <= 32) top[threadIdx.x] = tv;   // (its load was on its way with the rows')
    __syncthreads();
    if (threadIdx.x < 32) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) c += hist[w][threadIdx.x];
        total[threadIdx.x] = c;
        counts[(size_t)g * 32 + threadIdx.x] = c;
    }
    __syncthreads();
    if (threadIdx.x < 8) {   // range bucket threadIdx.x: as profile_select_kernel
        uint32_t best = 255u, best_count = 0;
#pragma unroll
        for (uint32_t d = 0; d < 32; ++d) {
            if (d < top[32] && top[d] == 8u + threadIdx.x && (best == 255u || total[d] > best_count)) { best = d; best_count = total[d]; }
        }
        sub[(size_t)g * 8 + threadIdx.x] = (uint8_t)best;
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

}  // namespace fb4
