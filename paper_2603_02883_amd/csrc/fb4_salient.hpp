// Attention-guided salient tokens (Sec. 3.3, App. F): the rows that the
// activation decomposition gives a second plane are, per tile of tokens, the one
// whose query attends most strongly on average -- the mean over the keys of
// its attention group of |Q.K^T| (spatial / 3D attention) or max(Q.K^T, 0)
// (temporal attention), pre-softmax.
//
// The scores are the one dense contraction of this library and run on the matrix
// cores: 32x32x16 bf16 MFMAs with fp32 accumulation computing S^T = K Q^T -- transposed
// so that a lane's 16 accumulators are 16 keys of ONE query: |.| or max(., 0)
// and the sum over keys then stay inside the lane, and the two half-wavefronts
// are only added up once at the very end.  Three kernels: groups of up to 64 tokens
// (attention_scores_short_kernel), longer ones with rows of up to 128 channels
// (attention_scores_dma_kernel) and of more (attention_scores_kernel).
//
// select_salient_kernel: per frame the head mean (in double, head by head), the
// best token of every tile (lowest index on ties, a NaN never wins), and the
// chosen tokens as ascending row numbers of the [frames * tokens] tensor.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

namespace fb4 {

typedef __bf16 mfma_bf16x8 __attribute__((ext_vector_type(8)));
typedef float mfma_f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t lds_u32x4 __attribute__((ext_vector_type(4)));

constexpr int kScoreThreads = 256;

// Workgroups are dealt to the eight XCDs in turn, and each XCD has its own L2.  The workgroups of one attention
// group read the same keys, so they should share an L2: workgroup b works on position (b % 8) * (n / 8) + b / 8
// of the launch, which puts consecutive positions on one XCD (the last n % 8 workgroups keep their own number).
__device__ __forceinline__ uint32_t xcd_local_position(uint32_t b, uint32_t n)
{
    const uint32_t chunk = n / 8u;
    return b < chunk * 8u ? (b % 8u) * chunk + b / 8u : b;
}
constexpr uint32_t kScoreShortGroup = 64;   // tokens of a short group at most

// A workgroup of four wavefronts takes 128 * kScoreQB queries of one group; every wavefront keeps its queries as B
// operands in registers for the whole pass and walks over the group's keys kScoreKeys at a time: the key block goes
// through LDS once for the four wavefronts (rows padded by 16 bytes so that the 16-byte operand reads of the 16 lanes
// of a pass fall into 16 different bank groups).  Long groups with rows of more than 128 channels: 64 queries per
// wavefront and 64 keys per barrier; short groups (scores_short_in_one_wave says which): 32 and 32.
// D32: channels / 32, rounded up (channels beyond `dim` are zero on both sides).  kRelu: max(., 0), else |.|.
// kScoreQB: blocks of 32 queries per wavefront; kScoreKeys: keys per barrier (a multiple of 32).
template <int D32, bool kRelu, int kScoreQB, int kScoreKeys>
__global__ __launch_bounds__(kScoreThreads) void attention_scores_kernel(const uint16_t* q, const uint16_t* k,
                                                                         uint32_t tokens, uint32_t dim,
                                                                         uint32_t blocks_per_group, uint32_t n_workgroups, float* scores)
{
    constexpr int kScoreQueries = 128 * kScoreQB;    // per workgroup
    constexpr int kSteps = D32 * 2;                  // MFMA steps of 16 channels
    constexpr int kRowBytes = D32 * 64 + 16;         // one key row in LDS: channels, then 16 bytes of padding
    __shared__ __align__(16) uint8_t lds[2][kScoreKeys * kRowBytes];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t pos = xcd_local_position(blockIdx.x, n_workgroups);
    const uint32_t g = pos / blocks_per_group;
    const uint32_t q0 = (pos - g * blocks_per_group) * kScoreQueries + wave * (32u * kScoreQB);
    const uint16_t* qg = q + (size_t)g * tokens * dim;
    const uint16_t* kg = k + (size_t)g * tokens * dim;
    const uint32_t half = lane >> 5, col = lane & 31u;

    // ---- this wavefront's queries as B operands: lane holds query q0 + lane % 32, channels 16 s + 8 (lane / 32) ..
    // (a query past the end reads the last one; a channel past `dim` is zero)
    mfma_bf16x8 qf[kScoreQB][kSteps];
#pragma unroll
    for (int b = 0; b < kScoreQB; ++b) {
        const uint16_t* row = qg + (size_t)min(q0 + 32u * b + col, tokens - 1u) * dim;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const uint32_t c = 16u * s + 8u * half;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (c + 8u <= dim) v = *reinterpret_cast<const uint4*>(row + c);   // dim is a multiple of 8
            qf[b][s] = __builtin_bit_cast(mfma_bf16x8, v);
        }
    }
    // ---- key blocks: 32 keys x dim channels; thread t stages 16-byte pieces t, t + 256, ...
    constexpr int kPiecesPerRow = D32 * 4;           // 16-byte pieces of a padded row's channel part
    constexpr int kPieces = kScoreKeys * kPiecesPerRow;
    constexpr int kPerThread = (kPieces + kScoreThreads - 1) / kScoreThreads;
    uint4 stage[kPerThread];
    auto fetch = [&](uint32_t kb) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const uint32_t piece = threadIdx.x + i * kScoreThreads;
            const uint32_t r = piece / kPiecesPerRow, c8 = (piece - r * kPiecesPerRow) * 8u;   // key row, first channel
            const uint32_t key = kb * kScoreKeys + r;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (piece < (uint32_t)kPieces && key < tokens && c8 + 8u <= dim)
                v = *reinterpret_cast<const uint4*>(kg + (size_t)key * dim + c8);
            stage[i] = v;
        }
    };
    auto deposit = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const uint32_t piece = threadIdx.x + i * kScoreThreads;
            const uint32_t r = piece / kPiecesPerRow, cb = (piece - r * kPiecesPerRow) * 16u;
            if (piece < (uint32_t)kPieces) {
                *reinterpret_cast<uint4*>(&lds[buf][r * kRowBytes + cb]) = stage[i];
            }
        }
    };
    const uint32_t n_kb = (tokens + kScoreKeys - 1) / kScoreKeys;
    fetch(0);
    deposit(0);
    __syncthreads();
    float sum[kScoreQB];   // over this lane's keys of f(S[query][key])
#pragma unroll
    for (int b = 0; b < kScoreQB; ++b) sum[b] = 0.0f;
    for (uint32_t kb = 0; kb < n_kb; ++kb) {
        const int buf = kb & 1;
        if (kb + 1 < n_kb) fetch(kb + 1);
#pragma unroll
        for (int kk = 0; kk < kScoreKeys / 32; ++kk) {   // 32 keys at a time
            mfma_f32x16 acc[kScoreQB];
#pragma unroll
            for (int b = 0; b < kScoreQB; ++b) acc[b] = mfma_f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                // A operand: key row lane % 32 of the 32 keys, channels 16 s + 8 (lane / 32) ..; one read feeds the
                // MFMAs of all the wavefront's query blocks (with one block per read the kernel is bound by LDS bandwidth)
                const uint4 a = *reinterpret_cast<const uint4*>(&lds[buf][(kk * 32 + col) * kRowBytes + s * 32 + half * 16]);
#pragma unroll
                for (int b = 0; b < kScoreQB; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(mfma_bf16x8, a), qf[b][s], acc[b], 0, 0, 0);
            }
#pragma unroll
            for (int b = 0; b < kScoreQB; ++b) {
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[b] += kRelu ? fmaxf(acc[b][r], 0.0f) : fabsf(acc[b][r]);
            }
        }
        if (kb + 1 < n_kb) deposit(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < kScoreQB; ++b) {
        const float total = sum[b] + __shfl_xor(sum[b], 32);   // the two half-wavefronts hold different keys of the same query
        const uint32_t qi = q0 + 32u * b + col;
        if (half == 0 && qi < tokens) scores[(size_t)g * tokens + qi] = total / (float)tokens;
    }
}

// Long groups of up to 128 channels: four blocks of 32 queries per wavefront (80 to 96 channels: six), so that one 16-byte
// operand read from LDS feeds as many MFMAs.  Channels are taken in steps of 16, not padded to 32: 72 channels are 5 steps.
// kP: 16-byte pieces per row (dim / 8).  Queries as B operands (16 registers per step) and four accumulator blocks
// leave no room to stage key blocks through registers: `global_load_lds_dwordx4` writes a wavefront's 64 x 16 bytes
// straight into LDS.  Those 1 KiB land contiguously, so rows cannot be padded; instead piece p of key row r sits at
// position p ^ ((r / (16 / G)) % G) of its row, G = gcd(kP, 16) (the load fetches the matching piece of global
// memory), which spreads the 16 rows that the lanes of one LDS pass read over all 64 banks.  With an odd kP the upper
// half of the last step lies past the row: its lanes read a zeroed piece behind the buffer.
// A workgroup of four wavefronts takes up to 2 * blocks_per_wave blocks of queries: wavefront w holds those of set
// w % 2 and walks the keys of half w / 2 of the group, 64 per barrier, from that half's own double-buffered LDS
// region; the two halves' sums meet in LDS at the end (always half 0 + half 1).  Queries that do not fill a workgroup
// are taken by one short workgroup per group; those are the last of the launch, so that they fill up its end.
// Measured (us in a graph; before: every row through registers into padded LDS rows, channels padded to 32, two MFMAs per
// operand read): 272 groups x 1350 tokens x 72 channels 120 -> 66 (71.4 GFLOP: 1.07 PFLOP/s), 64 channels 81 -> 58,
// 300 x 1000 x 96 74 -> 53, 300 x 1000 x 40 43 -> 28; 384 x 1024 x 128, which had a kernel of this kind, 88 -> 86.
// Then the sums of a block of queries moved beside the next block's MFMAs, and up to six blocks for 80 to 96 channels: 16 x
// 2000 x 72 12.6 -> 11.7, 8 x 8000 x 64 61.5 -> 55.4, 1000 x 300 x 96 30.3 -> 24.3, 12 x 16000 x 96 436 -> 403; 272 x 1350 x
// 72 67.4 -> 66.7, 384 x 1024 x 128 83.5 -> 82.5: full launches on ordinary data are held by the power limit, not by the
// schedule (2176 x 1350 x 72 510 us, the same on zeros 385).
constexpr int dma_max_blocks(int pieces) { return pieces >= 10 && pieces <= 12 ? 6 : 4; }   // of 32 queries per wavefront
constexpr int kDmaKeys = 64;               // per barrier and half
constexpr int kDmaMaxPieces = 16;
// Wavefronts per SIMD: three where 168 registers hold the kernel (up to 72 channels; 272 groups x 1350 tokens x 72, inputs
// changing: 76.6 us with two when all sums followed all MFMAs, 70.5 with three), else two, with up to six blocks of
// queries for 80 to 96 channels.
constexpr int dma_waves(int pieces) { return pieces <= 9 ? 3 : 2; }
// An operand of the next 32 keys is read right behind the last MFMA that uses the present one; 65 to 72 channels on three
// wavefronts per SIMD have no registers for that with more than two blocks of queries (14 would spill): theirs are read between
// two runs of 32 keys (with one or two blocks as well, 24 x 1000 x 72 took 7.1 us, now 6.9, and 16 x 1350 8.9 and 8.7).
constexpr bool dma_reads_early(int pieces) { return pieces != 9; }

template <int kP, bool kRelu>
__global__ __launch_bounds__(kScoreThreads) __attribute__((amdgpu_waves_per_eu(dma_waves(kP), dma_waves(kP))))
void attention_scores_dma_kernel(const uint16_t* q, const uint16_t* k, uint32_t groups, uint32_t tokens, uint32_t n_full,
                                 uint32_t blocks_per_wave, float* scores)
{
    constexpr int kSteps = (kP + 1) / 2;
    constexpr uint32_t kRowBytes = kP * 16;
    constexpr uint32_t kHalfBytes = kDmaKeys * kRowBytes;
    constexpr uint32_t kG = kP % 16 == 0 ? 16 : kP % 8 == 0 ? 8 : kP % 4 == 0 ? 4 : kP % 2 == 0 ? 2 : 1;
    // Two buffers per key half, as two arrays: the compiler then sees that the loads into one do not touch the
    // operand reads from the other and does not wait for them.
    __shared__ __align__(1024) uint8_t lds_a[2 * kHalfBytes + 16];   // [half], even steps; zeros
    __shared__ __align__(1024) uint8_t lds_b[2 * kHalfBytes + 16];   // [half], odd steps; zeros
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t qset = wave & 1u, kh = wave >> 1;
    const uint32_t n_blk = (tokens + 31u) / 32u;
    // ---- this workgroup's blocks of queries
    uint32_t g, first, cnt;
    if (blockIdx.x < groups * n_full) {
        const uint32_t pos = xcd_local_position(blockIdx.x, groups * n_full);
        g = pos / n_full;
        first = (pos - g * n_full) * 2u * blocks_per_wave;
        cnt = 2u * blocks_per_wave;
    } else {
        g = blockIdx.x - groups * n_full;
        first = n_full * 2u * blocks_per_wave;
        cnt = n_blk - first;
    }
    const uint32_t cnt0 = (cnt + 1u) / 2u;
    first += qset ? cnt0 : 0u;
    cnt = qset ? cnt - cnt0 : cnt0;
    // ---- this wavefront's keys: half 0 takes whole steps, half 1 the rest (at most as many steps)
    const uint32_t n_steps = (n_blk + 3u) / 4u;
    const uint32_t key_first = kh ? n_steps * kDmaKeys : 0u, my_steps = kh ? (n_blk - 2u * n_steps + 1u) / 2u : n_steps;
    const uint16_t* qg = q + (size_t)g * tokens * (kP * 8);
    const uint8_t* kg = reinterpret_cast<const uint8_t*>(k + (size_t)g * tokens * (kP * 8));
    const uint32_t half = lane >> 5, col = lane & 31u;

    // Position j (16 bytes) of a half's 64 rows: row j / kP.  kP loads of 64 positions, shared by the half's two
    // wavefronts.
    auto fetch = [&](uint32_t step, uint8_t* buffer) {
        if (step >= my_steps) return;
        // (opaque to the optimizer, which would otherwise keep every load's offset in a register of its own: with
        // 72 channels these registers spill, 81 us instead of 70)
        uint32_t l = lane;
        asm volatile("" : "+v"(l));
        const uint32_t key0 = key_first + step * kDmaKeys;
        const uint8_t* base = kg + (size_t)key0 * kRowBytes;   // wave-uniform
        auto piece_of = [&](uint32_t i, uint32_t& row) {   // the row and the piece that belong to load i's position of this lane
            const uint32_t j = 64u * i + l;
            row = j / kP;
            return (j - row * kP) ^ ((row / (16u / kG)) & (kG - 1u));
        };
        if (key0 + kDmaKeys <= tokens) {
#pragma unroll
            for (int i2 = 0; i2 < (kP + 1) / 2; ++i2) {
                const uint32_t i = 2u * i2 + qset;
                if (2 * i2 + 1 >= kP && i >= (uint32_t)kP) break;
                uint32_t row;
                const uint32_t piece = piece_of(i, row);
                const uint8_t* src = base + (row * kP + piece) * 16u;
                const uint32_t dst = __builtin_amdgcn_readfirstlane(kh * kHalfBytes + i * 1024u);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                 (__attribute__((address_space(3))) void*)(buffer + dst), 16, 0, 0);
            }
        } else {
            // the group's last step: zeros instead of the rows past its last key (their products add nothing).  (All of its
            // rows through registers, a load and a wait at a time: 2621 groups x 100 tokens x 128 channels 35.8 us instead of
            // 29.4.)
            const uint32_t valid = (tokens - key0) * kP;   // 16-byte positions
#pragma unroll 1
            for (uint32_t i = valid / 128u * 2u + qset; i < (uint32_t)kP; i += 2) {
                uint32_t zero = 0;
                asm volatile("" : "+v"(zero));   // (four registers for a moment, not for the whole pass)
                if (64u * i + l >= valid) *reinterpret_cast<uint4*>(buffer + kh * kHalfBytes + i * 1024u + l * 16u) = make_uint4(zero, zero, zero, zero);
            }
#pragma unroll 1
            for (uint32_t i = qset; 64u * i < valid; i += 2) {
                uint32_t row;
                const uint32_t piece = piece_of(i, row);
                if (64u * i + l < valid) {   // (a lane that takes no part leaves its 16 bytes alone)
                    const uint8_t* src = base + (row * kP + piece) * 16u;
                    const uint32_t dst = __builtin_amdgcn_readfirstlane(kh * kHalfBytes + i * 1024u);
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                                     (__attribute__((address_space(3))) void*)(buffer + dst), 16, 0, 0);
                }
            }
        }
    };
    // LDS offset of this lane's A operand of step s: key row lane % 32 of the first 32, piece 2 s + lane / 32
    const uint32_t row_at = kh * kHalfBytes + col * kRowBytes, swz = (col / (16u / kG)) & (kG - 1u);
    auto operand = [&](int s, int kk) -> uint32_t {
        const uint32_t at = row_at + ((((uint32_t)(2 * s) + half) ^ swz) << 4) + kk * 32u * kRowBytes;
        return (kP % 2 && s == kSteps - 1 && half) ? 2u * kHalfBytes : at;
    };
    float* meet = reinterpret_cast<float*>(lds_a);               // [query set][32 * dma_max_blocks(kP)]

    auto run = [&](auto blocks) {
        constexpr int NB = decltype(blocks)::value;
        // ---- this wavefront's queries as B operands (a query past the end reads the last one)
        mfma_bf16x8 qf[NB > 0 ? NB : 1][kSteps];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint16_t* row = qg + (size_t)min((first + b) * 32u + col, tokens - 1u) * (kP * 8);
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                uint4 v = make_uint4(0, 0, 0, 0);
                if (!(kP % 2 && s == kSteps - 1) || half == 0) v = *reinterpret_cast<const uint4*>(row + 16u * s + 8u * half);
                qf[b][s] = __builtin_bit_cast(mfma_bf16x8, v);
            }
        }
        float sum[NB > 0 ? NB : 1];
#pragma unroll
        for (int b = 0; b < NB; ++b) sum[b] = 0.0f;
        // Blocks of queries one after the other: the sums of one block's products (vector ALU) are formed while the next
        // block's MFMAs run, and two blocks' accumulators are enough.  `done`: the block whose sums are still to be formed
        // (zeros at first, which add nothing).
        mfma_f32x16 done = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        auto add_up = [&](float& s) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s += kRelu ? fmaxf(done[r], 0.0f) : fabsf(done[r]);
        };
        auto compute = [&](const uint8_t* buffer, uint32_t step) {
            if (NB == 0 || step >= my_steps) return;
            constexpr bool kEarly = dma_reads_early(kP) || NB <= 2;
            mfma_bf16x8 a[kSteps];   // operands of 32 keys
            auto read = [&](int s, int kk) { a[s] = __builtin_bit_cast(mfma_bf16x8, *reinterpret_cast<const uint4*>(buffer + operand(s, kk))); };
#pragma unroll
            for (int kk = 0; kk < kDmaKeys / 32; ++kk) {
                if (!kEarly || kk == 0) {
#pragma unroll
                    for (int s = 0; s < kSteps; ++s) read(s, kk);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const bool last = kEarly && b == NB - 1 && kk + 1 < kDmaKeys / 32;   // (an operand's last use with these keys)
                    mfma_f32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int s = 0; s < kSteps; ++s) {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], qf[b][s], acc, 0, 0, 0);
                        if (last) read(s, kk + 1);
                    }
                    add_up(sum[(b + NB - 1) % (NB > 0 ? NB : 1)]);
                    done = acc;
                    // The order: MFMA, operand read, a share of the sums.  The shares are the sums' instructions and no more: with
                    // room for others the scheduler filled it with this block's own sums, which wait for its MFMAs with no
                    // other block's behind them (us, 20 places / 16: 272 x 1350 x 72 65.3 / 64.9, 16 x 8000 x 72 115.8 / 112.7, 24 x
                    // 1000 x 72 6.84 / 6.55, 15 x 2048 x 112 17.4 / 15.8, 139 x 155 x 56 3.26 / 3.22: sums of |S|; twice the instructions
                    // with a maximum before each: 400 shapes of 65 to 6000 tokens in either mode 0.998 and 0.996 on average, none
                    // slower by more than 2 %).  One block of queries per
                    // wavefront has no other anyway: 20 (1 x 8192 x 96 33.1 / 33.6, 1 x 3600 x 128 19.7 / 20.0).
                    constexpr int kOps = kRelu ? 32 : 16, kParts = kSteps > 1 ? kSteps - 1 : 1, kEach = kOps / kParts;
                    constexpr int kFirst = NB == 1 ? (16 + kSteps - 1) / kSteps + 1 : kOps - kEach * (kParts - 1), kRest = NB == 1 ? kFirst : kEach;
#pragma unroll
                    for (int s = 0; s < kSteps; ++s) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        if (last) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                        if (s == (kSteps > 1 ? 1 : 0)) __builtin_amdgcn_sched_group_barrier(0x002, kFirst, 0);
                        else if (s > 1) __builtin_amdgcn_sched_group_barrier(0x002, kRest, 0);
                    }
                    if (kEarly) __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the first step's keys are in LDS
        __syncthreads();
        for (uint32_t step = 0; step < n_steps; step += 2) {
            if (step + 1 < n_steps) fetch(step + 1, lds_b);
            compute(lds_a, step);
            __builtin_amdgcn_s_waitcnt(0x0F70);   // the next step's keys have landed before anyone reads them
            __syncthreads();
            if (step + 1 < n_steps) {
                if (step + 2 < n_steps) fetch(step + 2, lds_a);
                compute(lds_b, step + 1);
                __builtin_amdgcn_s_waitcnt(0x0F70);
                __syncthreads();
            }
        }
        if (NB > 0) add_up(sum[NB > 0 ? NB - 1 : 0]);
        // ---- the two key halves meet: half 1 through LDS, then half 0 + half 1
#pragma unroll
        for (int b = 0; b < NB; ++b) sum[b] += __shfl_xor(sum[b], 32);   // the two half-wavefronts hold different keys
        if (kh == 1 && half == 0) {
#pragma unroll
            for (int b = 0; b < NB; ++b) meet[qset * (32u * dma_max_blocks(kP)) + 32u * b + col] = sum[b];
        }
        __syncthreads();
        if (kh == 0 && half == 0) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint32_t qi = (first + b) * 32u + col;
                if (qi < tokens) scores[(size_t)g * tokens + qi] = (sum[b] + meet[qset * (32u * dma_max_blocks(kP)) + 32u * b + col]) / (float)tokens;
            }
        }
    };
    fetch(0, lds_a);
    if (kP % 2 && threadIdx.x < 8) {   // the zeroed pieces
        reinterpret_cast<uint32_t*>((threadIdx.x & 4u ? lds_b : lds_a) + 2 * kHalfBytes)[threadIdx.x & 3u] = 0;
    }
    // (wave-uniform; every path meets the same barriers)
    switch (cnt) {
    case 0: run(std::integral_constant<int, 0>{}); break;
    case 1: run(std::integral_constant<int, 1>{}); break;
    case 2: run(std::integral_constant<int, 2>{}); break;
    case 3: run(std::integral_constant<int, 3>{}); break;
    case 5: if constexpr (dma_max_blocks(kP) > 4) run(std::integral_constant<int, 5>{}); break;
    case 6: if constexpr (dma_max_blocks(kP) > 4) run(std::integral_constant<int, 6>{}); break;
    default: run(std::integral_constant<int, 4>{}); break;
    }
}

// Short groups (temporal attention: a group is a handful of frames), bound by memory: Q and K are read once and a
// float per row comes back.  A wavefront takes kNB blocks of 32 rows at a time -- as many whole groups as fit 32
// rows (kNB = 1), or one group of 33 to 64 rows (kNB = 2); the tensors are contiguous, so those rows are one run of
// memory -- loads them straight into LDS of its own (pieces placed as in the kernel above), forms all products of the
// 32 queries with the 32 keys on the matrix cores and adds up those whose key lies in the query's group.  Nothing is
// shared between wavefronts, so there are no barriers; a wavefront requests the rows of its next task as soon as
// it has read its operands.  kP: 16-byte pieces per row; every row length is compiled, because dividing each load's
// position by a number not known before costs more than the products (8 groups x 32 tokens x 112 channels 3.34 us so, 2.73
// compiled; 16384 x 16 x 80 14.5 and 13.8).
// Measured (us; before: the first kernel above): 24576 groups x 16 tokens x 128 channels 53 -> 35.4 (5.7 TB/s), x 72
// channels 39 -> 20.5, 12000 x 21 x 64 15.2 -> 11.4, 6000 x 40 x 128 26.5 -> 23.9, 100000 x 4 x 64 95 -> 18.8.
// Which of the two: up to 32 tokens this one, except where the rows of five wavefronts fill a compute unit's LDS (8192 x
// 32 x 256: 44.2 against 37.8; with six, 13107 x 20 x 256: 40.0 against 45.7).  From 33 tokens on one wavefront's chain
// of loads and products is longer than four wavefronts' in the first kernel, and only many groups hide it (40 tokens x
// 72 channels, 6 / 409 / 1638 / 6553 groups: 3.4 / 3.6 / 4.4 / 14.9 us against 3.0 / 3.4 / 5.8 / 17.4), the less the
// fuller its two blocks of 32 are (4681 x 56 x 112: 20.7 against 18.7) and not for rows of more than 128 channels
// (5461 x 48 x 160: 29.2 against 26.7).
inline bool scores_short_in_one_wave(int64_t groups, int64_t tokens, int64_t dim, uint32_t waves_per_cu)
{
    if (tokens <= 32) return waves_per_cu > 5;
    return tokens <= 48 && dim <= 128 && groups >= 1024;
}
__host__ __device__ constexpr uint32_t short_region_bytes(uint32_t rows, uint32_t pieces)   // of one matrix: whole loads
{
    return (rows * pieces + 63u) / 64u * 1024u;
}
__host__ __device__ constexpr uint32_t short_wave_bytes(uint32_t rows, uint32_t pieces)
{
    return 2u * short_region_bytes(rows, pieces) + (pieces & 1u) * 16u;
}

template <int kP, int kNB>
__global__ __launch_bounds__(kScoreThreads) void attention_scores_short_kernel(const uint16_t* q, const uint16_t* k,
                                                                               uint32_t n_rows, uint32_t tokens,
                                                                               uint32_t rows_per_task, uint32_t n_tasks,
                                                                               uint32_t relu, uint32_t n_waves, uint32_t n_workgroups,
                                                                               float* scores)
{
    extern __shared__ __align__(1024) uint8_t short_lds[];
    constexpr uint32_t P = kP;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t half = lane >> 5, col = lane & 31u;
    constexpr uint32_t g_log = (uint32_t)__builtin_ctz(P | 16u);   // log2 of gcd(P, 16)
    const uint32_t region = short_region_bytes(rows_per_task, P);
    const uint32_t base = wave * short_wave_bytes(rows_per_task, P);
    uint8_t* lq = short_lds + base;
    uint8_t* lk = lq + region;
    if ((P & 1u) && lane < 4) reinterpret_cast<uint32_t*>(lk + region)[lane] = 0;   // the zeroed piece of an odd row's last step
    const uint8_t* qb = reinterpret_cast<const uint8_t*>(q);
    const uint8_t* kb = reinterpret_cast<const uint8_t*>(k);

    auto fetch = [&](uint32_t task) {
        const uint32_t row0 = task * rows_per_task;                          // wave-uniform
        const uint32_t n = min(rows_per_task, n_rows - row0);
        const uint8_t* q0 = qb + (size_t)row0 * (P * 16u);
        const uint8_t* k0 = kb + (size_t)row0 * (P * 16u);
#pragma unroll 4
        for (uint32_t i = 0; i * 64u < n * P; ++i) {
            const uint32_t j = 64u * i + lane, row = min(j / P, n - 1u);         // (past the last row: that row again)
            const uint32_t piece = (j % P) ^ ((row >> (4u - g_log)) & ((1u << g_log) - 1u));
            const uint32_t off = (row * P + piece) * 16u;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(k0 + off),
                                             (__attribute__((address_space(3))) void*)(lk + i * 1024u), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(q0 + off),
                                             (__attribute__((address_space(3))) void*)(lq + i * 1024u), 16, 0, 0);
        }
    };
    constexpr uint32_t steps = (P + 1u) / 2u;
    // this lane's 16 bytes of step s of row 32 b + lane % 32 (past the task's rows: of its last row; nobody uses the result)
    auto operand = [&](const uint8_t* m, uint32_t b, uint32_t s) {
        const uint32_t row = min(b * 32u + col, rows_per_task - 1u);
        const uint32_t swz = (row >> (4u - g_log)) & ((1u << g_log) - 1u);
        const uint32_t at = (row * P + ((2u * s + half) ^ swz)) * 16u;
        const bool past = (P & 1u) && s + 1u == steps && half;
        return __builtin_bit_cast(mfma_bf16x8, *reinterpret_cast<const uint4*>(past ? lk + region : m + at));
    };
    // a query's group: keys lo .. lo + tokens - 1 of the task's rows
    const uint32_t lo = kNB == 1 ? (col / tokens) * tokens : 0u;
    const float n_keys = (float)tokens;
    const uint32_t stride = n_workgroups * n_waves;
    uint32_t task = blockIdx.x * n_waves + wave;
    if (task >= n_tasks) return;
    fetch(task);
    while (true) {
        const uint32_t next = task + stride;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the task's rows are in LDS
        float sum[kNB];
#pragma unroll
        for (int b = 0; b < kNB; ++b) sum[b] = 0.0f;
        auto add_up = [&](const mfma_f32x16& acc, int keys, float& s) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                // accumulator r belongs to key 8 (r / 4) + 4 (lane / 32) + r % 4 of the block
                const float v = relu ? fmaxf(acc[r], 0.0f) : fabsf(acc[r]);
                s += (32u * keys + 8u * (r / 4) + 4u * half + (r % 4) - lo < tokens) ? v : 0.0f;
            }
        };
        auto refill = [&]() {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every operand of this task has been read
            if (next < n_tasks) fetch(next);
        };
        if constexpr (kNB == 1) {
            mfma_bf16x8 a[steps], bq[steps];
#pragma unroll
            for (uint32_t s = 0; s < steps; ++s) { a[s] = operand(lk, 0, s); bq[s] = operand(lq, 0, s); }
            refill();
            mfma_f32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (uint32_t s = 0; s < steps; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], bq[s], acc, 0, 0, 0);
            add_up(acc, 0, sum[0]);
        } else {
            mfma_f32x16 acc[kNB][kNB];
#pragma unroll
            for (int i = 0; i < kNB; ++i) {
#pragma unroll
                for (int b = 0; b < kNB; ++b) acc[i][b] = mfma_f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            }
#pragma unroll 2
            for (uint32_t s = 0; s < steps; ++s) {
                mfma_bf16x8 a[kNB], bq[kNB];
#pragma unroll
                for (int b = 0; b < kNB; ++b) { a[b] = operand(lk, b, s); bq[b] = operand(lq, b, s); }
#pragma unroll
                for (int i = 0; i < kNB; ++i) {
#pragma unroll
                    for (int b = 0; b < kNB; ++b) acc[i][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bq[b], acc[i][b], 0, 0, 0);
                }
            }
            refill();
#pragma unroll
            for (int b = 0; b < kNB; ++b) {
#pragma unroll
                for (int i = 0; i < kNB; ++i) add_up(acc[i][b], i, sum[b]);
            }
        }
        const uint32_t row0 = task * rows_per_task, n = min(rows_per_task, n_rows - row0);
#pragma unroll
        for (int b = 0; b < kNB; ++b) {
            const float total = sum[b] + __shfl_xor(sum[b], 32);   // the two half-wavefronts hold different keys of one query
            if (half == 0 && 32u * b + col < n) scores[(size_t)row0 + 32u * b + col] = total / n_keys;
        }
        if (next >= n_tasks) break;
        task = next;
    }
}

// Diagnostic: the rate at which this device sustains v_mfma_f32_32x32x16_bf16 on operands held in registers -- four
// independent accumulator chains per wavefront, no memory traffic inside the loop -- so that the attention
// kernel's rate can be read against what the matrix cores deliver at the clock the power management allows.
// random != 0: operands with random signs and mantissas (magnitudes in [0.5, 2)), as real activations toggle
// the datapath; random == 0: the same bit pattern in every element.
__global__ __launch_bounds__(256) void probe_mfma_rate_kernel(float* out, uint32_t iters, uint32_t random)
{
    auto word = [&](uint32_t i) {
        uint32_t h = (threadIdx.x * 2654435761u + i * 40503u + blockIdx.x) * 2246822519u;
        h ^= h >> 13;
        h *= 3266489917u;
        h ^= h >> 16;
        return random ? ((h & 0x80FF80FFu) | 0x3F003F00u) : 0x3F803F80u;   // two bf16 per word
    };
    const lds_u32x4 av = {word(1), word(2), word(3), word(4)}, bv = {word(5), word(6), word(7), word(8)};
    const mfma_bf16x8 a = __builtin_bit_cast(mfma_bf16x8, av), b = __builtin_bit_cast(mfma_bf16x8, bv);
    mfma_f32x16 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = mfma_f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (uint32_t i = 0; i < iters; ++i) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[c], 0, 0, 0);
        }
    }
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[c][r];
    }
    out[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}

// A workgroup takes some rows of tiles of a frame: their tokens are one run of memory, their chosen tokens one run of the
// ascending list.  Up to 24 head loads in flight, kLanes lanes per tile.  Bound by its chain of dependent steps -- loads,
// maxima, compaction --, so a few frames are spread over the compute units, one row of tiles each (but 64 tokens at least):
// 16 frames x 24 heads x 1024 tokens 5.1 us with a workgroup per frame, 3.1 so, 128 x 24 x 1350 6.4 and 4.8.  With more frames
// the instructions count and a workgroup takes a frame (256 x 24 x 1350 8.3 against 9.4), also where more threads than twice
// the chip holds would come of the split (128 frames of 90 x 90, tiles of 8 x 8, 9.6 against 18.1), past 384 frames (512 x 24 x
// 13 x 61, 8 x 8, 8.4 against 9.1) and, past 128 frames, where one wavefront takes a frame's tiles at once (256 x 8 x 16 x 16,
// 8 x 8, 3.5 against 3.7): 1024 threads with 16 lanes per tile up to 256 frames, else 256 and a thread per tile, unless one
// round of 16 lanes holds all tiles (1024 frames x 8 heads x 1024 tokens with 1024 x 16 / 256 x 16 / 256 x 1 15.5 / 9.5 / 6.8,
// 1024 x 8 x 256 9.1 / 4.2 / 4.4, 256 x 24 x 1350 7.9 / 11.7 / 9.3).
struct SelectShape { int threads, lanes; int64_t rows; };   // rows: of tiles per workgroup
inline SelectShape select_shape(int64_t frames, int64_t tile_rows, int64_t tile_columns, int64_t tile_tokens, int64_t row_tokens)
{
    const bool wide = tile_tokens > 4;   // 16 lanes per tile
    const int64_t rows = std::min((64 + row_tokens - 1) / row_tokens, tile_rows), n = rows * row_tokens;
    const int threads = n <= 128 ? 128 : n <= 512 ? 256 : 1024;
    const int64_t workgroups = frames * ((tile_rows + rows - 1) / rows);
    const bool one_round = tile_rows * tile_columns * (wide ? 16 : 1) <= 64;   // all tiles of a frame, by one wavefront
    if (workgroups <= 1600 && workgroups * threads <= 1 << 20 &&
        (rows < tile_rows ? frames <= 384 && !(one_round && frames > 128) : frames <= 256))
        return {threads, wide ? 16 : 1, rows};
    if (wide && tile_rows * tile_columns * 16 <= 256) return {256, 16, tile_rows};
    if (wide && frames <= 256) return {1024, 16, tile_rows};   // (256 compute units)
    return {256, 1, tile_rows};
}

// kMany: 24 heads at once.  Large frames with a thread per tile have a variant without, for fewer heads than that (64 frames x 8
// heads x 8100 tokens, tiles of 1 x 1, 27.0 us with and 26.2 without, 24 heads 38.7 and 55.6); elsewhere it costs nothing.
template <int kSelectThreads, int kLanes, int kMaxTokens, bool kMany>
__global__ __launch_bounds__(kSelectThreads) void select_salient_kernel(const float* scores, uint32_t heads,
                                                                        uint32_t grid_h, uint32_t grid_w, uint32_t tile_h,
                                                                        uint32_t tile_w, uint32_t th, uint32_t tw, uint32_t rows_per_workgroup,
                                                                        uint32_t per_frame, uint32_t first_workgroup, int32_t* rows_out)
{
    constexpr uint32_t kWaves = kSelectThreads / 64;
    __shared__ double mean[kMaxTokens];
    __shared__ uint8_t chosen[kMaxTokens];
    __shared__ uint32_t wave_total[kWaves];
    const uint32_t tokens = grid_h * grid_w;
    const uint32_t wg = first_workgroup + blockIdx.x, frame = per_frame == 1 ? wg : wg / per_frame, row0 = (wg - frame * per_frame) * rows_per_workgroup;
    const uint32_t y0 = row0 * tile_h, hh = min(rows_per_workgroup * tile_h, grid_h - y0), n = hh * grid_w;   // tokens of these rows of tiles
    const uint32_t n_tiles = min(rows_per_workgroup, th - row0) * tw;
    const float* sf = scores + (size_t)frame * heads * tokens + (size_t)y0 * grid_w;
    for (uint32_t t = threadIdx.x; t < n; t += kSelectThreads) {
        double m = 0.0;
        uint32_t h = 0;
        auto some = [&](auto count) {   // that many loads in flight, added in head order
            constexpr int N = decltype(count)::value;
            float v[N];
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] = sf[(size_t)(h + j) * tokens + t];
#pragma unroll
            for (int j = 0; j < N; ++j) m += (double)v[j];
            h += N;
        };
        if (kMany) {
            while (h + 24 <= heads) some(std::integral_constant<int, 24>{});
        }
        while (h + 8 <= heads) some(std::integral_constant<int, 8>{});
        while (h < heads) some(std::integral_constant<int, 1>{});
        mean[t] = m / (double)heads;
        chosen[t] = 0;
    }
    __syncthreads();
    const uint32_t part = threadIdx.x % kLanes;
    for (uint32_t tile = threadIdx.x / kLanes; tile < n_tiles; tile += kSelectThreads / kLanes) {
        const uint32_t ty = tile < tw ? 0u : tile / tw, yt = ty * tile_h, x0 = (tile - ty * tw) * tile_w;
        const uint32_t ht = min(tile_h, hh - yt), ww = min(tile_w, grid_w - x0);
        uint32_t best = 0xFFFFFFFFu;
        double best_v = 0.0;
        auto look = [&](uint32_t at) {   // (in ascending order: the first of equals stays)
            double v = mean[at];
            if (v != v) v = -__builtin_inf();
            if (best == 0xFFFFFFFFu || v > best_v) { best = at; best_v = v; }
        };
        if (kLanes == 1) {
            for (uint32_t y = yt; y < yt + ht; ++y)
                for (uint32_t x = x0; x < x0 + ww; ++x) look(y * grid_w + x);
        } else {
            for (uint32_t i = part; i < ht * ww; i += kLanes) look((yt + i / ww) * grid_w + x0 + i % ww);
        }
#pragma unroll
        for (int o = kLanes / 2; o > 0; o >>= 1) {   // (the lanes of a tile stay together)
            const uint32_t at = (uint32_t)__shfl_xor((int)best, o);
            const double v = __shfl_xor(best_v, o);
            // the lowest token on ties
            if (at != 0xFFFFFFFFu && (best == 0xFFFFFFFFu || v > best_v || (v == best_v && at < best))) { best = at; best_v = v; }
        }
        if (part == 0) chosen[best] = 1;   // (tiles are disjoint: no two threads write the same byte)
    }
    __syncthreads();
    // ascending compaction: thread t owns a contiguous run of tokens
    const uint32_t per = (n + kSelectThreads - 1) / kSelectThreads;
    const uint32_t first = min(n, threadIdx.x * per), last = min(n, first + per);
    uint32_t count = 0;
    for (uint32_t t = first; t < last; ++t) count += chosen[t];
    uint32_t incl = count;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = __shfl_up(incl, off);
        if ((int)(threadIdx.x & 63) >= off) incl += v;
    }
    if ((threadIdx.x & 63) == 63) wave_total[threadIdx.x >> 6] = incl;
    __syncthreads();
    uint32_t at = incl - count;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) at += w < (threadIdx.x >> 6) ? wave_total[w] : 0u;
    int32_t* out = rows_out + ((size_t)frame * th + row0) * tw;
    for (uint32_t t = first; t < last; ++t)
        if (chosen[t]) out[at++] = (int32_t)(frame * tokens + y0 * grid_w + t);
}
constexpr uint32_t kSelectMaxTokens = 8192;   // per frame (the head means sit in LDS)

// Sec. 3.4 ("Attention-Guided Semantic Relatedness Extraction"), the marking step: every anchor marks the tokens
// of a window x window (x window_t frames) box around it whose raw attention score from the anchor -- Q[anchor] .
// K[token], averaged over the heads -- exceeds a threshold.  The group of an anchor is the row-major number of the
// spatial tile it lies in (the per-frame candidates of a tile share one sub-formatbook); a token marked by anchors
// of several groups belongs to the highest group number (App. D: the subsequent anchor), an anchor to its own
// group.  Two small launches: the anchors' own groups and -1 elsewhere (seda_prepare_kernel; with many anchors
// seda_fill_kernel and seda_anchor_kernel instead), then the marks -- a maximum on the group number of every token
// that is no anchor (seda_mark_kernel, one workgroup per anchor and frame of the window).  Where one buffer is passed
// for both results its marks are no sign of an anchor: every token is marked then (anchor_group null), and
// seda_anchor_kernel puts the anchors' own groups back at the end.
// Token (frame f, head h, token t) of Q / K sits at ((f * stride_f + h * stride_h) + t) * dim: factorized
// attention [frames][heads][tokens][dim], 3D attention [heads][frames * tokens][dim].
constexpr int kAssignThreads = 256;

__device__ __forceinline__ uint32_t tile_of(uint32_t token, uint32_t grid_w, uint32_t tile_h, uint32_t tile_w)
{
    const uint32_t y = token / grid_w, x = token - y * grid_w;
    return (y / tile_h) * ((grid_w + tile_w - 1) / tile_w) + x / tile_w;
}

// A workgroup writes kPrepareRows rows and looks through all anchors for those among them, eight entries per thread: no
// second launch has to wait for the first.  More anchors cost more than that launch: the whole call with these / with
// seda_fill_kernel and seda_anchor_kernel, 16 frames x 1024 tokens, windows of one token: 1024 anchors 6.9 / 7.8 us, 2048
// 8.5 / 8.8, 3000 10.6 / 9.8, 16384 31.9 / 22.5; 64 x 4096 tokens, 2048 anchors 7.7 / 9.1, 16384 26.1 / 22.9.
constexpr uint32_t kPrepareRows = 1024;
constexpr uint32_t kPrepareMaxAnchors = 2048;

__global__ __launch_bounds__(kAssignThreads) void seda_prepare_kernel(const int32_t* anchors, uint32_t n_anchors, uint32_t n_rows,
                                                                      uint32_t tokens, uint32_t grid_w, uint32_t tile_h,
                                                                      uint32_t tile_w, int32_t* token_group, int32_t* anchor_group)
{
    __shared__ int32_t group[kPrepareRows];
    const uint32_t first = blockIdx.x * kPrepareRows, n = min(kPrepareRows, n_rows - first);
    for (uint32_t i = threadIdx.x; i < kPrepareRows; i += kAssignThreads) group[i] = -1;
    __syncthreads();
    if (n_anchors > 0) {
        constexpr uint32_t kRead = kPrepareMaxAnchors / kAssignThreads;   // entries per thread, all in flight
        int32_t row[kRead];
#pragma unroll
        for (uint32_t j = 0; j < kRead; ++j) row[j] = anchors[min(threadIdx.x + j * kAssignThreads, n_anchors - 1u)];   // (past the end: the last one again)
#pragma unroll
        for (uint32_t j = 0; j < kRead; ++j) {
            const uint32_t at = (uint32_t)row[j] - first;   // (a negative entry lies past any row)
            if (row[j] >= 0 && at < n) group[at] = (int32_t)tile_of((uint32_t)row[j] % tokens, grid_w, tile_h, tile_w);
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kAssignThreads) {
        token_group[first + i] = group[i];
        anchor_group[first + i] = group[i];
    }
}

__global__ __launch_bounds__(kAssignThreads) void seda_fill_kernel(int32_t* a, int32_t* b, uint32_t n)
{
    const uint32_t i = blockIdx.x * (uint32_t)kAssignThreads + threadIdx.x;
    if (i < n) {
        a[i] = -1;
        b[i] = -1;
    }
}

__global__ __launch_bounds__(kAssignThreads) void seda_anchor_kernel(const int32_t* anchors, uint32_t n, uint32_t frames,
                                                                     uint32_t grid_h, uint32_t grid_w, uint32_t tile_h,
                                                                     uint32_t tile_w, int32_t* token_group, int32_t* anchor_group)
{
    const uint32_t i = blockIdx.x * (uint32_t)kAssignThreads + threadIdx.x;
    if (i >= n) return;
    const uint32_t tokens = grid_h * grid_w;
    const int64_t row = anchors[i];
    if (row < 0 || row >= (int64_t)frames * tokens) return;
    const int32_t g = (int32_t)tile_of((uint32_t)row % tokens, grid_w, tile_h, tile_w);
    token_group[row] = g;    // (two entries naming one row write the same value)
    anchor_group[row] = g;
}

struct AssignParams {
    uint32_t frames, heads, grid_h, grid_w, dim, tile_h, tile_w, window, window_t;
    uint64_t stride_f, stride_h;   // in tokens
    float threshold;
};

// Adds up groups of kLanes neighbouring lanes (every lane ends with its group's sum; a fixed order).
template <int kLanes>
__device__ __forceinline__ float group_of_lanes_sum(float v)
{
    auto moved = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    if (kLanes >= 2) v += moved(v, std::integral_constant<int, 0xB1>{});     // quad_perm [1,0,3,2]
    if (kLanes >= 4) v += moved(v, std::integral_constant<int, 0x4E>{});     // quad_perm [2,3,0,1]
    if (kLanes >= 8) v += moved(v, std::integral_constant<int, 0x141>{});    // row_half_mirror
    if (kLanes >= 16) v += moved(v, std::integral_constant<int, 0x140>{});   // row_mirror
    return v;
}

// kLanes lanes share a row of K, 16 bytes each, 64 / kLanes window slots at a time, so that a load covers whole rows (and
// neighbouring slots are neighbouring rows); a wavefront takes every fourth head with the loads of two heads in
// flight, and a lane keeps its channels' sums over its heads: lanes and wavefronts are added up once at the end.
// kWindow: the window's side (slots and their places are then constants).  16 frames x 24 heads x 1024 tokens x 128
// channels, 1024 random anchors, 5 x 5 windows, with the preparation: 45.5 us with a thread per slot, which read its row 16
// bytes at a time, 26.5 so.
template <int kWindow, int kLanes>
__global__ __launch_bounds__(kAssignThreads) void seda_mark_kernel(const uint16_t* q, const uint16_t* k,
                                                                   const int32_t* anchors, AssignParams p,
                                                                   int32_t* token_group, const int32_t* anchor_group,
                                                                   float* scores)
{
    constexpr uint32_t slots = kWindow * kWindow, kRows = 64 / kLanes;
    constexpr int kSteps = (slots + kRows - 1) / kRows;
    __shared__ float partial[kAssignThreads / 64][kSteps * kRows];
    const uint32_t tokens = p.grid_h * p.grid_w;
    const uint32_t i = blockIdx.x, wt = blockIdx.y;
    const int64_t row = anchors[i];
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t sub = lane / kLanes, piece = lane % kLanes;
    const bool anchor_ok = row >= 0 && row < (int64_t)p.frames * tokens;   // otherwise: no token of the clip, marks nothing
    const uint32_t rc = anchor_ok ? (uint32_t)row : 0u;
    const uint32_t fa = rc / tokens, ac = rc - fa * tokens;
    const int32_t ay = (int32_t)(ac / p.grid_w), ax = (int32_t)(ac % p.grid_w);
    const int32_t f = (int32_t)fa + (int32_t)wt - (int32_t)(p.window_t / 2);
    const bool frame_ok = anchor_ok && f >= 0 && f < (int32_t)p.frames;
    if (!frame_ok && !scores) return;   // (the same for the whole workgroup)
    const uint32_t fc = frame_ok ? (uint32_t)f : fa;
    auto place = [&](uint32_t slot, uint32_t& t) {   // the slot's token; false (and the anchor's own) outside the clip
        const int32_t y = ay + (int32_t)(slot / kWindow) - kWindow / 2;
        const int32_t x = ax + (int32_t)(slot % kWindow) - kWindow / 2;
        const bool inside = slot < slots && frame_ok && y >= 0 && y < (int32_t)p.grid_h && x >= 0 && x < (int32_t)p.grid_w;
        t = inside ? (uint32_t)y * p.grid_w + (uint32_t)x : ac;
        return inside;
    };
    float acc[kSteps];
    uint32_t off[kSteps];   // of the slots' rows, in elements (the launcher checks tokens * dim < 2^31)
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        acc[j] = 0.0f;
        uint32_t t;
        place(kRows * j + sub, t);
        off[j] = t * p.dim;
    }
    if (frame_ok && wave < p.heads) {
        const uint32_t n16 = p.dim / 8u;
        for (uint32_t c = piece; c < n16; c += kLanes) {
#pragma unroll 2
            for (uint32_t h = wave; h < p.heads; h += kAssignThreads / 64) {
                const uint4 qv = *reinterpret_cast<const uint4*>(q + (fa * p.stride_f + h * p.stride_h + ac) * p.dim + c * 8u);
                const uint16_t* kh = k + (fc * p.stride_f + h * p.stride_h) * p.dim + c * 8u;
                uint4 kv[kSteps];
#pragma unroll
                for (int j = 0; j < kSteps; ++j) kv[j] = *reinterpret_cast<const uint4*>(kh + off[j]);
                const uint32_t qs[4] = {qv.x, qv.y, qv.z, qv.w};
#pragma unroll
                for (int j = 0; j < kSteps; ++j) {
                    const uint32_t ks[4] = {kv[j].x, kv[j].y, kv[j].z, kv[j].w};
                    float d0 = 0.0f, d1 = 0.0f;   // (short chains: their rounding errors stay those of small sums)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        d0 = __builtin_fmaf(__uint_as_float(qs[e] << 16), __uint_as_float(ks[e] << 16), d0);
                        d1 = __builtin_fmaf(__uint_as_float(qs[e] & 0xFFFF0000u), __uint_as_float(ks[e] & 0xFFFF0000u), d1);
                    }
                    acc[j] += d0 + d1;
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        const float v = group_of_lanes_sum<kLanes>(acc[j]);
        if (piece == 0) partial[wave][kRows * j + sub] = v;
    }
    __syncthreads();
    const uint32_t w = threadIdx.x;
    if (w < slots) {
        uint32_t t;
        const bool inside = place(w, t);
        // (in a fixed order; the four sums of a wavefront's heads are the largest terms: added in double)
        const float sc = (float)(((double)partial[0][w] + (double)partial[1][w]) + ((double)partial[2][w] + (double)partial[3][w])) / (float)p.heads;
        const size_t per = (size_t)p.window_t * slots;
        if (scores) scores[(size_t)i * per + (size_t)wt * slots + w] = inside ? sc : __builtin_nanf("");
        const size_t at = (size_t)fc * tokens + t;
        if (inside && sc > p.threshold && (!anchor_group || anchor_group[at] < 0))
            atomicMax(token_group + at, (int32_t)tile_of(ac, p.grid_w, p.tile_h, p.tile_w));
    }
}

// Sec. 3.4, factorized attention, step 2: one workgroup per spatial tile, one wavefront per frame at a time; or several
// workgroups per tile ("parts"), each of which finds the main anchor and prunes its own frames, with one or more wavefronts
// per frame.  Per frame the tile's candidate (the first entry of the frame's list that lies in this tile of this frame) and its
// temporal mean score averaged over the heads (in double, head by head); the main anchor is the best of them
// (earliest frame on ties, a NaN never wins); a frame stays if it is the main anchor's or if the raw temporal
// score from the main anchor to it -- Qt[p*][h][f*] . Kt[p*][h][f], head mean in fp32 -- exceeds the threshold.
// Every entry of `kept` is written exactly once, so no launch has to clear it first: a candidate's by the tile's part that has
// its frame, a later entry of the same tile and frame by the tile's first part, and an entry that lies in no tile of its
// frame by tile 0's first part.  `kept` may be `cand` in one part only: another part would still read what this one writes.
// The order in which a score's products are added depends on the number of wavefronts that share a frame.
// Bound by its chain of dependent loads (list, temporal scores, the two rows of every head): a wavefront per frame up
// to 16, the loads of four heads in flight, the best frame found by the lanes of one wavefront.  64 tiles x 16 frames x
// 24 heads x 128 channels: 30 us with four wavefronts, serial head sums and one frame after the other, 7.85 so, 7.05 in four parts
// (in a graph, inputs changing).
constexpr int kMainThreads = 256;       // seda_main_anchor_3d_kernel
constexpr int kMainMaxThreads = 1024;   // seda_main_anchor_kernel: 64 per frame, at most these (the launcher says when)
constexpr uint32_t kMainMaxFrames = 1024;
// How the pruning of a tile's frames is split: frames per part (of a tile: blockIdx.y), wavefronts per frame, and 256 / those, rounded
// up, which divides a wavefront's number (a division would take as long as a load).
inline uint32_t main_anchor_split(uint32_t per_part, uint32_t parts, uint32_t n_waves, uint32_t heads)
{
    const uint32_t shares = parts > 1 ? std::min(std::max(n_waves / per_part, 1u), (heads + 3) / 4) : 1u;
    return per_part | shares << 11 | ((256 + shares - 1) / shares) << 16;
}

// kParts: several workgroups per tile (blockIdx.y).
template <bool kParts>
__global__ __launch_bounds__(kMainMaxThreads) void seda_main_anchor_kernel(
    const float* temporal_scores, const uint16_t* qt, const uint16_t* kt, uint32_t frames, uint32_t heads, uint32_t grid_h,
    uint32_t grid_w, uint32_t dim, const int32_t* cand, uint32_t n_per_frame, uint32_t tile_h, uint32_t tile_w,
    float prune_threshold, int32_t* main_anchor, int32_t* kept, float* prune_scores, uint32_t n_waves, uint32_t tiles, uint32_t split)
{
    __shared__ double score[kMainMaxFrames];
    __shared__ int32_t slot[kMainMaxFrames], row_of[kMainMaxFrames];
    __shared__ int32_t best_frame;
    __shared__ float share_sum[kMainMaxThreads / 64];
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    const uint32_t tokens = grid_h * grid_w, tile = blockIdx.x, part = kParts ? blockIdx.y : 0u;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (uint32_t f = wave; f < frames; f += n_waves) {
        const int32_t* list = cand + (size_t)f * n_per_frame;
        int32_t* out = kept + (size_t)f * n_per_frame;
        uint32_t found = kNone;
        for (uint32_t j0 = 0; j0 < n_per_frame; j0 += 64) {
            const uint32_t j = j0 + lane;
            bool mine = false;
            if (j < n_per_frame) {
                const int64_t row = list[j];
                const bool valid = row >= (int64_t)f * tokens && row < (int64_t)(f + 1) * tokens;
                mine = valid && tile_of((uint32_t)(row - (int64_t)f * tokens), grid_w, tile_h, tile_w) == tile;
                if (!valid && tile == 0 && part == 0) out[j] = -1;
            }
            const unsigned long long m = __ballot(mine);
            const uint32_t first = m ? j0 + (uint32_t)__builtin_ctzll(m) : kNone;
            if (mine && part == 0 && (found != kNone || j != first)) out[j] = -1;   // a later entry of the same tile
            if (found == kNone) found = first;
        }
        double v = 0.0;
        int32_t row = -1;
        if (found != kNone) {
            row = list[found];
            const uint32_t pos = (uint32_t)(row - (int32_t)(f * tokens));
            for (uint32_t h0 = 0; h0 < heads; h0 += 64) {
                const uint32_t cnt = min(64u, heads - h0);
                const float own = lane < cnt ? temporal_scores[((size_t)pos * heads + h0 + lane) * frames + f] : 0.0f;
                for (uint32_t i = 0; i < cnt; ++i)   // head by head
                    v += (double)__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, own), (int)i));
            }
            v /= (double)heads;
            if (v != v) v = -__builtin_inf();
        }
        if (lane == 0) {
            slot[f] = found == kNone ? -1 : (int32_t)found;
            row_of[f] = row;
            score[f] = v;
        }
    }
    __syncthreads();
    if (wave == 0) {
        int32_t bf = -1;
        double bv = 0.0;
        auto offer = [&](int32_t f, double v) {   // the earliest frame on ties
            if (f >= 0 && (bf < 0 || v > bv || (v == bv && f < bf))) { bf = f; bv = v; }
        };
        for (uint32_t f = lane; f < frames; f += 64) offer(slot[f] >= 0 ? (int32_t)f : -1, score[f]);
        for (uint32_t o = 1; o < frames && o < 64; o <<= 1) {   // (lane 0 needs no more: lanes from `frames` on hold none)
            const int32_t of = __shfl_xor(bf, (int)o);
            const double ov = __shfl_xor(bv, (int)o);
            offer(of, ov);
        }
        if (lane == 0) {
            best_frame = bf;
            if (part == 0) main_anchor[tile] = bf < 0 ? -1 : row_of[bf];
        }
    }
    __syncthreads();
    const int32_t bf = __builtin_amdgcn_readfirstlane(best_frame);
    const uint32_t n16 = dim / 8;
    // this workgroup's frames
    const uint32_t per_part = split & 0x7FFu, shares = kParts ? (split >> 11) & 31u : 1u;
    const uint32_t f0 = kParts ? min(part * per_part, frames) : 0u, f1 = kParts ? min(f0 + per_part, frames) : frames;
    if (shares == 1u) {
        for (uint32_t f = f0 + wave; f < f1; f += n_waves) {
            float sc = __builtin_nanf("");
            if (slot[f] >= 0) {   // (then the tile has a main anchor)
                const uint32_t pos = (uint32_t)(row_of[bf] - (int32_t)((uint32_t)bf * tokens));
                // 16 lanes share a row's 16-byte pieces, four heads at a time; the wavefront's sum in a fixed order
                float acc = 0.0f;
                const size_t base = (size_t)pos * heads * frames;
                for (uint32_t c = lane & 15u; c < n16; c += 16) {
#pragma unroll 4
                    for (uint32_t h = lane >> 4; h < heads; h += 4) {
                        const uint4 a = reinterpret_cast<const uint4*>(qt + (base + (size_t)h * frames + (uint32_t)bf) * dim)[c];
                        const uint4 b = reinterpret_cast<const uint4*>(kt + (base + (size_t)h * frames + f) * dim)[c];
                        const uint32_t qs[4] = {a.x, a.y, a.z, a.w}, ks[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            acc = __builtin_fmaf(__uint_as_float(qs[i] << 16), __uint_as_float(ks[i] << 16), acc);
                            acc = __builtin_fmaf(__uint_as_float(qs[i] & 0xFFFF0000u), __uint_as_float(ks[i] & 0xFFFF0000u), acc);
                        }
                    }
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
                sc = acc / (float)heads;
                if (lane == 0)
                    kept[(size_t)f * n_per_frame + slot[f]] = ((int32_t)f == bf || sc > prune_threshold) ? row_of[f] : -1;
            }
            if (lane == 0 && prune_scores) prune_scores[(size_t)f * tiles + tile] = sc;
        }
    } else {
        // more wavefronts than frames: `shares` of them take a frame, every fourth of its heads in turn; addresses from scalar
        // parts and no work past the last head (with 16 wavefronts on a compute unit instructions cost as much as a round of loads)
        const uint32_t mine = (wave * (split >> 16)) >> 8, share = wave - mine * shares, f = f0 + mine;
        const bool ok = f < f1, anchored = ok && slot[min(f, frames - 1u)] >= 0;   // (then the tile has a main anchor)
        float sc = __builtin_nanf("");
        if (anchored) {
            const uint32_t pos = __builtin_amdgcn_readfirstlane((uint32_t)(row_of[bf] - (int32_t)((uint32_t)bf * tokens)));
            const size_t row0 = (size_t)pos * heads * frames, head = (size_t)frames * n16;
            const uint4* q0 = reinterpret_cast<const uint4*>(qt) + (row0 + (uint32_t)bf) * n16;
            const uint4* k0 = reinterpret_cast<const uint4*>(kt) + (row0 + f) * n16;
            const uint32_t own = lane >> 4, step = 4u * shares;
            float acc = 0.0f;
            for (uint32_t c = lane & 15u; c < n16; c += 16) {
                for (uint32_t h0 = 4u * share; h0 < heads; h0 += 2u * step) {   // (wave-uniform)
                    const bool two = h0 + step < heads;
                    uint4 a[2] = {}, b[2] = {};   // two heads' rows in flight (zeros past the last head)
                    if (h0 + own < heads) {
                        a[0] = q0[(h0 + own) * head + c];
                        b[0] = k0[(h0 + own) * head + c];
                    }
                    if (two && h0 + step + own < heads) {
                        a[1] = q0[(h0 + step + own) * head + c];
                        b[1] = k0[(h0 + step + own) * head + c];
                    }
#pragma unroll
                    for (uint32_t j = 0; j < 2; ++j) {
                        if (j && !two) break;
                        const uint32_t qs[4] = {a[j].x, a[j].y, a[j].z, a[j].w}, ks[4] = {b[j].x, b[j].y, b[j].z, b[j].w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            acc = __builtin_fmaf(__uint_as_float(qs[i] << 16), __uint_as_float(ks[i] << 16), acc);
                            acc = __builtin_fmaf(__uint_as_float(qs[i] & 0xFFFF0000u), __uint_as_float(ks[i] & 0xFFFF0000u), acc);
                        }
                    }
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
            sc = acc;
        }
        if (lane == 0) share_sum[wave] = sc;
        __syncthreads();
        if (ok && lane == 0 && share == 0) {
            for (uint32_t j = 1; j < shares; ++j) sc += share_sum[wave + j];
            sc /= (float)heads;   // (NaN without a candidate)
            if (anchored) kept[(size_t)f * n_per_frame + slot[f]] = ((int32_t)f == bf || sc > prune_threshold) ? row_of[f] : -1;
            if (prune_scores) prune_scores[(size_t)f * tiles + tile] = sc;
        }
    }
}

// Sec. 3.4, 3D attention: the main anchor of a spatial tile is the best token among its tile_h x tile_w x frames
// tokens by the head mean (double, head by head) of the clip-wide scores [heads][frames * tokens]; the lowest row
// on ties, a NaN never wins.  One workgroup per tile.
__global__ __launch_bounds__(kMainThreads) void seda_main_anchor_3d_kernel(const float* scores, uint32_t frames, uint32_t heads,
                                                                            uint32_t grid_h, uint32_t grid_w, uint32_t tile_h,
                                                                            uint32_t tile_w, int32_t* anchors)
{
    __shared__ double best_v[kMainThreads];
    __shared__ uint32_t best_row[kMainThreads];
    const uint32_t tokens = grid_h * grid_w, tile = blockIdx.x;
    const uint32_t tw = (grid_w + tile_w - 1) / tile_w;
    const uint32_t y0 = (tile / tw) * tile_h, x0 = (tile % tw) * tile_w;
    const uint32_t hh = min(tile_h, grid_h - y0), ww = min(tile_w, grid_w - x0);
    const uint32_t n = frames * hh * ww;
    const size_t total = (size_t)frames * tokens;
    double bv = 0.0;
    uint32_t br = 0xFFFFFFFFu;
    for (uint32_t i = threadIdx.x; i < n; i += kMainThreads) {   // ascending rows per thread
        const uint32_t f = i / (hh * ww), r = i - f * (hh * ww);
        const uint32_t row = f * tokens + (y0 + r / ww) * grid_w + x0 + r % ww;
        double v = 0.0;
        for (uint32_t h = 0; h < heads; ++h) v += (double)scores[(size_t)h * total + row];
        v /= (double)heads;
        if (v != v) v = -__builtin_inf();
        if (br == 0xFFFFFFFFu || v > bv) { br = row; bv = v; }
    }
    best_v[threadIdx.x] = bv;
    best_row[threadIdx.x] = br;
    __syncthreads();
    for (uint32_t s = kMainThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const double ov = best_v[threadIdx.x + s];
            const uint32_t orow = best_row[threadIdx.x + s];
            const double mv = best_v[threadIdx.x];
            const uint32_t mrow = best_row[threadIdx.x];
            const bool take = orow != 0xFFFFFFFFu && (mrow == 0xFFFFFFFFu || ov > mv || (ov == mv && orow < mrow));
            if (take) { best_v[threadIdx.x] = ov; best_row[threadIdx.x] = orow; }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) anchors[tile] = (int32_t)best_row[0];
}

}  // namespace fb4
