// logit_common.h -- reading one chunk of a logit row, shared by the token
// statistics and the speculative-sampling kernels.  Internal to the library.
#pragma once

#include "device_common.h"
#include "launch.h"

namespace ssl {
namespace lc {

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;

// Logits per 16-byte load and loads per thread (32 logits per thread).
template <bool kF32>
constexpr int per_load() { return kF32 ? 4 : 8; }
template <bool kF32>
constexpr int loads() { return 32 / per_load<kF32>(); }

// The row index of x[q] as load_chunk fills it: thread tid's loads j cover
// consecutive 16-byte blocks kThreads apart, so x[q] is element
// (blk0 + (q / per) * kThreads + tid) * per + q % per of the row.
template <bool kF32>
__device__ __forceinline__ int elem(int chunk, int q, int tid) {
    constexpr int per = per_load<kF32>();
    const int blk0 = chunk * (kLogitChunk / per);
    return (blk0 + (q / per) * kThreads + tid) * per + q % per;
}

// The 16-byte blocks of thread tid in chunk `chunk` of the row at `row_base`,
// all loads in flight together; loads are clamped into the row's last block.
template <bool kF32>
__device__ __forceinline__ void load_blocks(const void* row_base, int vocab, int chunk, int tid,
                                            uint4 (&raw)[loads<kF32>()]) {
    constexpr int per = per_load<kF32>();
    const int last_blk = (vocab - 1) / per;
    const int blk0 = chunk * (kLogitChunk / per);
    const char* base = static_cast<const char*>(row_base);
#pragma unroll
    for (int j = 0; j < loads<kF32>(); ++j) {
        const int blk = min(blk0 + j * kThreads + tid, last_blk);
        raw[j] = *reinterpret_cast<const uint4*>(base + (size_t)blk * 16);
    }
}

// The logits of one block, the thread's load j; elements at or past vocab read
// as -inf.
template <bool kF32>
__device__ __forceinline__ void unpack_block(const uint4& raw, int vocab, int chunk, int j, int tid,
                                             float (&x)[per_load<kF32>()]) {
    constexpr int per = per_load<kF32>();
    const int i0 = (chunk * (kLogitChunk / per) + j * kThreads + tid) * per;
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int e = 0; e < per; ++e) {
        const float v = kF32 ? __builtin_bit_cast(float, w[e])
                             : ((e & 1) ? bf16_hi(w[e >> 1]) : bf16_lo(w[e >> 1]));
        x[e] = i0 + e < vocab ? v : -INFINITY;
    }
}

// Runs f(j, raw blocks of load j) for the thread's loads in order, as a loop:
// the code of one block stays in the instruction cache, where the unrolled
// kernel's would be fetched once and run once.  The blocks are passed down a
// register queue, so that the loop needs no indexed registers.
template <int kN, int kArrays, typename F>
__device__ __forceinline__ void for_blocks(uint4 (&raw)[kArrays][kN], F&& f) {
#pragma unroll 1
    for (int j = 0; j < kN; ++j) {
        f(j);
#pragma unroll
        for (int r = 0; r < kArrays; ++r)
#pragma unroll
            for (int q = 0; q + 1 < kN; ++q) raw[r][q] = raw[r][q + 1];
    }
}

// The 32 logits of thread tid in chunk `chunk` of the row (bf16 or fp32).
template <bool kF32>
__device__ __forceinline__ void load_chunk(const void* row_base, int vocab, int chunk, int tid,
                                           float (&x)[32]) {
    constexpr int per = per_load<kF32>();
    uint4 raw[loads<kF32>()];
    load_blocks<kF32>(row_base, vocab, chunk, tid, raw);
#pragma unroll
    for (int j = 0; j < loads<kF32>(); ++j) {
        float y[per];
        unpack_block<kF32>(raw[j], vocab, chunk, j, tid, y);
#pragma unroll
        for (int e = 0; e < per; ++e) x[j * per + e] = y[e];
    }
}

}  // namespace lc
}  // namespace ssl
