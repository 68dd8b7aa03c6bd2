// hash.h -- the counter-based random choices of the count sketch (see
// hash.hip), shared by the table kernels and the list builder.
#pragma once

#include "internal.h"

namespace osk {

constexpr uint64_t kGoldenGamma = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ uint64_t splitmix64_output(uint64_t state) {
    uint64_t w = state;
    w = (w ^ (w >> 30)) * 0xBF58476D1CE4E5B9ull;
    w = (w ^ (w >> 27)) * 0x94D049BB133111EBull;
    return w ^ (w >> 31);
}

__device__ __forceinline__ uint64_t sketch_word(uint64_t seed, uint64_t blk, uint64_t k) {
    const uint64_t ctr = (blk << 40) | k;
    return splitmix64_output(seed + (ctr + 1ull) * kGoldenGamma);
}

__device__ __forceinline__ uint32_t word_bucket(uint64_t w, uint32_t b) {
    return (uint32_t)(((w >> 32) * (uint64_t)b) >> 32);
}

__device__ __forceinline__ uint32_t clamp_bucket(int32_t h, int32_t b) {
    return (uint32_t)(h < 0 ? 0 : (h >= b ? b - 1 : h));
}

// One packed entry of (block, index): bucket in bits 0..30, bit 31 = negative;
// from SplitMix64 of seed, or from the explicit tables h / sigma when h is set.
__device__ __forceinline__ uint32_t packed_entry(uint64_t seed, const int32_t* __restrict__ h,
                                                 const int8_t* __restrict__ sigma, int64_t blk,
                                                 int64_t k, int64_t n, int32_t b) {
    if (h) return clamp_bucket(h[blk * n + k], b) | (sigma[blk * n + k] < 0 ? 0x80000000u : 0u);
    const uint64_t w = sketch_word(seed, (uint64_t)blk, (uint64_t)k);
    return word_bucket(w, (uint32_t)b) | ((uint32_t)(w & 1ull) << 31);
}

}  // namespace osk
