// sketch_common.h -- constants and device helpers shared by the sketch kernel
// (sketch_kernel.h) and the list builders (sketch.hip).
#pragma once

#include <type_traits>

#include "internal.h"

namespace osk {

constexpr int kWin = kSketchWindow;    // sketched indices per window (8192)
constexpr int kLines = 4;              // lines per workgroup
constexpr int kThreads = 1024;         // 16 waves
constexpr int kWaves = kThreads / 64;
constexpr int kPerThread = kWin / kThreads;   // window positions staged per thread (8)
constexpr uint16_t kPad = (uint16_t)kWin;     // entry of the zero row, positive
// List chunks of a slot fetched ahead (before the next window's loads, which
// the chunks fetched after them wait for), and, for lists longer than that,
// chunks fetched ahead of the one that is summed.  Kernels of one slot have the
// registers for more, and need them: their lists are long (few buckets) and no
// other slot's work hides their latency (2 blocks of 64, 1000000 x 1: 1288 us,
// this 776; columns, 1000000 x 16: 1880, this 1236.  Rows with 2 chunks instead
// of 3: 100000 x 2500 into 4 blocks of 256 9 % slower.  Columns with 3 instead of
// 6, 1000000 x 16 into 4 blocks of 256: 1399 / 1291.  Two slots: no gain.)
template <int kSlots, bool kRows, int kQ>
constexpr int kAheadOf = kSlots > 1 || kQ > 1 ? 2 : (kRows ? 3 : 6);
template <int kSlots, int kQ>
constexpr int kTailOf = kSlots == 1 && kQ == 1 ? 4 : 0;
constexpr int kDist = 1;               // slots ahead whose lists are fetched

// LDS slot of window position p (p < kWin).  Thread t stages the quads of
// positions 4096u + 4t + j (j < 4); they go to slots 4096u + 1024j + t, so the
// lanes of one staging write touch consecutive slots.  List entries hold the
// slot of their position.
__device__ __forceinline__ int win_slot(int p) {
    return (p & ~4095) | ((p & 3) << 10) | ((p >> 2) & 1023);
}

// f(integral_constant<int, I>) for I = B .. E - 1, unrolled by the compiler
// whatever the size of f's body.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// Spread consecutive task ids over the 8 XCDs in contiguous runs (workgroup L
// runs on XCD L % 8), so neighbouring tasks share an XCD and its L2.
__device__ __forceinline__ int64_t xcd_task(int64_t L, int64_t tasks) {
    const int64_t q = tasks / 8, r = tasks % 8, x = L % 8;
    return x * q + min(x, r) + L / 8;
}

__device__ __forceinline__ uint64_t lanes_below() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x = max(x, (uint32_t)__shfl_xor((int)x, d));
    return x;
}

}  // namespace osk
