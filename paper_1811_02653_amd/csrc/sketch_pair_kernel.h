// sketch_pair_kernel.h -- the sketches of both operands of a product in one
// launch.  A small product has fewer tasks (groups of 4 lines) per operand
// than the device has CUs, and each of its kernels lasts a few microseconds,
// most of it latency: the two sketches side by side take the time of one (256
// x 4096 x 256, 5 blocks of 256: 9.3 + 10.3 us apart, 12.3 together; 128 x
// 2048 x 96, 4 blocks of 128: 7.9 + 7.7 us apart, 8.7 together).  Larger ones
// save a partial last round (launch_sketch_pair).  Included by one translation unit per
// output form.
#pragma once

#include "sketch_kernel.h"

namespace osk {
namespace {

// The first x.wgs workgroups take x's tasks, the rest y's.
template <int kSlots, typename TI, int kFp8Out>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void sketch_pair_kernel(SketchSide x, SketchSide y, int64_t n, int32_t qn, int32_t nwin,
                        int32_t nst, BlockList bl, int64_t RC,
                        const uint32_t* __restrict__ hdr, const uint4* __restrict__ ell,
                        int64_t ldo, int32_t npass, int32_t obp, int32_t omode, int64_t ozlo) {
    __shared__ float4 win[kWin + 1];
    const bool second = (int32_t)blockIdx.x >= x.wgs;
    const int64_t wg = second ? blockIdx.x - x.wgs : blockIdx.x;
    const SketchSide& s = second ? y : x;
    const TI* const X = static_cast<const TI*>(s.X);
    if constexpr (sizeof(TI) == 4) {
        if (s.rows) {
            sketch_tasks<kSlots, true, false, TI, kFp8Out>(
                win, wg, s.wgs, X, s.lines, n, s.ldx, 0, qn, nwin, nst, bl, RC, hdr, ell, s.out,
                ldo, npass, nullptr, obp, omode, ozlo);
            return;
        }
    }
    sketch_tasks<kSlots, false, false, TI, kFp8Out>(
        win, wg, s.wgs, X, s.lines, n, s.ldx, 0, qn, nwin, nst, bl, RC, hdr, ell, s.out, ldo,
        npass, nullptr, obp, omode, ozlo);
}

template <typename TI, int kFp8Out, int kMost>
hipError_t launch_pair(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                       const SketchSide& y) {
#define OSK_SLOT_CASE(S)                                                                          \
    if constexpr (S <= kMost)                                                                     \
        if (slots <= S) {                                                                         \
            hipLaunchKernelGGL((sketch_pair_kernel<S, TI, kFp8Out>),                              \
                               dim3((unsigned)(x.wgs + y.wgs)), dim3(kThreads), 0, st, x, y, a.n,  \
                               a.qn, a.nwin, a.nst, *a.bl, a.RC, a.hdr, a.ell, a.ldo,       \
                               a.npass, a.obp, a.omode, a.ozlo);                                  \
            return hipGetLastError();                                                             \
        }
    OSK_SLOT_CASE(1)
    OSK_SLOT_CASE(2)
    OSK_SLOT_CASE(3)
    OSK_SLOT_CASE(4)
    OSK_SLOT_CASE(6)
    OSK_SLOT_CASE(8)
    OSK_SLOT_CASE(10)
#undef OSK_SLOT_CASE
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace osk
