// sketch_fp8x3.hip -- the sketch kernel writing split FP8 copies.
#include "sketch_kernel.h"

namespace osk {

hipError_t sketch_rows_f32_fp8x3(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<true, false, float, 2>(slots, grid, st, a);
}

hipError_t sketch_rows_bf16_fp8x3(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<true, false, __bf16, 2>(slots, grid, st, a);
}

hipError_t sketch_cols_f32_fp8x3(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, false, float, 2>(slots, grid, st, a);
}

}  // namespace osk
