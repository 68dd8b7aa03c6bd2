// sketch_fp8.hip -- the sketch kernel writing FP8 copies.
#include "sketch_kernel.h"

namespace osk {

hipError_t sketch_rows_f32_fp8(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<true, false, float, 1>(slots, grid, st, a);
}

hipError_t sketch_rows_bf16_fp8(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<true, false, __bf16, 1>(slots, grid, st, a);
}

hipError_t sketch_cols_f32_fp8(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, false, float, 1>(slots, grid, st, a);
}

}  // namespace osk
