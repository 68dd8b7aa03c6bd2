// sketch_columns.hip -- the sketch kernel over columns of an FP32 matrix.
#include "sketch_kernel.h"

namespace osk {

hipError_t sketch_cols_f32(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, false, float>(slots, grid, st, a);
}

}  // namespace osk
