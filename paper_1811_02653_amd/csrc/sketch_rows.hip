// sketch_rows.hip -- the sketch kernel over rows of an FP32 matrix.
#include "sketch_kernel.h"

namespace osk {

hipError_t sketch_rows_f32(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<true, false, float>(slots, grid, st, a);
}

}  // namespace osk
