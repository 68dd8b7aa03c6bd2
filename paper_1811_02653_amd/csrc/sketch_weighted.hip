// sketch_weighted.hip -- the sketch kernel over weighted rows of an FP32 matrix.
#include "sketch_kernel.h"

namespace osk {

hipError_t sketch_rows_weighted(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<true, true, float>(slots, grid, st, a);
}

}  // namespace osk
