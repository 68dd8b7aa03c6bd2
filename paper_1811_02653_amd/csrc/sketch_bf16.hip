// sketch_bf16.hip -- the sketch kernel over rows, and columns, of a BF16 matrix.
#include "sketch_kernel.h"

namespace osk {

hipError_t sketch_rows_bf16(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<true, false, __bf16>(slots, grid, st, a);
}

hipError_t sketch_cols_bf16(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, false, __bf16, 0, kMaxWideSlots>(slots, grid, st, a);
}

}  // namespace osk
