// sketch_short.hip -- the sketch kernel over fewer than 4 columns, and over rows
// of fewer than 4 values.
#include "sketch_kernel.h"

namespace osk {

hipError_t sketch_narrow(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, false, float, 0, kMaxSlots, kNarrow>(slots, grid, st, a);
}

hipError_t sketch_short(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, false, float, 0, kMaxSlots, kShort>(slots, grid, st, a);
}

hipError_t sketch_short_weighted(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, true, float, 0, kMaxSlots, kShort>(slots, grid, st, a);
}

hipError_t sketch_short_bf16(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
    return launch_slots<false, false, __bf16, 0, kMaxSlots, kShort>(slots, grid, st, a);
}

}  // namespace osk
