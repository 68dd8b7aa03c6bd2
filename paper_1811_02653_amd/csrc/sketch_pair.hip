// sketch_pair.hip -- both sketches in one launch, FP32 or BF16 output.
#include "sketch_pair_kernel.h"

namespace osk {

hipError_t sketch_pair(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                       const SketchSide& y) {
    return launch_pair<float, 0, kMaxPairSlots>(slots, st, a, x, y);
}

}  // namespace osk
