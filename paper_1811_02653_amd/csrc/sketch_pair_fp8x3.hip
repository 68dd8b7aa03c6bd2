// sketch_pair_fp8x3.hip -- both sketches in one launch, split FP8 output.
#include "sketch_pair_kernel.h"

namespace osk {

hipError_t sketch_pair_fp8x3(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                             const SketchSide& y) {
    return launch_pair<float, 2, kMaxPairFp8Slots>(slots, st, a, x, y);
}

}  // namespace osk
