// sketch_pair_bf16.hip -- both sketches in one launch, columns of BF16 matrices.
#include "sketch_pair_kernel.h"

namespace osk {

hipError_t sketch_pair_bf16(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                            const SketchSide& y) {
    return launch_pair<__bf16, 0, kMaxWideSlots>(slots, st, a, x, y);
}

}  // namespace osk
