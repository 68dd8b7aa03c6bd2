// sketch_launch.h -- the sketch kernel's launchers, one per input form.
#pragma once

#include "sketch_common.h"

namespace osk {

// Slot counts compiled: 1, 2, 3, 4, 6, 8, 10, 12 (4 registers per slot).
constexpr int kMaxSlots = 12;
constexpr int kMaxFp8Slots = 10;       // with the FP8 epilogue
constexpr int kMaxWideSlots = 6;       // 8 BF16 column lines (8 registers per slot)

// Arguments of a sketch launch (see launch_sketch).
struct SketchArgs {
    const void* X;
    int64_t lines, n, ldx, ldk;
    int32_t qn, nwin, nst;
    const BlockList* bl;
    int64_t RC;
    const uint32_t* hdr;
    const uint4* ell;
    void* out;
    int64_t ldo;
    int32_t npass;
    const float* wd;
    int32_t obp, omode;
    int64_t ozlo;
};

constexpr int kMaxPairSlots = 10;      // both operands in one launch
constexpr int kMaxPairFp8Slots = 8;

// One operand of a pair launch.
struct SketchSide {
    const void* X;
    int64_t lines, ldx;
    void* out;
    int32_t wgs;       // its workgroups
    int32_t rows;      // lines are rows (else columns)
};
// Both sides of a product in one launch (a's fields X, lines, ldx, out, wd
// unused): FP32 operands with FP32 or BF16, FP8 and split FP8 output, and
// columns of BF16 operands with FP32 or BF16 output.
hipError_t sketch_pair(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                       const SketchSide& y);
hipError_t sketch_pair_bf16(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                            const SketchSide& y);
hipError_t sketch_pair_fp8(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                           const SketchSide& y);
hipError_t sketch_pair_fp8x3(int slots, hipStream_t st, const SketchArgs& a, const SketchSide& x,
                             const SketchSide& y);

// Launches the sketch kernel with at least `slots` slots per wave: rows of an
// FP32 X, rows weighted by sqrt(wd), rows of a BF16 X, columns of an FP32 X
// and of a BF16 one (8 lines per workgroup),
// and rows (FP32 or BF16) and columns writing the FP8 copy, plain or split.
// sketch_narrow: fewer than 4 columns (n >= 4).  sketch_short*: value (line, k) at
// X[line * ldx + k * ldk], loaded one at a time (n < 4).
hipError_t sketch_rows_f32(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_rows_weighted(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_rows_bf16(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_cols_f32(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_cols_bf16(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_narrow(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_short(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_short_weighted(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_short_bf16(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_rows_f32_fp8(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_rows_bf16_fp8(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_cols_f32_fp8(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_rows_f32_fp8x3(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_rows_bf16_fp8x3(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);
hipError_t sketch_cols_f32_fp8x3(int slots, dim3 grid, hipStream_t st, const SketchArgs& a);

}  // namespace osk
