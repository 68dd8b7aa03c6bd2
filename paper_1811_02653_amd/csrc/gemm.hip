// gemm.hip -- grouped FP32 MFMA product over the kept sketch blocks.
//
// Computes C = scale * sum_{j kept} At_j * Bt_j^T, where At_j (m x bp) and
// Bt_j (l x bp) are the j-th column blocks of the line-major sketches A S
// and (S^T B)^T.
// This is the computation phase and the reduction phase of Algorithm
// "OverSketch" fused into one K loop: the paper's b x b worker products
// A_tilde(i,k) B_tilde(k,j) for the blocks that returned (Fig. (bMM)) are
// summed in registers instead of through storage, and blocks that
// straggled are skipped by walking only the kept-block list.
//
// Design (gfx950; FP32 v_mfma_f32_32x32x2_f32, BF16 v_mfma_f32_32x32x16_bf16,
// FP8 v_mfma_scale_f32_32x32x64_f8f6f4):
//   - 256 x 256 output tile per workgroup of 8 waves, two per SIMD; wave
//     (wm, wn) owns a 128 x 64 sub-tile = 4 x 2 MFMA blocks of 32 x 32 (128
//     accumulators per lane).  With two waves on a SIMD one wave's memory
//     instructions issue while the other's MFMAs keep the pipe busy.
//   - K steps of 128 bytes of every tile row (32 FP32, 64 BF16 or 128 FP8
//     values).  Both operands are K-contiguous; a step's tiles go straight
//     from global memory into LDS (buffer_load_dwordx4 with the lds flag: no
//     VGPR staging, no LDS stores), unpadded, with the 16-byte chunk c of
//     row r at chunk c ^ key(r), key(r) = (r & 7) ^ ((r >> 3) & 1), so the
//     16 rows a fragment read serves at once hit 16 different bank groups.
//     Two step buffers per operand: step t + 1 is loaded into one while
//     step t is read from the other.
//   - Lane half h of every MFMA takes the K values at byte offset 64h + 16q
//     of the step's row (q = quad), so a lane's fragment is one 16-byte LDS
//     read; A and B use the same K order, so the dot products are unchanged
//     (only their summation order differs).
//   - The kept-block list is held in VGPRs and picked with v_readlane.
//   - Workgroup -> tile mapping keeps neighbouring tiles on one XCD (shared
//     L2) and rasterises in groups of kGroupM = 8 tile rows.
#include <algorithm>

#include "internal.h"

namespace osk {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int BM = 256;
constexpr int BN = 256;
constexpr int kStepBytes = 128; // K step: 128 bytes of each tile row (32 FP32 / 64 BF16 values)
// tiles are rasterised in groups of kGroupM tile rows (an XCD's 32
// concurrent tiles then share 8 row blocks of A; 8 measured 0.5 % faster
// than 4 on the full-size product)
constexpr int kGroupM = 8;

__device__ __forceinline__ int64_t xcd_task(int64_t L, int64_t tasks) {
    const int64_t q = tasks / 8, r = tasks % 8, x = L % 8;
    return x * q + min(x, r) + L / 8;
}

// Buffer resource of a matrix starting at p: no stride, no range limit
// (num_records = 2^32 - 1), the gfx9 data format word.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, -1, 0x00020000);
}

// ---------------------------------------------------------------------------
// Tiles loaded straight from global memory into LDS (buffer_load_dwordx4
// with the lds flag: no VGPR staging and no LDS store instructions, which
// each cost the MFMA pipe about one slot when issued in the K loop).  A tile
// of BT = 32 kU rows x 128 bytes (one K step) is stored unpadded: the
// 16-byte chunk c of row r sits at chunk c ^ key(r), key(r) = (r & 7) ^
// ((r >> 3) & 1).  A 16-byte fragment read is served 16 lanes (16
// consecutive rows, 256 bytes) at a time over the 64 four-byte banks: rows
// r and r + 8 share their (r & 7) and the parity of their 128-byte row
// offset, and the (r >> 3) term sends them to different chunks, so the 16
// reads of a pass hit 16 different bank groups (with key (r & 7) alone, they
// met in pairs: measured as half the LDS cycles spent in bank conflicts).
// Any 8 consecutive rows also take 8 different chunks.  Load u of wave w
// fills LDS rows 8(kU w + u) .. +7 (1 KiB, 16 bytes per lane): lane l takes
// row r = 8(kU w + u) + l/8 and physical chunk l % 8, i.e. logical chunk
// (l % 8) ^ key(r).  Rows past the matrix end are clamped to its last row
// (they only feed outputs that are not stored).
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ int chunk_key(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// (sub: LDS row r holds matrix row r - sub of the resource, for a tile
// whose rows start sub rows into the LDS array; a multiple of 16, so the
// key is that of r.)
template <int kU>
__device__ __forceinline__ void direct_offsets(uint32_t (&vo)[kU], int64_t ld_bytes, int last,
                                               int wave, int lane, int sub = 0) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int r = 8 * (kU * wave + u) + (lane >> 3);
        const int c = (lane & 7) ^ chunk_key(r);
        vo[u] = (uint32_t)((int64_t)min(r - sub, last) * ld_bytes + 16 * c);
    }
}

// The same for a split-precision step: chunks 0-3 of an LDS row hold 64 bytes
// of the high part, chunks 4-7 the 64 bytes lo_bytes further in the row.
template <int kU>
__device__ __forceinline__ void direct_offsets_pair(uint32_t (&vo)[kU], int64_t ld_bytes, int last,
                                                    int64_t lo_bytes, int wave, int lane) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int r = 8 * (kU * wave + u) + (lane >> 3);
        const int c = (lane & 7) ^ chunk_key(r);
        vo[u] = (uint32_t)((int64_t)min(r, last) * ld_bytes + 16 * (c & 3) + (c & 4 ? lo_bytes : 0));
    }
}

// (The builtin exists only for the device target; the host pass of a
// template kernel that names it would silently drop the kernel's launch
// stubs, hence the guard.)
template <int kU>
__device__ __forceinline__ void direct_issue(__amdgpu_buffer_rsrc_t rsrc, float* lds,
                                             const uint32_t (&vo)[kU], uint32_t kbyte, int wave) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int u = 0; u < kU; ++u)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsrc, (lds_void*)(lds + (kU * wave + u) * 256), 16, vo[u], kbyte, 0, 0);
#endif
}

// Float offset in a direct tile of the fragment of quad q for tile row
// rbase + 32 i (rbase = a wave's first row + lane % 32; 32 i changes no bit
// of the key): lane half h reads logical chunk 4h + q.
__device__ __forceinline__ int direct_frag_off(int rbase, int q, int lane) {
    return rbase * 32 + 4 * ((4 * (lane >> 5) + q) ^ chunk_key(rbase));
}

// The same in a pair step (high part in chunks 0-3, low part in chunks 4-7):
// fragment q of lane half h is chunk 2h + (q & 1) of the high part (q < 2) or
// of the low part.
__device__ __forceinline__ int pair_frag_off(int rbase, int q, int lane) {
    return rbase * 32 + 4 * ((4 * (q >> 1) + 2 * (lane >> 5) + (q & 1)) ^ chunk_key(rbase));
}

// Waits until at most kLoads of this wave's loads (the youngest) and none of
// its LDS accesses are outstanding, then for the workgroup's other waves.
// (__syncthreads() would wait for every load in flight, also those into LDS
// meant for later steps; the fence keeps later LDS reads below the barrier.)
template <int kLoads>
__device__ __forceinline__ void wait_step() {
    static_assert(kLoads >= 0 && kLoads < 64);
    if constexpr (kLoads == 0) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    } else {
#if defined(__HIP_DEVICE_COMPILE__)
        __builtin_amdgcn_s_waitcnt((kLoads & 15) | ((kLoads >> 4) << 14) | 0x70);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#endif
    }
}

__device__ __forceinline__ float comp(const float4& v, int c) {
    return c == 0 ? v.x : (c == 1 ? v.y : (c == 2 ? v.z : v.w));
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));


enum Kind { kF32, kBF16, kBF16X3, kFp8, kFp8X3 };   // operand precisions

// Operand precisions of the block product.  A K step is 128 bytes of a tile
// row in both: 32 FP32 values or 64 BF16 values.  A fragment is 16 bytes:
// lane half h of quad q holds the K values at byte offset 64h + 16q of the
// step's row (4 FP32 values feeding four 32x32x2 MFMAs, or 8 BF16 values
// feeding one 32x32x16 MFMA); A and B use the same K order.
// A quad's MFMAs come in kParts parts; the K loop issues the next quad's
// fragment reads after kHead parts and leaves the step's last kTail parts
// until after the step's barrier (they keep the MFMA pipe busy while the
// next step's first fragments are read).  Chosen by measurement: FP32 3 and
// 1, BF16 1 and 0 (BF16 3-4 % faster than the compiler's own placement,
// which read each quad's fragments just before its MFMAs; FP32 unchanged).
struct PrecF32 {
    static constexpr Kind kKind = kF32;
    static constexpr bool kPair = false;
    static constexpr int kElem = 4;
    static constexpr int kParts = 4;          // parts of a quad: the four K values kk
    static constexpr int kHead = 3;
    static constexpr int kTail = 1;
    template <int kI>
    static constexpr int parts = kParts;
    template <int kI, int kJ, int kLo = 0, int kHi = kParts>
    __device__ static __forceinline__ void mfma_quad(v16f (&acc)[kI][kJ], const float4 (&a)[kI],
                                                     const float4 (&b)[kJ]) {
#pragma unroll
        for (int kk = kLo; kk < kHi; ++kk)
#pragma unroll
            for (int i = 0; i < kI; ++i)
#pragma unroll
                for (int j = 0; j < kJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(a[i], kk), comp(b[j], kk),
                                                                     acc[i][j], 0, 0, 0);
    }
};

struct PrecBF16 {
    static constexpr Kind kKind = kBF16;
    static constexpr bool kPair = false;
    static constexpr int kElem = 2;
    static constexpr int kHead = 1;
    static constexpr int kTail = 0;
    template <int kI>
    static constexpr int parts = kI;          // parts of a quad: the row blocks i
    template <int kI, int kJ, int kLo = 0, int kHi = kI>
    __device__ static __forceinline__ void mfma_quad(v16f (&acc)[kI][kJ], const float4 (&a)[kI],
                                                     const float4 (&b)[kJ]) {
#pragma unroll
        for (int i = kLo; i < kHi; ++i)
#pragma unroll
            for (int j = 0; j < kJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[j]), acc[i][j],
                    0, 0, 0);
    }
};

// Split BF16 operands: a step holds 32 K values of both parts of every tile
// row (64 bytes high, 64 bytes low) and contributes hi*lo' + hi*hi' + lo*hi',
// so the three terms share one load of the four tiles and each fragment read
// (two thirds of the loads and LDS reads of three separate passes: 298 us
// against 333-361 for 4096 x 4096, K = 4096).
struct PrecBF16X3 : PrecBF16 {
    static constexpr Kind kKind = kBF16X3;
    static constexpr bool kPair = true;
};

// Per-C-block keep masks (cmask != nullptr, the paper's per-block
// stragglers): C is divided into cblk x cblk blocks, block (I, J) keeps the
// stored blocks j with cmask[(I * nbJ + J) * nstm + j] != 0 and is scaled by
// 1 / (their number); a block that keeps none is written as zero.  Tiles are
// laid on the C-block grid (ceil(cblk / 256) per block side, the last ones
// partial), so every tile lies in one block.
struct CMask {
    const uint8_t* mask;   // DEVICE [nbI][nbJ][nstm], or nullptr (one kept list)
    int64_t cblk;
    int32_t nbJ;
    int32_t nstm;
    int32_t tb;            // tiles per block side
};

// Split K loop (kSplit kernels, for products with few tiles): workgroup
// g = s * tiles + tile runs K steps s * chunk .. min(total, (s + 1) * chunk)
// - 1 of its tile and stores the unscaled partial tile at part + s * m * l
// (row-major, ld l); split_sum_kernel then adds the partials in split order.
struct SplitK {
    float* part;
    int32_t chunk;
};

// The part of a product that a launch computes: its tiles are the sub x sub
// parts of the tiles first, first + 1, ... (in raster order) of the tilesM x
// tilesN grid of sides sub * BT.  {0, 1}: all of it.
struct Part {
    int32_t first;
    int32_t sub;
};

// kOdd: the K step count may be odd (per-C-block masks, whose count varies
// per tile, with an odd bp / 32; split K loops): an odd last step runs
// alone after the step pairs.
// Eight waves per 256x256 tile, two per SIMD: wave (wm, wn) (wm < 2,
// wn < 4) computes rows 128 wm .. +127 and columns 64 wn .. +63 with 4x2
// MFMA blocks of 32x32 (128 accumulators).  With two waves on a SIMD, one
// wave's memory instructions issue while the other's MFMAs keep the pipe
// busy (one wave per SIMD left the pipe idle for about one MFMA slot per
// memory instruction).
// Tile forms.  128 (four waves of 64 x 64, two workgroups per CU) and 64 (four
// waves of 32 x 32, four workgroups per CU) run the same K loop; they read
// more LDS and L2 per flop (0.96 and 0.92 of the 256 form's FP32 rate at 4096
// x 4096 x 4096) but fill the CUs for products of few or ragged tiles: 2048 x
// 1536 over K = 4096, 917 us as 48 tiles of 256, 219 us as 768 of 64.  Every
// form sums an entry in the same order, bit for bit (pick_form chooses).
template <int BT_, int WR_, int WC_, int kEu_>
struct Tile {
    static constexpr int BT = BT_;                   // tile side
    static constexpr int WR = WR_;                   // waves along the rows
    static constexpr int WC = WC_;                   //   and the columns
    static constexpr int kWaves = WR * WC;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kI = BT / (32 * WR);        // 32x32 blocks per wave: rows
    static constexpr int kJ = BT / (32 * WC);        //   and columns
    static constexpr int kU = BT / (8 * kWaves);     // direct loads per wave and operand
    static constexpr int kEu = kEu_;                 // waves per SIMD
};
using Tile256 = Tile<256, 2, 4, 2>;
using Tile128 = Tile<128, 2, 2, 2>;
using Tile64 = Tile<64, 2, 2, 4>;

//
// Deep kernels (kDeep): a ring of four step buffers instead of two, loads
// issued three steps ahead, each step waiting for its own loads only.  For
// products with at most one workgroup per CU, whose short steps otherwise
// wait for the latency of a load each.  Steps run in fours, the last ones
// (any count) singly; the sums are the same.
template <typename P, typename S, bool kMask, bool kOdd, bool kSplit = false, bool kDeep = false>
__global__ __launch_bounds__(S::kThreads)
__attribute__((amdgpu_waves_per_eu(kDeep ? S::kEu / 2 : S::kEu, kDeep ? S::kEu / 2 : S::kEu)))
void gemm_kept_kernel(const void* __restrict__ At, int64_t ldat, const void* __restrict__ Bt,
                      int64_t ldbt, int64_t m, int64_t l, int32_t bp, BlockList kept,
                      int32_t nkept, int64_t lo_off, float scale,
                      float* __restrict__ C, int64_t ldc, int32_t tilesM, int32_t tilesN,
                      CMask cm, SplitK sk, Part pt) {
    // two K-step buffers per operand, separate arrays so that the compiler
    // can tell the tile loads in flight (into one) from the fragment reads
    // (from the other)
    constexpr int BT = S::BT;
    constexpr int kI = S::kI;
    constexpr int kJ = S::kJ;
    constexpr int kU = S::kU;
    constexpr int kParts = P::template parts<kI>;
    __shared__ __align__(1024) float As0[BT * 32];
    __shared__ __align__(1024) float As1[BT * 32];
    __shared__ __align__(1024) float Bs0[BT * 32];
    __shared__ __align__(1024) float Bs1[BT * 32];
    constexpr int kRing = kDeep ? BT * 32 : 1;
    __shared__ __align__(1024) float As2[kRing];
    __shared__ __align__(1024) float As3[kRing];
    __shared__ __align__(1024) float Bs2[kRing];
    __shared__ __align__(1024) float Bs3[kRing];
    constexpr int kLead = kDeep ? 3 : 1;         // steps ahead that loads are issued
    constexpr int kLoads = (kLead - 1) * 2 * kU; // loads of the steps after the next one
    __shared__ int32_t klist[kMask ? OS_MAX_BLOCKS + 1 : 1];   // per-tile kept list, count last

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar M0 and selects
    const int wm = wave / S::WC;
    const int wn = wave % S::WC;

    const int64_t ntiles = (int64_t)tilesM * tilesN;
    int32_t split = 0;
    int64_t T;
    int32_t sr = 0, sc = 0;              // part of the tile (sub > 1)
    if constexpr (kSplit) {
        split = (int32_t)(blockIdx.x / ntiles);
        T = (int64_t)blockIdx.x - (int64_t)split * ntiles;
    } else {
        T = xcd_task(blockIdx.x, gridDim.x);
        const int32_t c = (int32_t)(T % (pt.sub * pt.sub));
        T = pt.first + T / (pt.sub * pt.sub);
        sr = c / pt.sub;
        sc = c - sr * pt.sub;
    }
    const int64_t group = T / ((int64_t)kGroupM * tilesN);
    const int64_t first_m = group * kGroupM;
    const int64_t gsz = min((int64_t)kGroupM, (int64_t)tilesM - first_m);
    const int64_t in_group = T - group * kGroupM * tilesN;
    const int64_t tm = first_m + in_group % gsz;
    const int64_t tn = in_group / gsz;
    int64_t row0 = (tm * pt.sub + sr) * BT;
    int64_t col0 = (tn * pt.sub + sc) * BT;
    if constexpr (!kMask) {
        if (row0 >= m || col0 >= l) return;     // a part past the matrix (uniform)
    } else {
        // tile (tm, tn) of the C-block grid: block (I, J), tile (ti, tj) in it
        const int64_t I = tm / cm.tb, J = tn / cm.tb;
        row0 = I * cm.cblk + (tm % cm.tb * pt.sub + sr) * BT;
        col0 = J * cm.cblk + (tn % cm.tb * pt.sub + sc) * BT;
        m = min(m, (I + 1) * cm.cblk);          // rows and columns of this block only
        l = min(l, (J + 1) * cm.cblk);
        if (row0 >= m || col0 >= l) return;     // past a partial block's end (uniform)
        if (tid == 0) {
            const uint8_t* mk = cm.mask + (I * cm.nbJ + J) * cm.nstm;
            int32_t k = 0;
            for (int32_t j = 0; j < cm.nstm; ++j)
                if (mk[j]) klist[k++] = j;
            klist[OS_MAX_BLOCKS] = k;
        }
        __syncthreads();
        nkept = __builtin_amdgcn_readfirstlane(klist[OS_MAX_BLOCKS]);
        if (nkept == 0) {
            for (int64_t r = row0 + (tid >> 6); r < min(m, row0 + BT); r += S::kWaves)
                for (int64_t c = col0 + lane; c < min(l, col0 + BT); c += 64) C[r * ldc + c] = 0.f;
            return;
        }
        scale = 1.0f / (float)nkept;
    }
    // kept stored block of term index j: lane i of kv[q] holds entry 64q + i
    // of the kept list, read once here and picked with v_readlane, so the K
    // loop issues no scalar or LDS load for it (either would make the wave
    // wait for every LDS access in flight)
    int32_t kv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if constexpr (kMask)
            kv[q] = klist[64 * q + lane];
        else
            kv[q] = kept.idx[64 * q + lane];
    }
    auto kept_at = [&](int j) -> int32_t {
        const int32_t r0 = __builtin_amdgcn_readlane(kv[0], j & 63);
        const int32_t r1 = __builtin_amdgcn_readlane(kv[1], j & 63);
        const int32_t r2 = __builtin_amdgcn_readlane(kv[2], j & 63);
        const int32_t r3 = __builtin_amdgcn_readlane(kv[3], j & 63);
        return j < 64 ? r0 : (j < 128 ? r1 : (j < 192 ? r2 : r3));
    };

    v16f acc[kI][kJ];
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // K values per step
    constexpr int kStep = kStepBytes / P::kElem / (P::kPair ? 2 : 1);
    const int tpb = bp / kStep;                       // K steps per block
    int t_begin = 0;
    int t_end = nkept * tpb;                          // this workgroup's K steps
    if constexpr (kSplit) {
        t_begin = split * sk.chunk;
        t_end = min(t_end, t_begin + sk.chunk);
    }
    // byte offset of the first K column of step `step` in A's and B's rows
    auto step_k = [&](int step) -> uint32_t {
        return (uint32_t)(((int64_t)kept_at(step / tpb) * bp + (int64_t)(step % tpb) * kStep) *
                          P::kElem);
    };

    const __amdgpu_buffer_rsrc_t ra_src =
        tile_rsrc(static_cast<const char*>(At) + row0 * ldat * P::kElem);
    const __amdgpu_buffer_rsrc_t rb_src =
        tile_rsrc(static_cast<const char*>(Bt) + col0 * ldbt * P::kElem);
    uint32_t va[kU], vb[kU];
    const int alast = (int)min((int64_t)BT - 1, m - 1 - row0);
    const int blast = (int)min((int64_t)BT - 1, l - 1 - col0);
    if constexpr (P::kPair) {
        direct_offsets_pair<kU>(va, ldat * P::kElem, alast, lo_off * P::kElem, wave, lane);
        direct_offsets_pair<kU>(vb, ldbt * P::kElem, blast, lo_off * P::kElem, wave, lane);
    } else {
        direct_offsets<kU>(va, ldat * P::kElem, alast, wave, lane);
        direct_offsets<kU>(vb, ldbt * P::kElem, blast, wave, lane);
    }
    // fragment q of a lane half: K bytes 64 h + 16 q of the step, or (pair
    // steps) 32 h + 16 (q & 1) of the high (q < 2) or low part
    int fa_off[4], fb_off[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ra = wm * 32 * kI + (lane & 31), rb = wn * 32 * kJ + (lane & 31);
        fa_off[q] = P::kPair ? pair_frag_off(ra, q, lane) : direct_frag_off(ra, q, lane);
        fb_off[q] = P::kPair ? pair_frag_off(rb, q, lane) : direct_frag_off(rb, q, lane);
    }
    auto frag_a = [&](float4 (&a)[kI], const float* as, int q) {
#pragma unroll
        for (int i = 0; i < kI; ++i) a[i] = *reinterpret_cast<const float4*>(as + fa_off[q] + 1024 * i);
    };
    auto frag_b = [&](float4 (&b)[kJ], const float* bs, int q) {
#pragma unroll
        for (int j = 0; j < kJ; ++j) b[j] = *reinterpret_cast<const float4*>(bs + fb_off[q] + 1024 * j);
    };
    auto frag = [&](float4 (&a)[kI], float4 (&b)[kJ], const float* as, const float* bs, int q) {
        frag_a(a, as, q);
        frag_b(b, bs, q);
    };
    auto issue = [&](float* as, float* bs, int step) {
        const uint32_t k = step_k(step);
        direct_issue<kU>(ra_src, as, va, k, wave);
        direct_issue<kU>(rb_src, bs, vb, k, wave);
    };

    issue(As0, Bs0, t_begin);
    if constexpr (kDeep) {
        issue(As1, Bs1, min(t_begin + 1, t_end - 1));
        issue(As2, Bs2, min(t_begin + 2, t_end - 1));
    }
    wait_step<kLoads>();
    // (pair steps: fa, fb the high parts' fragments, ga, gb the low parts')
    float4 fa[kI], fb[kJ], ga[kI], gb[kJ];
    if constexpr (P::kPair) {
        frag_a(fa, As0, 0);
        frag_b(gb, Bs0, 2);
    } else {
        frag(fa, fb, As0, Bs0, 0);
    }
    // One K step: the next step's tiles go straight into the other buffers
    // (last read before the previous step's barrier) while this step's four
    // quads run; each quad's fragments are read during the previous quad's
    // MFMAs, after its first kHead parts, and the last quad's final kTail
    // parts run after the step's barrier, behind the reads of the next
    // step's first fragments (scheduling barriers pin this order).  The A
    // tile's loads are issued at the step's start and the B tile's after the
    // first quad, which halves the burst of line requests a CU sends at once
    // (the same loads; 2-3 % faster for BF16, 1 % for FP32); all are waited
    // for at the step's end.
    // Past the last step the tile loaded is step t_end - 1 again, a valid
    // address.  Steps run in pairs (one per buffer); when their count is odd
    // (kOdd kernels only) the last step runs alone after the pairs, from
    // the first buffer, where the last pair loaded it.
    auto quad = [&](float4 (&a)[kI], float4 (&b)[kJ], auto&& reads) {
        P::template mfma_quad<kI, kJ, 0, P::kHead>(acc, a, b);
        __builtin_amdgcn_sched_barrier(0);
        reads();
        __builtin_amdgcn_sched_barrier(0);
        P::template mfma_quad<kI, kJ, P::kHead, kParts>(acc, a, b);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mfma = [&](const float4 (&a)[kI], const float4 (&b)[kJ]) {
        P::template mfma_quad<kI, kJ>(acc, a, b);
        __builtin_amdgcn_sched_barrier(0);
    };
    // (as, bs: this step's buffers; xa, xb: the next step's; na, nb: those that
    // are loaded, the next step's unless kDeep)
    auto kstep = [&](const float* as, const float* bs, const float* xa, const float* xb, float* na,
                     float* nb, int t) {
        const uint32_t k = step_k(min(t + kLead, t_end - 1));
        direct_issue<kU>(ra_src, na, va, k, wave);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (P::kPair) {
            // per 16 K values: hi*lo', hi*hi', lo*hi'; each fragment is read
            // while the term before the one that needs it runs
            frag_b(fb, bs, 0);
            frag_a(ga, as, 2);
            __builtin_amdgcn_sched_barrier(0);
            mfma(fa, gb);
            direct_issue<kU>(rb_src, nb, vb, k, wave);
            frag_b(gb, bs, 3);
            __builtin_amdgcn_sched_barrier(0);
            mfma(fa, fb);
            frag_a(fa, as, 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma(ga, fb);
            frag_b(fb, bs, 1);
            frag_a(ga, as, 3);
            __builtin_amdgcn_sched_barrier(0);
            mfma(fa, gb);
            mfma(fa, fb);
            wait_step<kLoads>();
            frag_a(fa, xa, 0);
            frag_b(gb, xb, 2);
            __builtin_amdgcn_sched_barrier(0);
            mfma(ga, fb);
        } else {
            quad(fa, fb, [&] { frag(ga, gb, as, bs, 1); });
            direct_issue<kU>(rb_src, nb, vb, k, wave);
            __builtin_amdgcn_sched_barrier(0);
            quad(ga, gb, [&] { frag(fa, fb, as, bs, 2); });
            quad(fa, fb, [&] { frag(ga, gb, as, bs, 3); });
            P::template mfma_quad<kI, kJ, 0, kParts - P::kTail>(acc, ga, gb);
            __builtin_amdgcn_sched_barrier(0);
            wait_step<kLoads>();
            frag(fa, fb, xa, xb, 0);
            __builtin_amdgcn_sched_barrier(0);
            P::template mfma_quad<kI, kJ, kParts - P::kTail, kParts>(acc, ga, gb);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int t = t_begin;
    if constexpr (kDeep) {
        for (; t + 3 < t_end; t += 4) {
            kstep(As0, Bs0, As1, Bs1, As3, Bs3, t);
            kstep(As1, Bs1, As2, Bs2, As0, Bs0, t + 1);
            kstep(As2, Bs2, As3, Bs3, As1, Bs1, t + 2);
            kstep(As3, Bs3, As0, Bs0, As2, Bs2, t + 3);
        }
        if (t < t_end) kstep(As0, Bs0, As1, Bs1, As3, Bs3, t);
        if (t + 1 < t_end) kstep(As1, Bs1, As2, Bs2, As0, Bs0, t + 1);
        if (t + 2 < t_end) kstep(As2, Bs2, As3, Bs3, As1, Bs1, t + 2);
        __builtin_amdgcn_s_waitcnt(0);       // no load into LDS outlives the workgroup
    } else {
        for (; t + 1 < t_end; t += 2) {
            kstep(As0, Bs0, As1, Bs1, As1, Bs1, t);
            kstep(As1, Bs1, As0, Bs0, As0, Bs0, t + 1);
        }
        if constexpr (kOdd) {
            if (t < t_end) kstep(As0, Bs0, As1, Bs1, As1, Bs1, t);
        }
    }

    // 32x32 accumulator layout: register r of lane L holds row
    // 8*(r/4) + 4*(L/32) + r%4 and column L%32 of the block.
    float* out = C;
    int64_t ldo = ldc;
    if constexpr (kSplit) {
        out = sk.part + (int64_t)split * m * l;
        ldo = l;
        scale = 1.0f;
    }
#pragma unroll
    for (int i = 0; i < kI; ++i) {
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
            const int64_t col = col0 + wn * 32 * kJ + j * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = row0 + wm * 32 * kI + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (row < m && col < l) out[row * ldo + col] = acc[i][j][r] * scale;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Small products: one 32 x 32 tile of C per workgroup, the K steps dealt to
// its kSmallWaves waves (wave w takes steps w, w + kSmallWaves, ...), each
// wave's fragments loaded straight from the sketches into registers (a lane
// reads the 64 bytes of its row that its half of a step uses), the waves'
// partial tiles added in wave order through LDS; a wave sums even and odd
// quads apart (16 partial sums per entry: 600 x 300 over K = 832 FP32, relative
// error 1.84e-7 with 8, 1.39e-7, where the split K loop has 1.53e-7; the same
// time).  Bound by latency: a product
// of one or a few 256 tiles has too little work for tiles staged through LDS
// and a second launch for the sum of split partials.  (96 x 128 over K =
// 512: 26.4 us as one 256 tile split 8 ways and its sum, 7.1 us.)
// ---------------------------------------------------------------------------
constexpr int kSmallWaves = 8;
constexpr int kSmallSums = 2 * kSmallWaves;     // partial sums per entry
constexpr int kSmallTile = 32;

template <typename P>
__global__ __launch_bounds__(64 * kSmallWaves)
void gemm_small_kernel(const void* __restrict__ At, int64_t ldat, const void* __restrict__ Bt,
                       int64_t ldbt, int64_t m, int64_t l, int32_t bp, BlockList kept,
                       int32_t nkept, int64_t lo_off, float scale,
                       float* __restrict__ C, int64_t ldc, int32_t tilesM, int32_t tilesN) {
    __shared__ float red[kSmallWaves][kSmallTile * kSmallTile];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t T = xcd_task(blockIdx.x, (int64_t)tilesM * tilesN);
    const int64_t row0 = T / tilesN * kSmallTile;
    const int64_t col0 = T % tilesN * kSmallTile;

    int32_t kv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) kv[q] = kept.idx[64 * q + lane];
    auto kept_at = [&](int j) -> int32_t {
        const int32_t r0 = __builtin_amdgcn_readlane(kv[0], j & 63);
        const int32_t r1 = __builtin_amdgcn_readlane(kv[1], j & 63);
        const int32_t r2 = __builtin_amdgcn_readlane(kv[2], j & 63);
        const int32_t r3 = __builtin_amdgcn_readlane(kv[3], j & 63);
        return j < 64 ? r0 : (j < 128 ? r1 : (j < 192 ? r2 : r3));
    };
    constexpr int kStep = kStepBytes / P::kElem / (P::kPair ? 2 : 1);
    const int tpb = bp / kStep;
    const int total = nkept * tpb;
    // rows past the matrix read its last row (their sums are not stored)
    const int half = (P::kPair ? 32 : 64) * (lane >> 5);
    const char* pa = static_cast<const char*>(At) +
                     min(row0 + (lane & 31), m - 1) * ldat * P::kElem + half;
    const char* pb = static_cast<const char*>(Bt) +
                     min(col0 + (lane & 31), l - 1) * ldbt * P::kElem + half;
    auto load = [&](float4 (&a)[4], float4 (&b)[4], int step) {
        const int64_t k = ((int64_t)kept_at(step / tpb) * bp + (int64_t)(step % tpb) * kStep) *
                          P::kElem;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t at = k + (P::kPair ? 16 * (q & 1) + (q < 2 ? 0 : lo_off * P::kElem) : 16 * q);
            a[q] = *reinterpret_cast<const float4*>(pa + at);
            b[q] = *reinterpret_cast<const float4*>(pb + at);
        }
    };
    v16f acc[2][1][1];            // even and odd quads
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[h][0][0][r] = 0.f;
    auto sum = [&](const float4 (&a)[4], const float4 (&b)[4]) {
        auto term = [&](int qa, int qb) {
            const float4 x[1] = {a[qa]}, y[1] = {b[qb]};
            P::template mfma_quad<1, 1>(acc[qa & 1], x, y);
        };
        if constexpr (P::kPair) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                term(q, 2 + q);
                term(q, q);
                term(2 + q, q);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) term(q, q);
        }
    };
    if (wave < total) {
        float4 a0[4], b0[4], a1[4], b1[4];
        load(a0, b0, wave);
        int t = wave;
        // two steps in flight; past the end the last step is loaded again
        for (; t + kSmallWaves < total; t += 2 * kSmallWaves) {
            load(a1, b1, t + kSmallWaves);
            sum(a0, b0);
            load(a0, b0, min(t + 2 * kSmallWaves, total - 1));
            sum(a1, b1);
        }
        if (t < total) sum(a0, b0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
        red[wave][(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * kSmallTile + (lane & 31)] =
            acc[0][0][0][r] + acc[1][0][0][r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSmallTile * kSmallTile / (64 * kSmallWaves); ++u) {
        const int e = u * 64 * kSmallWaves + tid;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) v += red[w][e];
        const int64_t row = row0 + e / kSmallTile, col = col0 + e % kSmallTile;
        if (row < m && col < l) C[row * ldc + col] = v * scale;
    }
}

// C = scale * (sum of the nsplit partial products, in split order).
__global__ __launch_bounds__(256) void split_sum_kernel(const float* __restrict__ part,
                                                        int32_t nsplit, int64_t m, int64_t l,
                                                        float scale, float* __restrict__ C,
                                                        int64_t ldc) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= m * l) return;
    const int64_t row = i / l;
    // eight partials in flight (past the last one it is read again, not added)
    float v = 0.f;
    for (int32_t s = 0; s < nsplit; s += 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = part[(int64_t)min(s + u, nsplit - 1) * m * l + i];
#pragma unroll
        for (int u = 0; u < 8; ++u) v = s + u < nsplit ? v + x[u] : v;
    }
    C[row * ldc + (i - row * l)] = v * scale;
}

typedef int i32x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------
// FP8 (E4M3) operands with one E8M0 scale per 64 K values of a row, on the
// gfx950 scaled MFMA v_mfma_scale_f32_32x32x64_f8f6f4 (FP32 accumulation; the
// hardware multiplies the products by the row scales of A and B).  A row of
// an operand holds its codes, then one scale byte per 64 codes (`scales`
// bytes after the row's start).  The pipeline and the tile forms are
// gemm_kept_kernel's (a 64 form was slower than the 128 form throughout), K
// steps of 128 bytes of every tile row loaded straight into LDS, two step
// buffers.  A step is two 64-byte parts, one scale block each; lane half h
// holds the 32 codes at byte 64 p + 32 h of the step's row (two 16-byte LDS
// reads: logical chunks 4 p + 2 h and 4 p + 2 h + 1), both halves passing the
// block's scale.
//   plain (kPair = false): the parts are 128 consecutive codes, one scaled
//     MFMA per part and 32x32 block;
//   split (kPair): part 0 is 64 codes of the high part, part 1 the 64 codes
//     of the low part at the same columns (lo_off bytes on); hi*lo' + hi*hi'
//     + lo*hi', three MFMAs per block from one load of the four tiles
//     (4096 x 4096, K = 4096, blocks of 1024: 154 us, 2680 TFLOP/s, where
//     three separate passes of the K loop reached 2210-2310).
// Scale bytes: part p of a step has one byte per row, at column byte c / 64
// of the scale area (c = the part's first code column).  Every step each
// wave loads the aligned 4-byte word that holds it for 64 rows straight into
// LDS (plain: both parts' bytes are in one word; split: a word per part),
// laid out so that a fragment lane's kI A rows (or kJ B rows) are consecutive
// words.  (No branch around these loads: a wave-uniform one made the kernel
// spill 200-400 bytes per lane and run at less than half the speed.)
// Scale chunks: the scale loads above read 64 rows per instruction, one
// 4-byte piece each, and cost about as much as a whole step's tile loads;
// instead each wave loads kChunk bytes of its 64 rows at once (16: the
// scales of 8 steps, or of one part of 16 split steps, when the block stride
// is a multiple of 1024 codes and rows and the scale area are 16-byte
// aligned; 4: of 2 or 4 steps, when it is a multiple of 256), into one of two
// chunk buffers, and each step reads its scale bytes from there (a chunk is
// loaded during the first step of the one before it).
// (Split, 2048 x 2048, K = 2048, blocks of 512: 57 us loading every step, 48
// with 4-byte chunks; blocks of 1024 with 16-byte chunks: 46.)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int fp8_frag_off(int rbase, int s, int p, int lane) {
    return rbase * 32 + 4 * ((4 * s + 2 * (lane >> 5) + p) ^ chunk_key(rbase));
}

// kN (2 or 4) consecutive words of LDS, aligned to as many
template <int kN>
__device__ __forceinline__ void words(uint32_t (&d)[kN], const uint32_t* p) {
    if constexpr (kN == 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(p);
        d[0] = v.x;
        d[1] = v.y;
        d[2] = v.z;
        d[3] = v.w;
    } else {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        d[0] = v.x;
        d[1] = v.y;
    }
}

template <typename S, bool kPair, bool kOdd, bool kSplit = false, int kChunk = 0,
          bool kDeep = false>
__global__ __launch_bounds__(S::kThreads)
__attribute__((amdgpu_waves_per_eu(kDeep ? 1 : 2, kDeep ? 1 : 2)))
void gemm_kept_fp8d_kernel(const uint8_t* __restrict__ At, int64_t ldat,
                           const uint8_t* __restrict__ Bt, int64_t ldbt, int64_t scales,
                           int64_t m, int64_t l, int32_t bp, BlockList kept, int32_t nkept,
                           int64_t lo_off, float scale, float* __restrict__ C, int64_t ldc,
                           int32_t tilesM, int32_t tilesN, SplitK sk, Part pt) {
    constexpr int BT = S::BT;
    constexpr int kI = S::kI;
    constexpr int kJ = S::kJ;
    constexpr int kU = S::kU;
    __shared__ __align__(1024) float As0[BT * 32];
    __shared__ __align__(1024) float As1[BT * 32];
    __shared__ __align__(1024) float Bs0[BT * 32];
    __shared__ __align__(1024) float Bs1[BT * 32];
    constexpr int kRing = kDeep ? BT * 32 : 1;
    __shared__ __align__(1024) float As2[kRing];
    __shared__ __align__(1024) float As3[kRing];
    __shared__ __align__(1024) float Bs2[kRing];
    __shared__ __align__(1024) float Bs3[kRing];
    constexpr int kLead = kDeep ? 3 : 1;         // steps ahead that loads are issued
    constexpr int kLoads = (kLead - 1) * 2 * kU; // loads of the steps after the next one
    // scale words, two buffers: per row (A's, then B's) a word per loaded
    // part (kWords of them), or 16 bytes per row and loaded part
    constexpr int kWords = kPair ? 2 : 1;
    constexpr int kScaleBuf = kWords * 2 * BT * (kChunk == 16 ? 4 : 1);
    __shared__ __align__(16) uint32_t Sc[2 * kScaleBuf];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar M0 and selects
    const int wm = wave / S::WC;
    const int wn = wave % S::WC;

    const int64_t ntiles = (int64_t)tilesM * tilesN;
    int32_t split = 0;
    int64_t T;
    int32_t sr = 0, sc = 0;              // part of the tile (sub > 1)
    if constexpr (kSplit) {
        split = (int32_t)(blockIdx.x / ntiles);
        T = (int64_t)blockIdx.x - (int64_t)split * ntiles;
    } else {
        T = xcd_task(blockIdx.x, gridDim.x);
        const int32_t c = (int32_t)(T % (pt.sub * pt.sub));
        T = pt.first + T / (pt.sub * pt.sub);
        sr = c / pt.sub;
        sc = c - sr * pt.sub;
    }
    const int64_t group = T / ((int64_t)kGroupM * tilesN);
    const int64_t first_m = group * kGroupM;
    const int64_t gsz = min((int64_t)kGroupM, (int64_t)tilesM - first_m);
    const int64_t in_group = T - group * kGroupM * tilesN;
    const int64_t tm = first_m + in_group % gsz;
    const int64_t tn = in_group / gsz;
    const int64_t row0 = (tm * pt.sub + sr) * BT;
    const int64_t col0 = (tn * pt.sub + sc) * BT;
    if (row0 >= m || col0 >= l) return;         // a part past the matrix (uniform)

    int32_t kv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) kv[q] = kept.idx[64 * q + lane];
    auto kept_at = [&](int j) -> int32_t {
        const int32_t r0 = __builtin_amdgcn_readlane(kv[0], j & 63);
        const int32_t r1 = __builtin_amdgcn_readlane(kv[1], j & 63);
        const int32_t r2 = __builtin_amdgcn_readlane(kv[2], j & 63);
        const int32_t r3 = __builtin_amdgcn_readlane(kv[3], j & 63);
        return j < 64 ? r0 : (j < 128 ? r1 : (j < 192 ? r2 : r3));
    };

    v16f acc[kI][kJ];
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    constexpr int kStep = kPair ? 64 : 128;           // code columns per step
    constexpr int kPerChunk = kPair ? kChunk : kChunk / 2;   // steps per scale chunk
    // kDeep: as in gemm_kept_kernel, scales in chunks of at least four steps: a
    // chunk is loaded during the first step of the one before it, so that more
    // than kLoads later loads follow it by the end of that one.
    static_assert(!kDeep || (!kSplit && kPerChunk >= 4));
    const int tpb = bp / kStep;
    int t_begin = 0;
    int t_end = nkept * tpb;                          // this workgroup's K steps
    if constexpr (kSplit) {
        t_begin = split * sk.chunk;
        t_end = min(t_end, t_begin + sk.chunk);
    }
    // first code column (= byte) of step `step`
    auto step_k = [&](int step) -> uint32_t {
        return (uint32_t)((int64_t)kept_at(step / tpb) * bp + (int64_t)(step % tpb) * kStep);
    };

    const int alast = (int)min((int64_t)BT - 1, m - 1 - row0);
    const int blast = (int)min((int64_t)BT - 1, l - 1 - col0);
    const __amdgpu_buffer_rsrc_t ra_src = tile_rsrc(At + row0 * ldat);
    const __amdgpu_buffer_rsrc_t rb_src = tile_rsrc(Bt + col0 * ldbt);
    uint32_t va[kU], vb[kU];
    if constexpr (kPair) {
        direct_offsets_pair<kU>(va, ldat, alast, lo_off, wave, lane);
        direct_offsets_pair<kU>(vb, ldbt, blast, lo_off, wave, lane);
    } else {
        direct_offsets<kU>(va, ldat, alast, wave, lane);
        direct_offsets<kU>(vb, ldbt, blast, wave, lane);
    }
    // scale rows of this wave: word p = 64 (wave % (BT / 64)) + lane of A's
    // (the first BT / 64 waves) or B's (the next) area holds row srow (kI
    // consecutive words per A fragment lane: rows wm * 32 kI + 32 i + r; kJ per
    // B fragment lane).  Chunks keep rows in their natural order, so that the
    // 32 lanes of a fragment half read 16-byte-spaced entries (two lanes per
    // bank) instead of 16 kI-byte-spaced ones.
    constexpr int kSw = BT / 64;
    static_assert(2 * kSw == S::kWaves, "every wave loads the scales of 64 rows");
    const bool a_side = wave < kSw;
    const int p = 64 * (wave % kSw) + lane;
    constexpr int kIw = 32 * kI, kJw = 32 * kJ;
    const int srow = kChunk == 16 ? p
                     : a_side ? p / kIw * kIw + 32 * (p % kI) + ((p / kI) & 31)
                              : p / kJw * kJw + 32 * (p % kJ) + ((p / kJ) & 31);
    const uint32_t so = a_side ? (uint32_t)((int64_t)min(srow, alast) * ldat + scales)
                               : (uint32_t)((int64_t)min(srow, blast) * ldbt + scales);
    const __amdgpu_buffer_rsrc_t rs_src = a_side ? ra_src : rb_src;
    const int sbase = a_side ? 64 * (wave % kSw) : BT + 64 * (wave % kSw);

    // the scale words of a step (or the chunk it starts) into buffer `buf`
    auto issue_scales = [&](int buf, uint32_t k) {
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (kChunk == 16) {
            uint32_t* d = Sc + buf * kScaleBuf + 4 * sbase;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_src, (lds_void*)d, 16, so, k / kFp8Block,
                                                     0, 0);
            if constexpr (kPair)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rs_src, (lds_void*)(d + 8 * BT), 16, so,
                    (uint32_t)((k + lo_off) / kFp8Block), 0, 0);
        } else {
            uint32_t* d = Sc + buf * kScaleBuf + sbase;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_src, (lds_void*)d, 4, so,
                                                     (k / kFp8Block) & ~3u, 0, 0);
            if constexpr (kPair)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rs_src, (lds_void*)(d + 2 * BT), 4, so,
                    (uint32_t)((k + lo_off) / kFp8Block) & ~3u, 0, 0);
        }
#else
        (void)buf;
        (void)k;
        (void)so;
        (void)rs_src;
        (void)sbase;
#endif
    };

    int fa_off[2][2], fb_off[2][2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            fa_off[s2][q] = fp8_frag_off(wm * kIw + (lane & 31), s2, q, lane);
            fb_off[s2][q] = fp8_frag_off(wn * kJw + (lane & 31), s2, q, lane);
        }
    auto as_i32x8 = [](const float4& lo, const float4& hi) -> i32x8 {
        return i32x8{__float_as_int(lo.x), __float_as_int(lo.y), __float_as_int(lo.z),
                     __float_as_int(lo.w), __float_as_int(hi.x), __float_as_int(hi.y),
                     __float_as_int(hi.z), __float_as_int(hi.w)};
    };
    // A fragment of row block i of part s2; B fragments of part s2
    auto frag_a = [&](const float* as, int s2, int i) -> i32x8 {
        return as_i32x8(*reinterpret_cast<const float4*>(as + fa_off[s2][0] + 1024 * i),
                        *reinterpret_cast<const float4*>(as + fa_off[s2][1] + 1024 * i));
    };
    auto frag_b = [&](i32x8 (&b)[kJ], const float* bs, int s2) {
#pragma unroll
        for (int j = 0; j < kJ; ++j)
            b[j] = as_i32x8(*reinterpret_cast<const float4*>(bs + fb_off[s2][0] + 1024 * j),
                            *reinterpret_cast<const float4*>(bs + fb_off[s2][1] + 1024 * j));
    };
    // the step's scale bytes of the lane's A and B rows: part 0 in byte 0,
    // part 1 in byte 1
    uint32_t sa[kI], sb[kJ];
    auto read_scales = [&](int step, int buf, uint32_t k) {
        if constexpr (kChunk == 16) {
            const uint8_t* q = reinterpret_cast<const uint8_t*>(Sc + ((step / kPerChunk) & 1) * kScaleBuf);
            const int ra = wm * kIw + (lane & 31), rb = BT + wn * kJw + (lane & 31);
            auto at = [&](int row) -> uint32_t {
                if constexpr (kPair) {
                    const uint8_t* e = q + 16 * row + (step & 15);
                    return e[0] | (uint32_t)e[32 * BT] << 8;
                } else {
                    return *reinterpret_cast<const uint16_t*>(q + 16 * row + 2 * (step & 7));
                }
            };
#pragma unroll
            for (int i = 0; i < kI; ++i) sa[i] = at(ra + 32 * i);
#pragma unroll
            for (int j = 0; j < kJ; ++j) sb[j] = at(rb + 32 * j);
        } else {
            const uint32_t* q = Sc + (kChunk ? (step / kPerChunk) & 1 : buf) * kScaleBuf;
            const int wa = kI * (wm * 32 + (lane & 31)), wb = BT + kJ * (wn * 32 + (lane & 31));
            const uint32_t h0 = (k / kFp8Block & 3u) * 8u;
            words<kI>(sa, q + wa);
            words<kJ>(sb, q + wb);
#pragma unroll
            for (int i = 0; i < kI; ++i) sa[i] >>= h0;
#pragma unroll
            for (int j = 0; j < kJ; ++j) sb[j] >>= h0;
            if constexpr (kPair) {
                const uint32_t h1 = ((uint32_t)((k + lo_off) / kFp8Block) & 3u) * 8u;
                uint32_t la[kI], lb[kJ];
                words<kI>(la, q + 2 * BT + wa);
                words<kJ>(lb, q + 2 * BT + wb);
#pragma unroll
                for (int i = 0; i < kI; ++i) sa[i] = (sa[i] & 0xFFu) | (la[i] >> h1 & 0xFFu) << 8;
#pragma unroll
                for (int j = 0; j < kJ; ++j) sb[j] = (sb[j] & 0xFFu) | (lb[j] >> h1 & 0xFFu) << 8;
            }
        }
    };
    auto mfma = [&](v16f& c, const i32x8& a, const i32x8& b, uint32_t s_a, uint32_t s_b, int pa,
                    int pb) {
        c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0,
                                                            (int)((s_a >> (8 * pa)) & 0xFFu), 0,
                                                            (int)((s_b >> (8 * pb)) & 0xFFu));
    };

    {
        const uint32_t k = step_k(t_begin);
        direct_issue<kU>(ra_src, As0, va, k, wave);
        direct_issue<kU>(rb_src, Bs0, vb, k, wave);
        issue_scales(0, k);        // (t_begin is even, and 0 with chunks)
    }
    if constexpr (kDeep) {
        const uint32_t k1 = step_k(min(t_begin + 1, t_end - 1));
        direct_issue<kU>(ra_src, As1, va, k1, wave);
        direct_issue<kU>(rb_src, Bs1, vb, k1, wave);
        const uint32_t k2 = step_k(min(t_begin + 2, t_end - 1));
        direct_issue<kU>(ra_src, As2, va, k2, wave);
        direct_issue<kU>(rb_src, Bs2, vb, k2, wave);
    }
    wait_step<kLoads>();
    // plain: fa / fan one part's A fragment and the next one's, fb / fbn the
    // parts' B fragments; split: fa / ga one row block's high and low
    // fragments, fan / gan the next one's, fb / fbn the B parts
    i32x8 fa, fan, ga, gan, fb[kJ], fbn[kJ];
    fa = frag_a(As0, 0, 0);
    frag_b(fb, Bs0, 0);
    if constexpr (kPair) {
        ga = frag_a(As0, 1, 0);
        frag_b(fbn, Bs0, 1);
    }
    read_scales(t_begin, 0, step_k(t_begin));
    // One step: the next step's tiles and scale words go straight into the
    // other buffers while this step runs (the A tile and scales at the step's
    // start, the B tile after a quarter of its MFMAs, as in gemm_kept_kernel:
    // about 2 % faster); the A fragment of the next (part, row block) is
    // read during the current one's MFMAs, and part 1's B fragments during
    // part 0's last row block.  Steps run in pairs; an odd last step (kOdd)
    // runs alone after them.
    auto kstep = [&](const float* as, const float* bs, const float* xa, const float* xb, float* na,
                     float* nb, int nbuf, int t) {
        const uint32_t k = step_k(min(t + kLead, t_end - 1));
        direct_issue<kU>(ra_src, na, va, k, wave);
        if constexpr (kChunk != 0) {
            // (nbuf, kDeep: the step's place in its four; t_begin is 0)
            if ((!kDeep || nbuf == 0) && t % kPerChunk == 0 &&
                t + kPerChunk < t_end)
                issue_scales((t / kPerChunk + 1) & 1, step_k(t + kPerChunk));
        } else {
            issue_scales(nbuf, k);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kPair) {
#pragma unroll
            for (int i = 0; i < kI; ++i) {
                if (i + 1 < kI) {
                    fan = frag_a(as, 0, i + 1);
                    gan = frag_a(as, 1, i + 1);
                }
#pragma unroll
                for (int j = 0; j < kJ; ++j) mfma(acc[i][j], fa, fbn[j], sa[i], sb[j], 0, 1);
                if (i == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    direct_issue<kU>(rb_src, nb, vb, k, wave);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int j = 0; j < kJ; ++j) mfma(acc[i][j], fa, fb[j], sa[i], sb[j], 0, 0);
#pragma unroll
                for (int j = 0; j < kJ; ++j) mfma(acc[i][j], ga, fb[j], sa[i], sb[j], 1, 0);
                if (i + 1 < kI) {
                    fa = fan;
                    ga = gan;
                }
            }
        } else {
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
                for (int i = 0; i < kI; ++i) {
                    if (s2 == 0 && i == kI / 2) {
                        __builtin_amdgcn_sched_barrier(0);
                        direct_issue<kU>(rb_src, nb, vb, k, wave);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (i + 1 < kI) {
                        fan = frag_a(as, s2, i + 1);
                    } else if (s2 == 0) {
                        fan = frag_a(as, 1, 0);
                        frag_b(fbn, bs, 1);
                    }
#pragma unroll
                    for (int j = 0; j < kJ; ++j) mfma(acc[i][j], fa, fb[j], sa[i], sb[j], s2, s2);
                    if (i + 1 < kI || s2 == 0) fa = fan;
                }
                if (s2 == 0) {
#pragma unroll
                    for (int j = 0; j < kJ; ++j) fb[j] = fbn[j];
                }
            }
        }
        wait_step<kLoads>();
        fa = frag_a(xa, 0, 0);
        frag_b(fb, xb, 0);
        if constexpr (kPair) {
            ga = frag_a(xa, 1, 0);
            frag_b(fbn, xb, 1);
        }
        const int tn = min(t + 1, t_end - 1);
        read_scales(tn, nbuf, kDeep ? step_k(tn) : k);
    };
    int t = t_begin;
    if constexpr (kDeep) {
        for (; t + 3 < t_end; t += 4) {
            kstep(As0, Bs0, As1, Bs1, As3, Bs3, 0, t);
            kstep(As1, Bs1, As2, Bs2, As0, Bs0, 1, t + 1);
            kstep(As2, Bs2, As3, Bs3, As1, Bs1, 2, t + 2);
            kstep(As3, Bs3, As0, Bs0, As2, Bs2, 3, t + 3);
        }
        if (t < t_end) kstep(As0, Bs0, As1, Bs1, As3, Bs3, 0, t);
        if (t + 1 < t_end) kstep(As1, Bs1, As2, Bs2, As0, Bs0, 1, t + 1);
        if (t + 2 < t_end) kstep(As2, Bs2, As3, Bs3, As1, Bs1, 2, t + 2);
        __builtin_amdgcn_s_waitcnt(0);       // no load into LDS outlives the workgroup
    } else {
        for (; t + 1 < t_end; t += 2) {
            kstep(As0, Bs0, As1, Bs1, As1, Bs1, 1, t);
            kstep(As1, Bs1, As0, Bs0, As0, Bs0, 0, t + 1);
        }
        if constexpr (kOdd) {
            if (t < t_end) kstep(As0, Bs0, As1, Bs1, As1, Bs1, 1, t);
        }
    }

    float* out = C;
    int64_t ldo = ldc;
    if constexpr (kSplit) {
        out = sk.part + (int64_t)split * m * l;
        ldo = l;
        scale = 1.0f;
    }

#pragma unroll
    for (int i = 0; i < kI; ++i) {
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
            const int64_t col = col0 + wn * kJw + j * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = row0 + wm * kIw + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (row < m && col < l) out[row * ldo + col] = acc[i][j][r] * scale;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Grouped symmetric block product for a batch of sketched Gram matrices:
//   H_k = scale_k * S_k S_k^T, S_k the line-major sketch (m_k rows) of
//   problem k with only its kept blocks stored, so the sum over the kept
//   blocks runs over its first ksteps * 32 columns (padding columns are
//   zero; ksteps is even, the sketch carrying one more zero step when K*bp/32
//   is odd).  One persistent launch over a tile list that holds the
//   upper-triangle tiles (ti <= tj) of every problem.  Workgroup g takes
//   tiles starts[g] .. starts[g+1] - 1 (a static schedule balanced on the
//   host; every wave reaches its end), computing each with the same FP32
//   MFMA pipeline as above; an off-diagonal tile is also stored
//   transposed (mirror) when `full`.
// kWT = 4: 256 x 256 tiles, eight waves of 128 x 64 (two per SIMD, as in
// gemm_kept_kernel); kWT = 2: 128 x 128 tiles, four waves of 64 x 64 and two
// workgroups per CU (less padding on small problems).
// ---------------------------------------------------------------------------
template <int kWT>
struct TileShape {
    static constexpr int BT = 64 * kWT;                // tile side
    static constexpr int kWaves = 2 * kWT;             // 8 (256 tiles) or 4 (128 tiles)
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kI = kWT;                     // 32x32 blocks per wave: rows
    static constexpr int kJ = 2;                       //   and columns
    static constexpr int kU = BT / (8 * kWaves);       // direct loads per wave per operand
};


template <int kWT>
__global__ __launch_bounds__(TileShape<kWT>::kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_batch_sym_kernel(const BatchProblem* __restrict__ probs,
                           const int4* __restrict__ tiles, const int32_t* __restrict__ starts,
                           int full) {
    using TS = TileShape<kWT>;
    constexpr int BT = TS::BT;
    constexpr int kU = TS::kU;
    constexpr int kI = TS::kI;
    constexpr int kJ = TS::kJ;
    // direct tiles as in gemm_kept_kernel: separate arrays per buffer
    __shared__ __align__(1024) float As0[BT * 32];
    __shared__ __align__(1024) float As1[BT * 32];
    __shared__ __align__(1024) float Bs0[BT * 32];
    __shared__ __align__(1024) float Bs1[BT * 32];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / (TS::kWaves / 2);      // 2 waves along the rows
    const int wn = wave % (TS::kWaves / 2);      // kWaves / 2 along the columns
    int fa_off[4], fb_off[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        fa_off[q] = direct_frag_off(wm * 32 * kI + (lane & 31), q, lane);
        fb_off[q] = direct_frag_off(wn * 32 * kJ + (lane & 31), q, lane);
    }
    auto frag = [&](float4 (&a)[kI], float4 (&b)[kJ], const float* as, const float* bs, int q) {
#pragma unroll
        for (int i = 0; i < kI; ++i) a[i] = *reinterpret_cast<const float4*>(as + fa_off[q] + 1024 * i);
#pragma unroll
        for (int j = 0; j < kJ; ++j) b[j] = *reinterpret_cast<const float4*>(bs + fb_off[q] + 1024 * j);
    };

    const int32_t w_end = starts[blockIdx.x + 1];
    for (int32_t w = starts[blockIdx.x]; w < w_end; ++w) {
        const int4 tl = tiles[w];
        const BatchProblem pr = probs[tl.x];
        const int64_t m = pr.m;
        const int64_t row0 = (int64_t)tl.y * BT;
        const int64_t col0 = (int64_t)tl.z * BT;
        const int total = pr.ksteps;          // even: the sketch is padded to whole step pairs
        const __amdgpu_buffer_rsrc_t ra_src = tile_rsrc(pr.S + row0 * pr.ld);
        const __amdgpu_buffer_rsrc_t rb_src = tile_rsrc(pr.S + col0 * pr.ld);
        uint32_t va[kU], vb[kU];
        direct_offsets<kU>(va, pr.ld * 4, (int)min((int64_t)BT - 1, m - 1 - row0), wave, lane);
        direct_offsets<kU>(vb, pr.ld * 4, (int)min((int64_t)BT - 1, m - 1 - col0), wave, lane);
        auto issue = [&](float* as, float* bs, int step) {
            direct_issue<kU>(ra_src, as, va, (uint32_t)step * kStepBytes, wave);
            direct_issue<kU>(rb_src, bs, vb, (uint32_t)step * kStepBytes, wave);
        };

        v16f acc[kI][kJ];
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
            for (int j = 0; j < kJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();                       // the previous tile's last reads are done
        issue(As0, Bs0, 0);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();

        float4 fa[kI], fb[kJ], ga[kI], gb[kJ];
        frag(fa, fb, As0, Bs0, 0);
        // the order of gemm_kept_kernel's K step (FP32 head and tail parts)
        auto quad = [&](float4 (&a)[kI], float4 (&b)[kJ], auto&& reads) {
            PrecF32::mfma_quad<kI, kJ, 0, PrecF32::kHead>(acc, a, b);
            __builtin_amdgcn_sched_barrier(0);
            reads();
            __builtin_amdgcn_sched_barrier(0);
            PrecF32::mfma_quad<kI, kJ, PrecF32::kHead, PrecF32::kParts>(acc, a, b);
            __builtin_amdgcn_sched_barrier(0);
        };
        // (the B tile issued after the first quad, as in gemm_kept_kernel)
        auto kstep = [&](const float* as, const float* bs, float* na, float* nb, int t) {
            const uint32_t kn = (uint32_t)min(t + 1, total - 1) * kStepBytes;
            direct_issue<kU>(ra_src, na, va, kn, wave);
            __builtin_amdgcn_sched_barrier(0);
            quad(fa, fb, [&] { frag(ga, gb, as, bs, 1); });
            direct_issue<kU>(rb_src, nb, vb, kn, wave);
            __builtin_amdgcn_sched_barrier(0);
            quad(ga, gb, [&] { frag(fa, fb, as, bs, 2); });
            quad(fa, fb, [&] { frag(ga, gb, as, bs, 3); });
            PrecF32::mfma_quad<kI, kJ, 0, PrecF32::kParts - PrecF32::kTail>(acc, ga, gb);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            frag(fa, fb, na, nb, 0);
            __builtin_amdgcn_sched_barrier(0);
            PrecF32::mfma_quad<kI, kJ, PrecF32::kParts - PrecF32::kTail, PrecF32::kParts>(acc, ga,
                                                                                       gb);
            __builtin_amdgcn_sched_barrier(0);
        };
        for (int t = 0; t < total; t += 2) {
            kstep(As0, Bs0, As1, Bs1, t);
            kstep(As1, Bs1, As0, Bs0, t + 1);
        }

        const bool mirror = full && tl.y != tl.z;
#pragma unroll
        for (int i = 0; i < kI; ++i) {
#pragma unroll
            for (int j = 0; j < kJ; ++j) {
                const int64_t col = col0 + wn * 32 * kJ + j * 32 + (lane & 31);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t row = row0 + wm * 32 * kI + i * 32 + 8 * (r >> 2) +
                                        4 * (lane >> 5) + (r & 3);
                    if (row < m && col < m) {
                        const float v = acc[i][j][r] * pr.scale;
                        pr.H[row * pr.ldh + col] = v;
                        if (mirror) pr.H[col * pr.ldh + row] = v;
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Mixed-tile form of the batched symmetric product.  Eight waves per
// workgroup, one job at a time; a job is either
//   kind 0: one 256 x 256 tile, waves of 128 x 64 (as gemm_batch_sym_kernel
//           with kWT = 4), or
//   kind 1: one or two 128 x 128 tiles of one problem, waves 0-3 on the
//           first and 4-7 on the second, each wave a 64 x 64 quarter; the
//           LDS tiles hold the first tile's 128 rows then the second's.
// The host gives each upper triangle's interior to kind 0 and its diagonal
// band and ragged last tile column to kind 1, so a diagonal 256 tile (whose
// lower-left quarter is not needed) is three 128 tiles, and a last tile
// column of at most 128 live columns is computed 128 wide.  A job is two
// int4: {problem, kind, tile row, tile col} and {second tile row, second
// tile col, has second, 0}, tile indices in units of 256 (kind 0) or 128
// (kind 1) rows.  In a kind-1 job without a second tile, waves 4-7 load
// nothing and compute nothing; they keep to the barriers.
// ---------------------------------------------------------------------------

// One job's K loop and epilogue for one wave: kI x 2 MFMA blocks of 32 x 32
// whose A rows start at LDS row arow and B rows at brow, output origin
// (orow, ocol).  load: the wave issues its share of the tile loads (offsets
// va / vb against ra / rb); live: it computes and stores.
template <int kI>
__device__ __forceinline__ void mixed_job(float* As0, float* As1, float* Bs0, float* Bs1,
                                          __amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb,
                                          const uint32_t (&va)[4], const uint32_t (&vb)[4],
                                          bool load, bool live, int total, int arow, int brow,
                                          int wave, int lane, const BatchProblem& pr,
                                          int64_t orow, int64_t ocol, bool mirror) {
    constexpr int kJ = 2;
    int fa_off[4], fb_off[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        fa_off[q] = direct_frag_off(arow + (lane & 31), q, lane);
        fb_off[q] = direct_frag_off(brow + (lane & 31), q, lane);
    }
    auto frag = [&](float4 (&a)[kI], float4 (&b)[kJ], const float* as, const float* bs, int q) {
#pragma unroll
        for (int i = 0; i < kI; ++i) a[i] = *reinterpret_cast<const float4*>(as + fa_off[q] + 1024 * i);
#pragma unroll
        for (int j = 0; j < kJ; ++j) b[j] = *reinterpret_cast<const float4*>(bs + fb_off[q] + 1024 * j);
    };
    auto issue = [&](float* as, float* bs, int step) {
        if (load) {
            direct_issue<4>(ra, as, va, (uint32_t)step * kStepBytes, wave);
            direct_issue<4>(rb, bs, vb, (uint32_t)step * kStepBytes, wave);
        }
    };

    v16f acc[kI][kJ];
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();                           // the previous job's last reads are done
    issue(As0, Bs0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    float4 fa[kI], fb[kJ], ga[kI], gb[kJ];
    if (live) frag(fa, fb, As0, Bs0, 0);
    // the order of gemm_kept_kernel's K step (FP32 head and tail parts)
    auto quad = [&](float4 (&a)[kI], float4 (&b)[kJ], auto&& reads) {
        PrecF32::mfma_quad<kI, kJ, 0, PrecF32::kHead>(acc, a, b);
        __builtin_amdgcn_sched_barrier(0);
        reads();
        __builtin_amdgcn_sched_barrier(0);
        PrecF32::mfma_quad<kI, kJ, PrecF32::kHead, PrecF32::kParts>(acc, a, b);
        __builtin_amdgcn_sched_barrier(0);
    };
    // (the B tile issued after the first quad, as in gemm_kept_kernel)
    auto kstep = [&](const float* as, const float* bs, float* na, float* nb, int t) {
        const uint32_t kn = (uint32_t)min(t + 1, total - 1) * kStepBytes;
        if (load) direct_issue<4>(ra, na, va, kn, wave);
        __builtin_amdgcn_sched_barrier(0);
        if (live) quad(fa, fb, [&] { frag(ga, gb, as, bs, 1); });
        if (load) direct_issue<4>(rb, nb, vb, kn, wave);
        __builtin_amdgcn_sched_barrier(0);
        if (live) {
            quad(ga, gb, [&] { frag(fa, fb, as, bs, 2); });
            quad(fa, fb, [&] { frag(ga, gb, as, bs, 3); });
            PrecF32::mfma_quad<kI, kJ, 0, PrecF32::kParts - PrecF32::kTail>(acc, ga, gb);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (live) {
            frag(fa, fb, na, nb, 0);
            __builtin_amdgcn_sched_barrier(0);
            PrecF32::mfma_quad<kI, kJ, PrecF32::kParts - PrecF32::kTail, PrecF32::kParts>(acc, ga,
                                                                                       gb);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < total; t += 2) {
        kstep(As0, Bs0, As1, Bs1, t);
        kstep(As1, Bs1, As0, Bs0, t + 1);
    }
    if (!live) return;

    const int64_t m = pr.m;
#pragma unroll
    for (int i = 0; i < kI; ++i) {
#pragma unroll
        for (int j = 0; j < kJ; ++j) {
            const int64_t col = ocol + j * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = orow + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (row < m && col < m) {
                    const float v = acc[i][j][r] * pr.scale;
                    pr.H[row * pr.ldh + col] = v;
                    if (mirror) pr.H[col * pr.ldh + row] = v;
                }
            }
        }
    }
}

__global__ __launch_bounds__(TileShape<4>::kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_batch_mixed_kernel(const BatchProblem* __restrict__ probs,
                             const int4* __restrict__ jobs, const int32_t* __restrict__ starts,
                             int full) {
    constexpr int BT = 256;
    __shared__ __align__(1024) float As0[BT * 32];
    __shared__ __align__(1024) float As1[BT * 32];
    __shared__ __align__(1024) float Bs0[BT * 32];
    __shared__ __align__(1024) float Bs1[BT * 32];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave >> 2;

    const int32_t w_end = starts[blockIdx.x + 1];
    for (int32_t w = starts[blockIdx.x]; w < w_end; ++w) {
        const int4 j0 = jobs[2 * w];
        const int4 j1 = jobs[2 * w + 1];
        const BatchProblem pr = probs[j0.x];
        const int64_t m = pr.m;
        const bool big = j0.y == 0;
        // this wave's tile: rows ra.. of A's side, rows rb.. of B's side
        bool load = true;
        int64_t ra, rb;
        if (big) {
            ra = (int64_t)j0.z * 256;
            rb = (int64_t)j0.w * 256;
        } else if (half == 0) {
            ra = (int64_t)j0.z * 128;
            rb = (int64_t)j0.w * 128;
        } else {
            load = j1.z != 0;
            ra = (int64_t)(load ? j1.x : j0.z) * 128;
            rb = (int64_t)(load ? j1.y : j0.w) * 128;
        }
        const int span = big ? 256 : 128;
        const int sub = big ? 0 : 128 * half;
        uint32_t va[4], vb[4];
        direct_offsets<4>(va, pr.ld * 4, (int)min((int64_t)span - 1, m - 1 - ra), wave, lane, sub);
        direct_offsets<4>(vb, pr.ld * 4, (int)min((int64_t)span - 1, m - 1 - rb), wave, lane, sub);
        const __amdgpu_buffer_rsrc_t rsa = tile_rsrc(pr.S + ra * pr.ld);
        const __amdgpu_buffer_rsrc_t rsb = tile_rsrc(pr.S + rb * pr.ld);
        const bool mirror = full && ra != rb;
        if (big) {
            const int wm = wave >> 2, wn = wave & 3;
            mixed_job<4>(As0, As1, Bs0, Bs1, rsa, rsb, va, vb, true, true, pr.ksteps, wm * 128,
                         wn * 64, wave, lane, pr, ra + wm * 128, rb + wn * 64, mirror);
        } else {
            const int wm = (wave >> 1) & 1, wn = wave & 1;
            mixed_job<2>(As0, As1, Bs0, Bs1, rsa, rsb, va, vb, load, load, pr.ksteps,
                         sub + wm * 64, sub + wn * 64, wave, lane, pr, ra + wm * 64,
                         rb + wn * 64, mirror);
        }
    }
}

}  // namespace

bool plan_gemm_ok(int64_t m, int64_t l, int32_t bp, int64_t ldat, int64_t ldbt, int elem) {
    const int step = kStepBytes / elem;
    if (m < 1 || l < 1 || bp < step || bp % step) return false;
    if (ldat * elem > kMaxSketchLdBytes || ldbt * elem > kMaxSketchLdBytes) return false;
    const int64_t tilesM = (m + BM - 1) / BM;
    const int64_t tilesN = (l + BN - 1) / BN;
    return tilesM * tilesN <= 0x7fffffff;
}

namespace {

// Split K loop for products with few tiles: a single 256x256 tile runs on
// one CU, so a small product (for example 256 x 256 over K = 1024) would leave
// the other CUs idle.  Splits aim at kSplitSlots workgroups (the CU count of
// the device this is tuned for) with at least kSplitMinSteps K steps (one
// step pair) each.
constexpr int64_t kSplitSlots = 256;
constexpr int64_t kSplitMinSteps = 2;

int64_t tiles_of(int64_t m, int64_t l, int side) {
    return ((m + side - 1) / side) * ((l + side - 1) / side);
}

// Most splits a product over `steps` K steps takes (< 2: none).
int64_t split_bound(int64_t m, int64_t l, int64_t steps) {
    const int64_t tiles = tiles_of(m, l, BM);
    if (tiles * 2 > kSplitSlots) return 1;
    return std::min(kSplitSlots / tiles, steps / kSplitMinSteps);
}

// Splits and steps per split for `total` K steps of an m x l product (false:
// no split: enough tiles, too few steps, or too little partial space).
bool split_plan(int64_t m, int64_t l, int64_t total, const float* part, size_t part_bytes,
                int64_t& S, int64_t& chunk) {
    S = split_bound(m, l, total);
    if (S < 2 || !part) return false;
    chunk = (total + S - 1) / S;
    chunk += chunk & 1;                            // whole step pairs, the last split may be odd
    S = (total + chunk - 1) / chunk;               // every split has at least one step
    return S >= 2 && (size_t)S * (size_t)m * (size_t)l * 4u <= part_bytes;
}

// How a block product is run: tile side (256, 128 or 64; 32 = the small
// kernel), the split of its K loop (S = 1: none), and the side of the tiles of
// its last, partial round (0: as the others).
struct Form {
    int tile;
    int64_t S;
    int64_t chunk;
    int rest = 0;
    bool deep = false;         // the deep kernel (rest: for those tiles only)
};

// Tiles in whole rounds of the device, of `tiles`.
int64_t whole_rounds(int64_t tiles) { return tiles / kSplitSlots * kSplitSlots; }

// Predicted us per K step of `tiles` tiles of side f.tile, those past the
// whole rounds as tiles of side f.rest in a launch of their own (f.deep: by the
// deep kernel).  (A product
// of a few more than a multiple of 256 tiles leaves most CUs idle in its last
// round, and smaller tiles throughout cost 8 % (FP32) to 80 % (BF16) more LDS
// and L2 traffic.  K = 4096, us without / with: 5120 x 5120 FP32 1523 / 1473;
// 4500 x 4200 BF16 168 / 162, split BF16 475 / 410, FP8 120 / 109, split FP8
// 259 / 226; 7000 x 8000 split BF16 1080 / 1054, FP8 246 / 238; with deep
// kernels for the rest 4500 x 4200 BF16 156, split BF16 394, split FP8 221.)
double step_us(Kind kind, int tile, int64_t tiles);
double deep_us(Kind kind, int tile, int64_t tiles, int chunk);

double rest_us(Kind kind, int tile, int rest, int64_t tiles, int chunk, bool* deep) {
    const int64_t n1 = whole_rounds(tiles);
    const int64_t sub = tile / rest;
    const int64_t n2 = (tiles - n1) * sub * sub;
    const double us = step_us(kind, rest, n2), d = deep_us(kind, rest, n2, chunk);
    *deep = d > 0 && d < us;
    return step_us(kind, tile, n1) + (*deep ? d : us);
}

// f(tile, rest) for every remainder form of a product with tiles(side) tiles.
template <typename F, typename G>
void remainder_forms(bool fp8, G tiles, F f) {
    for (const int tile : {256, 128})
        for (const int rest : {128, 64}) {
            if (rest >= tile || (fp8 && rest == 64)) continue;
            const int64_t n = tiles(tile);
            const int64_t n1 = whole_rounds(n);
            if (n1 > 0 && n1 < n && n <= 0x7fffffff / 16) f(tile, rest, n);
        }
}

// Predicted microseconds per K step (128 bytes of every tile row) of
// `tiles` tiles of a side, from timings on an MI355X (256 CUs; r = the
// largest number of tiles on one CU).  A 256 tile has the least LDS and L2
// traffic per flop, but a product of few tiles leaves CUs idle, and one of a
// few more than a multiple of 256 tiles leaves most of them idle in its last
// round; smaller tiles fill both.  Measured at K = 4096, us with sides 256 /
// 128 / 64 / 32:
//                 512 x 512         1024 x 1024        2048 x 2048     4096 x 4096      5120 x 5120
//   FP32        906/250/80/37     909/255/84/136    915/278/276/-   922/959/1008/-  1830/1669/1576/-
//   BF16         82/36/39/20       84/50/41/72       86/53/58/-     113/126/207/-    196/229/323/-
//   split BF16  206/96/57/35      204/99/61/127     207/123/157/-   298/360/582/-    505/628/916/-
//   FP8          44/22             45/31             51/34           65/83           112/142
//   split FP8   111/52            111/64            114/73          153/202          267/330
double step_us(Kind kind, int tile, int64_t tiles) {
    const double r = (double)((tiles + kSplitSlots - 1) / kSplitSlots);
    const bool few = tiles <= 192;        // (256 tiles: less L2 contention, higher clock)
    if (tile == 32) return 0.25 * r + 0.04;
    switch (kind) {
        case kF32:
            return tile == 256 ? 7.1 * r : tile == 128 ? 1.87 * r + 0.1 : 0.49 * r + 0.15;
        case kBF16:
            return tile == 256   ? (few ? 1.4 : 1.75 * r)
                   : tile == 128 ? 0.5 * r + 0.3
                                 : std::max(0.62, 0.2 * r + 0.1);
        case kBF16X3:
            return tile == 256   ? (few ? 1.65 : 2.1 * r)
                   : tile == 128 ? 0.67 * r + 0.25
                                 : 0.28 * r + 0.17;
        case kFp8: return tile == 256 ? (few ? 1.5 : 1.9 * r) : 0.6 * r + 0.35;
        default: return tile == 256 ? (few ? 1.75 : 2.2 * r) : 0.7 * r + 0.35;
    }
}

// The same for the deep kernels, 0 where there is none or it does not pay:
// at most one workgroup of 128 tiles, or two of 64, per CU (chunk: bytes per
// FP8 scale chunk).  Measured us, two step buffers / four, K = 4096 (2048 *):
//                 512 x 512   1024 x 1024   1500 x 1500   2048 x 2048 *   300 x 6000 *
//   BF16   128       34/34         49/36         50/37          31/26          28/23
//           64       38/20         39/22         41/43          31/33          24/18
//   split  128       97/77        100/80        107/83          66/55          53/44
//           64       59/34         61/39         92/99          83/79          42/39
//   FP8    128       25/28         34/31         36/32          24/23          18/20
//     (blocks of 1024)             32/27                  K = 4096 36/30
//   split  128       56/51         65/53         70/56          47/38          43/33
//     (blocks of 1024)             64/49                  K = 4096 77/57
double deep_us(Kind kind, int tile, int64_t tiles, int chunk) {
    const bool few = tiles <= 160;
    if (tiles > (tile == 64 ? 512 : 256) || tile == 256) return 0;
    switch (kind) {
        case kBF16:
            return tile == 64 ? (tiles <= 256 ? 0.28 : 0.45) : (few ? 0.52 : 0.68);
        case kBF16X3:
            return tile == 64 ? (tiles <= 256 ? 0.27 : 0.58) : (few ? 0.62 : 0.8);
        case kFp8: return tile == 128 && chunk == 16 ? (few ? 0.7 : 0.8) : 0;
        case kFp8X3: return tile == 128 && chunk ? (few ? 0.75 : (chunk == 16 ? 0.83 : 1.0)) : 0;
        default: return 0;
    }
}

// The form predicted fastest.  Without partial space (part = nullptr) every
// entry is summed in step order whatever the tile, bit for bit the same.
// Where the split K loop serves a product, FP32 and split BF16 keep its split
// (the number of partial sums per entry, which their accuracy shows) whatever
// the tile, and take the small kernel only if that has as many.  BF16 and FP8
// products, plain or split FP8, may run unsplit: their error is the operands'
// rounding (against 64 bits, unsplit over split, 7 products of few tiles, 15 inputs
// each: BF16 1.00000 +- 0.00002, FP8 and split FP8 the same).
Form pick_form(Kind kind, int64_t m, int64_t l, int64_t total, const float* part,
               size_t part_bytes, int chunk_bytes = 0) {
    int64_t S = 1, chunk = total;
    if (!split_plan(m, l, total, part, part_bytes, S, chunk)) {
        S = 1;
        chunk = total;
    }
    const bool fp8 = kind == kFp8 || kind == kFp8X3;
    Form best{256, S, chunk};
    double t = 0;
    auto consider = [&](const Form& f) {
        const int64_t tiles = tiles_of(m, l, f.tile) * f.S;
        if (tiles > 0x7fffffff) return;
        // what 256 tiles add for first loads and epilogue: 2 us on few CUs, and,
        // where they fill them, 2 or 3 for rounds past the first (smaller tiles
        // write theirs while others run); 6 with partials, which are then summed.
        // (Fitted on 560 products of 1 to 128 steps in every form; with 6
        // throughout, products of few steps took smaller tiles than is best: 4096 x
        // 4096 over 4 steps, 128 / 256 tiles: BF16 23.2 / 21.0 us, split FP8 31.1 /
        // 25.1; 3000 x 4100 over 5, FP8 26.3 / 22.6.)
        double us = (f.deep ? deep_us(kind, f.tile, tiles, chunk_bytes)
                            : step_us(kind, f.tile, tiles)) * (double)f.chunk;
        if (f.tile == 256)
            us += f.S > 1         ? 6
                  : tiles <= 192 ? 2
                                 : std::min(3.0, 2.0 * (double)((tiles - 1) / kSplitSlots));
        if (f.S > 1) us += 4 + (double)f.S * (double)m * (double)l * 4 / 4e6;
        if (t == 0 || us < t) {
            t = us;
            best = f;
        }
    };
    for (const int tile : {256, 128, 64}) {
        if (tile == 64 && fp8) continue;
        consider(Form{tile, S, chunk});
        const bool whole = S == 1 || kind == kBF16 || fp8;     // (may run unsplit)
        if (S > 1 && whole) consider(Form{tile, 1, total});
        if (whole && deep_us(kind, tile, tiles_of(m, l, tile), chunk_bytes) > 0)
            consider(Form{tile, 1, total, 0, true});
    }
    if (part && !fp8 && (kind == kBF16 || S <= kSmallSums)) consider(Form{32, 1, total});
    if (best.S == 1)
        remainder_forms(fp8, [&](int side) { return tiles_of(m, l, side); },
                        [&](int tile, int rest, int64_t n) {
                            bool deep;
                            const double us =
                                rest_us(kind, tile, rest, n, chunk_bytes, &deep) * (double)total +
                                8;                     // (the second launch)
                            if (us < t) {
                                t = us;
                                best = Form{tile, 1, total, rest, deep};
                            }
                        });
    return best;
}

// C = scale * (the sum of the S partial products at part).
hipError_t launch_split_sum(const float* part, int64_t S, int64_t m, int64_t l, float scale,
                            float* C, int64_t ldc, hipStream_t s) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(split_sum_kernel, dim3((unsigned)((m * l + 255) / 256)), dim3(256), 0, s,
                       part, (int32_t)S, m, l, scale, C, ldc);
    return hipGetLastError();
}

// Operands of a block product (any precision).
struct Operands {
    const void* At;
    int64_t ldat;
    const void* Bt;
    int64_t ldbt;
    int64_t m, l;
    int32_t bp;
    const BlockList* kept;
    int32_t nkept;
    int64_t lo_off;
    float scale;
    float* C;
    int64_t ldc;
};

// Launches `count` tiles of side sub * S::BT, from tile `first` on, in parts of
// side S::BT (all of them: 0, tiles, 1).
template <typename P, typename S>
hipError_t launch_part(const Operands& o, const Form& f, int64_t total, float* part, int64_t first,
                       int64_t count, int sub, hipStream_t s) {
    const int64_t side = (int64_t)sub * S::BT;
    const int64_t tilesM = (o.m + side - 1) / side;
    const int64_t tilesN = (o.l + side - 1) / side;
    auto kern = f.S > 1      ? gemm_kept_kernel<P, S, false, true, true>
                : total % 2 ? gemm_kept_kernel<P, S, false, true>
                            : gemm_kept_kernel<P, S, false, false>;
    if constexpr (S::BT < 256 && P::kKind != kF32)
        if (f.deep && (!f.rest || sub > 1))
            kern = gemm_kept_kernel<P, S, false, true, false, true>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(f.S * count * sub * sub)), dim3(S::kThreads), 0, s,
                       o.At, o.ldat, o.Bt, o.ldbt, o.m, o.l, o.bp, *o.kept, o.nkept,
                       o.lo_off, o.scale, o.C, o.ldc, (int32_t)tilesM, (int32_t)tilesN,
                       CMask{nullptr, 0, 0, 0, 1}, SplitK{part, (int32_t)f.chunk},
                       Part{(int32_t)first, sub});
    return hipGetLastError();
}

template <typename P, typename S>
hipError_t launch_tile(const Operands& o, const Form& f, int64_t total, float* part,
                       hipStream_t s) {
    const int64_t tiles = tiles_of(o.m, o.l, S::BT);
    if constexpr (S::BT > 64) {
        if (f.rest) {
            const int64_t n1 = whole_rounds(tiles);
            const hipError_t e = launch_part<P, S>(o, f, total, part, 0, n1, 1, s);
            if (e != hipSuccess) return e;
            if constexpr (S::BT == 256)
                if (f.rest == 128)
                    return launch_part<P, Tile128>(o, f, total, part, n1, tiles - n1, 2, s);
            return launch_part<P, Tile64>(o, f, total, part, n1, tiles - n1, S::BT / 64, s);
        }
    }
    const hipError_t e = launch_part<P, S>(o, f, total, part, 0, tiles, 1, s);
    if (e != hipSuccess || f.S == 1) return e;
    return launch_split_sum(part, f.S, o.m, o.l, o.scale, o.C, o.ldc, s);
}

template <typename P>
hipError_t launch_form(const Operands& o, float* part, size_t part_bytes, hipStream_t s) {
    const int64_t total = (int64_t)o.nkept * (o.bp / (kStepBytes / P::kElem / (P::kPair ? 2 : 1)));
    const Form f = pick_form(P::kKind, o.m, o.l, total, part, part_bytes);
    if (f.tile == 256) return launch_tile<P, Tile256>(o, f, total, part, s);
    if (f.tile == 128) return launch_tile<P, Tile128>(o, f, total, part, s);
    if (f.tile == 64) return launch_tile<P, Tile64>(o, f, total, part, s);
    const int64_t tilesM = (o.m + kSmallTile - 1) / kSmallTile;
    const int64_t tilesN = (o.l + kSmallTile - 1) / kSmallTile;
    hipLaunchKernelGGL(gemm_small_kernel<P>, dim3((unsigned)(tilesM * tilesN)),
                       dim3(64 * kSmallWaves), 0, s, o.At, o.ldat, o.Bt, o.ldbt, o.m, o.l, o.bp,
                       *o.kept, o.nkept, o.lo_off, o.scale, o.C, o.ldc, (int32_t)tilesM,
                       (int32_t)tilesN);
    return hipGetLastError();
}

// As launch_part, tb = tiles of side sub * S::BT per C block side.
template <typename S>
hipError_t launch_cmask_part(const float* At, int64_t ldat, const float* Bt, int64_t ldbt,
                             int64_t m, int64_t l, int32_t bp, const CMask& cm, int64_t nbI,
                             int64_t first, int64_t count, int sub, float* C, int64_t ldc,
                             hipStream_t s) {
    BlockList none;
    for (int j = 0; j < OS_MAX_BLOCKS; ++j) none.idx[j] = 0;
    // a tile's step count is (its kept blocks) * bp / 32: always even when
    // bp / 32 is, and then the unmasked pair loop serves every tile
    auto kern = (bp / 32) % 2 == 0 ? gemm_kept_kernel<PrecF32, S, true, false>
                                   : gemm_kept_kernel<PrecF32, S, true, true>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(count * sub * sub)), dim3(S::kThreads), 0, s, At, ldat,
                       Bt, ldbt, m, l, bp, none, 0, (int64_t)0, 1.0f, C, ldc,
                       (int32_t)(nbI * cm.tb), (int32_t)(cm.nbJ * cm.tb), cm, SplitK{nullptr, 0},
                       Part{(int32_t)first, sub});
    return hipGetLastError();
}

}  // namespace

size_t gemm_split_bytes(int64_t m, int64_t l, int64_t max_steps) {
    if (m < 1 || l < 1) return 0;
    const int64_t S = split_bound(m, l, max_steps);
    return S >= 2 ? (size_t)S * (size_t)m * (size_t)l * 4u : 0;
}

hipError_t launch_gemm_kept(const float* At, int64_t ldat, const float* Bt, int64_t ldbt,
                            int64_t m, int64_t l, int32_t bp, const BlockList& kept,
                            int32_t nkept, float scale, float* C, int64_t ldc, float* part,
                            size_t part_bytes, hipStream_t s) {
    if (!plan_gemm_ok(m, l, bp, ldat, ldbt, 4) || nkept < 1) return hipErrorInvalidValue;
    return launch_form<PrecF32>(Operands{At, ldat, Bt, ldbt, m, l, bp, &kept, nkept, 0, scale, C, ldc},
                                part, part_bytes, s);
}

hipError_t launch_gemm_cmask(const float* At, int64_t ldat, const float* Bt, int64_t ldbt,
                             int64_t m, int64_t l, int32_t bp, int32_t nst, const uint8_t* cmask,
                             int64_t cblk, float* C, int64_t ldc, hipStream_t s) {
    if (!plan_gemm_ok(m, l, bp, ldat, ldbt, 4) || cblk < 1 || nst < 1 || nst > OS_MAX_BLOCKS)
        return hipErrorInvalidValue;
    const int64_t nbI = (m + cblk - 1) / cblk, nbJ = (l + cblk - 1) / cblk;
    // the form predicted fastest (every entry's sum is the same for all)
    auto tiles = [&](int side) -> int64_t {
        const int64_t tb = (cblk + side - 1) / side;
        return nbI * tb * nbJ * tb;
    };
    int side = 0, rest = 0;
    double t = 0;
    for (const int tile : {256, 128, 64}) {
        const int64_t live = tiles(tile);
        if (live > 0x7fffffff || nbJ > 0x7fffffff) continue;
        const double us = step_us(kF32, tile, live);
        if (!side || us < t) {
            t = us;
            side = tile;
        }
    }
    if (!side) return hipErrorInvalidValue;
    remainder_forms(false, tiles, [&](int tile, int part, int64_t n) {
        bool deep;
        const double us = rest_us(kF32, tile, part, n, 0, &deep);
        if (us < t) {
            t = us;
            side = tile;
            rest = part;
        }
    });
    const int64_t n = tiles(side);
    const CMask cm{cmask, cblk, (int32_t)nbJ, nst, (int32_t)((cblk + side - 1) / side)};
    auto run = [&](int bt, int64_t first, int64_t count, int sub) {
        auto launch = bt == 256   ? launch_cmask_part<Tile256>
                      : bt == 128 ? launch_cmask_part<Tile128>
                                  : launch_cmask_part<Tile64>;
        return launch(At, ldat, Bt, ldbt, m, l, bp, cm, nbI, first, count, sub, C, ldc, s);
    };
    if (!rest) return run(side, 0, n, 1);
    const int64_t n1 = whole_rounds(n);
    const hipError_t e = run(side, 0, n1, 1);
    return e != hipSuccess ? e : run(rest, n1, n - n1, side / rest);
}

hipError_t launch_gemm_batch_sym(const BatchProblem* probs, const int4* tiles,
                                 const int32_t* starts, int tile, int full, int32_t grid,
                                 hipStream_t s) {
    if (grid < 1) return hipErrorInvalidValue;
    if (tile == 256)
        hipLaunchKernelGGL(gemm_batch_sym_kernel<4>, dim3((unsigned)grid),
                           dim3(TileShape<4>::kThreads), 0, s,
                           probs, tiles, starts, full);
    else if (tile == 128)
        hipLaunchKernelGGL(gemm_batch_sym_kernel<2>, dim3((unsigned)grid),
                           dim3(TileShape<2>::kThreads), 0, s,
                           probs, tiles, starts, full);
    else if (tile == OS_GRAM_MIXED)
        hipLaunchKernelGGL(gemm_batch_mixed_kernel, dim3((unsigned)grid),
                           dim3(TileShape<4>::kThreads), 0, s,
                           probs, tiles, starts, full);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

int batch_sym_blocks_per_cu(int tile) {
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    if (tile == 256)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_batch_sym_kernel<4>,
                                                         TileShape<4>::kThreads, 0);
    else if (tile == 128)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_batch_sym_kernel<2>,
                                                         TileShape<2>::kThreads, 0);
    else if (tile == OS_GRAM_MIXED)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_batch_mixed_kernel,
                                                         TileShape<4>::kThreads, 0);
    return e == hipSuccess ? n : 0;
}

namespace {

// Bytes per scale chunk: whole chunks per block; 16-byte ones also need
// 16-byte aligned rows and scale area (with either the step count is even).
int scale_chunk(const Operands& o, int64_t scales) {
    if (o.bp % 1024 == 0 && o.ldat % 16 == 0 && o.ldbt % 16 == 0 && scales % 16 == 0) return 16;
    return o.bp % 256 == 0 && o.lo_off % 256 == 0 ? 4 : 0;
}

// (As launch_part and launch_tile.)
template <typename S, bool kPair>
hipError_t launch_fp8_part(const Operands& o, int64_t scales, const Form& f, int64_t total,
                           float* part, int64_t first, int64_t count, int sub, hipStream_t s) {
    const int64_t side = (int64_t)sub * S::BT;
    const int64_t tilesM = (o.m + side - 1) / side;
    const int64_t tilesN = (o.l + side - 1) / side;
    const int chunk = scale_chunk(o, scales);
    auto kern = f.S > 1       ? gemm_kept_fp8d_kernel<S, kPair, true, true>
                : chunk == 16 ? gemm_kept_fp8d_kernel<S, kPair, false, false, 16>
                : chunk == 4  ? gemm_kept_fp8d_kernel<S, kPair, false, false, 4>
                : total % 2  ? gemm_kept_fp8d_kernel<S, kPair, true>
                             : gemm_kept_fp8d_kernel<S, kPair, false>;
    if constexpr (S::BT == 128) {
        if (f.deep && (!f.rest || sub > 1)) {
            kern = gemm_kept_fp8d_kernel<S, kPair, false, false, 16, true>;
            if constexpr (kPair)
                if (chunk == 4) kern = gemm_kept_fp8d_kernel<S, kPair, false, false, 4, true>;
        }
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(f.S * count * sub * sub)), dim3(S::kThreads), 0, s,
                       static_cast<const uint8_t*>(o.At), o.ldat,
                       static_cast<const uint8_t*>(o.Bt), o.ldbt, scales, o.m, o.l, o.bp, *o.kept,
                       o.nkept, o.lo_off, o.scale, o.C, o.ldc, (int32_t)tilesM, (int32_t)tilesN,
                       SplitK{part, (int32_t)f.chunk}, Part{(int32_t)first, sub});
    return hipGetLastError();
}

template <typename S, bool kPair>
hipError_t launch_fp8_tile(const Operands& o, int64_t scales, const Form& f, int64_t total,
                           float* part, hipStream_t s) {
    const int64_t tiles = tiles_of(o.m, o.l, S::BT);
    if (f.rest) {                                     // (256 and 128 tiles only)
        const int64_t n1 = whole_rounds(tiles);
        const hipError_t e = launch_fp8_part<S, kPair>(o, scales, f, total, part, 0, n1, 1, s);
        if (e != hipSuccess) return e;
        return launch_fp8_part<Tile128, kPair>(o, scales, f, total, part, n1, tiles - n1,
                                               S::BT / 128, s);
    }
    const hipError_t e = launch_fp8_part<S, kPair>(o, scales, f, total, part, 0, tiles, 1, s);
    if (e != hipSuccess || f.S == 1) return e;
    return launch_split_sum(part, f.S, o.m, o.l, o.scale, o.C, o.ldc, s);
}

template <bool kPair>
hipError_t launch_fp8(const Operands& o, int64_t scales, float* part, size_t part_bytes,
                      hipStream_t s) {
    const int64_t total = (int64_t)o.nkept * (o.bp / (kPair ? 64 : 128));
    const Form f = pick_form(kPair ? kFp8X3 : kFp8, o.m, o.l, total, part, part_bytes,
                             scale_chunk(o, scales));
    return f.tile == 256 ? launch_fp8_tile<Tile256, kPair>(o, scales, f, total, part, s)
                         : launch_fp8_tile<Tile128, kPair>(o, scales, f, total, part, s);
}

}  // namespace

hipError_t launch_gemm_kept_fp8(const void* At, int64_t ldat, const void* Bt, int64_t ldbt,
                                int64_t scales, int64_t m, int64_t l, int32_t bp,
                                const BlockList& kept, int32_t nkept, int split, int64_t lo_off,
                                float scale, float* C, int64_t ldc, float* part,
                                size_t part_bytes, hipStream_t s) {
    if (!plan_gemm_ok(m, l, bp, ldat, ldbt, 1) || nkept < 1) return hipErrorInvalidValue;
    const Operands o{At, ldat, Bt, ldbt, m, l, bp, &kept, nkept, lo_off, scale, C, ldc};
    return split ? launch_fp8<true>(o, scales, part, part_bytes, s)
                 : launch_fp8<false>(o, scales, part, part_bytes, s);
}

hipError_t launch_gemm_kept_bf16(const void* At, int64_t ldat, const void* Bt, int64_t ldbt,
                                 int64_t m, int64_t l, int32_t bp, const BlockList& kept,
                                 int32_t nkept, int split, int64_t lo_off, float scale, float* C,
                                 int64_t ldc, float* part, size_t part_bytes, hipStream_t s) {
    if (!plan_gemm_ok(m, l, bp, ldat, ldbt, 2) || nkept < 1) return hipErrorInvalidValue;
    const Operands o{At, ldat, Bt, ldbt, m, l, bp, &kept, nkept, lo_off, scale, C, ldc};
    return split ? launch_form<PrecBF16X3>(o, part, part_bytes, s)
                 : launch_form<PrecBF16>(o, part, part_bytes, s);
}

}  // namespace osk
