// sketch_kernel.h -- the count-sketch kernel (see sketch.hip for the scheme)
// and its launch over the compiled slot counts.  Included by one translation
// unit per input form (sketch_rows.hip and the like), so that they compile in
// parallel.
#pragma once

#include <type_traits>

#include "sketch_launch.h"
#include "fp8.h"

namespace osk {

namespace {

// ---------------------------------------------------------------------------
// The sketch kernel.  Thread t stages window positions 4096u + 4t + j
// (u < 2, j < 4) into LDS slots win_slot(k) = 4096u + 1024j + t; list entries
// hold those slots.
//   kRowLines = true : lines are rows of X (lines x n, ld ldx, n >= 4): a
//                      line's 4 consecutive positions come with one load of 4
//                      values (16 bytes FP32, 1 KiB per wave; any element
//                      alignment): r[2*line + u] holds positions 4t + 4096u
//                      .. +3 of that line.  The quad that straddles the end of
//                      a window whose length is no multiple of 4 is loaded
//                      from the last 4 positions and shifted when it is staged.
//   kRowLines = false: lines are columns of X (n x lines, ld ldx, lines >= 4);
//                      r[4u + j] holds X[k][line0 .. line0+3] for position k =
//                      4096u + 4t + j, one 16-byte load.  The last group of
//                      lines starts at lines - 4 (lines that two groups hold
//                      are written twice with the same values).
//     BF16 columns   : the same with 8 lines (16 bytes) per workgroup; LDS
//                      keeps the 8 BF16 values of a position, converted as
//                      they are added.  Bound by those requests, a cache
//                      line each (16384 x 4096 into 4 blocks of 512: 85-90
//                      us, where the transpose and the sketch of its rows
//                      took 49 + 67).
// kForm (kRowLines = false), where loads of 4 values would leave the matrix:
//   kNarrow          : fewer than 4 columns (n >= 4), 16-byte loads as for
//                      columns, reading on into the next row; those that would
//                      end past the matrix are repeated by value.
//                      1000000 x 3 into 2 blocks of 64: 1250 us (a wave per line
//                      and 64 buckets, gathering from global memory, 6150).
//   kShort           : rows of fewer than 4 values, and anything as small: every
//                      value loaded by itself, as FP32, from X[line * ldx + k *
//                      ldk].  Bound by the writes of the sums (100000 rows of 3
//                      into 8 blocks of 1024: 700 us, 2700 gathering).
// kWeighted (row lines): every value at sketched index k is multiplied by
// sqrt(wd[k]) (a diagonal weight, as in A D^{1/2} S for a Hessian A D A^T);
// w[u] holds the weights of positions 4t + 4096u .. +3.  The weight is
// applied when the window is written to LDS, not when it is loaded, so the
// loads of the next window stay in flight while the current one is summed.
// ---------------------------------------------------------------------------
// Input values are held in registers as loaded (4 consecutive values of a
// line: a float4 for FP32, their 4 bit patterns in a uint2 for BF16) and
// converted to FP32 (exactly) when the window is written to LDS.
// A window's FP32 values and weights are read once: non-temporal loads keep
// them from displacing the bucket lists (which every line group reads) in
// the caches (the FP32 sketch of A 2-5 % faster).  Loads need only the
// alignment of an element (gfx950 loads 16 bytes at any dword).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef f32x4 f32x4_any2 __attribute__((aligned(2)));
__device__ __forceinline__ float4 load_stream(const float* __restrict__ p) {
    const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(p));
    return make_float4(t[0], t[1], t[2], t[3]);
}

template <typename TI>
struct RawQuad;
template <>
struct RawQuad<float> {
    using type = float4;
    static __device__ __forceinline__ float value(const type& v, int j) {
        return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
    }
    // the quad starting d values further (its last d values are not used)
    static __device__ __forceinline__ type shift(const type& v, int d) {
        return d == 1 ? make_float4(v.y, v.z, v.w, 0.f)
                      : (d == 2 ? make_float4(v.z, v.w, 0.f, 0.f)
                                : make_float4(v.w, 0.f, 0.f, 0.f));
    }
};
template <>
struct RawQuad<__bf16> {
    using type = uint2;
    typedef uint32_t pair2 __attribute__((ext_vector_type(2)));
    typedef pair2 pair2_any __attribute__((aligned(2)));
    static __device__ __forceinline__ type load(const __bf16* __restrict__ p) {
        const pair2 t = *reinterpret_cast<const pair2_any*>(p);
        return make_uint2(t[0], t[1]);
    }
    static __device__ __forceinline__ float value(const type& v, int j) {
        const uint32_t w = j < 2 ? v.x : v.y;
        return __uint_as_float((j & 1) ? (w & 0xFFFF0000u) : (w << 16));
    }
    static __device__ __forceinline__ type shift(const type& v, int d) {
        const uint64_t x = ((uint64_t)v.y << 32 | v.x) >> (16 * d);
        return make_uint2((uint32_t)x, (uint32_t)(x >> 32));
    }
};

// Lines per workgroup, and a piece of a window as loaded.
template <bool kRowLines, typename TI>
constexpr int kLinesOf = !kRowLines && sizeof(TI) == 2 ? 8 : kLines;
template <bool kRowLines, typename TI>
using Piece = std::conditional_t<kRowLines, typename RawQuad<TI>::type, float4>;

// Loads pieces p0 .. p1 - 1 of a window (piece 4u + q: r[2q + u] of row
// lines, r[4u + q] of column lines); all 8 pieces make the window.  p0 and p1
// are constants (the callers are unrolled).  Every
// load is unconditional (a branch around a load makes each use wait for all
// loads in flight): positions past the window's end are clamped to its last
// ones (no entry refers to them) and lines past the matrix to its last line
// (their sums are never stored).
template <bool kRowLines, typename TI>
__device__ __forceinline__ void load_window(Piece<kRowLines, TI> (&r)[kPerThread],
                                            const TI* __restrict__ X, int64_t lines, int64_t ldx,
                                            int64_t line0, int64_t k0, int kw, int p0, int p1) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (4 * u + q < p0 || 4 * u + q >= p1) continue;
            if constexpr (kRowLines) {
                // Uniform line bases plus a 32-bit lane offset (scalar-base
                // addressing: a piece issued late keeps one offset register
                // live, not a 64-bit address); the offset may be negative when
                // a last window has fewer than 4 positions
                const int off = min(4 * tid + 4096 * u, kw - 4);
                const TI* base = X + min(line0 + q, lines - 1) * ldx + k0;
                // (the FP32 load written here, not through a RawQuad helper:
                // through one the FP32 kernels took 20 more registers)
                if constexpr (sizeof(TI) == 4)
                    r[2 * q + u] = load_stream(base + off);
                else
                    r[2 * q + u] = RawQuad<TI>::load(base + off);
            } else {
                const int64_t kk = k0 + min(4 * tid + 4096 * u + q, kw - 1);
                f32x4 t;
                if constexpr (sizeof(TI) == 4)
                    t = *reinterpret_cast<const f32x4_any*>(X + kk * ldx + line0);
                else
                    t = *reinterpret_cast<const f32x4_any2*>(X + kk * ldx + line0);
                r[4 * u + q] = make_float4(t[0], t[1], t[2], t[3]);
            }
        }
    }
}

enum Form { kWhole, kNarrow, kShort };

// load_window of a kNarrow kernel (n positions of `lines` columns in all).
__device__ __forceinline__ void load_narrow(float4 (&r)[kPerThread], const float* __restrict__ X,
                                            int64_t lines, int64_t n, int64_t ldx, int64_t k0,
                                            int kw, int p0, int p1) {
#pragma unroll
    for (int p = 0; p < kPerThread; ++p) {
        if (p < p0 || p >= p1) continue;
        const int64_t k = k0 + min(4 * (int)threadIdx.x + 4096 * (p / 4) + p % 4, kw - 1);
        const f32x4 t = *reinterpret_cast<const f32x4_any*>(
            X + min(k * ldx, (n - 1) * ldx + lines - 4));
        r[p] = make_float4(t[0], t[1], t[2], t[3]);
    }
}

// The positions whose loads by load_narrow were moved down, loaded again one
// value at a time (window from k0 on, the last one).
__device__ __forceinline__ void reload_narrow(float4 (&r)[kPerThread], const float* __restrict__ X,
                                              int64_t lines, int64_t n, int64_t ldx, int64_t k0) {
#pragma unroll
    for (int p = 0; p < kPerThread; ++p) {
        const int64_t k = k0 + 4 * (int)threadIdx.x + 4096 * (p / 4) + p % 4;
        if (k < n && k * ldx > (n - 1) * ldx + lines - 4) {
            const float* x = X + k * ldx;
            r[p] = make_float4(x[0], x[min((int64_t)1, lines - 1)], x[lines - 1], 0.f);
        }
    }
}

// load_window of a kShort kernel.
template <typename TI>
__device__ __forceinline__ void load_short(float4 (&r)[kPerThread], const TI* __restrict__ X,
                                           int64_t lines, int64_t ldx, int64_t ldk, int64_t line0,
                                           int64_t k0, int kw, int p0, int p1) {
#pragma unroll
    for (int p = 0; p < kPerThread; ++p) {
        if (p < p0 || p >= p1) continue;
        const int64_t k = k0 + min(4 * (int)threadIdx.x + 4096 * (p / 4) + p % 4, kw - 1);
        auto at = [&](int q) { return (float)X[min(line0 + q, lines - 1) * ldx + k * ldk]; };
        r[p] = make_float4(at(0), at(1), at(2), at(3));
    }
}

__device__ __forceinline__ float comp4(const float4& v, int j) {
    return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
}

// The weights of this thread's positions of a window, as the loaded quads.
template <Form kForm>
__device__ __forceinline__ void load_weights(float4 (&w)[2], const float* __restrict__ wd,
                                             int64_t k0, int kw) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int t = 4 * (int)threadIdx.x + 4096 * u;
        if constexpr (kForm == kShort) {
            auto at = [&](int j) { return wd[k0 + min(t + j, kw - 1)]; };
            w[u] = make_float4(at(0), at(1), at(2), at(3));
        } else {
            w[u] = load_stream(wd + k0 + min(t, kw - 4));
        }
    }
}

__device__ __forceinline__ float4 weigh(float4 v, float w) {
    const float sw = sqrtf(w);
    return make_float4(v.x * sw, v.y * sw, v.z * sw, v.w * sw);
}

// Writes a loaded window of kw positions into LDS: win[win_slot(k)] = the 4
// lines' values at window position k (weighted when kWeighted).
template <bool kRowLines, bool kWeighted, typename TI>
__device__ __forceinline__ void stage_window(float4* __restrict__ win,
                                             Piece<kRowLines, TI> (&r)[kPerThread],
                                             float4 (&w)[2], int kw) {
    using R = RawQuad<TI>;
    const int tid = threadIdx.x;
    if constexpr (kRowLines) {
        if (kw & 3) {       // uniform: a last window that ends inside a quad
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int d = 4 * tid + 4096 * u - (kw - 4);
                if (d > 0 && d < 4) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) r[2 * q + u] = R::shift(r[2 * q + u], d);
                    if constexpr (kWeighted) w[u] = RawQuad<float>::shift(w[u], d);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float4 v = make_float4(R::value(r[u], j), R::value(r[2 + u], j),
                                       R::value(r[4 + u], j), R::value(r[6 + u], j));
                if constexpr (kWeighted) v = weigh(v, comp4(w[u], j));
                win[4096 * u + 1024 * j + tid] = v;      // slot of position 4096u + 4t + j
            }
        }
    } else {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float4 v = r[4 * u + j];
                if constexpr (kWeighted) v = weigh(v, comp4(w[u], j));
                win[4096 * u + 1024 * j + tid] = v;
            }
    }
}

// Adds 4 entries (16 bits each, two per word; sign bit 15 selects the sign of
// the FP32 +-1.0 factor).  All four LDS reads are issued before the first
// FMA so their latencies overlap.  kQ = 2: 8 BF16 lines per position.
template <int kQ>
__device__ __forceinline__ void add_half(float4 (&acc)[kQ], const float4* __restrict__ win,
                                         uint32_t w0, uint32_t w1) {
    const uint32_t w[2] = {w0, w1};
    float4 v[4];
    float s[4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        v[2 * u] = win[w[u] & 0x7FFFu];
        v[2 * u + 1] = win[(w[u] >> 16) & 0x7FFFu];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        s[2 * u] = __uint_as_float(0x3F800000u | ((w[u] << 16) & 0x80000000u));
        s[2 * u + 1] = __uint_as_float(0x3F800000u | (w[u] & 0x80000000u));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        float4 x[kQ];
        if constexpr (kQ == 1) {
            x[0] = v[u];
        } else {
            auto lo = [](float w) { return __uint_as_float(__float_as_uint(w) << 16); };
            auto hi = [](float w) { return __uint_as_float(__float_as_uint(w) & 0xFFFF0000u); };
            x[0] = make_float4(lo(v[u].x), hi(v[u].x), lo(v[u].y), hi(v[u].y));
            x[1] = make_float4(lo(v[u].z), hi(v[u].z), lo(v[u].w), hi(v[u].w));
        }
#pragma unroll
        for (int h = 0; h < kQ; ++h) {
            acc[h].x = fmaf(s[u], x[h].x, acc[h].x);
            acc[h].y = fmaf(s[u], x[h].y, acc[h].y);
            acc[h].z = fmaf(s[u], x[h].z, acc[h].z);
            acc[h].w = fmaf(s[u], x[h].w, acc[h].w);
        }
    }
}

// Adds the 8 entries of one chunk, four at a time (four waves per SIMD hide
// the LDS latency; eight reads in flight would spill).
template <int kQ>
__device__ __forceinline__ void add_chunk(float4 (&acc)[kQ], const float4* __restrict__ win,
                                          uint4 e) {
    add_half(acc, win, e.x, e.y);
    __builtin_amdgcn_sched_barrier(0);
    add_half(acc, win, e.z, e.w);
    __builtin_amdgcn_sched_barrier(0);
}

// One workgroup of 16 waves fills a CU's LDS, so each SIMD runs 4 waves of up
// to 128 VGPRs.  (8 waves of 256 VGPRs with whole chunks in flight: the FP32
// sketch of 8192 x 32768 into 10 blocks of 1024 took 506 us from rows and 785
// from columns, this 486 and 736.)
// sketch_tasks: the tasks of workgroup wg of nwg (win: its kWin + 1 rows of LDS).
template <int kSlots, bool kRowLines, bool kWeighted, typename TI, int kFp8Out, Form kForm = kWhole>
__device__ __forceinline__ void sketch_tasks(
    float4* __restrict__ win, int64_t wg, int64_t nwg, const TI* __restrict__ X, int64_t lines,
    int64_t n, int64_t ldx, int64_t ldk, int32_t qn, int32_t nwin, int32_t nst, const BlockList& bl,
    int64_t RC, const uint32_t* __restrict__ hdr, const uint4* __restrict__ ell,
    void* __restrict__ out, int64_t ldo, int32_t npass, const float* __restrict__ wd, int32_t obp,
    int32_t omode, int64_t ozlo) {
    // (row kWin of win stays zero)
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const uint32_t lane16 = 16 * (uint32_t)lane;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kL = kForm == kShort ? kLines : kLinesOf<kRowLines, TI>;
    constexpr int kQ = kL / 4;
    static_assert(kQ == 1 || (kFp8Out == 0 && !kWeighted));
    static_assert(kForm == kWhole || !kRowLines);
    constexpr int kAhead = kAheadOf<kSlots, kRowLines || kForm == kShort, kQ>;
    constexpr int kTail = kTailOf<kSlots, kQ>;
    static_assert(!kWeighted || kRowLines || kForm == kShort);
    auto load = [&](Piece<kRowLines, TI> (&r)[kPerThread], int64_t l0, int64_t k0, int kw, int p0,
                    int p1) {
        if constexpr (kForm == kNarrow)
            load_narrow(r, X, lines, n, ldx, k0, kw, p0, p1);
        else if constexpr (kForm == kShort)
            load_short(r, X, lines, ldx, ldk, l0, k0, kw, p0, p1);
        else
            load_window<kRowLines, TI>(r, X, lines, ldx, l0, k0, kw, p0, p1);
    };
    const int64_t groups = (lines + kL - 1) / kL;
    const int64_t tasks = groups * npass;
    const int gslots = nst * qn;         // groups of 64 buckets over the stored blocks
    if (tid == 0) win[kWin] = make_float4(0.f, 0.f, 0.f, 0.f);

    // Persistent: workgroup g takes tasks g, g + grid, ... (task = a group
    // of 4 lines and a pass); the first window of its next task is fetched
    // while the last window of the current one is summed, so only the first
    // task of a workgroup waits for its first window.
    //
    // Slot bookkeeping stays out of the scalar path (a scalar load in the
    // slot loop drains every LDS read in flight): lane s of each wave holds,
    // for its slot s, the header index of the slot's bucket group in window
    // 0 (hb, -1 for an unused slot), the region's chunk base in window 0
    // (eb), the group's first output column (col) and how many of its 64
    // buckets exist (lim, 0 for an unused slot).  A window's headers come in
    // with one vector load, issued before the window's values are fetched.
    auto line_of = [&](int64_t it) {
        const int64_t l0 = xcd_task(it, tasks) / npass * kL;
        return kRowLines || kForm != kWhole ? l0 : min(l0, lines - kL);
    };
    struct Meta {
        int32_t hb, eb, col, lim;
    };
    auto meta_of = [&](int64_t it) -> Meta {
        const int ps = (int)(xcd_task(it, tasks) % npass);
        const int G = (ps * kSlots + lane) * kWaves + wave;
        Meta m{-1, 0, 0, 0};
        if (lane < kSlots && G < gslots) {
            const int j = G / qn;
            const int q = G - j * qn;
            const int32_t i = bl.idx[j];
            m.hb = (i * nwin) * qn + q;
            m.eb = (int32_t)((int64_t)i * nwin * RC);
            m.col = j * obp + q * 64;
            m.lim = min(64, obp - q * 64);
        }
        return m;
    };
    auto headers = [&](int32_t hb, int w) -> uint32_t {
        const uint32_t h = hdr[max(hb, 0) + w * qn];     // unconditional: index valid
        return hb >= 0 ? h : 0u;
    };
    Piece<kRowLines, TI> pre[kPerThread];
    float4 wpre[2];
    uint32_t hnext = 0;
    if (wg < tasks) {
        hnext = headers(meta_of(wg).hb, 0);
        const int kw = (int)min((int64_t)kWin, n);
        load(pre, line_of(wg), 0, kw, 0, kPerThread);
        if constexpr (kWeighted) load_weights<kForm>(wpre, wd, 0, kw);
    }
    for (int64_t it = wg; it < tasks; it += nwg) {
    const int64_t line0 = line_of(it);
    const Meta meta = meta_of(it);      // (its loads complete with the window's, before staging)

    float4 acc[kSlots][kQ];
#pragma unroll
    for (int s = 0; s < kSlots; ++s)
#pragma unroll
        for (int h = 0; h < kQ; ++h) acc[s][h] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int w = 0; w < nwin; ++w) {
        __syncthreads();                 // the previous window is no longer read
        if constexpr (kForm == kNarrow) {
            if (w + 1 == nwin) reload_narrow(pre, X, lines, n, ldx, (int64_t)w * kWin);
        }
        stage_window<kRowLines, kWeighted, TI>(
            win, pre, wpre, (int)min((int64_t)kWin, n - (int64_t)w * kWin));
        __syncthreads();
        const uint32_t hv = hnext;       // this window's headers (lane s: slot s)
        // The list chunks of slot s + kDist (up to kAhead of them) are fetched
        // while slot s is summed.  Fetches are unconditional: chunk indices
        // past a slot's count repeat its last chunk, and an unused slot
        // (header 0) reads chunk 0 of block 0's region (never summed).
        const int64_t wrc = (int64_t)w * RC;
        // (List addresses stay scalar: uniform base plus the lane's 16 bytes.)
        auto slot_list = [&](int s, uint32_t& nch) -> const char* {
            const uint32_t h = (uint32_t)__builtin_amdgcn_readlane((int)hv, s);
            const int64_t eb = __builtin_amdgcn_readlane(meta.eb, s);
            nch = h >> 16;
            return reinterpret_cast<const char*>(ell) + ((eb + wrc + (h & 0xFFFFu)) << 10);
        };
        auto chunk_at = [&](const char* p, uint32_t c) -> uint4 {
            return *reinterpret_cast<const uint4*>(p + (c << 10) + lane16);
        };
        auto fetch = [&](uint4 (&d)[kAhead], const char* p, uint32_t nch) {
            const uint32_t last = nch > 0 ? nch - 1 : 0;
#pragma unroll
            for (int c = 0; c < kAhead; ++c) d[c] = chunk_at(p, min((uint32_t)c, last));
        };
        // The next window (this task's, else the first of the next task) is
        // loaded in kPerThread pieces spread over the slots, each issued
        // after the list fetch of its slot: a wave's loads complete in
        // order, so waiting for slot s's list waits only for pieces issued
        // kDist or more slots earlier, not for the whole window.  When no
        // window follows, the pieces read one quad of this window again
        // (every lane the same address; loads stay unconditional).
        int64_t l1 = line0, k1 = (int64_t)(w + 1) * kWin;
        int32_t hb1 = meta.hb;
        int kw1;
        if (w + 1 < nwin) {
            kw1 = (int)min((int64_t)kWin, n - k1);
        } else if (it + nwg < tasks) {
            hb1 = meta_of(it + nwg).hb;
            l1 = line_of(it + nwg);
            k1 = 0;
            kw1 = (int)min((int64_t)kWin, n);
        } else {
            k1 = 0;
            kw1 = (int)min((int64_t)4, n);
        }
        constexpr int kRing = kDist + 1;
        uint4 lst[kRing][kAhead];
        uint32_t nls[kRing];
        const char* pls[kRing];
#pragma unroll
        for (int s = 0; s < kDist && s < kSlots; ++s) {
            pls[s] = slot_list(s, nls[s]);
            fetch(lst[s], pls[s], nls[s]);
        }
        hnext = headers(hb1, (int)(k1 / kWin));
        constexpr int kSpreadSlots = kSlots < kPerThread ? kSlots : kPerThread;
        constexpr int kPer = (kPerThread + kSpreadSlots - 1) / kSpreadSlots;
        // (unrolled at compile time: acc[s] and the ring stay in registers
        // however large the body)
        static_for<0, kSlots>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if constexpr (s + kDist < kSlots) {
                constexpr int r = (s + kDist) % kRing;
                pls[r] = slot_list(s + kDist, nls[r]);
                fetch(lst[r], pls[r], nls[r]);
            }
            if constexpr (s < kSpreadSlots)
                load(pre, l1, k1, kw1, s * kPer,
                     (s + 1) * kPer < kPerThread ? (s + 1) * kPer : kPerThread);
            constexpr int r = s % kRing;
#pragma unroll
            for (int c = 0; c < kAhead; ++c)
                if ((uint32_t)c < nls[r]) add_chunk(acc[s], win, lst[r][c]);
            if constexpr (kTail > 0) {
                // (chunks ahead in the tail too)
                if (nls[r] > (uint32_t)kAhead) {
                    const uint32_t last = nls[r] - 1;
                    uint4 next[kTail];
#pragma unroll
                    for (int u = 0; u < kTail; ++u)
                        next[u] = chunk_at(pls[r], min((uint32_t)(kAhead + u), last));
                    for (uint32_t c = kAhead; c < nls[r]; c += kTail) {
                        uint4 e[kTail];
#pragma unroll
                        for (int u = 0; u < kTail; ++u) e[u] = next[u];
                        if (c + kTail < nls[r])
#pragma unroll
                            for (int u = 0; u < kTail; ++u)
                                next[u] = chunk_at(pls[r], min(c + kTail + u, last));
#pragma unroll
                        for (int u = 0; u < kTail; ++u)
                            if (c + u < nls[r]) add_chunk(acc[s], win, e[u]);
                    }
                }
            } else {
                for (uint32_t c = kAhead; c < nls[r]; ++c)
                    add_chunk(acc[s], win, chunk_at(pls[r], c));
            }
        });
        // (the next window's weights last: eight registers fewer during the
        // slots; every line group reads them, so they come from L2)
        if constexpr (kWeighted) load_weights<kForm>(wpre, wd, k1, kw1);
    }

    // Output: FP32 (omode 0, blocks obp = bp apart), or the copy the block
    // product reads, blocks obp = b rounded up to 64 apart:
    //   omode 1: BF16, each sum rounded to nearest even; omode 2: also the
    //            residual bf16(x - hi), ozlo values after the high part;
    //   omode 3: FP8 E4M3 codes (bytes) with one E8M0 scale per 64 codes,
    //            i.e. per slot group and line (its max over the wave's 64
    //            lanes); the scale bytes follow the codes (ozlo bytes into
    //            the row), in code order; omode 4: then the same for the
    //            residuals (codes, ozlo bytes after the first ones, and scales).
    // FP8 (separate instantiations: this code would make the FP32 and BF16
    // kernels with many slots spill).  Every lane of the wave holds a
    // bucket (lim is 64).  The maxima of a group's four lines are taken with
    // DPP moves and read into scalar registers; a lane's four codes (one per
    // line) are packed by the hardware conversion, transposed within each
    // quad of lanes, so that lane 4i + r holds line r's buckets 4i .. 4i + 3,
    // and stored with one instruction; lane s keeps slot s's four scales
    // until the end.  Bound: VALU issue (no other work overlaps it); with a
    // ds_bpermute butterfly, a software conversion and byte stores the sketch of
    // a 8192 x 32768 matrix into 10 blocks of 1024 took 690 us, now 492 (490
    // with FP32 output).  Split: 31.6 us for 2048 x 8192 into 5 blocks of 512,
    // where the FP32 sketch and its quantization took 29.9 + 8.8.
    if constexpr (kFp8Out != 0) {
        const int r4 = lane & 3;
        const uint32_t sel1 = (lane & 1) ? 0x03070105u : 0x06020400u;
        const uint32_t sel2 = (lane & 2) ? 0x03020706u : 0x05040100u;
        uint8_t* const rows = static_cast<uint8_t*>(out) + line0 * ldo;
        uint8_t* const mine = rows + r4 * ldo + 4 * (lane >> 2);
        const bool live = line0 + r4 < lines;
        constexpr bool kSplit = kFp8Out == 2;
        // the four lines' codes of v (one byte each), scale exponents e
        auto encode = [&](const float (&v)[4], int (&e)[4]) -> uint32_t {
            float y[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                uint32_t m = abs_bits(v[r]);
                m = dpp_max<0x111>(m);          // row_shr: 1, 2, 4, 8
                m = dpp_max<0x112>(m);
                m = dpp_max<0x114>(m);
                m = dpp_max<0x118>(m);
                m = dpp_max<0x142, 0xA>(m);     // row_bcast: 15, 31
                m = dpp_max<0x143, 0xC>(m);
                e[r] = e8m0_exponent((uint32_t)__builtin_amdgcn_readlane((int)m, 63));
                y[r] = ldexpf(v[r], -e[r]);
            }
            return e4m3_pack4(y[0], y[1], y[2], y[3]);
        };
        auto store = [&](uint32_t d, int64_t col) {
            uint32_t x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d, 0xB1, 0xF, 0xF, true);
            d = __builtin_amdgcn_perm(x, d, sel1);
            x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d, 0x4E, 0xF, 0xF, true);
            d = __builtin_amdgcn_perm(x, d, sel2);
            if (live) *reinterpret_cast<uint32_t*>(mine + col) = d;
        };
        auto scale_bytes = [](const int (&e)[4]) -> uint32_t {
            return (uint32_t)(e[0] + 127) | (uint32_t)(e[1] + 127) << 8 |
                   (uint32_t)(e[2] + 127) << 16 | (uint32_t)(e[3] + 127) << 24;
        };
        uint32_t scales = 0, scales_lo = 0;
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            if (__builtin_amdgcn_readlane(meta.lim, s) == 0) continue;      // uniform
            float v[4] = {acc[s][0].x, acc[s][0].y, acc[s][0].z, acc[s][0].w};
            const int64_t col = __builtin_amdgcn_readlane(meta.col, s);
            int e[4];
            const uint32_t d = encode(v, e);
            store(d, col);
            scales = lane == s ? scale_bytes(e) : scales;
            if constexpr (kSplit) {
                // the residuals, exact in FP32
                v[0] -= ldexpf(__builtin_amdgcn_cvt_f32_fp8((int)d, 0), e[0]);
                v[1] -= ldexpf(__builtin_amdgcn_cvt_f32_fp8((int)d, 1), e[1]);
                v[2] -= ldexpf(__builtin_amdgcn_cvt_f32_fp8((int)d, 2), e[2]);
                v[3] -= ldexpf(__builtin_amdgcn_cvt_f32_fp8((int)d, 3), e[3]);
                store(encode(v, e), ozlo + col);
                scales_lo = lane == s ? scale_bytes(e) : scales_lo;
            }
        }
        if (lane < kSlots && meta.lim > 0) {
            uint8_t* const sc = rows + ozlo * (kSplit ? 2 : 1) + meta.col / 64;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (line0 + r < lines) {
                    sc[r * ldo] = (uint8_t)(scales >> (8 * r));
                    if constexpr (kSplit) sc[r * ldo + ozlo / 64] = (uint8_t)(scales_lo >> (8 * r));
                }
        }
    } else
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        // lanes below lim hold buckets of the block (the last group may be partial)
        if (lane < __builtin_amdgcn_readlane(meta.lim, s)) {
#pragma unroll
            for (int h = 0; h < kQ; ++h) {
                const int64_t l4 = line0 + 4 * h;
                const int64_t o0 = l4 * ldo + __builtin_amdgcn_readlane(meta.col, s) + lane;
                const float v[4] = {acc[s][h].x, acc[s][h].y, acc[s][h].z, acc[s][h].w};
                if (omode == 0) {
                    float* o = static_cast<float*>(out) + o0;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r == 0 || l4 + r < lines) o[r * ldo] = v[r];
                } else {
                    __bf16* o = static_cast<__bf16*>(out) + o0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (r == 0 || l4 + r < lines) {
                            const __bf16 hi = (__bf16)v[r];
                            o[r * ldo] = hi;
                            if (omode == 2) o[r * ldo + ozlo] = (__bf16)(v[r] - (float)hi);
                        }
                    }
                }
            }
        }
    }
    }   // tasks
}

template <int kSlots, bool kRowLines, bool kWeighted, typename TI, int kFp8Out, Form kForm>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void sketch_kernel(const TI* __restrict__ X, int64_t lines, int64_t n, int64_t ldx, int64_t ldk,
                   int32_t qn, int32_t nwin, int32_t nst, BlockList bl, int64_t RC,
                   const uint32_t* __restrict__ hdr, const uint4* __restrict__ ell,
                   void* __restrict__ out, int64_t ldo, int32_t npass,
                   const float* __restrict__ wd, int32_t obp, int32_t omode, int64_t ozlo) {
    __shared__ float4 win[kWin + 1];
    sketch_tasks<kSlots, kRowLines, kWeighted, TI, kFp8Out, kForm>(
        win, blockIdx.x, gridDim.x, X, lines, n, ldx, ldk, qn, nwin, nst, bl, RC, hdr, ell, out,
        ldo, npass, wd, obp, omode, ozlo);
}

template <int S, bool R, bool W, typename TI, int Q8, Form F = kWhole>
hipError_t launch_one(dim3 grid, hipStream_t st, const SketchArgs& a) {
    hipLaunchKernelGGL((sketch_kernel<S, R, W, TI, Q8, F>), grid, dim3(kThreads), 0, st,
                       static_cast<const TI*>(a.X), a.lines, a.n, a.ldx, a.ldk, a.qn, a.nwin, a.nst,
                       *a.bl, a.RC, a.hdr, a.ell, a.out, a.ldo, a.npass, a.wd, a.obp, a.omode,
                       a.ozlo);
    return hipGetLastError();
}

template <bool R, bool W, typename TI, int Q8 = 0, int kMost = Q8 ? kMaxFp8Slots : kMaxSlots,
          Form F = kWhole>
hipError_t launch_slots(int slots, dim3 grid, hipStream_t st, const SketchArgs& a) {
#define OSK_SLOT_CASE(S) \
    if constexpr (S <= kMost) \
        if (slots <= S) return launch_one<S, R, W, TI, Q8, F>(grid, st, a);
    OSK_SLOT_CASE(1)
    OSK_SLOT_CASE(2)
    OSK_SLOT_CASE(3)
    OSK_SLOT_CASE(4)
    OSK_SLOT_CASE(6)
    OSK_SLOT_CASE(8)
    OSK_SLOT_CASE(10)
    OSK_SLOT_CASE(12)
#undef OSK_SLOT_CASE
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace osk
