// sketch.hip -- count-sketch kernels for gfx950.
//
// Both sketches apply the blocks of S (Eq. (sketch_matrix)) to one operand:
// every input element x at sketched index k is added, with sign sigma_i(k),
// into bucket h_i(k) of every stored block i (Algorithm "Calculating
// Count-sketch of a matrix A", applied block by block as in Algorithm "Over
// sketching A in parallel").
//
// A "line" is a vector over the sketched index: a row of A (m lines of
// length n) or a column of B (l lines of length n).  The sketch of a line is
// a row of the output: out[line][j*bp + c] = bucket c of stored block j
// (line-major; the sketch of A is A S, the sketch of B is (S^T B)^T).
//
// Scheme (read-once): a workgroup owns kLines = 4 lines and keeps ALL their
// buckets -- every stored block -- in registers (a pass covers up to
// 16 * kMaxSlots groups of 64 buckets; wider sketches take several passes).
// It walks the sketched index in windows of kWin = 8192: the window of its
// 4 lines is staged in LDS once as kWin float4 (the 4 lines' values at one
// k side by side), and every lane then adds, for each bucket it owns, the
// window entries hashed into that bucket: one 16-byte LDS read and four FMAs
// per entry.  Each input element is read from HBM once.  No atomics: every
// bucket of every line is summed by one lane, in ascending k.
//
// Which entries a lane adds comes from the prepared sketch, built once per
// (seed or tables, b, N, e, n): for every block i, window w and group q of 64
// consecutive buckets, a lane-interleaved list ("chunks" of 8 entries per
// lane, 1 KiB per chunk) padded to the longest bucket of the group.  An entry
// is 16 bits: the LDS slot of k's window offset (bits 0..14, a fixed
// permutation of the offset, see win_slot) and the sign (bit 15); the
// padding entry points at a zero row.
#include <algorithm>

#include "hash.h"
#include "sketch_launch.h"

namespace osk {
namespace {

// ---------------------------------------------------------------------------
// Prepared lists, built per region (window w, block i): by several waves, and
// workgroups, for block strides up to kBWMaxBp, else by one wave.
//   hdr[(i*nwin + w)*qn + q] = chunk base (bits 0..15) | chunk count (16..31)
//     of group q (buckets 64q .. 64q+63) within the (i, w) region;
//   ell region (i, w) = RC chunks of 64 lanes x 8 entries; lane L of group q
//     holds the entries of bucket 64q + L at positions 0, 1, ... (entry t in
//     chunk base + t/8, slot t%8), ascending k, then padding.
// The per-group chunk counts sum to at most ceil(kw/8) + qn = RC, because the
// longest bucket of a group holds at most the group's entries.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void ell_build_region(const uint32_t* __restrict__ table, int64_t n,
                                                 int64_t nt, int32_t bp, int32_t qn,
                                                 int32_t nwin, int64_t RC,
                                                 uint32_t* __restrict__ hdr,
                                                 uint16_t* __restrict__ ell, int w, int64_t i,
                                                 uint32_t* sm, const int32_t* __restrict__ inv) {
    uint32_t* cnt = sm;            // [bp] counts, then cursors
    uint32_t* qbase = sm + bp;     // [qn] chunk base of each group
    uint32_t* qlen = qbase + qn;   // [qn] chunk count of each group
    const int lane = threadIdx.x;
    const int64_t k0 = (int64_t)w * kWin;
    const int kw = (int)min((int64_t)kWin, n - k0);
    const uint32_t* row = table + i * nt + k0;
    uint32_t* H = hdr + (i * nwin + w) * qn;
    uint16_t* region = ell + (i * nwin + w) * RC * 512;
    // list position of a bucket (the bucket itself unless grouped), the
    // block's map copied to LDS after the counts and group fields
    uint32_t* pos = qlen + qn;
    uint32_t* tab = pos + bp;       // [kWin] the window's table entries
    auto at = [&](uint32_t e) -> uint32_t {
        const uint32_t h = e & 0x7FFFFFFFu;
        return inv ? pos[h] : h;
    };

    for (int c = lane; c < bp; c += 64) {
        cnt[c] = 0;
        if (inv) pos[c] = (uint32_t)inv[i * bp + c];
    }
    for (int t0 = 0; t0 < kw; t0 += 64 * 16) {
        uint32_t e[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) e[u] = row[min(t0 + 64 * u + lane, kw - 1)];
#pragma unroll
        for (int u = 0; u < 16; ++u) tab[t0 + 64 * u + lane] = e[u];
    }
    __syncthreads();
    for (int t = lane; t < kw; t += 64) atomicAdd(&cnt[at(tab[t])], 1u);
    __syncthreads();

    uint32_t base = 0;
    for (int q = 0; q < qn; ++q) {
        const int c = 64 * q + lane;
        const uint32_t x = c < bp ? cnt[c] : 0u;
        const uint32_t nch = (wave_max(x) + 7) / 8;
        if (lane == 0) {
            H[q] = base | (nch << 16);
            qbase[q] = base;
            qlen[q] = nch;
        }
        base += nch;
    }
    __syncthreads();
    for (int c = lane; c < bp; c += 64) cnt[c] = 0;
    __syncthreads();

    // Stable scatter: chunks of 64 consecutive k; lanes holding the same
    // bucket ("peers") are found bit by bit with ballots and ranked by lane.
    int nbits = 1;
    while ((1 << nbits) < bp) ++nbits;
    const uint64_t below = lanes_below();
    for (int t0 = 0; t0 < kw; t0 += 64) {
        const int t = t0 + lane;
        const bool valid = t < kw;
        const uint32_t e = valid ? tab[t] : 0u;
        const uint32_t h = valid ? at(e) : 0u;
        uint64_t peers = __ballot(valid);
        for (int bit = 0; bit < nbits; ++bit) {
            const bool set = (h >> bit) & 1u;
            const uint64_t B = __ballot(valid && set);
            peers &= set ? B : ~B;
        }
        uint32_t pos = 0;
        if (valid) {
            pos = cnt[h] + (uint32_t)__popcll(peers & below);
            const uint32_t chunk = qbase[h >> 6] + pos / 8;
            region[(int64_t)chunk * 512 + (h & 63) * 8 + (pos & 7)] =
                (uint16_t)(win_slot(t) | ((e >> 31) << 15));
        }
        __builtin_amdgcn_wave_barrier();
        // the highest peer advances the bucket's cursor (one writer per bucket)
        if (valid && (peers >> lane) == 1ull) cnt[h] += (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // padding up to each group's chunk count
    for (int q = 0; q < qn; ++q) {
        const int c = 64 * q + lane;
        const uint32_t have = c < bp ? cnt[c] : 0u;
        const uint32_t len = qlen[q] * 8;
        const uint32_t qb = qbase[q];
        for (uint32_t p = have; p < len; ++p)
            region[(int64_t)(qb + p / 8) * 512 + lane * 8 + (p & 7)] = kPad;
    }
}

// The same region built by kBW waves (bp <= kBWMaxBp): wave v
// scatters its own contiguous part of the window; its cursors start at
// the entries of the earlier parts (an exclusive scan over the parts' counts
// per bucket), so every bucket's list stays in ascending k.  With Z > 1, Z
// workgroups build one region: each counts the whole window, scatters the
// parts z * kBW .. z * kBW + kBW - 1 and pads every Z-th group (a prepare has
// few regions, 5 to 40 in the usual sizes, and one region is a long serial
// chain for its workgroup: counting takes about a third of it; n = 32768, 10
// blocks of 1024: 20.4 us with one, 14.7; n = 8192, 5 blocks of 512: 15.9 and
// 9.9).  LDS: per-wave
// cursors [kBW][bp], totals [bp], group bases and lengths [qn] each.  The
// single-sketch build takes 16 waves per region for bp <= 1024 and 8 up to
// 2048 (full-size lists, Z = 1: 26 us against 30 with 8 and 41 with 4);
// the batch build, which strides over many regions per workgroup, keeps 4
// (8 were 20 % slower there).
constexpr int kBWSingle = 8;
constexpr int kBWWide = 16;            // single-sketch regions with bp <= kBWWideMaxBp
constexpr int kBWWideMaxBp = 1024;
constexpr int kBWBatch = 4;
constexpr int kBWMaxBp = 2048;

template <int kBW, typename F>
__device__ __forceinline__ void ell_build_region_waves(F entry, int64_t n, int32_t bp, int32_t qn,
                                                       int32_t nwin, int64_t RC,
                                                       uint32_t* __restrict__ hdr,
                                                       uint16_t* __restrict__ ell, int w, int64_t i,
                                                       uint32_t* sm, const int32_t* __restrict__ inv,
                                                       int z = 0, int Z = 1) {
    uint32_t* cur = sm;                 // [kBW][bp] counts, then cursors
    uint32_t* tot = sm + kBW * bp;      // [bp] entries per bucket
    uint32_t* qbase = tot + bp;         // [qn] chunk base of each group
    uint32_t* qlen = qbase + qn;        // [qn] chunk count of each group
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = tid >> 6;
    const int64_t k0 = (int64_t)w * kWin;
    const int kw = (int)min((int64_t)kWin, n - k0);
    uint32_t* H = hdr + (i * nwin + w) * qn;
    uint16_t* region = ell + (i * nwin + w) * RC * 512;
    // this wave's part of the window: [t_beg, t_end)
    const int parts = kBW * Z;
    const int part = ((kw + parts - 1) / parts + 63) / 64 * 64;
    const int t_beg = min(kw, (z * kBW + wv) * part);
    const int t_end = min(kw, t_beg + part);
    uint32_t* mine = cur + wv * bp;
    uint32_t* pos = qlen + qn;          // [bp] the block's bucket -> position map
    uint32_t* tab = pos + bp;           // [kWin] the window's table entries
    auto at = [&](uint32_t e) -> uint32_t {
        const uint32_t h = e & 0x7FFFFFFFu;
        return inv ? pos[h] : h;
    };

    uint32_t* before = tab + kWin;      // [bp] (Z > 1) entries of the earlier workgroups' parts
    for (int c = tid; c < (kBW + 1) * bp; c += 64 * kBW) cur[c] = 0;
    if (Z > 1)
        for (int c = tid; c < bp; c += 64 * kBW) before[c] = 0;
    if (inv)
        for (int c = tid; c < bp; c += 64 * kBW) pos[c] = (uint32_t)inv[i * bp + c];
    {
        // the window's entries to LDS, every load issued before the first store
        constexpr int kU = kWin / (64 * kBW);
        uint32_t e[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (u * 64 * kBW < kw) e[u] = entry(k0 + min(u * 64 * kBW + tid, kw - 1));
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (u * 64 * kBW < kw) tab[u * 64 * kBW + tid] = e[u];
    }
    __syncthreads();
    if (Z == 1) {       // (each wave its own part: no division per 64 entries)
        for (int t = t_beg + lane; t < t_end; t += 64) atomicAdd(&mine[at(tab[t])], 1u);
    } else
    for (int t0 = 64 * wv; t0 < kw; t0 += 64 * kBW) {
        const int p = t0 / part - z * kBW;                  // (uniform: part is a multiple of 64)
        uint32_t* to = p < 0 ? before : (p < kBW ? cur + p * bp : tot);
        if (t0 + lane < kw) atomicAdd(&to[at(tab[t0 + lane])], 1u);
    }
    __syncthreads();
    for (int c = tid; c < bp; c += 64 * kBW) {
        uint32_t run = Z > 1 ? before[c] : 0u;
#pragma unroll
        for (int v = 0; v < kBW; ++v) {
            const uint32_t x = cur[v * bp + c];
            cur[v * bp + c] = run;
            run += x;
        }
        tot[c] += run;
    }
    __syncthreads();

    // chunk counts, a wave per group; then every wave adds up its bases
    for (int q = wv; q < qn; q += kBW) {
        const int c = 64 * q + lane;
        const uint32_t nch = (wave_max(c < bp ? tot[c] : 0u) + 7) / 8;
        if (lane == 0) qlen[q] = nch;
    }
    __syncthreads();
    for (int q0 = 0, base = 0; q0 < qn; q0 += 64) {      // (qn <= 32 for the builds in use)
        const int q = q0 + lane;
        const uint32_t len = q < qn ? qlen[q] : 0u;
        uint32_t sum = len;                               // inclusive scan over the lanes
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t up = (uint32_t)__shfl_up((int)sum, d);
            sum += lane >= d ? up : 0u;
        }
        if (q < qn) {
            const uint32_t first = (uint32_t)base + sum - len;
            if (wv == 0 && z == 0) H[q] = first | (len << 16);
            qbase[q] = first;                             // (the same value from every wave)
        }
        base += __shfl((int)sum, 63);
    }
    __syncthreads();

    // stable scatter of this wave's part, as in ell_build_region
    int nbits = 1;
    while ((1 << nbits) < bp) ++nbits;
    const uint64_t below = lanes_below();
    for (int t0 = t_beg; t0 < t_end; t0 += 64) {
        const int t = t0 + lane;
        const bool valid = t < t_end;
        const uint32_t e = valid ? tab[t] : 0u;
        const uint32_t h = valid ? at(e) : 0u;
        uint64_t peers = __ballot(valid);
        for (int bit = 0; bit < nbits; ++bit) {
            const bool set = (h >> bit) & 1u;
            const uint64_t B = __ballot(valid && set);
            peers &= set ? B : ~B;
        }
        if (valid) {
            const uint32_t pos = mine[h] + (uint32_t)__popcll(peers & below);
            const uint32_t chunk = qbase[h >> 6] + pos / 8;
            region[(int64_t)chunk * 512 + (h & 63) * 8 + (pos & 7)] =
                (uint16_t)(win_slot(t) | ((e >> 31) << 15));
        }
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers >> lane) == 1ull) mine[h] += (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }

    // padding up to each group's chunk count, groups spread over the waves
    // (other entries than the scatter's: no barrier between them)
    for (int q = wv * Z + z; q < qn; q += parts) {
        const int c = 64 * q + lane;
        const uint32_t have = c < bp ? tot[c] : 0u;
        const uint32_t len = qlen[q] * 8;
        const uint32_t qb = qbase[q];
        for (uint32_t p = have; p < len; ++p)
            region[(int64_t)(qb + p / 8) * 512 + lane * 8 + (p & 7)] = kPad;
    }
}

// table: the packed table, or nullptr to take every entry from the hash (or
// explicit tables) as it is needed; inv_out: where the identity position map
// goes (with table = nullptr; natural order only).
template <int kW>
__global__ __launch_bounds__(64 * kW) void ell_buildw_kernel(
    const uint32_t* __restrict__ table, uint64_t seed, const int32_t* __restrict__ h,
    const int8_t* __restrict__ sigma, int64_t n, int64_t nt, int32_t b, int32_t bp, int32_t qn,
    int32_t nwin, int64_t RC, uint32_t* __restrict__ hdr, uint16_t* __restrict__ ell,
    const int32_t* __restrict__ inv, int32_t* __restrict__ inv_out) {
    extern __shared__ uint32_t sm[];
    const int64_t i = blockIdx.y;
    const int z = (int)blockIdx.z, Z = (int)gridDim.z;
    if (table) {
        ell_build_region_waves<kW>([&](int64_t k) { return table[i * nt + k]; }, n, bp, qn, nwin,
                                   RC, hdr, ell, (int)blockIdx.x, i, sm, inv, z, Z);
    } else {
        if (inv_out && blockIdx.x == 0 && z == 0)
            for (int c = threadIdx.x; c < bp; c += 64 * kW) inv_out[i * bp + c] = c;
        ell_build_region_waves<kW>([&](int64_t k) { return packed_entry(seed, h, sigma, i, k, n, b); },
                                   n, bp, qn, nwin, RC, hdr, ell, (int)blockIdx.x, i, sm, nullptr, z,
                                   Z);
    }
}

__global__ __launch_bounds__(64) void ell_build_kernel(const uint32_t* __restrict__ table,
                                                       int64_t n, int64_t nt, int32_t bp,
                                                       int32_t qn, int32_t nwin, int64_t RC,
                                                       uint32_t* __restrict__ hdr,
                                                       uint16_t* __restrict__ ell,
                                                       const int32_t* __restrict__ inv) {
    extern __shared__ uint32_t sm[];
    ell_build_region(table, n, nt, bp, qn, nwin, RC, hdr, ell, (int)blockIdx.x,
                     (int64_t)blockIdx.y, sm, inv);
}

__global__ __launch_bounds__(64 * kBWBatch) void ell_build_batchw_kernel(
    const PrepDesc* __restrict__ descs, int32_t count, int64_t tasks) {
    extern __shared__ uint32_t sm[];
    for (int64_t t = blockIdx.x; t < tasks; t += gridDim.x) {
        const int32_t p = find_task(descs, count, t, [](const PrepDesc& d) {
            return d.ell_task0;
        });
        const PrepDesc& d = descs[p];
        const int64_t local = t - d.ell_task0;
        const int64_t i = local / d.nwin;
        const uint32_t* row = d.table + i * d.nt;
        ell_build_region_waves<kBWBatch>([&](int64_t k) { return row[k]; }, d.n, d.bp, d.qn, d.nwin,
                                         d.RC, d.hdr, d.ell, (int)(local % d.nwin), i, sm, d.inv);
        __syncthreads();
    }
}

// The same for many prepared sketches in one launch: task t (one wave) is
// region (block i, window w) of the descriptor whose ell_task0 range holds
// t; workgroups stride over the tasks.
__global__ __launch_bounds__(64) void ell_build_batch_kernel(const PrepDesc* __restrict__ descs,
                                                             int32_t count, int64_t tasks) {
    extern __shared__ uint32_t sm[];
    for (int64_t t = blockIdx.x; t < tasks; t += gridDim.x) {
        const int32_t p = find_task(descs, count, t, [](const PrepDesc& d) {
            return d.ell_task0;
        });
        const PrepDesc& d = descs[p];
        const int64_t local = t - d.ell_task0;
        ell_build_region(d.table, d.n, d.nt, d.bp, d.qn, d.nwin, d.RC, d.hdr, d.ell,
                         (int)(local % d.nwin), local / d.nwin, sm, d.inv);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Grouping the buckets of each block (one workgroup per block).  The sketch
// kernel's 64 lanes walk the lists of a group of 64 buckets in lockstep, so
// a group costs its longest list in every window.  Any fixed order of the
// buckets within a block serves the product (A's and B's sketches use the
// same order, and C sums over the buckets), so buckets of similar list
// lengths are put in one group: a recursive median split over the groups
// (a k-d partition), level d sorting each node's buckets by their count in
// the windows w with w % D == d (D levels for G = ceil(b / 64) groups), ties
// by their current position, and splitting the node in two halves of whole
// groups.  inv[i * bp + c] = the position of bucket c (c < b) in block i's
// sketch; positions b .. bp - 1 stay empty.
// ---------------------------------------------------------------------------
constexpr int kGroupThreads = 1024;
constexpr int kSortMax = 8192;        // >= OS_MAX_B, a power of two

__global__ __launch_bounds__(kGroupThreads) void group_kernel(const uint32_t* __restrict__ table,
                                                              int64_t n, int64_t nt, int32_t b,
                                                              int32_t bp, int32_t nwin,
                                                              int32_t* __restrict__ inv) {
    __shared__ uint64_t key[kSortMax];
    __shared__ uint32_t feat[kSortMax];
    __shared__ int32_t bucket_at[kSortMax];
    const int tid = threadIdx.x;
    const int64_t i = blockIdx.x;
    const uint32_t* row = table + i * nt;
    const int G = (b + 63) / 64;
    int D = 0;
    while ((1 << D) < G) ++D;
    int N = 1;
    while (N < b) N <<= 1;
    for (int p = tid; p < b; p += kGroupThreads) bucket_at[p] = p;
    __syncthreads();
    for (int d = 0; d < D; ++d) {
        for (int c = tid; c < b; c += kGroupThreads) feat[c] = 0;
        __syncthreads();
        for (int64_t w = d; w < nwin; w += D) {
            const int64_t k0 = w * (int64_t)kWin;
            const int64_t k1 = min(n, k0 + kWin);
            // the window's entries: all loads issued before the first atomic
            constexpr int kU = kWin / kGroupThreads;
            uint32_t e[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t k = k0 + u * kGroupThreads + tid;
                e[u] = row[min(k, k1 - 1)];
            }
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (k0 + u * kGroupThreads + tid < k1) atomicAdd(&feat[e[u] & 0x7FFFFFFFu], 1u);
        }
        __syncthreads();
        // key = (first group of the position's level-d node, count, position)
        for (int p = tid; p < N; p += kGroupThreads) {
            uint64_t kk = ~0ull;
            if (p < b) {
                int glo = 0, ghi = G;
                for (int lv = 0; lv < d; ++lv) {
                    const int gm = (glo + ghi) >> 1;
                    if ((p >> 6) < gm)
                        ghi = gm;
                    else
                        glo = gm;
                }
                kk = ((uint64_t)glo << 50) | ((uint64_t)feat[bucket_at[p]] << 14) | (uint64_t)p;
            }
            key[p] = kk;
        }
        __syncthreads();
        // bitonic sort of key[0, N), ascending.  Thread t exchanges the pair
        // (lo, lo + stride), lo = 2t - t % stride.  For strides up to 64 the
        // pairs of wave w lie in entries [128w, 128w + 128), so two such
        // stages in a row need only the wave's own LDS ordering (a wave's
        // LDS instructions execute in program order); a stage that crosses
        // waves (stride >= 128, or several pairs per thread) is fenced by
        // workgroup barriers on both sides.
        bool prev_cross = true;          // (the keys were just written by all waves)
        for (int size = 2; size <= N; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                const bool cross = stride >= 128 || N / 2 > kGroupThreads;
                if (cross || prev_cross) {
                    __syncthreads();
                } else {
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
                prev_cross = cross;
                for (int t = tid; t < N / 2; t += kGroupThreads) {
                    const int lo = 2 * t - (t & (stride - 1));
                    const int hi = lo + stride;
                    const bool up = (lo & size) == 0;
                    const uint64_t x = key[lo], y = key[hi];
                    if ((x > y) == up) {
                        key[lo] = y;
                        key[hi] = x;
                    }
                }
            }
        }
        __syncthreads();
        // the bucket now at position p was at position key[p] & 0x3FFF
        for (int p = tid; p < b; p += kGroupThreads) feat[p] = (uint32_t)bucket_at[key[p] & 0x3FFF];
        __syncthreads();
        for (int p = tid; p < b; p += kGroupThreads) bucket_at[p] = (int32_t)feat[p];
        __syncthreads();
    }
    for (int p = tid; p < b; p += kGroupThreads) inv[i * bp + bucket_at[p]] = p;
}

// bucket order of block i: order[i * bp + p] = the bucket at position p
// (p < b), p itself for the empty positions p >= b.
__global__ __launch_bounds__(256) void bucket_order_kernel(const int32_t* __restrict__ inv,
                                                           int32_t b, int32_t bp,
                                                           int32_t* __restrict__ order) {
    const int64_t i = blockIdx.y;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < bp; c += gridDim.x * blockDim.x) {
        if (c < b)
            order[i * bp + inv[i * bp + c]] = c;
        else
            order[i * bp + c] = c;
    }
}

__global__ __launch_bounds__(256) void identity_inv_kernel(int32_t bp, int32_t* __restrict__ inv) {
    const int64_t i = blockIdx.y;
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < bp; c += gridDim.x * blockDim.x)
        inv[i * bp + c] = c;
}

// ---------------------------------------------------------------------------
// Transpose: Y (cols x rows, ld ldy) = X^T for X rows x cols (ld ldx): FP32
// to FP32, or BF16 to BF16 (values copied exactly; staged through LDS as
// FP32, which holds every BF16 value).  A workgroup of 512 threads moves
// a 64 x 256 tile of X through LDS (row stride 257 floats: the column reads
// are conflict-free): every row of X contributes 256 consecutive values and
// every row of Y 64, each lane moving 4 values per access.
//   kWhole = true : the wr x wc whole tiles, X aligned to 4 values with
//                   ldx % 4 == 0: vector accesses with no bounds checks and
//                   no branches (a branch between the loads and their LDS
//                   writes, or between the LDS reads and the stores, costs
//                   8-10 % here);
//   kWhole = false: every other tile (the right and bottom strips, or all
//                   tiles when X is not aligned): loads clamped into the
//                   matrix, stores guarded.
// Y is aligned to 4 of its values with ldy % 4 == 0 (checked by the launcher).
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ float4 load4(const T* p);

template <>
__device__ __forceinline__ float4 load4<float>(const float* p) {
    return *reinterpret_cast<const float4*>(p);
}

template <>
__device__ __forceinline__ float4 load4<__bf16>(const __bf16* p) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
    return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
}

constexpr int kTrRows = 64;
constexpr int kTrCols = 256;

template <typename TO>
__device__ __forceinline__ void store4(TO* p, const float4& v);

template <>
__device__ __forceinline__ void store4<float>(float* p, const float4& v) {
    *reinterpret_cast<float4*>(p) = v;
}

template <>
__device__ __forceinline__ void store4<__bf16>(__bf16* p, const float4& v) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const bf16x4 w = {(__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
    *reinterpret_cast<bf16x4*>(p) = w;
}

template <typename T, bool kWhole, typename TO>
__global__ __launch_bounds__(512) void transpose_kernel(const T* __restrict__ X, int64_t rows,
                                                        int64_t cols, int64_t ldx,
                                                        TO* __restrict__ Y, int64_t ldy,
                                                        int64_t wr, int64_t wc) {
    __shared__ float t[kTrRows][kTrCols + 1];
    const int tid = threadIdx.x;
    int64_t r0, c0;
    if constexpr (kWhole) {
        const int64_t Tk = xcd_task(blockIdx.x, wr * wc);
        r0 = Tk / wc * kTrRows;
        c0 = Tk % wc * kTrCols;
    } else {
        // the right strip (tile rows < wr, tile columns >= wc), then the
        // bottom strip (tile rows >= wr, every tile column)
        const int64_t C = (cols + kTrCols - 1) / kTrCols;
        const int64_t right = wr * (C - wc);
        const int64_t k = blockIdx.x;
        if (k < right) {
            r0 = k / (C - wc) * kTrRows;
            c0 = (wc + k % (C - wc)) * kTrCols;
        } else {
            r0 = (wr + (k - right) / C) * kTrRows;
            c0 = (k - right) % C * kTrCols;
        }
    }
    // load: row sub + 8i of the tile, columns q .. q+3
    const int sub = tid >> 6;
    const int q = 4 * (tid & 63);
    float4 v[8];
    if constexpr (kWhole) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = load4<T>(X + (r0 + sub + 8 * i) * ldx + c0 + q);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const T* p = X + min(r0 + sub + 8 * i, rows - 1) * ldx;
            v[i].x = (float)p[min(c0 + q + 0, cols - 1)];
            v[i].y = (float)p[min(c0 + q + 1, cols - 1)];
            v[i].z = (float)p[min(c0 + q + 2, cols - 1)];
            v[i].w = (float)p[min(c0 + q + 3, cols - 1)];
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = sub + 8 * i;
        t[r][q + 0] = v[i].x;
        t[r][q + 1] = v[i].y;
        t[r][q + 2] = v[i].z;
        t[r][q + 3] = v[i].w;
    }
    __syncthreads();
    // store: row cs + 32i of the tile of Y (a column of X), columns p .. p+3
    const int cs = tid >> 4;
    const int p = 4 * (tid & 15);
    float4 w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = cs + 32 * i;
        w[i] = make_float4(t[p][c], t[p + 1][c], t[p + 2][c], t[p + 3][c]);
    }
    const int64_t yc = r0 + p;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int64_t yr = c0 + cs + 32 * i;
        TO* o = Y + yr * ldy + yc;
        if constexpr (kWhole) {
            store4<TO>(o, w[i]);
        } else if (yr < cols) {
            if (yc + 3 < rows) {
                store4<TO>(o, w[i]);
            } else {
                if (yc < rows) o[0] = (TO)w[i].x;
                if (yc + 1 < rows) o[1] = (TO)w[i].y;
                if (yc + 2 < rows) o[2] = (TO)w[i].z;
            }
        }
    }
}

struct Plan {
    int32_t qn;      // groups of 64 buckets per block
    int32_t nwin;    // windows over the sketched dimension
    int64_t RC;      // chunks per (block, window) region
};

Plan plan_of(int64_t n, int32_t bp) {
    Plan p;
    p.qn = (bp + 63) / 64;
    p.nwin = (int32_t)((n + kWin - 1) / kWin);
    p.RC = (min((int64_t)kWin, n) + 7) / 8 + p.qn;
    return p;
}

struct ListView {
    uint32_t* hdr;
    uint4* ell;
};

ListView carve_lists(void* lists, int32_t nblk, int64_t n, int32_t bp) {
    const Plan p = plan_of(n, bp);
    char* base = static_cast<char*>(lists);
    ListView v;
    v.hdr = reinterpret_cast<uint32_t*>(base);
    base += round_up((int64_t)nblk * p.nwin * p.qn * 4, 256);
    v.ell = reinterpret_cast<uint4*>(base);
    return v;
}

// Compute units of the current device (0 if unknown).
int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return cus;
}

// Passes and slots per pass for nst stored blocks: as few passes as the slots
// allow, and more (each a workgroup's own task) while the line groups leave
// CUs idle and the passes' waves hold more than one slot.
void pass_plan(int32_t nst, int32_t qn, int32_t* npass, int32_t* slots, int64_t groups = 0,
               int cus = 0) {
    const int64_t gs = (int64_t)nst * qn;
    const int64_t per = (int64_t)kWaves * kMaxSlots;
    int64_t P = (gs + per - 1) / per;
    while (groups > 0 && groups * (P + 1) <= cus && gs > P * kWaves) ++P;
    const int64_t need = (gs + P - 1) / P;               // groups per pass
    *npass = (int32_t)P;
    *slots = (int32_t)((need + kWaves - 1) / kWaves);
}

// X: FP32, or BF16 when bf16 (unweighted; its columns: out_mode 0 to 2 and
// sketch_rows_bf16_in_place_ok).  out_mode: 0 = FP32
// sketch (blocks bp apart); 1 = its BF16 rounding, 2 = BF16 and residual
// (nst blocks after), 3 = FP8 codes, then their scales, 4 = FP8 codes, the
// residuals' codes, then the scales of both (blocks round_up(bp, 64) apart).
hipError_t launch_sketch(bool row_lines, const void* X, bool bf16, int64_t lines, int64_t n,
                         int64_t ldx, const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                         const void* lists, void* out, int64_t ldo, hipStream_t s,
                         const float* wd = nullptr, int out_mode = 0) {
    const Plan p = plan_of(n, bp);
    const ListView v = carve_lists(const_cast<void*>(lists), nblk, n, bp);
    const bool wide = bf16 && !row_lines;
    const int L = wide ? 2 * kLines : kLines;
    const int64_t groups = (lines + L - 1) / L;
    const int cus = device_cus();
    int32_t npass, slots;
    pass_plan(nst, p.qn, &npass, &slots, groups, cus);
    // persistent workgroups: one per CU (a window fills a CU's LDS)
    int64_t nwg = groups * npass;
    if (cus > 0) nwg = std::min<int64_t>(nwg, cus);
    const dim3 grid((unsigned)nwg);
    if (out_mode < 0 || out_mode > 4) return hipErrorInvalidValue;
    const int32_t obp = out_mode ? p.qn * 64 : bp;
    const int64_t ozlo = out_mode >= 2 ? (int64_t)nst * obp : 0;
    SketchArgs a{X,     lines, n,   ldx,   0,  p.qn, p.nwin,   nst, &bl, p.RC, v.hdr,
                 v.ell, out,   ldo, npass, wd, obp,  out_mode, ozlo};
    if ((wide && (out_mode > 2 || lines < L || slots > kMaxWideSlots)) ||
        ((out_mode >= 3 || bf16) && wd))
        return hipErrorInvalidValue;
    if (row_lines ? n < 4 : lines < 4) {     // loads of 4 values would leave the matrix
        if (out_mode >= 3) return hipErrorInvalidValue;
        if (!row_lines && n >= 4) return sketch_narrow(slots, grid, s, a);
        a.ldx = row_lines ? ldx : 1;
        a.ldk = row_lines ? 1 : ldx;
        return wd     ? sketch_short_weighted(slots, grid, s, a)
               : bf16 ? sketch_short_bf16(slots, grid, s, a)
                      : sketch_short(slots, grid, s, a);
    }
    if (out_mode == 3)
        return bf16        ? sketch_rows_bf16_fp8(slots, grid, s, a)
               : row_lines ? sketch_rows_f32_fp8(slots, grid, s, a)
                           : sketch_cols_f32_fp8(slots, grid, s, a);
    if (out_mode == 4)
        return bf16        ? sketch_rows_bf16_fp8x3(slots, grid, s, a)
               : row_lines ? sketch_rows_f32_fp8x3(slots, grid, s, a)
                           : sketch_cols_f32_fp8x3(slots, grid, s, a);
    if (wide) return sketch_cols_bf16(slots, grid, s, a);
    if (bf16) return sketch_rows_bf16(slots, grid, s, a);
    if (!row_lines) return sketch_cols_f32(slots, grid, s, a);
    return wd ? sketch_rows_weighted(slots, grid, s, a) : sketch_rows_f32(slots, grid, s, a);
}

}  // namespace

size_t list_bytes(int32_t nblk, int64_t n, int32_t bp) {
    const Plan p = plan_of(n, bp);
    return (size_t)round_up((int64_t)nblk * p.nwin * p.qn * 4, 256) +
           (size_t)nblk * (size_t)p.nwin * (size_t)p.RC * 1024u;
}

void prep_desc_lists(PrepDesc& d, void* lists) {
    const Plan p = plan_of(d.n, d.bp);
    const ListView v = carve_lists(lists, d.nblk, d.n, d.bp);
    d.hdr = v.hdr;
    d.ell = reinterpret_cast<uint16_t*>(v.ell);
    d.qn = p.qn;
    d.nwin = p.nwin;
    d.RC = p.RC;
}

hipError_t launch_lists_batch(const PrepDesc* descs, int32_t count, int64_t tasks,
                              int32_t max_bp, hipStream_t s) {
    if (count < 1 || tasks < 1 || max_bp < 1) return hipErrorInvalidValue;
    const int32_t qn = (max_bp + 63) / 64;
    const unsigned grid = (unsigned)std::min<int64_t>(tasks, int64_t(1) << 20);
    if (max_bp <= kBWMaxBp) {
        const size_t lds = (size_t)((kBWBatch + 2) * max_bp + 2 * qn + kWin) * 4;
        hipLaunchKernelGGL(ell_build_batchw_kernel, dim3(grid), dim3(64 * kBWBatch), lds, s, descs,
                           count, tasks);
    } else {
        const size_t lds = (size_t)(2 * max_bp + 2 * qn + kWin) * 4;
        hipLaunchKernelGGL(ell_build_batch_kernel, dim3(grid), dim3(64), lds, s, descs, count,
                           tasks);
    }
    return hipGetLastError();
}

namespace {

// The wave-parallel builder (bp <= kBWMaxBp), from the packed table or (table
// = nullptr) from the hash or explicit tables.
hipError_t launch_lists_waves(const uint32_t* table, uint64_t seed, const int32_t* h,
                              const int8_t* sigma, int64_t n, int64_t nt, int32_t nblk, int32_t b,
                              int32_t bp, void* lists, const int32_t* inv, int32_t* inv_out,
                              hipStream_t s) {
    const Plan p = plan_of(n, bp);
    const ListView v = carve_lists(lists, nblk, n, bp);
    const bool wide = bp <= kBWWideMaxBp;
    const int waves = wide ? kBWWide : kBWSingle;
    // workgroups per region: up to 8 while the device has CUs for them, none
    // with less than one 64-entry part per wave
    int Z = 1;
    while (Z < 8 && (int64_t)2 * Z * p.nwin * nblk <= 256 &&
           2 * Z * waves * 64 <= std::min<int64_t>(n, kWin))
        Z *= 2;
    const size_t lds = (size_t)((waves + 2 + (Z > 1)) * bp + 2 * p.qn + kWin) * 4;
    auto kern = wide ? ell_buildw_kernel<kBWWide> : ell_buildw_kernel<kBWSingle>;
    hipLaunchKernelGGL(kern, dim3((unsigned)p.nwin, (unsigned)nblk, (unsigned)Z), dim3(64 * waves),
                       lds, s, table,
                       seed, h, sigma, n, nt, b, bp, p.qn, p.nwin, p.RC, v.hdr,
                       reinterpret_cast<uint16_t*>(v.ell), inv, inv_out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_build_lists(const uint32_t* table, int64_t n, int64_t nt, int32_t nblk,
                              int32_t bp, void* lists, hipStream_t s, const int32_t* inv) {
    if (bp <= kBWMaxBp)
        return launch_lists_waves(table, 0, nullptr, nullptr, n, nt, nblk, bp, bp, lists, inv,
                                  nullptr, s);
    const Plan p = plan_of(n, bp);
    const ListView v = carve_lists(lists, nblk, n, bp);
    const size_t lds = (size_t)(2 * bp + 2 * p.qn + kWin) * 4;
    hipLaunchKernelGGL(ell_build_kernel, dim3((unsigned)p.nwin, (unsigned)nblk), dim3(64), lds, s,
                       table, n, nt, bp, p.qn, p.nwin, p.RC, v.hdr,
                       reinterpret_cast<uint16_t*>(v.ell), inv);
    return hipGetLastError();
}

bool lists_need_table(int32_t bp) { return bp > kBWMaxBp; }

hipError_t launch_hash_lists(uint64_t seed, const int32_t* h, const int8_t* sigma, int64_t n,
                             int32_t nblk, int32_t b, int32_t bp, void* lists, int32_t* inv,
                             hipStream_t s) {
    if (lists_need_table(bp)) return hipErrorInvalidValue;
    return launch_lists_waves(nullptr, seed, h, sigma, n, 0, nblk, b, bp, lists, nullptr, inv, s);
}

hipError_t launch_group_buckets(const uint32_t* table, int64_t n, int64_t nt, int32_t nblk,
                                int32_t b, int32_t bp, int32_t* inv, hipStream_t s) {
    if (b < 1 || b > kSortMax || bp < b || nblk < 1) return hipErrorInvalidValue;
    const Plan p = plan_of(n, bp);
    if (b <= 64) {      // one group: nothing to order
        hipLaunchKernelGGL(identity_inv_kernel, dim3((unsigned)((bp + 255) / 256), (unsigned)nblk),
                           dim3(256), 0, s, bp, inv);
    } else {
        hipLaunchKernelGGL(group_kernel, dim3((unsigned)nblk), dim3(kGroupThreads), 0, s, table,
                           n, nt, b, bp, p.nwin, inv);
    }
    return hipGetLastError();
}

hipError_t launch_identity_inv(int32_t nblk, int32_t bp, int32_t* inv, hipStream_t s) {
    hipLaunchKernelGGL(identity_inv_kernel, dim3((unsigned)((bp + 255) / 256), (unsigned)nblk),
                       dim3(256), 0, s, bp, inv);
    return hipGetLastError();
}

hipError_t launch_bucket_order(const int32_t* inv, int32_t nblk, int32_t b, int32_t bp,
                               int32_t* order, hipStream_t s) {
    hipLaunchKernelGGL(bucket_order_kernel, dim3((unsigned)((bp + 255) / 256), (unsigned)nblk),
                       dim3(256), 0, s, inv, b, bp, order);
    return hipGetLastError();
}

bool plan_sketch_ok(int64_t lines, int32_t nst, int32_t bp, int64_t n) {
    if (lines < 1 || nst < 1 || nst > OS_MAX_BLOCKS || bp < kBlockAlign || bp % kBlockAlign ||
        n < 1 || n > kMaxSketchedLen)
        return false;
    const Plan p = plan_of(n, bp);
    int32_t npass, slots;
    pass_plan(nst, p.qn, &npass, &slots);
    const int64_t groups = (lines + kLines - 1) / kLines;
    return groups * npass <= 0x7fffffff && slots <= kMaxSlots;
}

hipError_t launch_sketch_rows(const float* X, int64_t n, int64_t cols, int64_t ldx,
                              const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                              const void* lists, float* out, int64_t ldo, hipStream_t s) {
    if (!plan_sketch_ok(cols, nst, bp, n)) return hipErrorInvalidValue;
    return launch_sketch(false, X, false, cols, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s);
}

bool sketch_rows_in_place_ok(int64_t n, int64_t cols, int64_t ldx, int32_t nst, int32_t bp) {
    const Plan p = plan_of(n, bp);
    const int64_t groups = (cols + kLines - 1) / kLines;
    const int cus = device_cus();
    if (cus < 1) return true;
    int32_t npass, slots;
    pass_plan(nst, p.qn, &npass, &slots, groups, cus);
    const double rounds = (double)((groups * npass + cus - 1) / cus);
    const double window = (double)n * (double)ldx <= (double)(1 << 20) ? 2.0 : 6.0;
    const double extra = rounds * ((double)n / kWin) * window * std::min(1.0, (double)ldx / 24);
    return extra <= 8 + (double)n * (double)cols * 1.3e-6;
}

bool sketch_rows_bf16_in_place_ok(int64_t n, int64_t cols, int32_t nst, int32_t bp) {
    const Plan p = plan_of(n, bp);
    int32_t npass, slots;
    pass_plan(nst, p.qn, &npass, &slots);
    if (cols < 2 * kLines || slots > kMaxWideSlots) return false;
    return p.nwin == 1 || cols / kLines >= device_cus();
}

hipError_t launch_sketch_rows_bf16(const void* X, int64_t n, int64_t cols, int64_t ldx,
                                   const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                                   const void* lists, void* out, int64_t ldo, int out_mode,
                                   hipStream_t s) {
    if (!plan_sketch_ok(cols, nst, bp, n)) return hipErrorInvalidValue;
    return launch_sketch(false, X, true, cols, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s,
                         nullptr, out_mode);
}

bool sketch_pair_fits(int64_t m, int64_t l, int64_t n, int32_t nst, int32_t bp) {
    const Plan p = plan_of(n, bp);
    const int cus = device_cus();
    const int64_t groups = (m + kLines - 1) / kLines + (l + kLines - 1) / kLines;
    int32_t npass, slots;
    pass_plan(nst, p.qn, &npass, &slots, groups, cus);
    return groups * npass <= cus;
}

bool launch_sketch_pair(bool bf16, const void* A, bool a_rows, int64_t m, int64_t lda, void* outA,
                        const void* B, bool b_rows, int64_t l, int64_t ldb, void* outB, int64_t n,
                        const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                        const void* lists, int64_t ldo, int out_mode, hipStream_t s,
                        hipError_t* err) {
    const Plan p = plan_of(n, bp);
    const int L = bf16 ? 2 * kLines : kLines;
    const int64_t ga = (m + L - 1) / L, gb = (l + L - 1) / L;
    const int cus = device_cus();
    int32_t npass, slots;
    pass_plan(nst, p.qn, &npass, &slots, ga + gb, cus);
    const int most = bf16 ? kMaxWideSlots : (out_mode >= 3 ? kMaxPairFp8Slots : kMaxPairSlots);
    if (cus < 16 || slots > most || out_mode < 0 || out_mode > (bf16 ? 2 : 4) ||
        (out_mode >= 3 && !sketch_fp8_fusable(bp, nst)))
        return false;
    // (BF16: columns only, both in place by the rule for one, on their sum)
    if (bf16 && (a_rows || b_rows || !sketch_rows_bf16_in_place_ok(n, m + l, nst, bp)))
        return false;
    if ((a_rows ? n : m) < L || (b_rows ? n : l) < L || !plan_sketch_ok(m, nst, bp, n) ||
        !plan_sketch_ok(l, nst, bp, n))
        return false;
    // Workgroups of each side: one per task when they fit, else the split of
    // the CUs that ends first, in multiples of the 8 XCDs (a workgroup's tasks
    // then stay on one XCD); a task of columns lasts 1.5 times one of rows.
    // The two launches one by one leave CUs idle in two last rounds; apart /
    // together, whole product, us: 1100 x 10000 x 1100 FP8, 5 blocks of 500,
    // 111 / 80; 1500 x 8000 x 1300 BF16, 5 of 700, 98 / 86; 512 x 8192 x 300,
    // 9 of 512, 76 / 68; BF16 columns, 9000 x 1001 (both), 4 of 400, 84 / 61,
    // 4096 x 1024 and 300, 3 of 256, 40 / 32; where less than a fifteenth is predicted (3333 x
    // 20011 x 2777, 5 of 900, 840 / 849) they stay apart.
    const int64_t ta = ga * npass, tb = gb * npass;
    const double ca = a_rows ? 1 : 1.5, cb = b_rows ? 1 : 1.5;
    int64_t wa = ta, wb = tb;
    if (ta + tb > cus) {
        auto rounds = [](int64_t t, int64_t w) { return (double)((t + w - 1) / w); };
        auto alone = [&](int64_t g) {                    // (a pass is its share of a task)
            int32_t P, ns;
            pass_plan(nst, p.qn, &P, &ns, g, cus);
            return rounds(g * P, cus) * npass / P;
        };
        const double apart = ca * alone(ga) + cb * alone(gb);
        double best = 0;
        for (int64_t w = 8; w < cus; w += 8) {
            const double t = std::max(ca * rounds(ta, w), cb * rounds(tb, cus - w));
            if (best == 0 || t < best) {
                best = t;
                wa = w;
            }
        }
        if (best >= 0.93 * apart) return false;
        wb = std::min(cus - wa, tb);
        wa = std::min(wa, ta);
    }
    const ListView v = carve_lists(const_cast<void*>(lists), nblk, n, bp);
    const int32_t obp = out_mode ? p.qn * 64 : bp;
    const SketchArgs a{nullptr, 0,     n,     0,       0,   p.qn,  p.nwin,  nst, &bl,
                       p.RC,    v.hdr, v.ell, nullptr, ldo, npass, nullptr, obp, out_mode,
                       out_mode >= 2 ? (int64_t)nst * obp : 0};
    const SketchSide x{A, m, lda, outA, (int32_t)wa, a_rows ? 1 : 0};
    const SketchSide y{B, l, ldb, outB, (int32_t)wb, b_rows ? 1 : 0};
    *err = bf16            ? sketch_pair_bf16(slots, s, a, x, y)
           : out_mode == 4   ? sketch_pair_fp8x3(slots, s, a, x, y)
           : out_mode == 3 ? sketch_pair_fp8(slots, s, a, x, y)
                           : sketch_pair(slots, s, a, x, y);
    return true;
}

hipError_t launch_sketch_rows_q(const float* X, int64_t n, int64_t cols, int64_t ldx,
                                const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                                const void* lists, void* out, int64_t ldo, int split,
                                hipStream_t s) {
    if (!plan_sketch_ok(cols, nst, bp, n)) return hipErrorInvalidValue;
    return launch_sketch(false, X, false, cols, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s,
                         nullptr, split ? 2 : 1);
}

hipError_t launch_sketch_rows_fp8(const float* X, int64_t n, int64_t cols, int64_t ldx,
                                  const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                                  const void* lists, void* out, int64_t ldo, int split,
                                  hipStream_t s) {
    if (!plan_sketch_ok(cols, nst, bp, n) || !sketch_fp8_fusable(bp, nst))
        return hipErrorInvalidValue;
    return launch_sketch(false, X, false, cols, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s,
                         nullptr, split ? 4 : 3);
}

size_t transpose_bytes(int64_t rows, int64_t cols) {
    return (size_t)round_up(cols * round_up(rows, 4) * 4, 256);
}

template <typename T, typename TO>
hipError_t launch_transpose_t(const T* X, int64_t rows, int64_t cols, int64_t ldx, TO* Y,
                              int64_t ldy, hipStream_t s) {
    const int64_t R = (rows + kTrRows - 1) / kTrRows;
    const int64_t C = (cols + kTrCols - 1) / kTrCols;
    if (R * C > 0x7fffffff || ldy % 4 || (reinterpret_cast<uintptr_t>(Y) % (4 * sizeof(TO))))
        return hipErrorInvalidValue;
    const bool vec = (reinterpret_cast<uintptr_t>(X) % (4 * sizeof(T))) == 0 && (ldx & 3) == 0;
    const int64_t wr = vec ? rows / kTrRows : 0;     // whole tiles: wr x wc
    const int64_t wc = vec ? cols / kTrCols : 0;
    if (wr * wc > 0)
        hipLaunchKernelGGL((transpose_kernel<T, true, TO>), dim3((unsigned)(wr * wc)), dim3(512),
                           0, s, X, rows, cols, ldx, Y, ldy, wr, wc);
    if (R * C > wr * wc)
        hipLaunchKernelGGL((transpose_kernel<T, false, TO>), dim3((unsigned)(R * C - wr * wc)),
                           dim3(512), 0, s, X, rows, cols, ldx, Y, ldy, wr, wc);
    return hipGetLastError();
}

hipError_t launch_transpose(const float* X, int64_t rows, int64_t cols, int64_t ldx, float* Y,
                            int64_t ldy, hipStream_t s) {
    return launch_transpose_t(X, rows, cols, ldx, Y, ldy, s);
}

hipError_t launch_transpose_bf16_raw(const void* X, int64_t rows, int64_t cols, int64_t ldx,
                                     void* Y, int64_t ldy, hipStream_t s) {
    return launch_transpose_t(static_cast<const __bf16*>(X), rows, cols, ldx,
                              static_cast<__bf16*>(Y), ldy, s);
}

hipError_t launch_sketch_cols(const float* X, int64_t rows, int64_t n, int64_t ldx,
                              const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                              const void* lists, float* out, int64_t ldo, hipStream_t s,
                              const float* wd) {
    if (!plan_sketch_ok(rows, nst, bp, n)) return hipErrorInvalidValue;
    return launch_sketch(true, X, false, rows, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s, wd);
}

hipError_t launch_sketch_cols_bf16(const void* X, int64_t rows, int64_t n, int64_t ldx,
                                   const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                                   const void* lists, float* out, int64_t ldo, hipStream_t s) {
    if (!plan_sketch_ok(rows, nst, bp, n)) return hipErrorInvalidValue;
    return launch_sketch(true, X, true, rows, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s);
}

hipError_t launch_sketch_cols_q(const void* X, bool x_bf16, int64_t rows, int64_t n, int64_t ldx,
                                const BlockList& bl, int32_t nst, int32_t nblk, int32_t bp,
                                const void* lists, void* out, int64_t ldo, int split,
                                hipStream_t s) {
    if (!plan_sketch_ok(rows, nst, bp, n)) return hipErrorInvalidValue;
    return launch_sketch(true, X, x_bf16, rows, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s,
                         nullptr, split ? 2 : 1);
}

bool sketch_fp8_fusable(int32_t b, int32_t nst) {
    if (round_up(b, 64) != block_stride_fp8(b)) return false;
    // (the 12-slot kernel with the FP8 epilogue would spill)
    int32_t npass, slots;
    pass_plan(nst, (int32_t)(round_up(b, kBlockAlign) + 63) / 64, &npass, &slots);
    return slots <= kMaxFp8Slots;
}

hipError_t launch_sketch_cols_fp8(const void* X, bool x_bf16, int64_t rows, int64_t n,
                                  int64_t ldx, const BlockList& bl, int32_t nst, int32_t nblk,
                                  int32_t bp, const void* lists, void* out, int64_t ldo,
                                  int split,
                                  hipStream_t s) {
    if (!plan_sketch_ok(rows, nst, bp, n) || !sketch_fp8_fusable(bp, nst))
        return hipErrorInvalidValue;
    return launch_sketch(true, X, x_bf16, rows, n, ldx, bl, nst, nblk, bp, lists, out, ldo, s,
                         nullptr, split ? 4 : 3);
}

}  // namespace osk
