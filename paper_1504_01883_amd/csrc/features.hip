// Fused depth-masked LBP + regional histogram + L1 normalisation, gfx950.
//
// One workgroup (4 wave64) per face crop; every step runs inside one launch:
//   1. exact lower median m of the crop's non-zero depth (the depth region of
//      interest of the paper's fusion);
//   2. for every interior pixel whose depth d satisfies d != 0 and
//      |d - m| < window, the 3x3 LBP code of the grey and of the depth plane
//      (Sec. 2.4, Eq. 2: neighbour p has weight 2^p and its bit is set when it
//      is >= the centre; p0 = top-left neighbour, then clockwise);
//   3. code -> uniform-59 bin through a 256-entry LDS table;
//   4. increments of the regional histograms (Eq. 3) held in LDS;
//   5. the row written once to HBM as count / T, T = channels * n_in, each
//      quotient the correctly rounded IEEE single division (and optionally the
//      raw counts).
//
// Kernels:
//   k_features_fast       -- the default configuration (uniform-59 bins, both
//                            channels, window 1..255 mm), one workgroup per
//                            crop. Crops up to 256 px wide in one panel of the
//                            lane path below, wider ones in several; crops
//                            whose median lies within the window of 0 pixel by
//                            pixel, inside the same launch.
//   k_features_persistent -- the same per crop, a fixed grid taking crops
//                            from a self-resetting work queue (ragged batches).
//   k_split_*             -- the same configuration, several workgroups per
//                            crop, for few or large crops.
//   k_features_any        -- every other configuration (256 bins, one channel,
//                            mask off, wide windows, coarse grids).
//
// Default configuration, per crop:
//   * Median: the four waves each estimate it from 64 pixels of a 16 x 16
//     sampling grid; one pass over the crop then histograms the 64 mm window
//     (where several workgroups share a crop, a wider one if the estimates
//     disagree) around the combined estimate (1 mm bins, LDS atomics) and counts
//     non-zero pixels and pixels above the window's start in packed 16-bit
//     registers; when the median falls in the window the histogram gives
//     it, otherwise an exact two-level radix select (high byte, then low
//     byte) runs.
//   * Codes: lanes own 4 adjacent columns and walk down a band of rows with a
//     3-row register window. Each pixel is packed as (grey | d' << 16) with
//     d' = clamp(d - (m - window), 0, 2 window) (0 for d = 0): clamping keeps
//     every comparison against an in-window centre unchanged and makes the
//     depth fit 9 bits, so ONE packed 16-bit subtraction per neighbour yields
//     both channels' comparisons: the sign bit of each 16-bit half. Byte
//     permutes gather the sign bits of two neighbours per instruction and
//     masked AND-ORs merge them into one word holding both channels'
//     comparison bytes. Halo columns come from the neighbouring lanes through
//     DPP wave shifts.
//   * Counters: one LDS word per (cell, bin), the grey count in its low 16
//     bits and the depth count in its high 16 bits.
//   * Normalisation: count / T is tabulated once per crop for every count a
//     cell can hold, then the row is written by table lookup.
#include "lbpf_internal.h"

#include <algorithm>

namespace lbpf {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kFastMaxW = 256;    // 64 lanes x 4 columns
constexpr int kQuot = 1088;       // tabulated quotients (cells up to 32 x 34 px)
constexpr int kU59 = 59;

// Neighbour p of the centre (y, x) is (y + kDy[p], x + kDx[p]).
__constant__ int8_t kDy[8] = {-1, -1, -1, 0, 1, 1, 1, 0};
__constant__ int8_t kDx[8] = {-1, 0, 1, 1, 1, 0, -1, -1};

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b));
}
__device__ __forceinline__ uint32_t pk_sub_sat(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, a),
                                                                      __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, int lane) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t t = __shfl_up(v, off, 64);
        if (lane >= off) v += t;
    }
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

struct MedianScratch {
    uint32_t hist[256];
    int32_t bin;
    uint32_t rank;
    uint32_t est[4];  // median estimates of the first four waves
};

// On wave 0: find the bin of a 256-bin LDS histogram that holds 0-based rank
// `rank`, and the rank inside that bin. rank >= total leaves ms.bin at -1.
__device__ __forceinline__ void select_bin(MedianScratch &ms, uint32_t rank, int lane) {
    const uint32_t c0 = ms.hist[4 * lane + 0], c1 = ms.hist[4 * lane + 1],
                   c2 = ms.hist[4 * lane + 2], c3 = ms.hist[4 * lane + 3];
    const uint32_t s = c0 + c1 + c2 + c3;
    const uint32_t incl = wave_inclusive_scan(s, lane);
    const uint32_t excl = incl - s;
    if (lane == 0) ms.bin = -1;
    if (excl <= rank && rank < incl) {
        uint32_t r = rank - excl;
        int b = 4 * lane;
        if (r >= c0) {
            r -= c0;
            b += 1;
            if (r >= c1) {
                r -= c1;
                b += 1;
                if (r >= c2) {
                    r -= c2;
                    b += 1;
                }
            }
        }
        ms.bin = b;
        ms.rank = r;
    }
}

__device__ __forceinline__ bool centre_in_mask(uint32_t d, int32_t m, int32_t window) {
    if (window <= 0) return true;
    if (m < 0 || d == 0) return false;
    const int32_t diff = (int32_t)d - m;
    return diff < window && -diff < window;
}

template <typename T>
__device__ __forceinline__ uint32_t lbp_code(const T *p, int32_t pitch, int y, int x) {
    const uint32_t c = p[(size_t)y * pitch + x];
    uint32_t code = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t g = p[(size_t)(y + kDy[k]) * pitch + (x + kDx[k])];
        code |= (g >= c ? 1u : 0u) << k;
    }
    return code;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Load through the global address space at a 32-bit byte offset from a
// workgroup-uniform base (global_load with an SGPR base). Unaligned
// addresses are fine on gfx950.
template <typename T>
__device__ __forceinline__ T gld(const void *base, uint32_t byte_off) {
    typedef __attribute__((address_space(1))) const T gT;
    return *(const gT *)((const __attribute__((address_space(1))) char *)base + byte_off);
}

// Streaming (non-temporal) store: the feature rows are not read again by this
// kernel, and kept out of L2's reuse they do not evict the depth lines that
// the code pass reads a second time.
template <typename T>
__device__ __forceinline__ void st_nt(T *p, T v) {
    __builtin_nontemporal_store(v, p);
}
// (a & m) | c with m in an SGPR: one VALU instruction (gfx9 VOP3 takes no
// literal, so the compiler would otherwise split it into AND + OR).
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t m, uint32_t c) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(m), "v"(c));
    return r;
}

// a + b + c in one instruction; written out because the compiler otherwise
// shares a + b between two such sums and spends three adds on them.
__device__ __forceinline__ uint32_t add3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}

// Depth pixels x0..x0+7 of crop row y as four u16 pairs; pixels at x >= w
// read as 0. A chunk that ends past the right edge of a crop that may not be
// over-read is loaded from column w - 8 instead (crops at least 8 wide), and
// the pixels before x0 are zeroed as well: the median pass does not count a
// zero, so every pixel still counts once, and the chunk is one load.
__device__ __forceinline__ u32x4 depth_chunk(const CropDesc &c, int y, int x0) {
    const bool inside = (c.flags & kCropOverReadOk) || x0 + 8 <= c.w;
    if (inside || c.w >= 8) {
        const int xs = inside ? x0 : c.w - 8;
        u32x4 q = gld<u32x4>(c.depth, ((uint32_t)y * (uint32_t)c.depth_pitch + (uint32_t)xs) * 2u);
        if (x0 + 8 > c.w) {
            // Element e (column xs + e) is kept iff x0 <= xs + e < w.
            const int lo = x0 - xs, hi = c.w - xs;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t keep = (2 * i >= lo && 2 * i < hi ? 0x0000FFFFu : 0u) |
                                      (2 * i + 1 >= lo && 2 * i + 1 < hi ? 0xFFFF0000u : 0u);
                q[i] &= keep;
            }
        }
        return q;
    }
    const uint16_t *row = c.depth + (size_t)y * c.depth_pitch;
    u32x4 q;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = (x0 + 2 * i < c.w) ? row[x0 + 2 * i] : 0u;
        const uint32_t b = (x0 + 2 * i + 1 < c.w) ? row[x0 + 2 * i + 1] : 0u;
        q[i] = a | (b << 16);
    }
    return q;
}

constexpr int kMedBatch = 8;  // 16-byte chunks in flight per thread

// f(v) for the eight depth pixels v[8] of every chunk of the crop that falls to
// this thread of kNT (0: no depth, or outside the crop), four chunks in flight.
template <int kNT, typename F>
__device__ __forceinline__ void each_chunk(const CropDesc &c, F &&f) {
    const int cpr = (c.w + 7) >> 3;              // 8-pixel chunks per row (<= 128)
    const int rows_par = kNT / cpr;              // rows visited in parallel
    const int cx = threadIdx.x % cpr, ry0 = threadIdx.x / cpr;
    const int nk = ry0 < rows_par ? max(0, (c.h - ry0 + rows_par - 1) / rows_par) : 0;
    constexpr int kBatch = 4;  // more would cost the kernels a workgroup per CU (VGPRs)
    for (int kb = 0; kb < nk; kb += kBatch) {
        u32x4 buf[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            buf[u] = depth_chunk(c, ry0 + min(kb + u, nk - 1) * rows_par, 8 * cx);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (kb + u >= nk) break;
            uint32_t v[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i] = buf[u][i] & 0xFFFFu;
                v[2 * i + 1] = buf[u][i] >> 16;
            }
            f(v);
        }
    }
}

// The value of rank `rank` among the crop's depths in [base, base + 2^k), k <= 8.
// All kNT threads of the block call it.
template <int kNT>
__device__ __forceinline__ int32_t median_refine(const CropDesc &c, MedianScratch &ms, int32_t base,
                                              uint32_t k, uint32_t rank) {
    for (int i = threadIdx.x; i < 256; i += kNT) ms.hist[i] = 0;
    __syncthreads();
    each_chunk<kNT>(c, [&](const uint32_t (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (v[i] != 0 && v[i] - (uint32_t)base < (1u << k)) atomicAdd(&ms.hist[v[i] - base], 1u);
    });
    __syncthreads();
    if (threadIdx.x < 64) select_bin(ms, rank, threadIdx.x);
    __syncthreads();
    const int32_t m = base + ms.bin;
    __syncthreads();
    return m;
}

// Exact lower median of the non-zero depth values of the crop by two 256-bin
// passes (high byte, then low byte), -1 if none: for the rare crop whose median
// the window of the estimate misses. All kNT threads of the block call it.
template <int kNT = kThreads>
__device__ __noinline__ int32_t crop_median(const CropDesc c, MedianScratch &ms) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < 256; i += kNT) ms.hist[i] = 0;
    __syncthreads();
    each_chunk<kNT>(c, [&](const uint32_t (&v)[8]) {
        // One atomic for the pixels that share the chunk's middle key.
        const uint32_t key = (v[3] ? v[3] : v[4]) >> 8;
        uint32_t same = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) same += (v[i] != 0 && (v[i] >> 8) == key) ? 1u : 0u;
        if (same) atomicAdd(&ms.hist[key], same);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (v[i] != 0 && (v[i] >> 8) != key) atomicAdd(&ms.hist[v[i] >> 8], 1u);
    });
    __syncthreads();
    if (wave == 0) {
        const uint32_t tot = wave_sum(ms.hist[4 * lane] + ms.hist[4 * lane + 1] +
                                      ms.hist[4 * lane + 2] + ms.hist[4 * lane + 3]);
        if (tot > 0) {
            select_bin(ms, (tot - 1) / 2, lane);
        } else if (lane == 0) {
            ms.bin = -1;
        }
    }
    __syncthreads();
    const int32_t hi = ms.bin;
    const uint32_t rank_in_hi = ms.rank;
    __syncthreads();
    if (hi < 0) return -1;
    return median_refine<kNT>(c, ms, hi << 8, 8, rank_in_hi);
}

// Window of the median pass: bins of 2^k mm from lo on, k = 0 and kMedWin bins
// centred on the estimate where the four wave estimates agree within kMedAgree
// mm; else (two surfaces of about equal share, as where boxes overlap) 256 bins
// that span all four.
constexpr uint32_t kMedWin = 64;
constexpr int32_t kMedAgree = 48;
struct MedWindow {
    int32_t lo;
    uint32_t k;
    bool wide;
};

// One u16 pair of the median pass: per-half counts of v >= lo (ge2) and of
// v != 0 (nz2), and the window's histogram. one2 holds 0x10001 (kept opaque to
// the compiler, see median_rows).
template <bool kWide>
__device__ __forceinline__ void median_count(uint32_t q, uint32_t lolo, uint32_t lm1,
                                             uint32_t one2, uint32_t k, uint32_t &ge2, uint32_t &nz2,
                                             MedianScratch &ms) {
    // v >= lo iff v - (lo - 1) saturates above 0 (lo >= 1, so 0 is not).
    ge2 += pk_min(pk_sub_sat(q, lm1), one2);
    nz2 += pk_min(q, one2);
    const uint32_t t = pk_sub(q, lolo);  // v - lo; past the window for v < lo
    const uint32_t t0 = kWide ? (t & 0xFFFFu) >> k : t & 0xFFFFu, t1 = kWide ? t >> (16 + k) : t >> 16;
    if (t0 < (kWide ? 256u : kMedWin)) atomicAdd(&ms.hist[t0], 1u);
    if (t1 < (kWide ? 256u : kMedWin)) atomicAdd(&ms.hist[t1], 1u);
}

// End of the median pass for a block of kNW waves: totals over the block,
// then the lower median's rank looked up in the window histogram. Returns the
// bin, -1 when the crop has no depth, -2 when the median lies outside the window;
// ms.rank is its rank within the bin. All threads call it; it ends with a
// barrier.
template <int kNW>
__device__ __forceinline__ int32_t median_finish(MedianScratch &ms, uint32_t *sh_red,
                                                 uint32_t ge2, uint32_t nz2) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t nnz = wave_sum((nz2 & 0xFFFFu) + (nz2 >> 16));
    const uint32_t below = nnz - wave_sum((ge2 & 0xFFFFu) + (ge2 >> 16));
    if (lane == 0) {
        sh_red[wave] = below;
        sh_red[kNW + wave] = nnz;
    }
    __syncthreads();
    uint32_t tb = 0, tn = 0;
#pragma unroll
    for (int i = 0; i < kNW; ++i) {
        tb += sh_red[i];
        tn += sh_red[kNW + i];
    }
    if (tn == 0) return -1;  // uniform: every thread sees the same totals
    const uint32_t rank = (tn - 1) / 2;
    if (wave == 0) {
        if (rank >= tb) {
            select_bin(ms, rank - tb, lane);  // -1 when the rank lies above the window
        } else if (lane == 0) {
            ms.bin = -1;
        }
    }
    __syncthreads();
    const int32_t bin = ms.bin;
    __syncthreads();
    return bin >= 0 ? bin : -2;
}

// The median from a bin of the window (or -1, -2: see median_finish).
template <int kNT>
__device__ __forceinline__ int32_t median_of_bin(const CropDesc &c, MedianScratch &ms,
                                                 const MedWindow &win, int32_t bin) {
    if (bin == -1) return -1;
    if (bin == -2) return crop_median<kNT>(c, ms);
    const int32_t v = win.lo + (bin << win.k);
    return win.k == 0 ? v : median_refine<kNT>(c, ms, v, win.k, ms.rank);
}

// One wave's 64-sample estimate of the median: the lower median of the
// non-zero values among `v` (one per lane), or 1000 when all are zero. A binary
// search over the value range finds the smallest t with more than `rank`
// non-zero samples <= t, each count a ballot (16 steps of one compare).
__device__ __forceinline__ uint32_t median_estimate(uint32_t v) {
    const int nz = __popcll(__ballot(v != 0));
    if (nz == 0) return 1000u;
    const uint32_t rank = (uint32_t)(nz - 1) / 2;
    const uint32_t vm1 = v - 1u;  // v = 0 wraps above every bound
    uint32_t lo = 1, hi = 65535;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((uint32_t)__popcll(__ballot(vm1 < mid)) > rank)
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// The window from the four wave estimates (the wide one with kWide only: its
// branch costs the kernels of large batches 1%, and their workgroups overlap
// the rare radix select). lo >= 1, and lo + (bins << k) <= 65536,
// so a value below lo (0 among them) wraps past the window.
template <bool kWide>
__device__ __forceinline__ MedWindow median_window(const MedianScratch &ms) {
    const int32_t ea = min(ms.est[0], ms.est[1]), eb = max(ms.est[0], ms.est[1]);
    const int32_t ec = min(ms.est[2], ms.est[3]), ed = max(ms.est[2], ms.est[3]);
    const int32_t e0 = min(ea, ec), e3 = max(eb, ed);
    MedWindow win;
    win.wide = kWide && e3 - e0 > kMedAgree;
    win.k = 0;
    if (!win.wide) {
        // Centred on the mean of the middle two.
        win.lo = ((max(ea, ec) + min(eb, ed)) >> 1) - (int32_t)kMedWin / 2;
        win.lo = min(max(win.lo, 1), 65536 - (int32_t)kMedWin);
    } else {
        win.lo = max(e0 - 32, 1);
        while (win.k < 7 && (e3 + 32 - win.lo) >> win.k >= 256) ++win.k;
        win.lo = min(win.lo, 65536 - (256 << win.k));
    }
    return win;
}

// The median pass of a block of kNT threads over rows ya .. yb - 1 of a crop:
// clears ms.hist, estimates the crop's median and places the window, then
// counts the rows. Returns the window, the same in every thread and for every
// range of the crop's rows; ge2, nz2: this thread's packed counts of v >= lo and
// v != 0; ms.hist: the window's histogram, complete after the caller's next
// barrier.
template <int kNT, bool kWide>
__device__ __forceinline__ MedWindow median_rows(const CropDesc &c, int ya, int yb, MedianScratch &ms,
                                               uint32_t &ge2, uint32_t &nz2) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cpr = (c.w + 7) >> 3;
    const int rows_par = kNT / cpr;
    const int cx = tid % cpr, ry0 = ya + tid / cpr;
    const int nk = tid / cpr < rows_par ? max(0, (yb - ry0 + rows_par - 1) / rows_par) : 0;
    const int x0 = 8 * cx;
    // The first batch of chunks does not depend on the estimate: issue its
    // loads before the estimate is taken so the two latencies overlap.
    u32x4 buf[kMedBatch];
#pragma unroll
    for (int u = 0; u < kMedBatch; ++u)
        if (nk > 0) buf[u] = depth_chunk(c, ry0 + min(u, nk - 1) * rows_par, x0);
    // select_bin scans all 256 bins; the pass fills the first kMedWin.
    for (int i = tid; i < 256; i += kNT) ms.hist[i] = 0;
    if (kNT == 256 || wave < 4) {
        // Wave w samples grid rows w, w + 4, ... of a 16 x 16 grid over the
        // crop, so each wave's estimate covers the whole crop.
        const int gr = 4 * (lane >> 4) + wave, gc = lane & 15;
        const int sy = ((2 * gr + 1) * c.h) >> 5, sx = ((2 * gc + 1) * c.w) >> 5;
        const uint32_t e = median_estimate(c.depth[(size_t)sy * c.depth_pitch + sx]);
        if (lane == 0) ms.est[wave] = e;
    }
    __syncthreads();
    const MedWindow win = median_window<kWide>(ms);
    const uint32_t lolo = (uint32_t)win.lo * 0x10001u;
    const uint32_t lm1 = (uint32_t)(win.lo - 1) * 0x10001u;
    // A 1 in each half that the compiler cannot see: with a visible constant
    // it turns each packed min below into two compares and selects.
    uint32_t one2 = 0x10001u;
    asm volatile("" : "+s"(one2));

    ge2 = nz2 = 0;  // per-half counts of v >= lo and of v != 0
    for (int kb = 0; kb < nk; kb += kMedBatch) {
        if (kb > 0) {
#pragma unroll
            for (int u = 0; u < kMedBatch; ++u)
                buf[u] = depth_chunk(c, ry0 + min(kb + u, nk - 1) * rows_par, x0);
        }
#pragma unroll
        for (int u = 0; u < kMedBatch; ++u) {
            if (kb + u >= nk) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (kWide && win.wide) median_count<true>(buf[u][i], lolo, lm1, one2, win.k, ge2, nz2, ms);
                else median_count<false>(buf[u][i], lolo, lm1, one2, 0u, ge2, nz2, ms);
            }
        }
    }
    return win;
}

// Exact lower median of the crop's non-zero depth, -1 if none.
//  1. Each wave estimates it as the lower median of the non-zero values
//     among 64 pixels of a 16 x 16 sampling grid (wave w takes the grid rows
//     w, w + 4, ...); the estimate is the mean of the middle two of the four.
//  2. One pass over the crop: the histogram of a window around the estimates
//     (LDS atomics), and per-thread counts of the non-zero pixels and of those
//     below the window (packed 16-bit arithmetic, no atomics).
//  3. When the median's rank falls inside the window, its bin gives it (after
//     a pass over the bin's values where bins are wider than 1 mm); otherwise
//     the two-level radix select runs.
// All kNT threads of the block call it.
template <int kNT, bool kWide>
__device__ __forceinline__ int32_t crop_median_fast(const CropDesc &c, MedianScratch &ms,
                                                   uint32_t *sh_red) {
    uint32_t ge2, nz2;
    const MedWindow win = median_rows<kNT, kWide>(c, 0, c.h, ms, ge2, nz2);
    return median_of_bin<kNT>(c, ms, win, median_finish<kNT / 64>(ms, sh_red, ge2, nz2));
}

// Columns x0..x0+3 of one row as loaded: grey bytes in G, depth u16 pairs
// in Z0 (x0, x0+1) and Z1 (x0+2, x0+3). Every lane issues the same two loads,
// from column xl = x0, or, for a lane that hangs over the right edge of a crop
// that may not be over-read, from xl = w - 4; make_row then shifts that
// lane's columns down by s = x0 - xl. Columns past the crop are never used.
struct RawRow {
    uint32_t G, Z0, Z1;
};

__device__ __forceinline__ RawRow load_row(const CropDesc &c, int y, int xl) {
    RawRow r;
    r.G = gld<uint32_t>(c.grey, (uint32_t)y * (uint32_t)c.grey_pitch + (uint32_t)xl);
    const u32x2 z =
        gld<u32x2>(c.depth, ((uint32_t)y * (uint32_t)c.depth_pitch + (uint32_t)xl) * 2u);
    r.Z0 = z.x;
    r.Z1 = z.y;
    return r;
}

// load_row at byte offsets goff (grey plane) and doff (depth plane) from the
// crop's origin.
__device__ __forceinline__ RawRow load_row_at(const CropDesc &c, uint32_t goff, uint32_t doff) {
    RawRow r;
    r.G = gld<uint32_t>(c.grey, goff);
    const u32x2 z = gld<u32x2>(c.depth, doff);
    r.Z0 = z.x;
    r.Z1 = z.y;
    return r;
}

// d' = clamp(d - lo, 0, span) on a pair of u16, for lo >= 0 (so d = 0 maps
// to 0).
__device__ __forceinline__ uint32_t to_window(uint32_t z, uint32_t lolo, uint32_t span2) {
    return pk_min(pk_sub_sat(z, lolo), span2);
}

// Row of 6 packed pixels (grey | d' << 16): columns [x0-1, x0 .. x0+3, x0+4].
struct Row6 {
    uint32_t p[6];
};

// s8 = 8 s and s16 = 16 s for the column shift s of load_row.
__device__ __forceinline__ Row6 make_row(const RawRow &raw, uint32_t lolo, uint32_t span2,
                                         uint32_t s8, uint32_t s16) {
    const uint32_t G = raw.G >> s8;
    const uint64_t Z = ((((uint64_t)raw.Z1) << 32) | raw.Z0) >> s16;
    const uint32_t D0 = to_window((uint32_t)Z, lolo, span2);
    const uint32_t D1 = to_window((uint32_t)(Z >> 32), lolo, span2);
    Row6 r;
    r.p[1] = __builtin_amdgcn_perm(G, D0, 0x01000C04u);
    r.p[2] = __builtin_amdgcn_perm(G, D0, 0x03020C05u);
    r.p[3] = __builtin_amdgcn_perm(G, D1, 0x01000C06u);
    r.p[4] = __builtin_amdgcn_perm(G, D1, 0x03020C07u);
    // Left halo = previous lane's last pixel, right halo = next lane's first.
    // bound_ctrl: the lane with no source (0, resp. 63) reads 0, and no old
    // value has to be set up first.
    r.p[0] = __builtin_amdgcn_mov_dpp(r.p[4], 0x138, 0xF, 0xF, true);  // wave_shr:1
    r.p[5] = __builtin_amdgcn_mov_dpp(r.p[1], 0x130, 0xF, 0xF, true);  // wave_shl:1
    return r;
}

// Byte 0 | byte 1 and byte 2 | byte 3 of x, one SDWA instruction each.
__device__ __forceinline__ uint32_t or_b01(uint32_t x) {
    uint32_t r;
    asm("v_or_b32_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:BYTE_1"
        : "=v"(r)
        : "v"(x));
    return r;
}
__device__ __forceinline__ uint32_t or_b23(uint32_t x) {
    uint32_t r;
    asm("v_or_b32_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:BYTE_3"
        : "=v"(r)
        : "v"(x));
    return r;
}

// Comparison bits of the centre B[j] against its 8 neighbours in rows A
// (y-1), B (y), C (y+1). A set bit means the neighbour is BELOW the centre:
// the sign of the packed 16-bit difference neighbour - centre, bit 15 for
// grey and bit 31 for depth. v_perm's selectors 8-11 replicate those sign
// bits into whole bytes, so each perm gathers the four signs of two
// neighbours (bytes: grey of the first, grey of the second, depth of the
// first, depth of the second); the masks then keep bit p for neighbour p.
// Grey index = byte 0 | byte 1, depth index = byte 2 | byte 3 (or_b01,
// or_b23): bit p <-> neighbour p in both.
template <typename Row>
__device__ __forceinline__ uint32_t compare_bits(const Row &A, const Row &B, const Row &C, int j) {
    const uint32_t c = B.p[j];
    // All eight differences first: a packed result read by the very next
    // instruction costs a wait state on gfx950.
    const uint32_t d0 = pk_sub(A.p[j - 1], c), d1 = pk_sub(A.p[j], c), d2 = pk_sub(A.p[j + 1], c);
    const uint32_t d3 = pk_sub(B.p[j + 1], c), d4 = pk_sub(C.p[j + 1], c), d5 = pk_sub(C.p[j], c);
    const uint32_t d6 = pk_sub(C.p[j - 1], c), d7 = pk_sub(B.p[j - 1], c);
    // perm(hi, lo, sel): 8 = sign of lo[15], 9 = lo[31], 10 = hi[15], 11 = hi[31].
    constexpr uint32_t kSel = 0x090B080Au;
    uint32_t acc = __builtin_amdgcn_perm(d0, d1, kSel) & 0x02010201u;
    acc = and_or(__builtin_amdgcn_perm(d2, d3, kSel), 0x08040804u, acc);
    acc = and_or(__builtin_amdgcn_perm(d4, d5, kSel), 0x20102010u, acc);
    acc = and_or(__builtin_amdgcn_perm(d6, d7, kSel), 0x80408040u, acc);
    return acc;
}

// Centre pixels [xa, xb) x [ya, yb) of a crop.
struct Region {
    int xa, xb, ya, yb;
};

constexpr int kPanel = kFastMaxW - 2;  // centre columns of a panel: 256 columns loaded

// How a region's centre rows fall on the lanes of a block: a stream is the L
// lanes across the region's columns (4 each, one halo column on either side),
// S streams share its rows. Every lane of the block steps through n_step rows,
// so the row loop is uniform; rows past a stream's own are coded but not
// counted, and stay inside the region: floor(s R / S) + ceil(R / S) <= R.
struct Lanes {
    int x0, xl;        // first column of this lane, and the column its loads start at
    int yb, n_own;     // first centre row, rows of its own
    int n_step;
    uint32_t s8;       // 8 (x0 - xl): the shift that undoes xl
};
template <int kNT>
__device__ __forceinline__ Lanes lanes_of(const CropDesc &c, const Region &rg) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int L = (rg.xb - rg.xa + 2 + 3) >> 2, spw = 64 / L, sw = lane / L;
    const int S = kNT / 64 * spw, s = wave * spw + (sw < spw ? sw : 0), R = rg.yb - rg.ya;
    Lanes l;
    l.x0 = rg.xa - 1 + 4 * (lane - sw * L);
    const bool full = (c.flags & kCropOverReadOk) || l.x0 + 4 <= c.w;
    l.xl = full ? l.x0 : c.w - 4;
    l.s8 = 8u * (uint32_t)(l.x0 - l.xl);
    l.yb = rg.ya + (s * R) / S;
    l.n_own = sw < spw ? rg.ya + ((s + 1) * R) / S - l.yb : 0;
    l.n_step = (R + S - 1) / S;
    return l;
}

// Word offset of column x's cell in a row band's counters.
__device__ __forceinline__ uint32_t column_offset(const CropDesc &c, const FeatParams &fp, int x) {
    return (uint32_t)(((min(x, c.w - 1) + 1) * fp.grid_x - 1) / c.w * fp.nbins);
}

// Byte offset of a comparison byte's bin: the table's (4 x bin), or, with 256
// bins, of the code itself, the byte's complement.
template <bool kFull, typename L>
__device__ __forceinline__ uint32_t bin_offset(const L *lut4, uint32_t below) {
    return kFull ? 1020u - 4u * below : (uint32_t)lut4[below];
}

// Counters of the grey and of the depth channel. Grey counts grow by 1 at
// counter (cell, bin); depth counts by dinc at doff bytes further. A counter
// may have 2^copies words, one for every 2^copies-th lane (base is the lane's),
// so that fewer lanes of an instruction meet on a word; rowoff and the bin
// table hold offsets in bytes of such counters.
struct Counters {
    char *base;
    const uint16_t *rowoff;  // of row y's band
    uint32_t dinc, doff;
    uint32_t copies = 0;
};

// Per-pixel histogram loop over a region of any crop in any configuration,
// for what the lane path does not take: each thread takes pixels in row order
// and increments its bins with LDS atomics.
template <int kNT, typename L>
__device__ void code_pixels(const CropDesc c, const FeatParams &fp, int32_t m, const Region rg,
                            const L *lut4, const Counters &ct) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int y = rg.ya + wave; y < rg.yb; y += kNT / 64) {
        for (int x = rg.xa + lane; x < rg.xb; x += 64) {
            const uint32_t dc = c.depth[(size_t)y * c.depth_pitch + x];
            if (!centre_in_mask(dc, m, fp.window)) continue;
            char *cell = ct.base + ct.rowoff[y] + (column_offset(c, fp, x) << (2 + ct.copies));
            // The table maps comparison bytes (set bits: neighbours below).
            if (fp.use_grey)
                atomicAdd(reinterpret_cast<uint32_t *>(
                              cell + lut4[255u ^ lbp_code(c.grey, c.grey_pitch, y, x)]), 1u);
            if (fp.use_depth)
                atomicAdd(reinterpret_cast<uint32_t *>(
                              cell + ct.doff + lut4[255u ^ lbp_code(c.depth, c.depth_pitch, y, x)]),
                          ct.dinc);
        }
    }
}

// Codes and counts a region with both channels in one pass, for a window of
// 1 .. 255 and a median m >= window: each pixel packed as grey | d' << 16, so
// that one packed subtraction compares both channels (see the file's head).
template <bool kFull, int kPF, int kNT, typename L>
__device__ __forceinline__ void code_both(const CropDesc &c, const FeatParams &fp, int32_t m,
                                          const Region &rg, const L *lut4, const Counters &ct) {
    const Lanes l = lanes_of<kNT>(c, rg);
    const uint32_t lolo = (uint32_t)(m - fp.window) * 0x10001u;
    const uint32_t span2 = (uint32_t)(2 * fp.window) * 0x10001u;
    const uint32_t in_hi = (uint32_t)(2 * fp.window - 1) << 16;
    const uint32_t s8 = l.s8, s16 = 2u * l.s8;
    const RawRow rawA = load_row(c, l.yb - 1, l.xl), rawB = load_row(c, l.yb, l.xl);
    RawRow ring[kPF];
#pragma unroll
    for (int u = 0; u < kPF; ++u) ring[u] = load_row(c, min(l.yb + 1 + u, rg.yb), l.xl);
    uint32_t colg[4], cold[4], thr[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        colg[k] = column_offset(c, fp, l.x0 + k) << (2 + ct.copies);
        cold[k] = colg[k] + ct.doff;
        thr[k] = (l.x0 + k >= rg.xa && l.x0 + k < rg.xb) ? in_hi : 0u;
    }
    Row6 A = make_row(rawA, lolo, span2, s8, s16), B = make_row(rawB, lolo, span2, s8, s16);
    auto step = [&](int t, const RawRow &raw) {
        const Row6 C = make_row(raw, lolo, span2, s8, s16);
        const uint32_t bias = t < l.n_own ? 0xFFFF0000u : 0x7FFF0000u;
        const uint32_t row4 = ct.rowoff[l.yb + t];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t bits = compare_bits(A, B, C, k + 1);
            if (B.p[k + 1] + bias < thr[k]) {
                const uint32_t og = bin_offset<kFull>(lut4, or_b01(bits));
                const uint32_t od = bin_offset<kFull>(lut4, or_b23(bits));
                atomicAdd(reinterpret_cast<uint32_t *>(ct.base + add3(row4, colg[k], og)), 1u);
                atomicAdd(reinterpret_cast<uint32_t *>(ct.base + add3(row4, cold[k], od)), ct.dinc);
            }
        }
        A = B;
        B = C;
    };
    int t = 0;
    for (; t + kPF <= l.n_step; t += kPF) {
#pragma unroll
        for (int u = 0; u < kPF; ++u) {
            const RawRow raw = ring[u];
            ring[u] = load_row(c, min(l.yb + t + u + 1 + kPF, rg.yb), l.xl);
            step(t + u, raw);
        }
    }
#pragma unroll
    for (int u = 0; u < kPF - 1; ++u) {
        if (t + u >= l.n_step) break;  // uniform
        step(t + u, ring[u]);
    }
}

// Columns x0-1 .. x0+4 of one row as u16 pairs (x0-1, x0), (x0, x0+1), ..,
// (x0+3, x0+4); out: per centre pair (x0, x0+1), (x0+2, x0+3) a 1 in the half
// of each pixel outside the mask.
struct Row5 {
    uint32_t p[5];
    uint32_t out[2];
};

// Codes and counts a region with one channel (depth when kDepth, else grey), in
// any window (kMask: pixels outside it, or with no depth, are not counted).
// Two pixels to a word: every packed instruction compares two centre pixels.
// Grey compares by the sign of the difference; depth uses all 16 bits, so its
// comparison is a saturating subtraction.
template <bool kDepth, bool kMask, bool kFull, int kPF, int kNT, typename L>
__device__ __forceinline__ void code_one(const CropDesc &c, const FeatParams &fp, int32_t m,
                                         const Region &rg, const L *lut4, const Counters &ct) {
    const Lanes l = lanes_of<kNT>(c, rg);
    // In the mask: d in [first, last], d != 0.
    const int32_t first = max(m - fp.window + 1, 1), last = min(m + fp.window - 1, 65535);
    const uint32_t first2 = (uint32_t)first * 0x10001u;
    const uint32_t span2 = (uint32_t)(last - first) * 0x10001u;
    const uint32_t s8 = l.s8, s16 = 2u * l.s8;
    const uint32_t inc = kDepth ? ct.dinc : 1u;
    uint32_t one2 = 0x10001u;  // opaque, as in median_rows
    asm volatile("" : "+s"(one2));
    auto load = [&](int y) {
        RawRow r{0u, 0u, 0u};
        if (!kDepth)
            r.G = gld<uint32_t>(c.grey, (uint32_t)y * (uint32_t)c.grey_pitch + (uint32_t)l.xl);
        if (kDepth || kMask) {
            const u32x2 z = gld<u32x2>(c.depth, ((uint32_t)y * (uint32_t)c.depth_pitch + (uint32_t)l.xl) * 2u);
            r.Z0 = z.x;
            r.Z1 = z.y;
        }
        return r;
    };
    auto make = [&](const RawRow &raw) {
        const uint64_t Z = ((((uint64_t)raw.Z1) << 32) | raw.Z0) >> s16;
        const uint32_t z0 = (uint32_t)Z, z1 = (uint32_t)(Z >> 32);
        Row5 r;
        if (kDepth) {
            const uint32_t zl = __builtin_amdgcn_mov_dpp(z1, 0x138, 0xF, 0xF, true);  // wave_shr:1
            const uint32_t zr = __builtin_amdgcn_mov_dpp(z0, 0x130, 0xF, 0xF, true);  // wave_shl:1
            r.p[0] = __builtin_amdgcn_alignbit(z0, zl, 16);
            r.p[1] = z0;
            r.p[2] = __builtin_amdgcn_alignbit(z1, z0, 16);
            r.p[3] = z1;
            r.p[4] = __builtin_amdgcn_alignbit(zr, z1, 16);
        } else {
            const uint32_t G = raw.G >> s8;
            const uint32_t gl = __builtin_amdgcn_mov_dpp(G, 0x138, 0xF, 0xF, true);
            const uint32_t gr = __builtin_amdgcn_mov_dpp(G, 0x130, 0xF, 0xF, true);
            // perm(hi, lo, sel): bytes 0-3 are lo's, 4-7 hi's, 0x0C is 0.
            r.p[0] = __builtin_amdgcn_perm(G, gl, 0x0C040C03u);
            r.p[1] = __builtin_amdgcn_perm(G, G, 0x0C010C00u);
            r.p[2] = __builtin_amdgcn_perm(G, G, 0x0C020C01u);
            r.p[3] = __builtin_amdgcn_perm(G, G, 0x0C030C02u);
            r.p[4] = __builtin_amdgcn_perm(gr, G, 0x0C040C03u);
        }
        r.out[0] = r.out[1] = 0u;
        if (kMask) {
            // d - first wraps above the span for d < first (first + span <= 65535).
            r.out[0] = pk_min(pk_sub_sat(pk_sub(z0, first2), span2), one2);
            r.out[1] = pk_min(pk_sub_sat(pk_sub(z1, first2), span2), one2);
        }
        return r;
    };
    RawRow ring[kPF];
    const RawRow rawA = load(l.yb - 1), rawB = load(l.yb);
#pragma unroll
    for (int u = 0; u < kPF; ++u) ring[u] = load(min(l.yb + 1 + u, rg.yb));
    uint32_t col4[4], cut[2] = {0u, 0u};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        col4[k] = 4u * column_offset(c, fp, l.x0 + k) + (kDepth ? ct.doff : 0u);
        if (l.x0 + k < rg.xa || l.x0 + k >= rg.xb) cut[k >> 1] |= 1u << (16 * (k & 1));
    }
    Row5 A = make(rawA), B = make(rawB);
    auto step = [&](int t, const RawRow &raw) {
        const Row5 C = make(raw);
        const uint32_t other = t < l.n_own ? 0u : 0x10001u;
        const uint32_t row4 = ct.rowoff[l.yb + t];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = 2 * j + 1;
            uint32_t b0, b1;  // comparison bytes of the pair's pixels
            if (kDepth) {
                const uint32_t v = B.p[i];
                const uint32_t n[8] = {A.p[i - 1], A.p[i], A.p[i + 1], B.p[i + 1],
                                       C.p[i + 1], C.p[i], C.p[i - 1], B.p[i - 1]};
                uint32_t bits = 0;
#pragma unroll
                for (int q = 0; q < 8; ++q) bits |= pk_min(pk_sub_sat(v, n[q]), one2) << q;
                b0 = bits & 0xFFFFu;
                b1 = bits >> 16;
            } else {
                const uint32_t bits = compare_bits(A, B, C, i);
                b0 = or_b01(bits);
                b1 = or_b23(bits);
            }
            const uint32_t out = B.out[j] | cut[j] | other;
            if (!(out & 0xFFFFu))
                atomicAdd(reinterpret_cast<uint32_t *>(
                              ct.base + add3(row4, col4[2 * j], bin_offset<kFull>(lut4, b0))), inc);
            if (!(out >> 16))
                atomicAdd(reinterpret_cast<uint32_t *>(
                              ct.base + add3(row4, col4[2 * j + 1], bin_offset<kFull>(lut4, b1))), inc);
        }
        A = B;
        B = C;
    };
    int t = 0;
    for (; t + kPF <= l.n_step; t += kPF) {
#pragma unroll
        for (int u = 0; u < kPF; ++u) {
            const RawRow raw = ring[u];
            ring[u] = load(min(l.yb + t + u + 1 + kPF, rg.yb));
            step(t + u, raw);
        }
    }
#pragma unroll
    for (int u = 0; u < kPF - 1; ++u) {
        if (t + u >= l.n_step) break;  // uniform
        step(t + u, ring[u]);
    }
}

// The lane path's loads need w >= 4 unless the crop may be over-read.
__device__ __forceinline__ bool lanes_ok(const CropDesc &c) {
    return c.w >= 4 || (c.flags & kCropOverReadOk);
}

// LDS of the fast path, about 23 KB: six workgroups fit a CU's LDS.
struct FastShared {
    // cells * 59 words: the grey count of (cell, bin) in the low half, the
    // depth count in the high half (a cell holds fewer than 65536 pixels).
    __attribute__((aligned(16))) uint32_t hist[64 * kU59];
    MedianScratch ms;
    uint8_t lut[256];    // comparison byte (bit p: neighbour p below) -> 4 x bin
    uint8_t colband[LBPF_MAX_SIDE];
    uint16_t rowoff[LBPF_MAX_SIDE];  // byte offset of row y's band in hist
    float q[kQuot];
    uint32_t red[2 * kWaves];
    int32_t next;
};

__device__ __forceinline__ void load_tables(FastShared &sh, const uint8_t *tables) {
    for (int i = threadIdx.x; i < 256; i += kThreads)
        sh.lut[i] = (uint8_t)(4 * tables[256 + i]);  // bins <= 58: byte offsets fit
}

// Normalisation and output of one crop by a block of kNT threads, after the
// counting (the caller's barrier): n_in = total of the grey counts, T = 2 n_in,
// grey count / T to out[0 .. half), depth count / T to out[half .. 2 half),
// raw counts to cout when it is not null. maxc bounds every count, so when it
// is below kQuot the quotients are tabulated once in q. red holds kNT / 64
// words.
template <int kNT>
__device__ __forceinline__ void finish_crop(const uint32_t *hist, int half, int maxc, float *q,
                                            uint32_t *red, float *out, uint32_t *cout) {
    constexpr int kNW = kNT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t part = 0;
    for (int i = tid; i < half; i += kNT) part += hist[i] & 0xFFFFu;
    part = wave_sum(part);
    if (lane == 0) red[wave] = part;
    __syncthreads();
    uint32_t n_in = 0;
#pragma unroll
    for (int i = 0; i < kNW; ++i) n_in += red[i];
    const float T = (float)(2u * n_in);
    const bool tab = maxc < kQuot;
    if (tab) {
        for (int v = tid; v <= maxc; v += kNT) q[v] = n_in ? (float)v / T : 0.0f;
        __syncthreads();
    }
    const bool vec = (half & 3) == 0 && ((uintptr_t)out & 15) == 0 && ((uintptr_t)cout & 15) == 0;
    if (vec && tab) {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        for (int i = 4 * tid; i < half; i += 4 * kNT) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(&hist[i]);
            const u32x4 g = v & 0xFFFFu, d = v >> 16;
            st_nt(reinterpret_cast<f32x4 *>(out + i), f32x4{q[g.x], q[g.y], q[g.z], q[g.w]});
            st_nt(reinterpret_cast<f32x4 *>(out + half + i), f32x4{q[d.x], q[d.y], q[d.z], q[d.w]});
            if (cout) {
                *reinterpret_cast<u32x4 *>(cout + i) = g;
                *reinterpret_cast<u32x4 *>(cout + half + i) = d;
            }
        }
    } else {
        for (int i = tid; i < half; i += kNT) {
            const uint32_t v = hist[i], g = v & 0xFFFFu, d = v >> 16;
            out[i] = tab ? q[g] : (n_in ? (float)g / T : 0.0f);
            out[half + i] = tab ? q[d] : (n_in ? (float)d / T : 0.0f);
            if (cout) {
                cout[i] = g;
                cout[half + i] = d;
            }
        }
    }
}

// Features of one crop by the whole workgroup: row `out` (and `cout` when
// not null) of length fp.dim. The tables must already be in LDS; the caller
// separates consecutive crops with a barrier. kPF = rows loaded ahead.
template <int kPF, bool kEarly>
__device__ void fast_crop(const CropDesc &cd, const FeatParams &fp, FastShared &sh, float *out,
                          uint32_t *cout) {
    // A private copy: the descriptor then lives in registers and is not
    // re-read after every LDS atomic that might alias it.
    const CropDesc c = cd;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w = c.w, h = c.h;
    const int gx = fp.grid_x, gy = fp.grid_y, cells = gx * gy;

    const int half = cells * kU59;  // words of sh.hist; half of dim
    // 64 * 59 is a multiple of 4, so the rounded-up clear stays in the array.
    for (int i = 4 * tid; i < half; i += 4 * kThreads)
        *reinterpret_cast<u32x4 *>(&sh.hist[i]) = u32x4{0u, 0u, 0u, 0u};
    // Coordinate y lies in band floor(((y + 1) g - 1) / n) of a side of length n.
    for (int y = tid; y < h; y += kThreads)
        sh.rowoff[y] = (uint16_t)(((y + 1) * gy - 1) / h * gx * kU59 * 4);  // < 64 * 59 * 4
    for (int x = tid; x < w; x += kThreads) sh.colband[x] = (uint8_t)(((x + 1) * gx - 1) / w);

    // Stream geometry of the code phase. Its first rows do not depend on the
    // median: with kEarly their loads are issued now and land while the
    // median is computed (at the price of registers held across it).
    // The lane loads need w >= 4 unless the crop may be over-read.
    const bool fast = w <= kFastMaxW && (w >= 4 || (c.flags & kCropOverReadOk));
    const int L = (w + 3) >> 2;           // lanes per stream (<= 64 when fast)
    const int spw = fast ? 64 / L : 1;    // streams per wave
    const int sw = lane / L;              // stream of this lane within the wave
    const int x0 = 4 * (lane - sw * L);
    const int S = kWaves * spw;
    const int s = wave * spw + (sw < spw ? sw : 0);
    const int rows = h - 2;
    // Stream s owns rows yb .. yb + n_own - 1. Every lane of the block steps
    // through n_step >= n_own rows, so the row loop is uniform; the rows past
    // a lane's own are loaded and coded but not counted. They stay inside the
    // crop: floor(s R / S) + ceil(R / S) <= R, so the last centre row
    // yb + n_step - 1 <= h - 2 and its lower neighbour row <= h - 1.
    const int yb = 1 + (s * rows) / S;
    const int n_own = (fast && sw < spw) ? 1 + ((s + 1) * rows) / S - yb : 0;
    const int n_step = (rows + S - 1) / S;
    const bool full = (c.flags & kCropOverReadOk) || x0 + 4 <= w;
    const int xl = full ? x0 : w - 4;
    const uint32_t s8 = 8u * (uint32_t)(x0 - xl), s16 = 2u * s8;
    RawRow rawA, rawB, ring[kPF];
    auto prime = [&]() {
        rawA = load_row(c, yb - 1, xl);
        rawB = load_row(c, yb, xl);
#pragma unroll
        for (int u = 0; u < kPF; ++u) ring[u] = load_row(c, min(yb + 1 + u, h - 1), xl);
    };
    if (kEarly && fast) prime();

    // Ends with a barrier; the same value in every lane.
    const int32_t m = __builtin_amdgcn_readfirstlane(crop_median_fast<kThreads, false>(c, sh.ms, sh.red));
    const int32_t lo = m - fp.window;
    // The packed window arithmetic needs lo >= 0.
    if (fast && (m < 0 || lo >= 0)) {
        if (m >= 0) {
            if (!kEarly) prime();
            const uint32_t lolo = (uint32_t)lo * 0x10001u;
            const uint32_t span2 = (uint32_t)(2 * fp.window) * 0x10001u;
            const uint32_t in_hi = (uint32_t)(2 * fp.window - 1) << 16;

            // Per column: histogram column offset (bytes) and in-window
            // threshold (0 for border or out-of-crop columns: never counted).
            // A pixel counts when its packed word plus the row's bias is
            // below the threshold: the bias subtracts 1 from d' in rows the
            // lane owns (so 1 <= d' < 2 window passes) and lifts d' above
            // every threshold in the others.
            uint32_t col4[4], thr[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int x = x0 + k;
                col4[k] = (uint32_t)(sh.colband[min(x, w - 1)] * kU59) * 4u;
                thr[k] = (x >= 1 && x <= w - 2) ? in_hi : 0u;
            }
            char *hbase = reinterpret_cast<char *>(sh.hist);

            Row6 A = make_row(rawA, lolo, span2, s8, s16);
            Row6 B = make_row(rawB, lolo, span2, s8, s16);
            // Byte offsets of the next row to refill, kept running so the loop
            // has no multiplies; rows past h - 1 clamp to it (the offsets
            // grow with the row).
            const uint32_t gstep = (uint32_t)c.grey_pitch, dstep = 2u * (uint32_t)c.depth_pitch;
            const uint32_t r0 = (uint32_t)(yb + 1 + kPF), rl = (uint32_t)(h - 1);
            uint32_t gnext = r0 * gstep + (uint32_t)xl, dnext = r0 * dstep + 2u * (uint32_t)xl;
            const uint32_t gmax = rl * gstep + (uint32_t)xl, dmax = rl * dstep + 2u * (uint32_t)xl;
            // One row: code the centre row B against A and C = the row in
            // `slot`, count it, then refill `slot` kPF rows ahead.
            auto step = [&](const int tt, RawRow &slot, const bool refill) {
                const int yy = yb + tt;
                const Row6 C = make_row(slot, lolo, span2, s8, s16);
                if (refill) slot = load_row_at(c, min(gnext, gmax), min(dnext, dmax));
                gnext += gstep;
                dnext += dstep;
                const uint32_t bias = tt < n_own ? 0xFFFF0000u : 0x7FFF0000u;
                const uint32_t row4 = sh.rowoff[yy];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t bits = compare_bits(A, B, C, k + 1);
                    if (B.p[k + 1] + bias < thr[k]) {
                        // The table holds 4 x bin: byte offsets.
                        const uint32_t og = sh.lut[or_b01(bits)];
                        const uint32_t od = sh.lut[or_b23(bits)];
                        atomicAdd(reinterpret_cast<uint32_t *>(hbase + add3(row4, col4[k], og)), 1u);
                        atomicAdd(reinterpret_cast<uint32_t *>(hbase + add3(row4, col4[k], od)),
                                  0x10000u);
                    }
                }
                A = B;
                B = C;
            };
            // Whole groups of kPF rows in a loop with no other exit, so the
            // wait for each ring slot counts exactly the loads issued after
            // it; then the remaining rows, which need no refill.
            int t = 0;
            for (; t + kPF <= n_step; t += kPF) {
#pragma unroll
                for (int u = 0; u < kPF; ++u) step(t + u, ring[u], true);
            }
#pragma unroll
            for (int u = 0; u < kPF - 1; ++u) {
                if (t + u >= n_step) break;  // uniform
                step(t + u, ring[u], false);
            }
        }
    } else if (m >= 0) {
        // Wider crops by panels; a median within the window of 0, or crops
        // too narrow for the lane loads, pixel by pixel.
        const Counters ct{reinterpret_cast<char *>(sh.hist), sh.rowoff, 0x10000u, 0u};
        if (lo >= 0 && w > kFastMaxW)
            for (int xa = 1; xa < w - 1; xa += kPanel)
                code_both<false, 2, kThreads>(c, fp, m, Region{xa, min(xa + kPanel, w - 1), 1, h - 1},
                                              sh.lut, ct);
        else
            code_pixels<kThreads>(c, fp, m, Region{1, w - 1, 1, h - 1}, sh.lut, ct);
    }
    __syncthreads();

    finish_crop<kThreads>(sh.hist, half, ((h + gy - 1) / gy) * ((w + gx - 1) / gx), sh.q, sh.red,
                          out, cout);
}

// One workgroup per crop.
template <int kPF>
__global__ __launch_bounds__(kThreads) void k_features_fast(const CropDesc *__restrict__ crops,
                                                            FeatParams fp,
                                                            const uint8_t *__restrict__ tables,
                                                            float *__restrict__ hist,
                                                            uint32_t *__restrict__ counts) {
    __shared__ FastShared sh;
    load_tables(sh, tables);
    const size_t i = blockIdx.x;
    fast_crop<kPF, true>(crops[i], fp, sh, hist + i * fp.dim, counts ? counts + i * fp.dim : nullptr);
}

// Persistent: a fixed grid of workgroups takes crops from a work queue in the
// order `order` (largest first balances ragged batches) until it runs dry.
// queue[0] is the next position, queue[1] counts finished workgroups; the
// last workgroup to finish resets both, so the kernel can be relaunched (or
// replayed from a graph) with no memset in between.
template <int kPF>
__global__ __launch_bounds__(kThreads, 4) void k_features_persistent(
    const CropDesc *__restrict__ crops, const int32_t *__restrict__ order, int32_t n,
    FeatParams fp, const uint8_t *__restrict__ tables, float *__restrict__ hist,
    uint32_t *__restrict__ counts, uint32_t *__restrict__ queue,
    const int32_t *__restrict__ n_dev) {
    __shared__ FastShared sh;
    if (n_dev) n = *n_dev;  // a batch count kept in device memory (graph replays)
    load_tables(sh, tables);
    if (threadIdx.x == 0) sh.next = (int32_t)atomicAdd(&queue[0], 1u);
    __syncthreads();
    for (;;) {
        // Every thread read the same j; readfirstlane tells the compiler so,
        // and the crop's descriptor is then fetched with scalar loads.
        const int32_t j = __builtin_amdgcn_readfirstlane(sh.next);
        if (j >= n) break;
        // The next position is taken now and published after this crop, so
        // the atomic's latency overlaps the crop (a workgroup takes one
        // position past the end on its way out).
        uint32_t next = 0;
        if (threadIdx.x == 0) next = atomicAdd(&queue[0], 1u);
        const size_t i = order ? (size_t)order[j] : (size_t)j;
        fast_crop<kPF, false>(crops[i], fp, sh, hist + i * fp.dim, counts ? counts + i * fp.dim : nullptr);
        if (threadIdx.x == 0) sh.next = (int32_t)next;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&queue[1], 1u) == gridDim.x - 1) {
            atomicExch(&queue[0], 0u);
            atomicExch(&queue[1], 0u);
        }
    }
}

// --- few or large crops: several workgroups a crop -------------------------------
//
// One workgroup per crop leaves most of the GPU idle when there are fewer crops
// than CUs, and makes a call as long as its largest crop (a 256 x 256 face takes
// 40 us on one workgroup). Here a crop is shared by parts_of(c) workgroups in
// three launches: the median's counts by rows, the codes by row bands and
// column panels, the normalisation (5 faces of 48-256 px 50 -> 22 us a call; 128
// crops of 257-1024 px 4170 -> 150 us, of which the median 38, the codes 97: 560
// px a ns, bound by LDS atomics on flat patches and VALU issue). Nothing but the crop's own row of `hist` is
// written: until the last launch it holds the packed counters (words 0 ..
// half - 1, added to atomically) and, behind them, kMedWords words of median
// counts per part.

constexpr int kSplitMinPx = 2048, kSplitMaxPx = 16384;  // pixels a part
constexpr int kMedWords = 132;    // 256 16-bit bins, non-zero pixels, those >= lo, the window

// The crop table: in device memory, or (a frame's few faces) in the kernel's
// arguments, so that no copy precedes the launch.
struct CropArgs {
    CropDesc c[kArgCrops];
};
__device__ __forceinline__ CropDesc crop_at(const CropDesc *t, int32_t i) { return t[i]; }
__device__ __forceinline__ CropDesc crop_at(const CropArgs &t, int32_t i) { return t.c[i]; }

__device__ __forceinline__ int parts_of(const CropDesc &c, const SplitCfg &sc, const int32_t *n_dev) {
    const int px = n_dev ? min(max(*n_dev * sc.px, kSplitMinPx), kSplitMaxPx) : sc.px;
    return min(sc.parts, ((int)c.w * c.h + px - 1) / px);
}

// Parts of a crop that hold median counts: 8 (each part of the code launch sums
// them with its loads in one flight), or one per 32 K pixels (so that a part's
// counts fit its 16-bit bins), at most what fits behind the counters.
__device__ __forceinline__ int median_parts(const CropDesc &c, int parts, int half) {
    return min(parts, min(max(8, (int)c.w * c.h >> 15), half / kMedWords));
}

struct SplitShared {
    __attribute__((aligned(16))) uint32_t hist[64 * kU59];
    MedianScratch ms;
    uint16_t lut[256];               // comparison byte -> offset of its bin
    uint16_t rowoff[LBPF_MAX_SIDE];  // offset of row y's band
    uint32_t red[2];
};

// Crop of a workgroup: rotated by the part, so that a large crop's parts spread
// over the XCDs (workgroups are dealt to them in turn).
__device__ __forceinline__ int32_t split_crop() {
    return (int32_t)((blockIdx.x + blockIdx.y) % gridDim.x);
}

// Part p of a crop: a column panel and a range of rows. With at least one range
// per grid row, each lies within one grid row, so that the part's few counters
// leave room for copies.
__device__ __forceinline__ bool part_region(const CropDesc &c, int gy, int parts, int p, Region &rg) {
    const int panels = (c.w - 2 + kPanel - 1) / kPanel;
    int bands = max(1, parts / panels);
    const int sub = bands / gy;  // ranges per grid row
    if (sub > 0) bands = sub * gy;
    if (p >= bands * panels) return false;
    const int band = p / panels, panel = p % panels;
    rg.xa = 1 + panel * (c.w - 2) / panels;
    rg.xb = 1 + (panel + 1) * (c.w - 2) / panels;
    if (sub > 0) {
        const int g = band / sub, k = band % sub;
        const int y0 = max(g * c.h / gy, 1), y1 = min((g + 1) * c.h / gy, c.h - 1);
        rg.ya = y0 + k * (y1 - y0) / sub;
        rg.yb = y0 + (k + 1) * (y1 - y0) / sub;
    } else {
        rg.ya = 1 + band * (c.h - 2) / bands;
        rg.yb = 1 + (band + 1) * (c.h - 2) / bands;
    }
    return rg.yb > rg.ya;
}

template <typename Table>
__global__ __launch_bounds__(kThreads) void k_split_median(Table crops, SplitCfg sc, FeatParams fp,
                                                           float *__restrict__ hist,
                                                           const int32_t *__restrict__ n_dev) {
    __shared__ MedianScratch ms;
    __shared__ uint32_t red[2 * kWaves];
    const int32_t p = blockIdx.y, i = split_crop();
    if (n_dev && i >= *n_dev) return;  // uniform
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = fp.grid_x * fp.grid_y * kU59;
    const CropDesc c = crop_at(crops, i);
    const int parts = parts_of(c, sc, n_dev), mparts = median_parts(c, parts, half);
    if (p >= parts) return;  // uniform
    uint32_t *row = reinterpret_cast<uint32_t *>(hist + (size_t)i * fp.dim);
    for (int w = p * half / parts + tid; w < (p + 1) * half / parts; w += kThreads) row[w] = 0u;
    if (p >= mparts) return;
    uint32_t ge2, nz2;
    const MedWindow win =
        median_rows<kThreads, true>(c, p * c.h / mparts, (p + 1) * c.h / mparts, ms, ge2, nz2);
    const uint32_t nnz = wave_sum((nz2 & 0xFFFFu) + (nz2 >> 16));
    const uint32_t nge = wave_sum((ge2 & 0xFFFFu) + (ge2 >> 16));
    if (lane == 0) {
        red[wave] = nnz;
        red[kWaves + wave] = nge;
    }
    __syncthreads();
    uint32_t *part = row + half + p * kMedWords;
    if (tid < (win.wide ? 128 : (int)kMedWin / 2))
        part[tid] = ms.hist[2 * tid] | (ms.hist[2 * tid + 1] << 16);
    if (tid == 0) {
        uint32_t a = 0, b = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            a += red[w];
            b += red[kWaves + w];
        }
        part[128] = a;
        part[129] = b;
        part[130] = (uint32_t)win.lo;
        part[131] = win.k | (win.wide ? 256u : 0u);
    }
}

template <typename Table>
__global__ __launch_bounds__(kThreads) void k_split_code(Table crops, SplitCfg sc, FeatParams fp,
                                                         const uint8_t *__restrict__ tables,
                                                         float *__restrict__ hist,
                                                         const int32_t *__restrict__ n_dev) {
    __shared__ SplitShared sh;
    const int32_t p = blockIdx.y, i = split_crop();
    if (n_dev && i >= *n_dev) return;  // uniform
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gx = fp.grid_x, gy = fp.grid_y, half = gx * gy * kU59;
    const CropDesc c = crop_at(crops, i);
    const int parts = parts_of(c, sc, n_dev), mparts = median_parts(c, parts, half);
    Region rg;
    if (!part_region(c, gy, parts, p, rg)) return;  // uniform
    uint32_t *row = reinterpret_cast<uint32_t *>(hist + (size_t)i * fp.dim);
    // Counters of the grid rows this part touches, in as many copies (at most
    // 8) as fit: large crops have flat patches, whose lanes would otherwise
    // meet on one word.
    const int w0 = ((rg.ya + 1) * gy - 1) / c.h * gx * kU59;
    const int w1 = ((rg.yb * gy - 1) / c.h + 1) * gx * kU59;
    const uint32_t cp = min(31 - __builtin_clz(64 * kU59 / (w1 - w0)), 3);
    // 64 * 59 is a multiple of 4, so the rounded-up clear stays in the array.
    for (int w = 4 * tid; w < (w1 - w0) << cp; w += 4 * kThreads)
        *reinterpret_cast<u32x4 *>(&sh.hist[w]) = u32x4{0u, 0u, 0u, 0u};
    for (int k = tid; k < 256; k += kThreads) sh.lut[k] = (uint16_t)((uint32_t)tables[256 + k] << (2 + cp));
    for (int y = rg.ya + tid; y < rg.yb; y += kThreads)
        sh.rowoff[y] = (uint16_t)((((y + 1) * gy - 1) / c.h * gx * kU59 - w0) << (2 + cp));
    // The median from the parts' counts, as median_finish: thread t sums bin t,
    // eight loads in flight.
    static_assert(kThreads == 256, "a thread per bin");
    const uint32_t *med = row + half;
    const MedWindow win{(int32_t)med[130], med[131] & 255u, (med[131] & 256u) != 0};
    uint32_t bins = 0, tot = 0;
    for (int q0 = 0; q0 < mparts; q0 += 8) {
        uint32_t v[8], u[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t *part = med + min(q0 + k, mparts - 1) * kMedWords;
            v[k] = part[tid >> 1] >> (16 * (tid & 1)) & 0xFFFFu;
            u[k] = part[128 + (tid & 1)];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            bins += q0 + k < mparts ? v[k] : 0u;
            tot += q0 + k < mparts ? u[k] : 0u;
        }
    }
    sh.ms.hist[tid] = win.wide || tid < (int)kMedWin ? bins : 0u;  // (the rest was not written)
    if (tid < 2) sh.red[tid] = tot;
    __syncthreads();
    const uint32_t nnz = sh.red[0], below = nnz - sh.red[1];
    int32_t m = -1;
    if (nnz > 0) {  // uniform
        const uint32_t rank = (nnz - 1) / 2;
        if (wave == 0) {
            if (rank >= below) select_bin(sh.ms, rank - below, lane);
            else if (lane == 0) sh.ms.bin = -1;
        }
        __syncthreads();
        const int32_t bin = sh.ms.bin;
        __syncthreads();
        m = median_of_bin<kThreads>(c, sh.ms, win, bin >= 0 ? bin : -2);
    }
    m = __builtin_amdgcn_readfirstlane(m);
    if (m < 0) return;
    const Counters ct{reinterpret_cast<char *>(sh.hist + (lane & ((1u << cp) - 1u))), sh.rowoff,
                      0x10000u, 0u, cp};
    if (m >= fp.window && lanes_ok(c))
        code_both<false, 2, kThreads>(c, fp, m, rg, sh.lut, ct);
    else
        code_pixels<kThreads>(c, fp, m, rg, sh.lut, ct);
    __syncthreads();
    for (int w = tid; w < w1 - w0; w += kThreads) {
        uint32_t v = sh.hist[w << cp];
        if (cp == 1) v += sh.hist[2 * w + 1];
        if (cp >= 2) {
            u32x4 t = *reinterpret_cast<const u32x4 *>(&sh.hist[w << cp]);
            if (cp == 3) t += *reinterpret_cast<const u32x4 *>(&sh.hist[(w << cp) + 4]);
            v = t.x + t.y + t.z + t.w;
        }
        if (v) atomicAdd(&row[w0 + w], v);
    }
}

template <typename Table>
__global__ __launch_bounds__(kThreads) void k_split_finish(Table crops, FeatParams fp,
                                                           float *__restrict__ hist,
                                                           uint32_t *__restrict__ counts,
                                                           const int32_t *__restrict__ n_dev) {
    __shared__ __attribute__((aligned(16))) uint32_t cnt[64 * kU59];
    __shared__ float q[kQuot];
    __shared__ uint32_t red[kWaves];
    const size_t i = blockIdx.x;
    if (n_dev && (int32_t)i >= *n_dev) return;  // uniform
    const CropDesc c = crop_at(crops, (int32_t)i);
    const int w = c.w, h = c.h;
    const int gx = fp.grid_x, gy = fp.grid_y, half = gx * gy * kU59;
    float *out = hist + i * fp.dim;
    for (int k = threadIdx.x; k < half; k += kThreads)
        cnt[k] = reinterpret_cast<const uint32_t *>(out)[k];
    __syncthreads();
    finish_crop<kThreads>(cnt, half, ((h + gy - 1) / gy) * ((w + gx - 1) / gx), q, red, out,
                          counts ? counts + i * fp.dim : nullptr);
}

// --- every other configuration --------------------------------------------------
//
// 256 bins, one channel, mask off, wide windows, coarse grids: one workgroup of
// 8 waves per crop on the same lane path, counters in dynamic LDS. Both channels
// share a counter word when a cell's counts fit 16 bits (packed); with a window
// outside 1 .. 255 mm they are coded in two passes, since the packed pixels of
// code_both hold the depth clamped to the window. Bound by VALU issue (67% of it)
// and the LDS; 1024 crops of 200 x 200, 256 bins of grey: 74 us, 2.6 TB/s of
// input and output, against 331 one pixel a thread with 18 loads a pixel.
enum class Channels { kGrey, kDepth, kBothNarrow, kBothWide };
constexpr int kAnyThreads = 512;

template <Channels kCh, bool kMask, bool kFull>
__global__ __launch_bounds__(kAnyThreads) void k_features_any(const CropDesc *__restrict__ crops,
                                                              FeatParams fp, bool packed,
                                                              const uint8_t *__restrict__ tables,
                                                              float *__restrict__ hist,
                                                              uint32_t *__restrict__ counts) {
    extern __shared__ __attribute__((aligned(16))) uint32_t cnt[];
    __shared__ MedianScratch ms;
    __shared__ uint16_t lut[256];                 // comparison byte -> 4 x bin
    __shared__ uint16_t rowoff[LBPF_MAX_SIDE];    // < 64 * 256 * 4
    __shared__ float q[kQuot];
    __shared__ uint32_t red[2 * (kAnyThreads / 64)];
    constexpr int kNT = kAnyThreads, kNW = kNT / 64;
    constexpr bool kBoth = kCh == Channels::kBothNarrow || kCh == Channels::kBothWide;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const CropDesc c = crops[blockIdx.x];
    const int gx = fp.grid_x, gy = fp.grid_y, per = gx * gy * fp.nbins;
    const int words = kBoth && !packed ? 2 * per : per;
    for (int i = tid; i < words; i += kNT) cnt[i] = 0u;
    for (int i = tid; i < 256; i += kNT) lut[i] = (uint16_t)(4 * tables[256 + i]);
    for (int y = tid; y < c.h; y += kNT)
        rowoff[y] = (uint16_t)(((y + 1) * gy - 1) / c.h * gx * fp.nbins * 4);
    int32_t m = 0;
    if (kMask) m = __builtin_amdgcn_readfirstlane(crop_median_fast<kNT, true>(c, ms, red));
    __syncthreads();
    if (m >= 0) {
        const Counters ct{reinterpret_cast<char *>(cnt), rowoff, kBoth && packed ? 0x10000u : 1u,
                          kBoth && !packed ? 4u * per : 0u};
        if (!lanes_ok(c) || (kCh == Channels::kBothNarrow && m < fp.window)) {
            code_pixels<kNT>(c, fp, m, Region{1, c.w - 1, 1, c.h - 1}, lut, ct);
        } else {
            for (int xa = 1; xa < c.w - 1; xa += kPanel) {
                const Region rg{xa, min(xa + kPanel, c.w - 1), 1, c.h - 1};
                if constexpr (kCh == Channels::kBothNarrow) {
                    code_both<kFull, 2, kNT>(c, fp, m, rg, lut, ct);
                } else {
                    if constexpr (kCh != Channels::kDepth)
                        code_one<false, kMask, kFull, 4, kNT>(c, fp, m, rg, lut, ct);
                    if constexpr (kCh != Channels::kGrey)
                        code_one<true, kMask, kFull, 4, kNT>(c, fp, m, rg, lut, ct);
                }
            }
        }
    }
    __syncthreads();

    const uint32_t low = kBoth && packed ? 0xFFFFu : ~0u;
    uint32_t part = 0;
    for (int i = tid; i < per; i += kNT) part += cnt[i] & low;
    part = wave_sum(part);
    if (lane == 0) red[wave] = part;
    __syncthreads();
    uint32_t n_in = 0;
#pragma unroll
    for (int w = 0; w < kNW; ++w) n_in += red[w];
    const float T = (float)(fp.nch * n_in);
    const int maxc = ((c.h + gy - 1) / gy) * ((c.w + gx - 1) / gx);
    const bool tab = maxc < kQuot;
    if (tab) {
        for (int v = tid; v <= maxc; v += kNT) q[v] = n_in ? (float)v / T : 0.0f;
        __syncthreads();
    }
    float *out = hist + (size_t)blockIdx.x * fp.dim;
    uint32_t *cout = counts ? counts + (size_t)blockIdx.x * fp.dim : nullptr;
    for (int i = tid; i < fp.dim; i += kNT) {
        uint32_t v;
        if (kBoth && packed) v = i < per ? cnt[i] & 0xFFFFu : cnt[i - per] >> 16;
        else v = cnt[i];
        st_nt(out + i, tab ? q[v] : (n_in ? (float)v / T : 0.0f));
        if (cout) cout[i] = v;
    }
}

__global__ __launch_bounds__(kThreads) void k_debug_codes(const CropDesc *__restrict__ crop,
                                                          FeatParams fp, uint8_t *gcodes,
                                                          uint8_t *dcodes, uint8_t *mask) {
    __shared__ MedianScratch ms;
    const CropDesc c = *crop;
    const int32_t m = fp.window > 0 ? crop_median(c, ms) : -1;
    for (int i = threadIdx.x; i < c.w * c.h; i += kThreads) {
        const int y = i / c.w, x = i % c.w;
        uint8_t g = 0, d = 0, k = 0;
        if (y >= 1 && y <= c.h - 2 && x >= 1 && x <= c.w - 2) {
            if (c.grey) g = (uint8_t)lbp_code(c.grey, c.grey_pitch, y, x);
            d = (uint8_t)lbp_code(c.depth, c.depth_pitch, y, x);
            k = centre_in_mask(c.depth[(size_t)y * c.depth_pitch + x], m, fp.window) ? 1 : 0;
        }
        gcodes[i] = g;
        dcodes[i] = d;
        mask[i] = k;
    }
}

}  // namespace

// Packed 16-bit counters: a cell of the largest crop holds < 65536 pixels.
static bool packed_cells(const FeatParams &fp) {
    return (int64_t)((LBPF_MAX_SIDE + fp.grid_x - 1) / fp.grid_x) *
               ((LBPF_MAX_SIDE + fp.grid_y - 1) / fp.grid_y) < 65536;
}

bool fast_path_ok(const FeatParams &fp) {
    return fp.nbins == kU59 && fp.use_grey && fp.use_depth && fp.window >= 1 &&
           fp.window <= 255 && fp.grid_x * fp.grid_y <= 64 && packed_cells(fp);
}

// Whether the median parts that fit behind a row's counters (median_parts) hold a
// crop of `largest` px: fewer than 60000 px each, whole rows of at most 1024 more.
static bool median_parts_fit(int32_t largest, const FeatParams &fp) {
    return (int64_t)(fp.grid_x * fp.grid_y * kU59 / kMedWords) * 60000 >= largest;
}

// Whether a call of these crops is split, from the two launches' times in us as
// measured: one workgroup per crop takes 5.5 + 0.72 per 1000 px of the largest
// crop, or 8 + 1 per 620 K px in all (twice that for crops wider than a panel);
// split, 18.5 + 1 per 450 K px. Whole calls, one workgroup / split: 5 crops of
// 48-256 px 50 / 22, 64 x 200 x 200 37 / 25, 256 x 200 x 200 38 / 40, 256 x 128
// x 128 18 / 28, 128 of 257-1024 px 984 / 139, 512 of 257-1024 px 1404 / 455,
// 512 of 100-300 px 100 / 95, 2048 of 100-300 px 208 / 267.
SplitCfg split_for(const CropDesc *crops, int32_t n, const FeatParams &fp) {
    SplitCfg sc;
    if (n <= 0 || !fast_path_ok(fp)) return sc;
    int64_t total = 0, wide = 0;
    int32_t largest = 0, widest = 0;
    for (int32_t i = 0; i < n; ++i) {
        const int32_t px = (int32_t)crops[i].w * crops[i].h;
        total += px;
        if (crops[i].w > kFastMaxW) wide += px;
        largest = std::max(largest, px);
        widest = std::max<int32_t>(widest, crops[i].w);
    }
    const double one = std::max(5.5 + 0.72e-3 * largest, 8.0 + (double)(total + wide) / 620e3);
    if (18.5 + (double)total / 450e3 >= one) return sc;
    if (!median_parts_fit(largest, fp)) return sc;
    sc.px = (int32_t)std::min<int64_t>(std::max<int64_t>(total / 512, kSplitMinPx), kSplitMaxPx);
    sc.parts = std::max((largest + sc.px - 1) / sc.px, (widest - 2 + kPanel - 1) / kPanel);
    return sc;
}

SplitCfg split_for_device_count(int32_t max_n, const FeatParams &fp) {
    SplitCfg sc;
    if (max_n > 512 || !fast_path_ok(fp) || !median_parts_fit(LBPF_MAX_SIDE * LBPF_MAX_SIDE, fp))
        return sc;
    sc.parts = 32;
    sc.px = 52;  // 27 K px a crop on average, 512 parts in all
    return sc;
}

template <bool kFull>
static hipError_t launch_any(const CropDesc *crops, int32_t n, const FeatParams &fp,
                             const uint8_t *d_tables, float *hist, uint32_t *counts,
                             hipStream_t s) {
    const bool both = fp.use_grey && fp.use_depth, mask = fp.window > 0;
    const bool packed = both && packed_cells(fp);
    const size_t lds = sizeof(uint32_t) * (size_t)fp.grid_x * fp.grid_y * fp.nbins *
                       (both && !packed ? 2 : 1);
    auto go = [&](auto kern) {
        // The opt-in above 64 KB of LDS in all (the 256-bin mapping on 8 x 8 cells).
        hipError_t e = hipFuncSetAttribute((const void *)kern,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(n), dim3(kAnyThreads), lds, s, crops, fp, packed, d_tables,
                           hist, counts);
        return hipGetLastError();
    };
    using C = Channels;
    if (!both && fp.use_grey)
        return mask ? go(k_features_any<C::kGrey, true, kFull>)
                    : go(k_features_any<C::kGrey, false, kFull>);
    if (!both)
        return mask ? go(k_features_any<C::kDepth, true, kFull>)
                    : go(k_features_any<C::kDepth, false, kFull>);
    if (mask && fp.window <= 255) return go(k_features_any<C::kBothNarrow, true, kFull>);
    return mask ? go(k_features_any<C::kBothWide, true, kFull>)
                : go(k_features_any<C::kBothWide, false, kFull>);
}

hipError_t launch_features(const CropDesc *crops, int32_t n, const FeatParams &fp,
                           const uint8_t *d_tables, float *hist, uint32_t *counts,
                           hipStream_t s, const SplitCfg &split, const LaunchCfg &lc,
                           const int32_t *order, uint32_t *queue, int32_t num_cus,
                           const int32_t *n_dev, const CropDesc *h_crops) {
    if (n <= 0) return hipSuccess;
    if (!fast_path_ok(fp)) {
        if (n_dev) return hipErrorInvalidValue;  // device counts: the fast configuration only
        return fp.nbins == kU59 ? launch_any<false>(crops, n, fp, d_tables, hist, counts, s)
                                : launch_any<true>(crops, n, fp, d_tables, hist, counts, s);
    }
    const int pf = lc.row_prefetch <= 2 ? 2 : (lc.row_prefetch <= 4 ? 4 : 8);
    if (split.parts > 0 && !lc.persistent) {
        const dim3 grid(n, split.parts);
        auto go = [&](auto table) {
            using T = decltype(table);
            hipLaunchKernelGGL(k_split_median<T>, grid, dim3(kThreads), 0, s, table, split, fp,
                               hist, n_dev);
            hipLaunchKernelGGL(k_split_code<T>, grid, dim3(kThreads), 0, s, table, split, fp,
                               d_tables, hist, n_dev);
            hipLaunchKernelGGL(k_split_finish<T>, dim3(n), dim3(kThreads), 0, s, table, fp, hist,
                               counts, n_dev);
        };
        if (h_crops) {
            CropArgs args;
            std::copy(h_crops, h_crops + n, args.c);
            go(args);
        } else {
            go(crops);
        }
    } else if (lc.persistent && queue) {
        const int grid = std::min<int>(n, std::max(1, lc.wg_per_cu) * num_cus);
        const int32_t *ord = lc.sorted ? order : nullptr;
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), 0, s, crops, ord, n, fp,
                               d_tables, hist, counts, queue, n_dev);
        };
        if (pf == 2) go(k_features_persistent<2>);
        else if (pf == 4) go(k_features_persistent<4>);
        else go(k_features_persistent<8>);
    } else {
        if (n_dev) return hipErrorInvalidValue;  // device counts: not one workgroup per crop
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(n), dim3(kThreads), 0, s, crops, fp, d_tables, hist,
                               counts);
        };
        if (pf == 2) go(k_features_fast<2>);
        else if (pf == 4) go(k_features_fast<4>);
        else go(k_features_fast<8>);
    }
    return hipGetLastError();
}

hipError_t launch_debug_codes(const CropDesc *crop, const FeatParams &fp, uint8_t *gcodes,
                              uint8_t *dcodes, uint8_t *mask, int32_t, int32_t, hipStream_t s) {
    hipLaunchKernelGGL(k_debug_codes, dim3(1), dim3(kThreads), 0, s, crop, fp, gcodes, dcodes,
                       mask);
    return hipGetLastError();
}

}  // namespace lbpf
