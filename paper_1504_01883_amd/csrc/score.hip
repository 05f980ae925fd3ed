// SVM decision values S = X W^T + b on gfx950 matrix cores, and the per-row
// argmax (Sec. 2.5: one hyperplane per enrolled person, the largest decision
// value names the person).
//
// FP32 paths:
//   * k_score_f32_rows (few rows or few identities, D a multiple of 4): operands
//     straight to registers, D shared by the waves of a workgroup;
//   * k_score_f32_bf16x3 (D a multiple of 32, 16-byte aligned rows): each value
//     split exactly into three BF16 parts, six of the nine BF16 products, FP32 sums;
//   * k_score_f32_tiles (the same shapes, for callers that keep one order of
//     summation, and row counts on the device): FP32 MFMA, tiles through LDS;
//   * k_score_f32 (any D): v_mfma_f32_16x16x4f32 (D[m][n] += sum_k A[m][k]
//     B[k][n] over a 16 x 16 x 4 block; lane l supplies A[l % 16][l / 16] and
//     B[l / 16][l % 16] and receives D[4 (l / 16) + t][l % 16], t = 0..3).
//     Operands go straight from global memory (L2) into VGPRs as float4: lane
//     l loads row (l % 16) of a block at columns d0 + 4 (l / 16) .. +3, and
//     MFMA c (c = 0..3) consumes component c, so four MFMAs cover 16
//     consecutive d exactly once for both operands.
#include "lbpf_internal.h"

#include <algorithm>
#include <type_traits>

namespace lbpf {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int kTile = 64;
constexpr int kRowsWaves = 8;      // waves of k_score_f32_rows
constexpr int kRowsMaxSplits = 8;  // its ranges of D at most

// Four consecutive operands d .. d+3 of row `row` (zeros past `nrows` rows or
// past `d_end`); `ld` is the row stride. kVec: 16-byte aligned rows and
// d_end a multiple of 4, so a quad is either fully inside or fully outside.
template <bool kVec>
__device__ __forceinline__ floatx4 load_frag(const float *__restrict__ base, int32_t row,
                                             int32_t nrows, int32_t d_end, int32_t d, int32_t ld) {
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    if (row < nrows) {
        const float *p = base + (size_t)row * ld + d;
        if (kVec) {
            if (d + 3 < d_end) v = *reinterpret_cast<const floatx4 *>(p);
        } else {
            if (d + 0 < d_end) v.x = p[0];
            if (d + 1 < d_end) v.y = p[1];
            if (d + 2 < d_end) v.z = p[2];
            if (d + 3 < d_end) v.w = p[3];
        }
    }
    return v;
}

// A workgroup of 8 wave64 owns a 64 x 64 tile of S. Wave w computes rows
// 32 (w & 1) .. +32 of the tile over one quarter of the feature dimension
// (w >> 1), as 2 x 4 blocks of 16 x 16; the quarters are summed in a fixed
// order through LDS at the end. Two waves per SIMD hide each other's load
// latency. Each iteration covers 32 feature columns (2 sub-steps of
// 16) and the operands of the next iteration are loaded before the MFMAs of
// the current one are issued, so a global load has a full iteration of MFMA
// work (64 instructions) to land.
template <bool kVec>
__global__ __launch_bounds__(512) void k_score_f32(const float *__restrict__ X, int32_t N,
                                                   const float *__restrict__ W,
                                                   const float *__restrict__ bias, int32_t K,
                                                   int32_t D, float *__restrict__ S) {
    __shared__ floatx4 partial[3][2][2][4][64];  // [quarter-1][row half][i][j][lane]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int rh = wave & 1, kq = wave >> 1;
    const int32_t n0 = blockIdx.x * kTile + rh * 32;
    const int32_t k0 = blockIdx.y * kTile;
    const int32_t dq = ((D + 127) / 128) * 32;  // quarter length, a multiple of 32
    const int32_t d_begin = min(kq * dq, D);
    const int32_t d_end = min(d_begin + dq, D);

    floatx4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // Operands of one 32-column iteration: [sub-step][block].
    floatx4 xa[2][2], wb[2][4];
    auto load_iter = [&](int32_t d, floatx4 (&xo)[2][2], floatx4 (&wo)[2][4]) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int32_t du = d + 16 * u + 4 * q;
#pragma unroll
            for (int i = 0; i < 2; ++i) xo[u][i] = load_frag<kVec>(X, n0 + 16 * i + r, N, d_end, du, D);
#pragma unroll
            for (int j = 0; j < 4; ++j) wo[u][j] = load_frag<kVec>(W, k0 + 16 * j + r, K, d_end, du, D);
        }
    };
    load_iter(d_begin, xa, wb);
    for (int32_t d0 = d_begin; d0 < d_end; d0 += 32) {
        floatx4 xn[2][2], wn[2][4];
        load_iter(d0 + 32, xn, wn);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[u][i][c], wb[u][j][c],
                                                                         acc[i][j], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int i = 0; i < 2; ++i) xa[u][i] = xn[u][i];
#pragma unroll
            for (int j = 0; j < 4; ++j) wb[u][j] = wn[u][j];
        }
    }

    // Waves of quarters 1..3 hand their sums to the quarter-0 wave of the same rows.
    if (kq > 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) partial[kq - 1][rh][i][j][lane] = acc[i][j];
    }
    __syncthreads();
    if (kq > 0) return;
    // Lane l holds S[n0 + 16 i + 4 q + t][k0 + 16 j + r] in acc[i][j][t].
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int32_t k = k0 + 16 * j + r;
        if (k >= K) continue;
        const float bk = bias[k];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const floatx4 s = ((acc[i][j] + partial[0][rh][i][j][lane]) +
                               partial[1][rh][i][j][lane]) + partial[2][rh][i][j][lane];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int32_t n = n0 + 16 * i + 4 * q + t;
                if (n < N) S[(size_t)n * K + k] = s[t] + bk;
            }
        }
    }
}

// --- Close decisions -----------------------------------------------------------------
//
// Where a row's best scores lie within what two orders of summation differ by, those
// scores are summed again in one fixed order, written over the others and compared:
// the order of the FP32 MFMA tiles (per range of D, each eight columns as 0 4 1 5 2 6
// 3 7, an FMA each; the ranges' sums in order; the bias), or, where D is not a
// multiple of 32, that of k_score_f32. So the named identity does not follow the
// kernel that made the scores.
//
// Within: each score may be off by 2^-23 sqrt(D) |x| |w|, 4.8 standard deviations of
// D roundings of sums as large as |x| |w| (no partial sum is larger), and by 2^-22 of
// itself for the bias's addition. Of |x| the scoring kernels leave the value or an
// upper bound. Where the weights' norms are not known, 2^-13 of |x w| stands for the
// first: 60 times the usual difference, but too little where x is nearly at right
// angles to all the weights close to the best.
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));

struct Window {
    // An identity's share: reach |of[k] - from v|, of the norms of the weights' rows,
    // reach = 2^-23 sqrt(D) |x|, from = 0; or of the biases, reach = 2^-13, from = 1.
    // reach no number: no score is settled.
    float reach, from;
    const float *__restrict__ of;
    // xn: |x|, or more.
    __device__ Window(const float *norm, const float *bias, float xn, int32_t D)
        : reach(norm ? 0x1p-23f * sqrtf((float)D) * xn : 0x1p-13f), from(norm ? 0.0f : 1.0f),
          of(norm ? norm : bias) {
        if (!(reach < 1e30f)) reach = NAN;
    }
    __device__ __forceinline__ float off(float v, float of_k) const {
        return reach * fabsf(of_k - from * v) + 0x1p-22f * fabsf(v);
    }
    // The most a score may be in another order; itself where that makes no sense.
    __device__ __forceinline__ float upper(float v, float of_k) const {
        return fabsf(v) < 1e37f ? v + off(v, of_k) : v;
    }
};

struct Closest {
    float best = -INFINITY, most = -INFINITY;   // the best score and its upper
    float top = -INFINITY, second = -INFINITY;  // the highest uppers
    int32_t arg;  // larger than any valid index at first
    bool nan = false;
    __device__ explicit Closest(int32_t K) : arg(K) {}
    __device__ __forceinline__ void see(float v, float upper, int32_t k, int32_t K) {
        second = fmaxf(second, fminf(upper, top));
        top = fmaxf(top, upper);
        nan |= v != v;
        if (v > best || arg == K) {
            best = v;
            most = upper;
            arg = k;
        }
    }
    __device__ __forceinline__ void take(float ob, float om, int32_t oa, float ot, float os) {
        second = fmaxf(fmaxf(second, os), fminf(top, ot));
        top = fmaxf(top, ot);
        if (ob > best || (ob == best && oa < arg)) {
            best = ob;
            most = om;
            arg = oa;
        }
    }
    __device__ __forceinline__ void reduce_wave() {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float ob = __shfl_xor(best, off, 64), om = __shfl_xor(most, off, 64),
                        ot = __shfl_xor(top, off, 64), os = __shfl_xor(second, off, 64);
            take(ob, om, __shfl_xor(arg, off, 64), ot, os);
        }
        nan = __ballot(nan) != 0;
    }
    // Scores whose uppers reach this are close; no number where none is to be settled.
    // After reduce_wave, and alike in all lanes (a row without NaN).
    __device__ __forceinline__ float floor(const Window &w) const {
        if (nan || !(fabsf(best) < 1e37f) || !(w.reach >= 0.0f)) return NAN;
        return best - (most - best);
    }
};

constexpr int kSettleRows = 3;       // candidates a turn
constexpr int kSettleAsk = 4;        // as many close ones at most are asked for their partial sums
constexpr int kSettlePieces = 2;     // of 256 columns a step
constexpr int kSettleStride = 532;   // floats of LDS a row, its 1, 2 or 4 ranges 4 apart
constexpr int kSettleLds = (1 + kSettleRows) * kSettleStride + 16;

// The fixed order's ranges: 1, 2 or 4 of equal length, D a multiple of 32 times that;
// or (order < 0) k_score_f32's four quarters, the last ones shorter or empty.
struct Ranges {
    int n;
    int32_t len;
    __device__ Ranges(int order, int32_t D)
        : n(order < 0 ? 4 : order), len(order < 0 ? ((D + 127) / 128) * 32 : D / order) {}
    __device__ __forceinline__ int32_t own(int r, int32_t D) const { return min(len, max(D - r * len, 0)); }
};

// 16 columns onto a sum, in the fixed order.
template <bool kQuarters>
__device__ __forceinline__ float chain16(const floatx4 (&x)[4], const floatx4 (&w)[4], float acc) {
    if constexpr (kQuarters) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int h = 0; h < 4; ++h) acc = __builtin_fmaf(x[h][e], w[h][e], acc);
    } else {
#pragma unroll
        for (int h = 0; h < 4; h += 2)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc = __builtin_fmaf(x[h][e], w[h][e], acc);
                acc = __builtin_fmaf(x[h + 1][e], w[h + 1][e], acc);
            }
    }
    return acc;
}

// One wave: up to kSettleRows scores (lane c: identity cand of candidate c) in the
// fixed order; lane c * ranges + r returns range r's sum of candidate c. A chain of
// FMAs in one lane a sum, its operands staged in LDS by all lanes (lane l copies
// columns 4 (l % per) .. + 3 of a piece of range l / per) and read 16 columns ahead:
// 25 us over 7552 columns in one range, 7 in four.
template <bool kQuarters>
__device__ __forceinline__ float settle_few(const float *__restrict__ x, const float *__restrict__ W,
                                            int32_t D, const Ranges &rg, int32_t cand, int n, float *lds) {
    const int lane = threadIdx.x & 63;
    const int per = 64 / rg.n, cols = 4 * per * kSettlePieces;  // of a range, a step
    const int32_t at = 4 * (lane % per), from = (lane / per) * rg.len, own = rg.own(lane / per, D);
    const int to = (lane / per) * (cols + 4) + at;
    const int mine = lane % rg.n, of = lane / rg.n;
    float acc = 0.0f;
    floatx4 v[1 + kSettleRows][kSettlePieces];
    auto load = [&](int32_t c0) {
#pragma unroll
        for (int c = 0; c <= kSettleRows; ++c) {
            // Fewer than kSettleRows: the first candidate again.
            const float *src =
                c == 0 ? x : W + (size_t)__builtin_amdgcn_readlane(cand, c <= n ? c - 1 : 0) * D;
#pragma unroll
            for (int p = 0; p < kSettlePieces; ++p) {
                const int32_t d = c0 + 4 * per * p + at;
                v[c][p] = *reinterpret_cast<const floatx4 *>(src + min(from + d, D - 4));
                if (d >= own) v[c][p] = floatx4{};  // nothing to add
            }
        }
    };
    load(0);
    for (int32_t c0 = 0; c0 < rg.len; c0 += cols) {
#pragma unroll
        for (int c = 0; c <= kSettleRows; ++c) {
#pragma unroll
            for (int p = 0; p < kSettlePieces; ++p)
                *reinterpret_cast<floatx4 *>(lds + c * kSettleStride + to + 4 * per * p) = v[c][p];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (c0 + cols < rg.len) load(c0 + cols);
        if (of < n) {
            const float *px = lds + mine * (cols + 4), *pw = px + (1 + of) * kSettleStride;
            // An LDS read's time is that of 16 columns' FMAs: read as far ahead
            // (past the row's end at last, into what the buffer has room for).
            floatx4 x0[4], w0[4], x1[4], w1[4];
            auto read = [&](floatx4(&xs)[4], floatx4(&ws)[4], int j) {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    xs[h] = *reinterpret_cast<const floatx4 *>(px + j + 4 * h);
                    ws[h] = *reinterpret_cast<const floatx4 *>(pw + j + 4 * h);
                }
            };
            read(x0, w0, 0);
            for (int j = 0; j < cols; j += 32) {
                read(x1, w1, j + 16);
                __builtin_amdgcn_sched_barrier(0);
                acc = chain16<kQuarters>(x0, w0, acc);
                __builtin_amdgcn_sched_barrier(0);
                read(x0, w0, j + 32);
                __builtin_amdgcn_sched_barrier(0);
                acc = chain16<kQuarters>(x1, w1, acc);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    return acc;
}

// As settle_few for up to 64 / ranges scores at a time (lane c * ranges + r: candidate
// c's identity), 16 columns a step, two steps on their way: 60 us a turn over 7552
// columns in one range, 15 in four, mostly the latency of LDS.
template <bool kQuarters>
__device__ __forceinline__ float settle_many(const float *__restrict__ x, const float *__restrict__ W,
                                             int32_t D, const Ranges &rg, int32_t cand, float *lds) {
    constexpr int kStride = 20;  // floats of LDS a sum's columns: reads in all banks
    static_assert((64 + 4) * kStride <= kSettleLds, "a wave's LDS");
    const int lane = threadIdx.x & 63;
    // Lane l copies columns 4 (l % 4) .. + 3 for the sums of lanes l / 4 + 16 i, and x's
    // for range l / 4. 16 is a multiple of the ranges: all of one range.
    const int q = lane >> 2, r = q % rg.n, at = 4 * (lane & 3);
    const int32_t from = r * rg.len, own = rg.own(r, D);
    const float *src[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) src[i] = W + (size_t)__shfl(cand, q + 16 * i, 64) * D;
    floatx4 w0[4], w1[4], x0, x1;
    auto load = [&](int32_t j, floatx4(&w)[4], floatx4 &xs) {
        const int32_t d = min(from + j + at, D - 4);
        const bool in = j + at < own;  // else nothing to add
        xs = *reinterpret_cast<const floatx4 *>(x + d);
        if (!in) xs = floatx4{};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = *reinterpret_cast<const floatx4 *>(src[i] + d);
            if (!in) w[i] = floatx4{};
        }
    };
    float acc = 0.0f;
    const float *pw = lds + lane * kStride, *px = lds + (64 + lane % rg.n) * kStride;
    auto step = [&](int32_t j, floatx4(&w)[4], floatx4 &xs) {
        float *to = lds + q * kStride + at;
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<floatx4 *>(to + 16 * i * kStride) = w[i];
        if (q < rg.n) *reinterpret_cast<floatx4 *>(to + 64 * kStride) = xs;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        load(j + 32, w, xs);
        floatx4 a[4], b[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            a[h] = *reinterpret_cast<const floatx4 *>(px + 4 * h);
            b[h] = *reinterpret_cast<const floatx4 *>(pw + 4 * h);
        }
        acc = chain16<kQuarters>(a, b, acc);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    load(0, w0, x0);
    load(16, w1, x1);
#pragma unroll 1
    for (int32_t j = 0; j < rg.len; j += 32) {
        step(j, w0, x0);
        step(j + 16, w1, x1);
    }
    return acc;
}

// Sum over a wave's lanes up to this one.
__device__ __forceinline__ float scan_wave(float v) {
    auto add = [&](auto ctrl, auto rows) {
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value,
                                                        decltype(rows)::value, 0xF, false));
    };
    using std::integral_constant;
    const integral_constant<int, 0xF> all;
    add(integral_constant<int, 0x111>(), all);                             // row_shr:1
    add(integral_constant<int, 0x112>(), all);                             // row_shr:2
    add(integral_constant<int, 0x114>(), all);                             // row_shr:4
    add(integral_constant<int, 0x118>(), all);                             // row_shr:8
    add(integral_constant<int, 0x142>(), integral_constant<int, 0xA>());  // row_bcast:15
    add(integral_constant<int, 0x143>(), integral_constant<int, 0xC>());  // row_bcast:31
    return v;
}

// One wave: what two orders of summation of x u and of x w differ by, from the partial
// sums themselves (every fourth): twice Window's share of the root of their squares'
// sum. Where the terms have either sign that is 50 times less than Window's bound by
// the norms, so that few of the rows the norms alone would have settled are (0.5% to
// 0.9% of rows against 256 to 8192 random weights; by the bound sqrt(D) max|x|, which
// is 16 times the norm of a histogram, 8% to 14% come here). About 6 us, where
// settle_few takes 15 to 25.
template <bool kQuarters>
__device__ __forceinline__ floatx2 spread(const float *__restrict__ x, const float *__restrict__ u,
                                          const float *__restrict__ w, int32_t D, const Ranges &rg) {
    constexpr int kFly = 4;  // 256 columns each, on their way at a time
    const int lane = threadIdx.x & 63;
    floatx2 sum{0.0f, 0.0f};
    for (int r = 0; r < rg.n; ++r) {
        const int32_t from = r * rg.len, own = rg.own(r, D);
        floatx2 before{0.0f, 0.0f};
        floatx4 a[2][kFly], b[2][kFly], c[2][kFly];
        auto load = [&](int g, int32_t d0) {
#pragma unroll
            for (int f = 0; f < kFly; ++f) {
                const int32_t at = min(from + d0 + 256 * f + 4 * lane, D - 4);
                a[g][f] = *reinterpret_cast<const floatx4 *>(x + at);
                b[g][f] = *reinterpret_cast<const floatx4 *>(u + at);
                c[g][f] = *reinterpret_cast<const floatx4 *>(w + at);
            }
        };
        auto add = [&](int g, int32_t d0) {
#pragma unroll
            for (int f = 0; f < kFly; ++f) {
                const bool in = d0 + 256 * f + 4 * lane < own;
                const floatx4 s = a[g][f] * b[g][f], t = a[g][f] * c[g][f];
                const floatx2 v{scan_wave(in ? s.x + s.y + (s.z + s.w) : 0.0f),
                                scan_wave(in ? t.x + t.y + (t.z + t.w) : 0.0f)};
                const floatx2 p = before + v;
                if (in) sum += p * p;
                before += floatx2{__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v.x), 63)),
                                  __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v.y), 63))};
            }
        };
        load(0, 0);
        for (int32_t d0 = 0; d0 < own; d0 += 512 * kFly) {
            load(1, d0 + 256 * kFly);
            add(0, d0);
            load(0, d0 + 512 * kFly);
            add(1, d0 + 256 * kFly);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        sum += floatx2{__shfl_xor(sum.x, off, 64), __shfl_xor(sum.y, off, 64)};
    return floatx2{0x1p-22f * sqrtf(4.0f * sum.x), 0x1p-22f * sqrtf(4.0f * sum.y)};
}

// One wave: |x|.
__device__ __forceinline__ float norm_of(const float *__restrict__ x, int32_t D) {
    constexpr int kFly = 8;
    const int lane = threadIdx.x & 63;
    float sum = 0.0f;
    for (int32_t d0 = 0; d0 < D; d0 += 256 * kFly) {
        floatx4 a[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u)
            a[u] = *reinterpret_cast<const floatx4 *>(x + min(d0 + 256 * u + 4 * lane, D - 4));
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const floatx4 t = a[u] * a[u];
            sum += d0 + 256 * u + 4 * lane < D ? t.x + t.y + (t.z + t.w) : 0.0f;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
    return sqrtf(sum);
}

// One wave: row S_n's close scores again, and the identity. order: see Ranges.
//
// Whole calls in us, D = 7552 (FP32 MFMA tiles throughout / this), weights normal and
// rows uniform: no row close 5 x 1024 131 / 18, 4096 x 256 135 / 106, 16384 x 1024 1847
// / 1295; as they come (26 of 4096 rows and 212 of 16384 within the first window, 0 and
// 6 within the second) 132 / 17, 135 / 112, 1847 / 1314; in every row two copies within
// rounding 135 / 46, 137 / 174, 1845 / 1770; in every row 64 copies 138 / 170, 140 / 651,
// 1846 / 3150 (three at a time by settle_few: 473, 1211 and 12305).
template <bool kQuarters>
__device__ __forceinline__ int32_t settle(const float *__restrict__ x, const float *__restrict__ W,
                                          const float *__restrict__ b, float *S_n, int32_t K,
                                          int32_t D, int order, const Closest &row, float row_floor,
                                          const Window &row_win, float *lds) {
    const int lane = threadIdx.x & 63;
    const Ranges rg(order, D);
    // Alike in all lanes.
    auto uniform = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
    float floor = uniform(row_floor);
    const float row_best = uniform(row.best);
    const int32_t row_arg = __builtin_amdgcn_readfirstlane(row.arg);
    Window win = row_win;
    win.reach = uniform(row_win.reach);
    __threadfence_block();  // the row's scores, written by other lanes
    auto score = [&](int32_t k) { return k < K ? S_n[min(k, K - 1)] : -INFINITY; };
    auto close = [&](float v, int32_t k) { return k < K && win.upper(v, win.of[min(k, K - 1)]) >= floor; };
    int32_t many = 0;
    bool alike = true;
    uint64_t blocks = 0;  // of 64 scores, the first 64 blocks: with a close one
    auto count = [&]() {
        many = 0;
        alike = true;
        blocks = 0;
#pragma unroll 4
        for (int32_t k0 = 0; k0 < K; k0 += 64) {
            const float v = score(k0 + lane);
            const bool is = close(v, k0 + lane);
            const uint64_t m = __ballot(is);
            many += __builtin_popcountll(m);
            if (m && k0 < 64 * 64) blocks |= 1ull << (k0 / 64);
            alike = alike && __ballot(is && v != row_best) == 0;
        }
    };
    count();
    if (many > kSettleAsk && win.from == 0.0f) {
        // The norm itself, where the window may be of a bound of it.
        win = Window(win.of, b, uniform(norm_of(x, D)), D);
        floor = row_best - win.off(row_best, win.of[row_arg]);
        count();
    }
    // More than a wave's worth, all alike: rows of W or X that are the same, not chance.
    if (many < 2 || (many > 64 && alike)) return row_arg;
    if (many <= kSettleAsk) {  // once more by their own partial sums
        bool other = false;
        for (int32_t k0 = 0; k0 < K && !other; k0 += 64) {
            if (k0 < 64 * 64 && !((blocks >> (k0 / 64)) & 1)) continue;
            uint64_t m = __ballot(close(score(k0 + lane), k0 + lane) && k0 + lane != row_arg);
            for (; m && !other; m &= m - 1) {
                const int32_t k = k0 + __builtin_ctzll(m);
                const float v = S_n[k];
                const floatx2 off = spread<kQuarters>(x, W + (size_t)row_arg * D, W + (size_t)k * D, D, rg);
                other = v + 0x1p-22f * fabsf(v) + off.y >= row_best - 0x1p-22f * fabsf(row_best) - off.x;
            }
        }
        if (!other) return row_arg;
    }
    // A few at a time by settle_few; more than two turns' worth by settle_many.
    const int turn = many > 2 * kSettleRows ? 64 / rg.n : kSettleRows;

    float best = -INFINITY;
    int32_t arg = K;
    int32_t cand = 0;
    int32_t k0 = 0;
    uint64_t m = 0;  // close ones of the block before k0, not taken yet
    for (;;) {
        int n = 0;
        for (; n < turn; ++n) {
            while (m == 0 && k0 < K) {
                if (k0 >= 64 * 64 || (blocks >> (k0 / 64)) & 1) m = __ballot(close(score(k0 + lane), k0 + lane));
                k0 += 64;
            }
            if (m == 0) break;
            const int32_t k = k0 - 64 + __builtin_ctzll(m);
            if (turn == kSettleRows ? lane == n : lane / rg.n == n) cand = k;
            m &= m - 1;
        }
        if (n == 0) return arg;
        const float acc = turn == kSettleRows ? settle_few<kQuarters>(x, W, D, rg, cand, n, lds)
                                              : settle_many<kQuarters>(x, W, D, rg, cand, lds);
        for (int c = 0; c < n; ++c) {
            float t = __shfl(acc, c * rg.n, 64);
            for (int r = 1; r < rg.n; ++r) t += __shfl(acc, c * rg.n + r, 64);
            const int32_t k = __builtin_amdgcn_readlane(cand, turn == kSettleRows ? c : c * rg.n);
            t += b[k];
            if (lane == 0) S_n[k] = t;
            if (t > best || arg == K) {
                best = t;
                arg = k;
            }
        }
    }
}

template <bool kSettle>
__global__ __launch_bounds__(256) void k_argmax(float *S, int32_t N, int32_t K, int32_t *out,
                                                const int32_t *__restrict__ n_dev,
                                                const float *__restrict__ X,
                                                const float *__restrict__ W,
                                                const float *__restrict__ b,
                                                const float *__restrict__ norm, int32_t D, int order) {
    const int lane = threadIdx.x & 63;
    if (n_dev) N = *n_dev;
    const int32_t n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;
    float *row = S + (size_t)n * K;
    Closest c(K);
    const bool vec = (K & 3) == 0 && ((uintptr_t)S & 15) == 0;
    // The first scores are asked for before the bound of the row's norm, which the
    // scoring kernel left where the identity goes, is waited for.
    constexpr int kFirst = kSettle ? 4 : 0;
    const float *ofs = norm ? norm : b;
    floatx4 v[kFirst + 1], of[kFirst + 1];
    if (vec) {
#pragma unroll
        for (int j = 0; j < kFirst; ++j) {
            const int32_t k = min(4 * lane + 256 * j, K - 4);
            v[j] = *reinterpret_cast<const floatx4 *>(row + k);
            of[j] = *reinterpret_cast<const floatx4u *>(ofs + k);
        }
    }
    const float xn = kSettle ? __int_as_float(out[n]) : 0.0f;
    __builtin_amdgcn_sched_barrier(0);
    const Window win(norm, b, xn, D);
    if (vec) {
        // Four consecutive identities a lane per step (16-byte loads), still
        // scanned in increasing order within the lane.
        auto see4 = [&](int32_t k, const floatx4 &vs, const floatx4 &os) {
#pragma unroll
            for (int e = 0; e < 4; ++e) c.see(vs[e], kSettle ? win.upper(vs[e], os[e]) : vs[e], k + e, K);
        };
#pragma unroll
        for (int j = 0; j < kFirst; ++j)
            if (4 * lane + 256 * j < K) see4(4 * lane + 256 * j, v[j], of[j]);
#pragma unroll 4
        for (int32_t k = 4 * lane + 256 * kFirst; k < K; k += 256) {
            floatx4 os{};
            if constexpr (kSettle) os = *reinterpret_cast<const floatx4u *>(win.of + k);
            see4(k, *reinterpret_cast<const floatx4 *>(row + k), os);
        }
    } else {
        for (int32_t k = lane; k < K; k += 64)
            c.see(row[k], kSettle ? win.upper(row[k], win.of[k]) : row[k], k, K);
    }
    c.reduce_wave();
    if constexpr (kSettle) {
        __shared__ float lds[4][kSettleLds];
        const float floor = c.floor(win);
        if (c.second >= floor)  // uniform
            c.arg = settle<false>(X + (size_t)n * D, W, b, row, K, D, order, c, floor, win,
                                  lds[threadIdx.x >> 6]);
    }
    if (lane == 0) out[n] = c.arg;
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void glb_void_t;
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

template <int kVm>
__device__ __forceinline__ void wait_vm() {
    static_assert(kVm >= 0 && kVm < 64, "vmcnt range");
    // gfx9 s_waitcnt: vmcnt[3:0], expcnt[6:4], lgkmcnt[11:8], vmcnt[15:14].
    __builtin_amdgcn_s_waitcnt((kVm & 15) | (7 << 4) | (15 << 8) | ((kVm >> 4) << 14));
}

// Barrier that orders LDS only: this wave's LDS reads have returned
// (lgkmcnt 0) before it arrives. __syncthreads would also drain the copies of
// the stages still in flight.
__device__ __forceinline__ void barrier_lds() {
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// --- FP32 MFMA, 128 x 128 or 128 x 256 tiles ---------------------------------------
//
// For callers that keep one order of summation (the trainer's Gram products,
// whose coordinate steps follow their last bits) and for row counts read on the
// device. A workgroup of 4 waves owns a 128 x 128 tile of S; wave w computes the
// 64 x 64 quarter (rows 64 (w & 1), columns 64 (w >> 1)) as 2 x 2 blocks of 32 x
// 32 (four independent accumulator chains). 128-byte slices of the 128 X rows and
// 128 W rows stream through a ring of kRingN 32 KB stages (global_load_lds; each
// wave copies 32 rows of each; chunk c of row r at position c ^ (r % 8)), and
// a stage's fragments are read one stage ahead. The barrier per stage orders
// LDS only (barrier_lds), so the copies of later stages stay in flight.
// kGram: X = W and no bias, so S is its own mirror image to the last bit; tiles
// below the diagonal are left out and the others written twice (5120 x 5120 x
// 7552: 3460 us for all tiles, 2040 so).

template <int kRingN, int kTK, bool kGram>
__global__ __launch_bounds__(256) void k_score_f32_tiles(
    const float *__restrict__ X, int32_t N, const float *__restrict__ W,
    const float *__restrict__ bias, int32_t K, int32_t D, float *__restrict__ S,
    const int32_t *__restrict__ n_dev) {
    // Tile: 128 feature rows x kTK identities (kTK = 256, 128 or 64); wave w owns
    // rows 64 (w & 1) .. +64 and identities (kTK / 2) (w >> 1) .. + kTK / 2 as
    // 2 x kJB blocks of 32 x 32.
    constexpr int kSlice = 128, kTM = 128;
    constexpr int kJB = kTK / 64;                          // 32-wide blocks per wave
    constexpr int kWRows = kTK / 4;                        // W rows each wave copies
    constexpr int kCopies = 4 + kWRows / 8;                // 1 KB copies per wave and stage
    constexpr int kStage = (kTM + kTK) * kSlice;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kRingN * kStage];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int32_t n0 = blockIdx.x * kTM, k0 = blockIdx.y * kTK;
    if (n_dev) N = *n_dev;  // the grid covers the most rows; tiles past N leave
    if (n0 >= N) return;    // uniform
    if (kGram && k0 + kTK <= n0) return;  // the mirror image of another tile
    const int nst = D / (kSlice / 4);
    auto swz = [](int row, int chunk) { return chunk ^ (row & 7); };

    // Copy role: X rows 32 w .. +31 (4 copies of 8 rows) and W rows
    // kWRows w .. + kWRows; lane i -> row i / 8 of its kilobyte, position i % 8.
    const int rr = lane >> 3, pos = lane & 7;
    const float *src[kCopies];
    int dst[kCopies];
#pragma unroll
    for (int j = 0; j < kCopies; ++j) {
        const bool isx = j < 4;
        const int row = isx ? wave * 32 + j * 8 + rr : wave * kWRows + (j - 4) * 8 + rr;
        const int32_t g = isx ? min(n0 + row, N - 1) : min(k0 + row, K - 1);
        src[j] = (isx ? X : W) + (size_t)g * D + 4 * swz(row, pos);
        dst[j] = isx ? (wave * 32 + j * 8) * kSlice : kTM * kSlice + (wave * kWRows + (j - 4) * 8) * kSlice;
    }
    // Copy j of stage st into ring slot st % kRingN. Stages past the last one
    // re-read the last stage's slice into a slot nobody reads again, so every
    // step issues the same copies: the loop body has no branch and the copies
    // can be spread between its matrix instructions.
    auto copy1 = [&](int st, int j) {
        uint8_t *stage = lds + (st % kRingN) * kStage;
        const int sg = min(st, nst - 1);
        __builtin_amdgcn_global_load_lds((glb_void_t *)(src[j] + sg * (kSlice / 4)),
                                         (lds_void_t *)(stage + dst[j]), 16, 0, 0);
    };

    const int fr = lane & 31, fq = lane >> 5;
    int oa[2][4], ob[kJB][4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int ra = wm * 64 + 32 * i + fr;
            oa[i][p] = ra * kSlice + 16 * swz(ra, 2 * p + fq);
        }
#pragma unroll
        for (int j = 0; j < kJB; ++j) {
            const int rb = wn * (kTK / 2) + 32 * j + fr;
            ob[j][p] = kTM * kSlice + rb * kSlice + 16 * swz(rb, 2 * p + fq);
        }
    }
    struct Frag {
        floatx4 a[2][4], b[kJB][4];
    };
    // Fragments of feature chunk p (4 floats of each lane's row) of stage st.
    auto read_p = [&](int st, Frag &f, int p) {
        const uint8_t *stage = lds + (st % kRingN) * kStage;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            f.a[i][p] = *reinterpret_cast<const floatx4 *>(stage + oa[i][p]);
#pragma unroll
        for (int j = 0; j < kJB; ++j)
            f.b[j][p] = *reinterpret_cast<const floatx4 *>(stage + ob[j][p]);
    };
    floatx16 acc[2][kJB];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < kJB; ++j) acc[i][j] = floatx16{};
    auto mma_p = [&](const Frag &f, int p) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < kJB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[i][p][c], f.b[j][p][c],
                                                                      acc[i][j], 0, 0, 0);
    };
    auto mma = [&](const Frag &f) {
#pragma unroll
        for (int p = 0; p < 4; ++p) mma_p(f, p);
    };
    // Stage st's buffer is free once its fragments are in registers (read
    // during the previous step, before this step's barrier), so the copy of
    // stage st + kRingN goes there: kRingN - 1 stages stay in flight. With a
    // single wave per SIMD the matrix core idles whenever this wave stalls on
    // issuing memory instructions, so each step runs as four groups, one per
    // feature chunk p: a share of the copies, the next stage's chunk-p
    // fragments, and the current stage's chunk-p MFMAs. The scheduling
    // barriers keep the groups apart.
    auto step = [&](int st, const Frag &cur, Frag &nxt) {
        wait_vm<(kRingN - 2) * kCopies>();
        barrier_lds();
#pragma unroll
        for (int p = 0; p < 4; ++p) {
#pragma unroll
            for (int j = 0; j < kCopies; ++j)
                if (j % 4 == p) copy1(st + kRingN, j);
            read_p(st + 1, nxt, p);
            mma_p(cur, p);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int st = 0; st < kRingN; ++st)
#pragma unroll
        for (int j = 0; j < kCopies; ++j) copy1(st, j);
    Frag f0, f1;
    wait_vm<(kRingN - 1) * kCopies>();
    barrier_lds();
#pragma unroll
    for (int p = 0; p < 4; ++p) read_p(0, f0, p);
    int st = 0;
    for (; st + 2 < nst; st += 2) {
        step(st, f0, f1);
        step(st + 1, f1, f0);
    }
    if (st + 1 < nst) {
        step(st, f0, f1);
        mma(f1);
    } else {
        mma(f0);
    }
    // The copies past the last stage must land before the workgroup's LDS
    // is released.
    wait_vm<0>();

    // 32 x 32 block layout: register r of lane l is row 8 (r / 4) + 4 (l / 32)
    // + r % 4, column l % 32.
    auto for_each = [&](auto &&f) {
#pragma unroll
        for (int j = 0; j < kJB; ++j) {
            const int32_t k = k0 + wn * (kTK / 2) + 32 * j + (lane & 31);
            if (k >= K) continue;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int32_t n = n0 + wm * 64 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                    if (n < N) f(i, j, r, n, k);
                }
        }
    };
    for_each([&](int i, int j, int r, int32_t n, int32_t k) {
        const float v = acc[i][j][r] + bias[k];
        S[(size_t)n * K + k] = v;
        if constexpr (kGram) S[(size_t)k * K + n] = v;
    });
}

// --- FP32 on the BF16 matrix cores -------------------------------------------------
//
// An FP32 value is the exact sum of three BF16 values: h = bf16(v), m =
// bf16(v - h), l = v - h - m (8 + 8 + 8 significant bits, each remainder exact
// in FP32). Of the nine partial products of x w six are kept, h h, h m, m h, h l,
// l h, m m; left out are m l and l m, at most 2^-25 of |x w| each and with either
// sign (2^-27.4 in root mean square, both), and l l. Six BF16 MFMA take 6 / 16 of the FP32 MFMA's cycles.
//
// h h and the five smaller terms are summed apart (lead, rest): an MFMA rounds its
// sum to FP32, so in one accumulator six roundings a product would fall on the
// large sum; apart, one does, none while the 16-bit products h h fit 24 bits, and
// the others fall on 2^-8 of it. Every kFlush stages lead is added to a running
// sum and starts again from zero; rest joins at the end. Error against 64 bits
// relative to the condition scale, root mean square, against the FP32 MFMA
// kernel's (all in one accumulator), 2048 x 1024 x 7552, normal weights: dense
// uniform rows 1.8e-9 / 1.8e-8 (4.2e-9), 64 values that are not 0 a row 9.4e-9 /
// 1.9e-8 (1.8e-8), 8 2.3e-8 / 2.4e-8 (3.2e-8), 2 2.9e-8 / 2.8e-8 (3.7e-8, and a
// largest error of 2.6e-7 where the others have 1.2e-7). The third set of
// accumulators takes the registers to 256 a lane; the loads' addresses are kept in
// one register each for it.
//
// A workgroup of 8 waves owns 64 kWN feature rows x 64 kWK identities (256 x 128
// or 128 x 256) over one of `splits` ranges of the 32-column stages of D; each
// wave computes 64 x 64 of them as 2 x 2 blocks of 32 x 32. Per stage each thread
// loads 24 floats (two stages ahead), splits them and writes the three planes into
// one of two 72 KB LDS buffers (16-byte chunk c of a row at c ^ ((row / 2) % 4));
// one plane is read by as many waves as a BF16 product's operand would be, but
// multiplied twice as often. Whole calls, this / one accumulator / FP32 MFMA in
// 128 x 256 tiles: 16384 x 1024 x 7552 1230 / 1281 / 1850 us, 4096 x 256 108 / 112 /
// 135: 1.24 PFLOP/s of BF16. With one accumulator, waves out of step, raised wave
// priority during the MFMAs, or VALU work interleaved by scheduling barriers gained
// nothing (1330-1370 us against 1300).
//
// A tile is computed again by FP32 MFMAs on operands straight from memory where
// the split does not hold: a result is not finite (h rounds to infinity, or m =
// inf - inf), or so small that BF16's last bit, 2^-133, may count: below 2^-96 of
// the tile's largest value and not 0, or 0 where that is above 2^30 (D up to 2^14
// keeps 24 bits then).
constexpr int kX3Waves = 8, kX3MaxSplits = 16;
// A tile's operands are addressed in 32 bits from its first row: 256 rows of 4 D bytes.
constexpr int32_t kX3MaxD = 1 << 21;
static bool x3_takes(int32_t D) { return D % 32 == 0 && D <= kX3MaxD; }

__device__ __forceinline__ bool finite_f32(float v) {
    return fabsf(v) <= 3.402823466e38f;
}

template <int kWN, int kWK>
__global__ __launch_bounds__(64 * kX3Waves) void k_score_f32_bf16x3(
    const float *__restrict__ X, int32_t N, const float *__restrict__ W,
    const float *__restrict__ bias, int32_t K, int32_t D, float *__restrict__ S, int32_t splits,
    float *__restrict__ part, float *__restrict__ xn) {
    static_assert(kWN * kWK == kX3Waves, "64 x 64 per wave");
    constexpr int kT = 64 * kX3Waves, kFlush = 8, kTN = 64 * kWN, kTK = 64 * kWK;
    constexpr int kRows = kTN + kTK;              // X rows, then W rows
    constexpr int kGroups = kRows * 4 / kT;       // 8-column groups a thread splits
    static_assert(kRows * 4 % kT == 0, "whole groups");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[2][3][kRows * 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % kWN, wk = wave / kWN;
    // Tile order: consecutive workgroups are dealt round-robin to the 8 XCDs;
    // each XCD takes a contiguous range of logical tiles, walked in groups of
    // 4 row tiles x all identity tiles, which share their operands in its L2.
    const int32_t sp = blockIdx.y;
    const uint32_t KT = (uint32_t)(K + kTK - 1) / kTK, NT = (uint32_t)(N + kTN - 1) / kTN;
    const uint32_t nwg = gridDim.x, pid = blockIdx.x;
    const uint32_t xcd = pid & 7u, per = nwg >> 3, rem = nwg & 7u;
    const uint32_t L = xcd * per + min(xcd, rem) + (pid >> 3);
    constexpr uint32_t kGroupN = 4;
    const uint32_t g = L / (kGroupN * KT), i_g = L - g * (kGroupN * KT);
    const uint32_t gn = min(kGroupN, NT - g * kGroupN);
    const int32_t n0 = (int32_t)(g * kGroupN + i_g % gn) * kTN;
    const int32_t k0 = (int32_t)(i_g / gn) * kTK;
    const int32_t stages = D >> 5;
    const int32_t st0 = (int32_t)((int64_t)stages * sp / splits);
    const int32_t st1 = (int32_t)((int64_t)stages * (sp + 1) / splits);

    auto swz = [](int row, int chunk) { return chunk ^ ((row >> 1) & 3); };
    // Group i's rows are all X's or all W's. Rows past the matrices' ends re-read the
    // last one (not stored).
    static_assert(kTN * 4 % kT == 0, "a group of X rows or of W rows");
    constexpr int kOfX = kTN * 4 / kT;
    const float *Xt = X + (size_t)n0 * D, *Wt = W + (size_t)k0 * D;
    uint32_t src[kGroups];  // bytes from the tile's first row
    const int dst = (tid >> 2) * 64 + 16 * swz(tid >> 2, tid & 3);  // group 0's, then 8 KB apart
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const int row = (i * kT + tid) >> 2, c = tid & 3;
        const int32_t r = i < kOfX ? min(row, N - 1 - n0) : min(row - kTN, K - 1 - k0);
        src[i] = ((uint32_t)r * (uint32_t)D + 8 * c) * 4;
    }
    floatx4 raw[kGroups][2];
    auto load = [&](int32_t st) {
        typedef __attribute__((address_space(1))) const char gchar;
        const auto *x = (gchar *)(Xt + 32 * st), *w = (gchar *)(Wt + 32 * st);
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            asm volatile("" : "+v"(src[i]));  // one register, not a 64-bit sum kept for the loop
#pragma unroll
            for (int h = 0; h < 2; ++h)
                raw[i][h] = *(__attribute__((address_space(1))) const floatx4 *)((i < kOfX ? x : w) + src[i] + 16 * h);
        }
    };
    const int fr = lane & 31, fq = lane >> 5;
    floatx16 lead[2][2], rest[2][2], sum[2][2];  // [identity block][row block]

    float top[2] = {};  // largest |v| of this thread's rows of X, and of W
    auto store = [&](int b) {
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            uintx4 hv, mv, lv;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const floatx2 v = {raw[i][e >> 1][2 * (e & 1)], raw[i][e >> 1][2 * (e & 1) + 1]};
                asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(top[i < kOfX ? 0 : 1]) : "v"(v[0]), "v"(v[1]));
                // Two a conversion; the pair's halves are floats as they are.
                auto pack = [](floatx2 f) {
                    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
                };
                auto rest = [](floatx2 f, uint32_t h) {
                    return floatx2{f[0] - __uint_as_float(h << 16),
                                   f[1] - __uint_as_float(h & 0xffff0000u)};
                };
                hv[e] = pack(v);
                const floatx2 r = rest(v, hv[e]);
                mv[e] = pack(r);
                lv[e] = pack(rest(r, mv[e]));
            }
            *reinterpret_cast<uintx4 *>(&lds[b][0][dst + 16 * kT * i]) = hv;
            *reinterpret_cast<uintx4 *>(&lds[b][1][dst + 16 * kT * i]) = mv;
            *reinterpret_cast<uintx4 *>(&lds[b][2][dst + 16 * kT * i]) = lv;
        }
    };
    // lead[..]: h h; rest[..]: the terms 2^-8 of it and below.
    auto stage = [&](int b) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            bf16x8 xh[2], wh[2], xo[2], wo[2];
            auto read = [&](int q, int row, bf16x8(&v)[2]) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int r = row + 32 * i + fr;
                    v[i] = *reinterpret_cast<const bf16x8 *>(&lds[b][q][r * 64 + 16 * swz(r, 2 * s + fq)]);
                }
            };
            auto mul = [&](const bf16x8(&w)[2], const bf16x8(&x)[2], floatx16(&to)[2][2]) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        to[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[j], x[i], to[j][i], 0, 0, 0);
            };
            const int rx = wn * 64, rw = kTN + wk * 64;
            read(0, rx, xh);
            read(0, rw, wh);
            read(2, rw, wo);
            mul(wh, xh, lead);
            mul(wo, xh, rest);
            read(2, rx, xo);
            mul(wh, xo, rest);
            read(1, rx, xo);
            mul(wh, xo, rest);
            read(1, rw, wo);
            mul(wo, xh, rest);
            mul(wo, xo, rest);
        }
    };
    auto flush = [&](bool first) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (first) sum[j][i] = rest[j][i] = floatx16{};
                else sum[j][i] += lead[j][i];
                lead[j][i] = floatx16{};
            }
    };
    flush(true);
    load(st0);
    store(0);
    if (st0 + 1 < st1) load(st0 + 1);
    __syncthreads();
    for (int32_t st = st0; st < st1; ++st) {
        const int b = (st - st0) & 1;
        if (st + 1 < st1) store(b ^ 1);
        if (st + 2 < st1) load(st + 2);
        stage(b);
        if ((st - st0) % kFlush == kFlush - 1) flush(false);
        __syncthreads();
    }
    flush(false);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) sum[j][i] += rest[j][i];

    // A bound of each row's norm over this range, for Window, by the tiles of the first
    // identities. (The norms themselves, 16 FMAs a stage here, cost 3% of the call.)
    if (xn && k0 == 0) {
        float v = top[0];  // of 8 in each 32 columns; a row's four lanes are neighbours
        v = fmaxf(v, __shfl_xor(v, 1, 64));
        v = fmaxf(v, __shfl_xor(v, 2, 64));
#pragma unroll
        for (int i = 0; i < kOfX; ++i) {
            const int32_t n = n0 + ((i * kT + tid) >> 2);
            if ((tid & 3) == 0 && n < N) xn[(size_t)sp * N + n] = sqrtf(32.0f * (float)(st1 - st0)) * v;
        }
    }

    // A split value is off by 2^-134 at most, so a result by 2^-134 D max |v|.
    uint32_t *most = reinterpret_cast<uint32_t *>(&lds[0][0][0]);
    if (tid == 0) *most = 0;
    const float mine = fmaxf(top[0], top[1]);
    __syncthreads();
    atomicMax(most, __float_as_uint(mine));
    __syncthreads();
    const float all = __uint_as_float(*most);
    const float small = all * 0x1p-96f, none = all > 0x1p30f ? -1.0f : 0.0f;
    bool again = false;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float v = fabsf(sum[j][i][r]);
                again |= !finite_f32(v) || (v < small && v > none);
            }
    if (__syncthreads_or(again)) {
        const float *px[2], *pw[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            px[i] = X + (size_t)min(n0 + wn * 64 + 32 * i + fr, N - 1) * D + 4 * fq;
            pw[i] = W + (size_t)min(k0 + wk * 64 + 32 * i + fr, K - 1) * D + 4 * fq;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) sum[j][i] = floatx16{};
        // MFMA c covers columns c and 4 + c of eight.
        for (int32_t d = 32 * st0; d < 32 * st1; d += 8) {
            floatx4 x[2], w[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                x[i] = *reinterpret_cast<const floatx4 *>(px[i] + d);
                w[i] = *reinterpret_cast<const floatx4 *>(pw[i] + d);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        sum[j][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[j][c], x[i][c],
                                                                         sum[j][i], 0, 0, 0);
        }
    }
    // Register 4 q + t of lane l: identity 8 q + 4 (l / 32) + t, row l % 32.
    float *out = sp > 0 ? part + (size_t)(sp - 1) * N * K : S;
    const bool vec = (K & 3) == 0 && ((uintptr_t)out & 15) == 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int32_t n = n0 + wn * 64 + 32 * i + fr;
        if (n >= N) continue;
        float *row = out + (size_t)n * K;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int32_t k = k0 + wk * 64 + 32 * j + 8 * q + 4 * fq;
                floatx4 v;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    v[t] = sum[j][i][4 * q + t];
                    if (splits == 1 && k + t < K) v[t] += bias[k + t];
                }
                if (vec && k + 3 < K) {
                    *reinterpret_cast<floatx4 *>(row + k) = v;
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (k + t < K) row[k + t] = v[t];
                }
            }
    }
}

// Split-D epilogue, one wave per row: S = (((S + part_0) + part_1) + ...) + b in
// split order (the first range's sums are in S, the others' in part), and (optionally) the row's argmax, ties to the lowest index as
// in k_argmax.
// kVec: K a multiple of 4 and 16-byte aligned rows, so each lane takes four
// consecutive identities per step as float4.
template <bool kVec>
__global__ __launch_bounds__(256) void k_reduce_argmax(const float *__restrict__ part,
                                                       int32_t splits, int32_t N, int32_t K,
                                                       const float *__restrict__ bias,
                                                       float *S, int32_t *__restrict__ out,
                                                       const float *__restrict__ X,
                                                       const float *__restrict__ W,
                                                       const float *__restrict__ norm,
                                                       const float *__restrict__ xn, int32_t D,
                                                       int order) {
    const int lane = threadIdx.x & 63;
    const int32_t n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;
    const size_t plane = (size_t)N * K, row = (size_t)n * K;
    Closest c(K);
    const float *ofs = norm ? norm : bias;
    float xx = xn && lane < splits ? xn[(size_t)lane * N + n] : 0.0f;  // a lane a range
    static_assert(kX3MaxSplits <= 64, "a lane a range");
    auto sum4 = [&](int32_t k) {
        floatx4 v = *reinterpret_cast<const floatx4 *>(S + row + k);
        for (int q = 0; q < splits - 1; ++q)
            v += *reinterpret_cast<const floatx4 *>(part + (size_t)q * plane + row + k);
        return v + *reinterpret_cast<const floatx4 *>(bias + k);
    };
    auto sum1 = [&](int32_t k) {
        float v = S[row + k];
        for (int q = 0; q < splits - 1; ++q) v += part[(size_t)q * plane + row + k];
        return v + bias[k];
    };
    // The first sums before the norms are waited for.
    const int32_t first = kVec ? min(4 * lane, K - 4) : min(lane, K - 1);
    floatx4 v4{}, of4{};
    float v1 = 0.0f;
    if constexpr (kVec) {
        v4 = sum4(first);
        of4 = *reinterpret_cast<const floatx4u *>(ofs + first);
    } else {
        v1 = sum1(first);
    }
    __builtin_amdgcn_sched_barrier(0);
    xx *= xx;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) xx += __shfl_xor(xx, off, 64);
    const Window win(norm, bias, sqrtf(xx), D);
    if constexpr (kVec) {
        for (int32_t k = 4 * lane; k < K;) {
            *reinterpret_cast<floatx4 *>(S + row + k) = v4;
#pragma unroll
            for (int e = 0; e < 4; ++e)  // ascending: the first is kept
                c.see(v4[e], win.upper(v4[e], of4[e]), k + e, K);
            k += 256;
            if (k >= K) break;
            v4 = sum4(k);
            of4 = *reinterpret_cast<const floatx4u *>(ofs + k);
        }
    } else {
        for (int32_t k = lane; k < K;) {
            S[row + k] = v1;
            c.see(v1, win.upper(v1, ofs[k]), k, K);
            k += 64;
            if (k >= K) break;
            v1 = sum1(k);
        }
    }
    if (!out) return;
    c.reduce_wave();
    __shared__ float lds[4][kSettleLds];
    const float floor = xn ? c.floor(win) : NAN;
    if (c.second >= floor)  // uniform
        c.arg = settle<false>(X + (size_t)n * D, W, bias, S + row, K, D, order, c, floor, win,
                              lds[threadIdx.x >> 6]);
    if (lane == 0) out[n] = c.arg;
}

// --- FP32, few feature rows ---------------------------------------------------------
//
// Bound by reading W once (a frame's faces: 5 x 1024 x 7552 reads 31 MB of W
// for 77 MFLOP). A workgroup of 8 wave64 owns 32 identities x 16 kNB feature
// rows over one of `splits` ranges of the 32-column steps of D; its waves take
// the steps in turn (step s by wave s % 8) and their sums meet in LDS in wave
// order. Operands go straight from global memory to registers: of each 128-byte
// step of a row, lane quarter q = l / 16 holds columns 8 q .. 8 q + 7, and
// MFMA c (c = 0..7) multiplies column 8 q + c of every quarter, so the eight
// MFMAs cover the step once for both operands. W is the first operand: a lane
// then holds four consecutive identities of one feature row. kU steps are
// loaded before the first of them is multiplied. 5 x 8192 x 7552: 51 us a call,
// 4.9 TB/s of W (128 x 128 tiles: 167 us); 5 x 1024 x 7552: 15 us, mostly
// launches (130 us).
template <int kNB, bool kTail>
__global__ __launch_bounds__(512) void k_score_f32_rows(
    const float *__restrict__ X, int32_t N, const float *__restrict__ W,
    const float *__restrict__ bias, int32_t K, int32_t D, float *__restrict__ S, int32_t splits,
    float *__restrict__ part, const int32_t *__restrict__ n_dev, float *__restrict__ xn) {
    constexpr int kWB = 2, kU = kNB == 4 ? 2 : 4;
    __shared__ floatx4 red[kRowsWaves][kWB][kNB][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int32_t k0 = blockIdx.x * 16 * kWB, n0 = blockIdx.y * 16 * kNB, sp = blockIdx.z;
    if (n_dev) N = *n_dev;
    if (n0 >= N) return;  // uniform
    if (xn && k0 >= K) {  // a workgroup behind the identities': the rows' norms, for Window
        const int32_t lo = 32 * (int32_t)((int64_t)((D + 31) >> 5) * sp / splits);
        const int32_t hi = min(32 * (int32_t)((int64_t)((D + 31) >> 5) * (sp + 1) / splits), D);
        for (int j = wave; j < 16 * kNB && n0 + j < N; j += kRowsWaves) {
            const float *x = X + (size_t)(n0 + j) * D;
            float v = 0.0f;
#pragma unroll 4
            for (int32_t d = lo + 4 * lane; d < hi; d += 256) {
                const floatx4 t = *reinterpret_cast<const floatx4 *>(x + d);
                v += t.x * t.x + t.y * t.y + (t.z * t.z + t.w * t.w);
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            if (lane == 0) xn[(size_t)sp * N + n0 + j] = sqrtf(v);
        }
        return;
    }
    const float *wp[kWB], *xp[kNB];
#pragma unroll
    for (int i = 0; i < kWB; ++i) wp[i] = W + (size_t)min(k0 + 16 * i + r, K - 1) * D + 8 * q;
#pragma unroll
    for (int j = 0; j < kNB; ++j) xp[j] = X + (size_t)min(n0 + 16 * j + r, N - 1) * D + 8 * q;
    const int32_t steps = (D + 31) >> 5;
    const int32_t s_end = (int32_t)((int64_t)steps * (sp + 1) / splits);
    floatx4 acc[kWB][kNB];
#pragma unroll
    for (int i = 0; i < kWB; ++i)
#pragma unroll
        for (int j = 0; j < kNB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Columns 32 s + 8 q .. + 7 of a row (p points at its column 8 q); zeros
    // past D, a multiple of 4 (kTail: D % 32 != 0). No branch: a guarded load
    // would be waited for before the next one is issued.
    auto load8 = [&](const float *p, int32_t s, floatx4 (&v)[2]) {
        const int32_t d = 32 * s;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int32_t at = d + 8 * q + 4 * h;
            v[h] = *reinterpret_cast<const floatx4 *>(p + (kTail ? min(at, D - 4) - 8 * q : d + 4 * h));
            if (kTail && at >= D) v[h] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
    };
    for (int32_t s = (int32_t)((int64_t)steps * sp / splits) + wave; s < s_end;
         s += kRowsWaves * kU) {
        floatx4 wv[kU][kWB][2], xv[kU][kNB][2];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            // Past the range: any step before D, loaded but not multiplied.
            const int32_t su = min(s + kRowsWaves * u, s_end - 1);
#pragma unroll
            for (int i = 0; i < kWB; ++i) load8(wp[i], su, wv[u][i]);
#pragma unroll
            for (int j = 0; j < kNB; ++j) load8(xp[j], su, xv[u][j]);
        }
        __builtin_amdgcn_sched_barrier(0);  // every load issued before the first wait
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (s + kRowsWaves * u >= s_end) break;  // uniform
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int i = 0; i < kWB; ++i)
#pragma unroll
                    for (int j = 0; j < kNB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            wv[u][i][c >> 2][c & 3], xv[u][j][c >> 2][c & 3], acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < kWB; ++i)
#pragma unroll
        for (int j = 0; j < kNB; ++j) red[wave][i][j][lane] = acc[i][j];
    __syncthreads();
    // Lane l of block (i, j): S[n0 + 16 j + l % 16][k0 + 16 i + 4 (l / 16) + t].
    for (int e = threadIdx.x; e < kWB * kNB * 64; e += 64 * kRowsWaves) {
        const int l = e & 63, j = (e >> 6) % kNB, i = (e >> 6) / kNB;
        floatx4 v = red[0][i][j][l];
#pragma unroll
        for (int w = 1; w < kRowsWaves; ++w) v += red[w][i][j][l];
        const int32_t n = n0 + 16 * j + (l & 15), k = k0 + 16 * i + 4 * (l >> 4);
        if (n >= N) continue;
        float *out = splits > 1 ? part + ((size_t)sp * N + n) * K : S + (size_t)n * K;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (k + t < K) out[k + t] = splits > 1 ? v[t] : v[t] + bias[k + t];
    }
}

// One workgroup per row, for few rows: as k_reduce_argmax (splits > 1: the
// partials summed in split order, the bias added, S written) or k_argmax
// (splits == 1: S read), with 512 lanes on a row and every partial of an
// identity in flight at once. A wave per row (k_argmax, k_reduce_argmax) walks
// the row in dependent steps of memory latency, which pays only once there are
// rows enough to fill the GPU with waves.
template <bool kQuarters>
__global__ __launch_bounds__(512) void k_row_argmax(const float *__restrict__ part, int32_t splits,
                                                     int32_t N, int32_t K,
                                                     const float *__restrict__ bias, float *S,
                                                     int32_t *out,
                                                     const int32_t *__restrict__ n_dev,
                                                     const float *__restrict__ X,
                                                     const float *__restrict__ W,
                                                     const float *__restrict__ norm,
                                                     const float *xn, int32_t D, int order) {
    __shared__ float sv[8], sm[8], st[8], ss[8];
    __shared__ bool sn[8];
    __shared__ int32_t sa[8];
    __shared__ float lds[kSettleLds];
    const int32_t n = blockIdx.x;
    if (n_dev) N = *n_dev;
    if (n >= N) return;  // uniform
    const size_t plane = (size_t)N * K, row = (size_t)n * K;
    Closest c(K);
    constexpr int kTwo = 2;
    float p[kTwo][kRowsMaxSplits], bk[kTwo], of[kTwo];
    const float *ofs = norm ? norm : bias;
    auto load = [&](int32_t k0) {
#pragma unroll
        for (int u = 0; u < kTwo; ++u) {
            const int32_t k = min(k0 + u * (int32_t)blockDim.x, K - 1);
            of[u] = ofs[k];
            bk[u] = bias[k];
            if (splits == 1) {
                p[u][0] = S[row + k];
            } else {
#pragma unroll
                for (int q = 0; q < kRowsMaxSplits; ++q)
                    p[u][q] = part[(size_t)min(q, splits - 1) * plane + row + k];
            }
        }
    };
    load(threadIdx.x);
    float xx = 0.0f;
    if (xn) {  // one split: where the identity goes
        float t[kRowsMaxSplits];
#pragma unroll
        for (int q = 0; q < kRowsMaxSplits; ++q) t[q] = xn[(size_t)min(q, splits - 1) * N + n];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kRowsMaxSplits; ++q) xx += q < splits ? t[q] * t[q] : 0.0f;
    }
    const Window win(norm, bias, sqrtf(xx), D);
    for (int32_t k0 = threadIdx.x; k0 < K;) {
#pragma unroll
        for (int u = 0; u < kTwo; ++u) {
            const int32_t k = k0 + u * (int32_t)blockDim.x;
            float v = p[u][0];
            if (splits > 1) {
#pragma unroll
                for (int q = 1; q < kRowsMaxSplits; ++q)
                    if (q < splits) v += p[u][q];  // uniform
                v += bk[u];
                if (k < K) S[row + k] = v;
            }
            if (k < K) c.see(v, win.upper(v, of[u]), k, K);
        }
        k0 += kTwo * (int32_t)blockDim.x;
        if (k0 < K) load(k0);
    }
    if (!out) return;
    c.reduce_wave();
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sv[wave] = c.best;
        sm[wave] = c.most;
        st[wave] = c.top;
        ss[wave] = c.second;
        sn[wave] = c.nan;
        sa[wave] = c.arg;
    }
    __syncthreads();
    if (wave != 0) return;
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
        c.take(sv[w], sm[w], sa[w], st[w], ss[w]);
        c.nan |= sn[w];
    }
    const float floor = xn ? c.floor(win) : NAN;
    if (c.second >= floor)  // uniform
        c.arg = settle<kQuarters>(X + (size_t)n * D, W, bias, S + row, K, D, order, c, floor, win, lds);
    if (threadIdx.x == 0) out[n] = c.arg;
}

// Euclidean norms of the rows of W, one workgroup a row, summed in FP64 (weights near
// FP32's ends have a norm as well).
__global__ __launch_bounds__(256) void k_weight_norms(const float *__restrict__ W, int32_t D,
                                                      float *__restrict__ norm) {
    __shared__ double red[4];
    const float *w = W + (size_t)blockIdx.x * D;
    double acc = 0.0;
    for (int32_t d = threadIdx.x; d < D; d += 256) acc += (double)w[d] * (double)w[d];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) norm[blockIdx.x] = (float)sqrt(red[0] + red[1] + red[2] + red[3]);
}

}  // namespace

hipError_t launch_row_norms(const float *W, int32_t K, int32_t D, float *norm, hipStream_t s) {
    hipLaunchKernelGGL(k_weight_norms, dim3(K), dim3(256), 0, s, W, D, norm);
    return hipGetLastError();
}

// Products of few rows (at most 32) or of few 64 x 32 blocks run
// k_score_f32_rows: below the line a call's time is W's one pass, above it the
// blocks' own operand traffic passes that of the tiles. Where k_score_f32_bf16x3
// serves the others (x3), up to 3 blocks per 8 CUs, else one per CU. Whole calls
// in us, rows / x3 / FP32 tiles, D = 7552: 5 x 1024 15 / 63 / 130, 32 x 8192 80 /
// 190 / 169, 128 x 1024 (64 blocks) 47 / 65 / 134, 512 x 256 (64) 47 / 53 / 131,
// 256 x 1024 (128) 72 / 68 / 135, 1024 x 256 (128) 73 / 57 / 132, 512 x 1024 (256)
// 130 / 73 / 139, 64 x 8192 (256) 144 / 160 / 171, 128 x 8192 (512) 251 / 161 / 170.
static bool few_rows(int32_t N, int32_t K, int32_t D, int32_t num_cus, bool x3) {
    return D % 4 == 0 && (N <= 32 || (int64_t)((N + 63) / 64) * ((K + 31) / 32) <=
                                         (x3 ? num_cus * 3 / 8 : num_cus));
}
// 16-row blocks of X per workgroup of k_score_f32_rows.
static int32_t rows_blocks(int32_t N) { return N <= 16 ? 1 : (N <= 32 ? 2 : 4); }

// Split of k_score_f32_bf16x3 with the least time as measured: 2.8 us a stage and
// round of tiles (of the shape that needs fewer rounds, see launch_score_f32),
// and the reduce's traffic at 4 TB/s.
static int32_t x3_splits(int32_t N, int32_t K, int32_t D, int32_t num_cus, size_t part_elems) {
    const auto tiles = [&](int64_t tn, int64_t tk) { return ((N + tn - 1) / tn) * ((K + tk - 1) / tk); };
    const int64_t t = std::min(tiles(256, 128), tiles(128, 256));
    const int32_t stages = D / 32;
    int32_t best = 1;
    double least = 0.0;
    for (int32_t sp = 1; sp <= std::min(kX3MaxSplits, stages); ++sp) {
        // S holds one range's sums; a bound of each row's norm for each range.
        if (sp > 1 && (size_t)(sp - 1) * (size_t)N * (size_t)K + (size_t)sp * (size_t)N > part_elems) break;
        const double us = 2.8 * (double)((t * sp + num_cus - 1) / num_cus) * ((stages + sp - 1) / sp) +
                          (sp > 1 ? 4.0 + 8.0 * sp * (double)N * (double)K / 4e6 : 0.0);
        if (sp == 1 || us < least) {
            least = us;
            best = sp;
        }
    }
    return best;
}

int32_t score_f32_splits(int32_t N, int32_t K, int32_t D, int32_t num_cus, size_t part_elems) {
    if (few_rows(N, K, D, num_cus, x3_takes(D))) {
        // Two workgroups a CU, each wave with at least four 32-column steps.
        const int32_t nb = 16 * rows_blocks(N);
        const int64_t groups = (int64_t)((K + 31) / 32) * ((N + nb - 1) / nb);
        int64_t sp = std::min<int64_t>({(2 * (int64_t)num_cus + groups - 1) / groups, kRowsMaxSplits,
                                        std::max(1, (D + 31) / 32 / (4 * kRowsWaves)),
                                        (int64_t)(part_elems / ((size_t)N * ((size_t)K + 1)))});
        return (int32_t)std::max<int64_t>(sp, 1);
    }
    return x3_takes(D) ? x3_splits(N, K, D, num_cus, part_elems) : 1;
}

int32_t score_f32_order(int32_t N, int32_t K, int32_t D, int32_t num_cus, size_t part_elems) {
    if (D % 32 != 0) return D % 4 == 0 ? -1 : 0;
    const int64_t tiles = (int64_t)((N + 127) / 128) * ((K + 127) / 128);
    int32_t best = 1;
    for (int32_t sp = 2; sp <= 4; sp *= 2) {
        if (tiles * best >= num_cus || D % (32 * sp) != 0 ||
            (size_t)sp * (size_t)N * (size_t)K > part_elems)
            break;
        best = sp;
    }
    return best;
}

// The partials' sum in split order, the bias and the argmax (argmax may be null).
static hipError_t launch_reduce(const float *part, int32_t splits, int32_t N, int32_t K,
                                const float *b, float *S, int32_t *argmax, hipStream_t s,
                                const float *X, const float *W, const float *norm,
                                const float *xn, int32_t D, int order) {
    const bool v4 = K % 4 == 0 && ((uintptr_t)S % 16 == 0) && ((uintptr_t)b % 16 == 0) &&
                    ((uintptr_t)part % 16 == 0);
    if (v4)
        hipLaunchKernelGGL(k_reduce_argmax<true>, dim3((N + 3) / 4), dim3(256), 0, s, part, splits,
                           N, K, b, S, argmax, X, W, norm, xn, D, order);
    else
        hipLaunchKernelGGL(k_reduce_argmax<false>, dim3((N + 3) / 4), dim3(256), 0, s, part, splits,
                           N, K, b, S, argmax, X, W, norm, xn, D, order);
    return hipGetLastError();
}

hipError_t launch_score_f32(const float *X, int32_t N, const float *W, const float *b, int32_t K,
                            int32_t D, float *S, int32_t *argmax, hipStream_t s, int32_t splits,
                            float *part, const int32_t *n_dev, bool one_order, int32_t order,
                            const float *norm) {
    if (N <= 0 || K <= 0) return hipSuccess;
    const bool aligned = ((uintptr_t)X % 16 == 0) && ((uintptr_t)W % 16 == 0);
    int cus = 256;
    {
        int dev = 0;
        if (hipGetDevice(&dev) == hipSuccess)
            (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        cus = std::max(cus, 1);
    }
    const bool x3 = !n_dev && x3_takes(D);
    // Where the rows' norms (or bounds of them) go: behind the partial sums, or (one range) where
    // the identities go after them.
    const auto norms_at = [&](float *behind) {
        return !argmax || !order ? nullptr : splits > 1 ? behind : reinterpret_cast<float *>(argmax);
    };
    if (!one_order && aligned && splits >= 1 && few_rows(N, K, D, cus, x3) && (splits == 1 || part)) {
        const int32_t nb = rows_blocks(N);
        float *xn = norms_at(part + (size_t)splits * N * K);
        const dim3 g((K + 31) / 32 + (xn ? 1 : 0), (N + 16 * nb - 1) / (16 * nb), splits);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, g, dim3(64 * kRowsWaves), 0, s, X, N, W, b, K, D, S, splits,
                               part, n_dev, xn);
        };
        const bool tail = D % 32 != 0;
        if (nb == 1) tail ? go(k_score_f32_rows<1, true>) : go(k_score_f32_rows<1, false>);
        else if (nb == 2) tail ? go(k_score_f32_rows<2, true>) : go(k_score_f32_rows<2, false>);
        else tail ? go(k_score_f32_rows<4, true>) : go(k_score_f32_rows<4, false>);
        auto best = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(N), dim3(K > 256 ? 512 : 256), 0, s, part, splits, N, K, b, S,
                               argmax, n_dev, X, W, norm, xn, D, order);
        };
        if (splits > 1 || argmax) order < 0 ? best(k_row_argmax<true>) : best(k_row_argmax<false>);
        return hipGetLastError();
    }
    if (!one_order && aligned && x3 && splits >= 1 && (splits == 1 || part)) {
        // The shape that goes with this many splits.
        float *xn = norms_at(part + (size_t)(splits - 1) * N * K);
        const auto tiles = [&](int tn, int tk) { return ((N + tn - 1) / tn) * ((K + tk - 1) / tk); };
        const auto rounds = [&](int t) { return ((int64_t)t * splits + cus - 1) / cus; };
        const int tall = tiles(256, 128), wide = tiles(128, 256);
        if (rounds(tall) <= rounds(wide))
            hipLaunchKernelGGL((k_score_f32_bf16x3<4, 2>), dim3(tall, splits), dim3(64 * kX3Waves),
                               0, s, X, N, W, b, K, D, S, splits, part, xn);
        else
            hipLaunchKernelGGL((k_score_f32_bf16x3<2, 4>), dim3(wide, splits), dim3(64 * kX3Waves),
                               0, s, X, N, W, b, K, D, S, splits, part, xn);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (splits > 1)
            return launch_reduce(part, splits, N, K, b, S, argmax, s, X, W, norm, xn, D, order);
        if (!argmax) return hipSuccess;
        if (!xn) return launch_argmax(S, N, K, argmax, s);
        hipLaunchKernelGGL(k_argmax<true>, dim3((N + 3) / 4), dim3(256), 0, s, S, N, K, argmax, n_dev,
                           X, W, b, norm, D, order);
        return hipGetLastError();
    }
    if (aligned && D % 32 == 0 && splits >= 1) {
        // 128 x 256 tiles (48 KB stages, two-stage ring, one workgroup of 434
        // registers a lane per CU), 4/3 the matrix work per copied byte of the
        // 128 x 128 tile, where they fill the CUs in fewer rounds: a round of
        // them takes about 1.91 rounds of 128 x 128 ones (16384 x 1024 x 7552:
        // 1858 us in 2 rounds against 1941-1947 in 4), so when 1.91 r256 < r128
        // (on 5120 x 5120 x 7552, 4 wide rounds against 7: 3.8 ms against 3.45).
        const size_t nt = (size_t)((N + 127) / 128);
        const size_t r128 = (nt * (size_t)((K + 127) / 128) + cus - 1) / cus;
        const size_t r256 = (nt * (size_t)((K + 255) / 256) + cus - 1) / cus;
        const bool wide = K >= 256 && 191 * r256 < 100 * r128;
        const dim3 g((N + 127) / 128, wide ? (K + 255) / 256 : (K + 127) / 128);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, g, dim3(256), 0, s, X, N, W, b, K, D, S, n_dev);
        };
        // 128 x 128 tiles, at least two per CU (512 on the 256-CU MI355X): a
        // two-stage ring (64 KB of LDS; the workgroup's 270 registers a lane
        // still leave one workgroup per CU, and a shallower ring measured faster
        // than four stages: 1940-1946 us against 1960-1964 on 16384 x 1024 x
        // 7552). Fewer tiles: a four-stage ring.
        const bool gram = one_order && X == W && N == K;
        if (wide) gram ? go(k_score_f32_tiles<2, 256, true>) : go(k_score_f32_tiles<2, 256, false>);
        else if ((size_t)g.x * g.y >= 512)
            gram ? go(k_score_f32_tiles<2, 128, true>) : go(k_score_f32_tiles<2, 128, false>);
        else gram ? go(k_score_f32_tiles<4, 128, true>) : go(k_score_f32_tiles<4, 128, false>);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || !argmax) return e;
        return launch_argmax(S, N, K, argmax, s, n_dev);
    }
    if (n_dev) return hipErrorInvalidValue;  // device row counts: the tiled kernel only
    dim3 grid((N + kTile - 1) / kTile, (K + kTile - 1) / kTile);
    const bool vec = (D % 4 == 0) && ((uintptr_t)X % 16 == 0) && ((uintptr_t)W % 16 == 0);
    if (vec)
        hipLaunchKernelGGL(k_score_f32<true>, grid, dim3(512), 0, s, X, N, W, b, K, D, S);
    else
        hipLaunchKernelGGL(k_score_f32<false>, grid, dim3(512), 0, s, X, N, W, b, K, D, S);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !argmax) return e;
    return launch_argmax(S, N, K, argmax, s);
}

hipError_t launch_argmax(const float *S, int32_t N, int32_t K, int32_t *argmax, hipStream_t s,
                         const int32_t *n_dev) {
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_argmax<false>, dim3((N + 3) / 4), dim3(256), 0, s, const_cast<float *>(S), N,
                       K, argmax, n_dev, nullptr, nullptr, nullptr, nullptr, 0, 0);
    return hipGetLastError();
}

}  // namespace lbpf
