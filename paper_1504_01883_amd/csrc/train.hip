// On-device SVM training (Sec. 2.5: one max-margin hyperplane per person, that
// person against all others; the paper trains on the CPU, Sec. 3).
//
// Problem per class k: L2-regularised hinge loss with C, the bias as an extra
// constant feature 1, features scaled by sigma = 1 / (lower median of the
// sample norms). Solver: dual coordinate descent (Hsieh et al., ICML 2008),
// in FP64, visiting the samples of every epoch in a seeded random order:
//   G  = y_i w.x_i - 1
//   PG = G, except min(G, 0) at alpha_i = 0 and max(G, 0) at alpha_i = C
//   alpha_i <- clamp(alpha_i - G / Q_ii, 0, C), Q_ii = x_i.x_i (+1 for the bias)
//   w <- w + (alpha_i' - alpha_i) y_i x_i
// until max |PG| over an epoch is below eps, or max_epochs. W = sigma w, b =
// the bias weight.
//
// Order of the samples: epoch e of class k is a Fisher-Yates shuffle of
// 0..N-1 (i from N-1 down to 1 swaps i with r mod (i+1)) drawing r from the
// splitmix64 stream (Steele, Lea and Flood, OOPSLA 2014: state += golden
// gamma, output = the variant-13 mix of the state) seeded with
// seed XOR (k+1) * 0x5851F42D4C957F2D; epoch e uses draws e(N-1) .. e(N-1)+N-2
// (splitmix64 is counter based: draw m is the mix of state0 + (m+1) gamma).
// One thread shuffles while the others wait at the barrier; it costs a few
// percent of an epoch.
//
// Layout: one workgroup per class. Thread t owns coordinates d = t + 256 j
// (j < kJ) of w, held in registers; the sample row is read as FP32 straight
// from the feature matrix (coalesced, one row ahead), scaled in FP64. alpha
// and the epoch's order live in LDS. One barrier per coordinate step (the
// dot product's cross-wave sum, double-buffered).
#include "gram.h"
#include "lbpf_internal.h"

#include <algorithm>

namespace lbpf {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Squared norms of the rows (one wave per row) and, with sigma given, the
// diagonal Q_ii = sum (sigma x)^2 + 1.
__global__ __launch_bounds__(kThreads) void k_row_norms(const float *__restrict__ X, int32_t N,
                                                        int32_t D, const double *__restrict__ sigma,
                                                        double *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int32_t i = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (i >= N) return;
    const float *x = X + (size_t)i * D;
    const double s = sigma ? *sigma : 1.0;
    double acc = 0.0;
    for (int d = lane; d < D; d += 64) {
        const double v = s * (double)x[d];
        acc += v * v;
    }
    acc = wave_sum_f64(acc);
    if (lane == 0) out[i] = sigma ? acc + 1.0 : sqrt(acc);
}

// sigma = 1 / (lower median of the norms), 1 when that median is 0: the
// element of rank (N-1)/2, ranks broken by index so exactly one qualifies.
__global__ __launch_bounds__(kThreads) void k_sigma(const double *__restrict__ norms, int32_t N,
                                                    double *__restrict__ sigma) {
    const uint32_t want = (uint32_t)(N - 1) / 2;
    for (int32_t i = threadIdx.x; i < N; i += kThreads) {
        const double v = norms[i];
        uint32_t rank = 0;
        for (int32_t j = 0; j < N; ++j) {
            const double u = norms[j];
            rank += (u < v || (u == v && j < i)) ? 1u : 0u;
        }
        if (rank == want) *sigma = v > 0.0 ? 1.0 / v : 1.0;
    }
}

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t state0, uint64_t m) {
    // Output of draw m (0-based) of a stream whose state starts at state0.
    uint64_t z = state0 + (m + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

struct TrainArgs {
    const float *X;
    const int32_t *labels;
    const double *sigma, *qii;
    int32_t N, D, K;
    double C, eps;
    int32_t max_epochs;
    uint64_t seed;
    int32_t warm;
    double *alpha;   // [K][N]: warm start in, final values out (may be null)
    float *W;        // [K][D]
    float *b;        // [K]
    double *W64;     // [K][D] or null
    double *b64;     // [K] or null
    int32_t *epochs; // [K] or null
};

template <int kJ>
__device__ __forceinline__ void load_row(const float *__restrict__ X, int32_t i, int32_t D, int tid,
                                         float (&x)[kJ]) {
    const float *row = X + (size_t)i * D;
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        const int d = tid + kThreads * j;
        x[j] = d < D ? row[d] : 0.0f;
    }
}

// One workgroup per class. Dynamic LDS: alpha (N doubles), order (N ints).
template <int kJ>
__global__ __launch_bounds__(kThreads) void k_train(TrainArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    double *alpha = reinterpret_cast<double *>(smem);
    int32_t *order = reinterpret_cast<int32_t *>(alpha + a.N);
    __shared__ double red[2][kWaves];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t k = blockIdx.x;
    const int32_t N = a.N, D = a.D;
    const double sigma = *a.sigma, C = a.C;
    const bool warm = a.warm && a.alpha;

    // w: coordinates tid + 256 j in registers; the bias weight wb is kept
    // by every thread (its updates are uniform).
    double w[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) w[j] = 0.0;
    double wb = 0.0;
    for (int32_t i = tid; i < N; i += kThreads) alpha[i] = warm ? a.alpha[(size_t)k * N + i] : 0.0;
    __syncthreads();
    if (warm) {
        // w = sum_i alpha_i y_i x_i over the scaled, augmented samples.
        for (int32_t i = 0; i < N; ++i) {
            const double ai = alpha[i];
            if (ai == 0.0) continue;
            const double ay = a.labels[i] == k ? ai : -ai;
            float x[kJ];
            load_row<kJ>(a.X, i, D, tid, x);
#pragma unroll
            for (int j = 0; j < kJ; ++j) w[j] += ay * (sigma * (double)x[j]);
            wb += ay;
        }
    }

    const uint64_t state0 = a.seed ^ (0x5851F42D4C957F2Dull * (uint64_t)(k + 1));
    int32_t epoch = 0;
    while (epoch < a.max_epochs) {
        if (tid == 0) {
            const uint64_t base = (uint64_t)epoch * (uint64_t)(N - 1);
            for (int32_t i = 0; i < N; ++i) order[i] = i;
            for (int32_t i = N - 1; i > 0; --i) {
                const uint64_t r = splitmix64_at(state0, base + (uint64_t)(N - 1 - i));
                const int32_t j = (int32_t)(r % (uint64_t)(i + 1));
                const int32_t t = order[i];
                order[i] = order[j];
                order[j] = t;
            }
        }
        __syncthreads();

        double max_pg = 0.0;
        float xn[kJ];
        load_row<kJ>(a.X, order[0], D, tid, xn);
        for (int32_t s = 0; s < N; ++s) {
            const int32_t i = order[s];
            float xc[kJ];
#pragma unroll
            for (int j = 0; j < kJ; ++j) xc[j] = xn[j];
            if (s + 1 < N) load_row<kJ>(a.X, order[s + 1], D, tid, xn);
            const double a_old = alpha[i];  // read before this step's barrier
            const double y = a.labels[i] == k ? 1.0 : -1.0;
            const double q = a.qii[i];
            double part = 0.0;
#pragma unroll
            for (int j = 0; j < kJ; ++j) part += w[j] * (sigma * (double)xc[j]);
            part = wave_sum_f64(part);
            if (lane == 0) red[s & 1][wave] = part;
            __syncthreads();
            double wx = red[s & 1][0];
#pragma unroll
            for (int v = 1; v < kWaves; ++v) wx += red[s & 1][v];
            wx += wb;
            const double G = y * wx - 1.0;
            double PG = G;
            if (a_old <= 0.0) PG = G < 0.0 ? G : 0.0;
            else if (a_old >= C) PG = G > 0.0 ? G : 0.0;
            max_pg = fmax(max_pg, fabs(PG));
            if (PG != 0.0 && q > 0.0) {
                const double a_new = fmin(fmax(a_old - G / q, 0.0), C);
                if (tid == 0) alpha[i] = a_new;
                const double step = (a_new - a_old) * y;
                if (step != 0.0) {
#pragma unroll
                    for (int j = 0; j < kJ; ++j) w[j] += step * (sigma * (double)xc[j]);
                    wb += step;
                }
            }
        }
        ++epoch;
        __syncthreads();  // order and alpha are rewritten next
        if (max_pg < a.eps) break;  // uniform: every thread holds the same max_pg
    }

#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        const int d = tid + kThreads * j;
        if (d < D) {
            const double v = sigma * w[j];
            a.W[(size_t)k * D + d] = (float)v;
            if (a.W64) a.W64[(size_t)k * D + d] = v;
        }
    }
    if (tid == 0) {
        a.b[k] = (float)wb;
        if (a.b64) a.b64[k] = wb;
        if (a.epochs) a.epochs[k] = epoch;
    }
    if (a.alpha)
        for (int32_t i = tid; i < N; i += kThreads) a.alpha[(size_t)k * N + i] = alpha[i];
}

template <int kJ>
hipError_t launch_train_j(const TrainArgs &a, hipStream_t s) {
    const size_t lds = (size_t)a.N * (sizeof(double) + sizeof(int32_t));
    hipError_t e = hipFuncSetAttribute((const void *)k_train<kJ>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_train<kJ>, dim3(a.K), dim3(kThreads), lds, s, a);
    return hipGetLastError();
}

// --- Gram form (FP32) ----------------------------------------------------------
//
// The same dual coordinate descent, restated on the Gram matrix G = X X^T of
// the unscaled features (one FP32 matrix-core GEMM). With s2 = sigma^2, the
// margin of sample i under the current duals is
//   w.x_i = s2 g_i + c,   g_i = sum_j alpha_j y_j G_ij,   c = sum_j alpha_j y_j
// (c is the bias feature's share), and a step on alpha_i moves g by
// (alpha_i' - alpha_i) y_i times row i of G (N values) and c by the same
// scalar. Most steps change nothing: a sample whose projected gradient is 0
// leaves alpha and g as they are. The solver wave therefore tests the next
// 64 samples of the epoch's order at once (one LDS read of g per lane), takes
// the first whose projected gradient is not 0, updates, and tests again from
// the sample after it: the same steps as visiting the samples one by one.
// Other waves draw the next epochs' orders meanwhile. FP32 throughout.

__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

typedef float gf4 __attribute__((ext_vector_type(4)));
typedef float gf4u __attribute__((ext_vector_type(4), aligned(4)));  // a row of G

// Four 16-byte pieces of LDS kStride bytes apart, waited for in the same block: the
// results land in distinct registers, so the reads go out back to back. The outputs
// are early-clobber: a read that returns while later ones are still being issued
// must not land in the address register.
template <int kStride>
__device__ __forceinline__ void lds_read4(uint32_t addr, gf4 &a, gf4 &b, gf4 &c, gf4 &d) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:%5\n\t"
        "ds_read_b128 %2, %4 offset:%6\n\t"
        "ds_read_b128 %3, %4 offset:%7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d)
        : "v"(addr), "n"(kStride), "n"(2 * kStride), "n"(3 * kStride)
        : "memory");
}

__device__ __forceinline__ float readlane_f(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

// The zero bias row of the Gram products.
__global__ __launch_bounds__(256) void k_gram_zero(float *__restrict__ z, int32_t n) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) z[i] = 0.0f;
}

// Row norms sqrt(G_ii).
__global__ __launch_bounds__(256) void k_gram_diag(const float *__restrict__ G, int32_t N,
                                                   float *__restrict__ norms) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < N) norms[i] = sqrtf(G[(size_t)i * N + i]);
}

// sigma = 1 / (lower median of the norms), 1 when that median is 0: the
// element of rank (N-1)/2, ties ranked by index. 16 elements a workgroup, each
// compared with all by 16 lanes (a lane for each element and N serial loads: 293 us
// at N = 5120, 17 us so).
__global__ __launch_bounds__(256) void k_gram_sigma(const float *__restrict__ norms, int32_t N,
                                                    float *__restrict__ sigma) {
    __shared__ uint32_t rank[16];
    const int e = threadIdx.x & 15, part = threadIdx.x >> 4;
    const int32_t i = min((int32_t)blockIdx.x * 16 + e, N - 1);
    if (threadIdx.x < 16) rank[threadIdx.x] = 0;
    __syncthreads();
    const float v = norms[i];
    uint32_t r = 0;
#pragma unroll 8
    for (int32_t j = part; j < N; j += 16) {
        const float u = norms[j];
        r += (u < v || (u == v && j < i)) ? 1u : 0u;
    }
    atomicAdd(&rank[e], r);
    __syncthreads();
    if (part == 0 && rank[e] == (uint32_t)(N - 1) / 2) *sigma = v > 0.0f ? 1.0f / v : 1.0f;
}

// A[k][i] = alpha[k][i] y_ki, the left operand of a warm start's margins.
__global__ __launch_bounds__(256) void k_gram_alpha_y(const float *__restrict__ alpha,
                                                      const int32_t *__restrict__ labels,
                                                      int32_t N, int32_t K, float *__restrict__ A) {
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (size_t)N * K) return;
    const int32_t k = (int32_t)(e / (size_t)N), i = (int32_t)(e % (size_t)N);
    A[e] = labels[i] == k ? alpha[e] : -alpha[e];
}

constexpr size_t kGramLds = 160 * 1024 - 64;  // dynamic LDS of k_train_gram at most

struct GramArgs {
    const float *G;          // [N][N]
    const int32_t *labels;
    const float *sigma;
    const float *g0;         // [K][N] margins sum_j alpha_j y_j G_ij of a warm start, or null
    int32_t N, K;
    float C, eps;
    int32_t max_epochs;
    uint64_t seed;
    float *alpha;            // [K][N]: warm start in (with g0), final values out
    float *b;                // [K]
    int32_t *epochs;         // [K] or null
};

// Segment `seg` of `nseg` of epoch e's order (N entries): Fisher-Yates from
// the identity, i = N-1 down to 1 swapping i with r mod (i+1), r = draw
// e(N-1) + (N-1-i) of the class's splitmix64 stream; segment s takes the
// steps i in [max(1, N - (s+1) L), N-1 - s L], L = ceil((N-1) / nseg), and
// segment 0 first writes the identity. One wave, 64 swaps at a time: a swap waits
// for the last one before it that touched one of its two entries, and runs of swaps
// that wait for none of their own run go at once.
__device__ void gram_order(int16_t *ord, int32_t N, uint64_t state0, int32_t e, int seg, int nseg,
                           int lane) {
    if (seg == 0)
        for (int32_t p = lane; p < N; p += 64) ord[p] = (int16_t)p;
    const int32_t L = (N - 1 + nseg - 1) / nseg;
    const int32_t hi = N - 1 - seg * L, lo = max(1, N - (seg + 1) * L);
    const uint64_t base = (uint64_t)e * (uint64_t)(N - 1);
    for (int32_t top = hi; top >= lo; top -= 64) {
        const int32_t i = top - lane;
        int32_t j = -1;
        if (i >= lo) {
            const uint64_t r = splitmix64_at(state0, base + (uint64_t)(N - 1 - i));
            j = (int32_t)(r % (uint64_t)(i + 1));
        }
        const int cnt = min(64, top - lo + 1);
        // Entry i of a swap is touched before only as an earlier one's j.
        int last = -1;
        for (int t = 0; t < cnt; ++t) {
            const int32_t jt = __builtin_amdgcn_readlane(j, t);
            if (lane > t && (j == jt || i == jt)) last = t;
        }
        for (int t = 0; t < cnt;) {  // swaps t .. end - 1
            const uint64_t wait = __ballot(lane > t && lane < cnt && last >= t);
            const int end = wait ? __builtin_ctzll(wait) : cnt;
            if (lane >= t && lane < end) {
                const int16_t u = ord[i], v = ord[j];
                ord[i] = v;
                ord[j] = u;
            }
            t = end;
        }
    }
}

// A block of 64 samples of the epoch's order, one a lane, and G of the header
// comment under the present g and c. An update's time is its instructions and
// their latency, so what the block fixes is worked out once.
struct GramBlock {
    int32_t i;
    float y, al, q, G;
    uint64_t lower, upper, inside;  // lanes with alpha <= 0, >= C, between; valid ones
};

// One workgroup per class: waves 0..kS-1 solve, waves kS..kS+W-1 draw epoch orders
// (W = blockDim / 64 - kS). The order of epoch f is built by order wave f mod W
// in W segments during the W epochs before f, so each wave does 1/W of an
// order per epoch and every epoch ends at one barrier; W + 1 order buffers
// (epoch f in buffer f mod (W + 1)).
//
// An update is a serial chain: g of the next 64 samples from LDS, the first of
// them with a projected gradient, its step, its row of G, d times that row added
// to g. The solver waves run the chain alike, each on its own; only the row is
// shared out (wave w: columns 256 (kS u + w) + 4 lane .. + 3, u < kU). kTwo: from
// one of two copies of g into the other, and one hand-shake an update tells that
// all parts are written (a wave is one update ahead of another at most, and writes
// the copy that no one reads any more); else in place, with a hand-shake before the
// writes too. The rows of the next two samples, as things stand, are on their way
// to registers. The order of every sum is that of a single wave.
//
// 256 classes x 5120 samples (35 thousand updates in the longest class, rows of
// 20 KB out of the 105 MB matrix, 2.9 TB/s): 32 ms, 0.92 us an update; 51 ms with
// one solver wave, no row ahead and one swap of an order at a time. Whole trainings,
// before and after: 64 x 640 17.1 / 9.5 ms, 13 x 91 4.4 / 3.5, 254 x 5842 191 / 51,
// 330 x 7920 (in place) 273 / 149. Up to 1024 samples one wave: a row is 4 pieces
// then, about what a hand-shake takes (280 cycles).
//
// Dynamic LDS, N4 = N rounded up to 4: g (two copies if kTwo), alpha, the diagonal
// s2 G_ii + 1 (FP32 each), the orders (int16), y (int8). Entries of g past N hold
// what follows a row in memory and are not used.
template <int kS, int kU, bool kTwo>
__global__ __launch_bounds__(64 * (kS + 4)) void k_train_gram(GramArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int32_t N = a.N, N4 = (N + 3) & ~3;
    const int W = (int)(blockDim.x >> 6) - kS, B = W + 1;
    float *g = reinterpret_cast<float *>(smem);  // the present copy
    float *g_next = kTwo ? g + N4 : g;
    float *al = g_next + N4;
    float *qd = al + N4;
    int16_t *ord = reinterpret_cast<int16_t *>(qd + N4);  // [W + 1][N4]
    int8_t *ys = reinterpret_cast<int8_t *>(ord + (size_t)B * N4);
    __shared__ int32_t done[2];
    __shared__ uint32_t marks[4];  // hand-shakes each solver wave has come to

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t k = blockIdx.x;
    const float sig = *a.sigma, s2 = sig * sig, C = a.C;
    const bool warm = a.g0 != nullptr;
    for (int32_t i = tid; i < N; i += (int32_t)blockDim.x) {
        ys[i] = a.labels[i] == k ? 1 : -1;
        al[i] = warm ? a.alpha[(size_t)k * N + i] : 0.0f;
        g[i] = warm ? a.g0[(size_t)k * N + i] : 0.0f;
        qd[i] = s2 * a.G[(size_t)i * N + i] + 1.0f;
    }
    if (tid < 4) marks[tid] = 0;
    const uint64_t state0 = a.seed ^ (0x5851F42D4C957F2Dull * (uint64_t)(k + 1));
    __syncthreads();

    float c = 0.0f;  // solver waves: sum alpha y (the bias weight)
    if (wave < kS && warm) {
        float part = 0.0f;
        for (int32_t i = lane; i < N; i += 64) part += ys[i] > 0 ? al[i] : -al[i];
        c = wave_sum_f32(part);
    }
    gf4 r0[kU], r1[kU], r2[kU];  // rows id0, id1, id2 of G, or on their way
    int32_t id0 = -1, id1 = -1, id2 = -1;
    int32_t col[kU];  // columns past the end repeat the last ones
#pragma unroll
    for (int u = 0; u < kU; ++u) col[u] = min(256 * (kS * u + wave) + 4 * lane, N4 - 4);
    const int whole = (N4 / 256 - wave + kS - 1) / kS;  // pieces inside for every lane
    auto load = [&](int32_t i, gf4(&r)[kU]) {
        const float *row = a.G + (size_t)i * N;
#pragma unroll
        for (int u = 0; u < kU; ++u) r[u] = *reinterpret_cast<const gf4u *>(row + col[u]);
    };
    uint32_t mark = 0;
    // All solver waves are here, with their LDS reads and writes done. They make
    // the same updates, so each comes.
    auto meet = [&]() {
        ++mark;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0)
            __hip_atomic_store(&marks[wave], mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (__ballot((int32_t)(__hip_atomic_load(&marks[lane & (kS - 1)], __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_WORKGROUP) - mark) < 0)) {
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    int32_t epoch = a.max_epochs;
    // e < 0: the first orders only.
    for (int32_t e = -W; e < a.max_epochs; ++e) {
        if (wave < kS) {
            if (e >= 0) {
                const int16_t *od = ord + (size_t)(e % B) * N4;
                // The present block and the one after it, whose duals no step of
                // the present one changes; the samples of the block after that.
                GramBlock now, after;
                int32_t far;
                auto read = [&](GramBlock &w, int32_t i, int32_t p) {
                    const bool valid = p < N;
                    w.i = i;
                    w.y = ys[i] > 0 ? 1.0f : -1.0f;
                    w.al = al[i];
                    w.q = qd[i];
                    const uint64_t v = __ballot(valid), lo = __ballot(w.al <= 0.0f);
                    const uint64_t up = __ballot(w.al >= C) & ~lo;
                    w.lower = v & lo;
                    w.upper = v & up;
                    w.inside = v & ~(lo | up);
                };
                // Lanes whose projected gradient is not 0.
                auto test = [&](GramBlock &w, float gi) {
                    w.G = w.y * (s2 * gi + c) - 1.0f;
                    return (__ballot(w.G < 0.0f) & w.lower) | (__ballot(w.G > 0.0f) & w.upper) |
                           (__ballot(w.G != 0.0f) & w.inside);
                };
                int32_t s = 0;
                float max_pg = 0.0f;  // of the samples this lane held
                const int32_t i0 = lane < N ? od[lane] : 0, i1 = 64 + lane < N ? od[64 + lane] : 0;
                far = 128 + lane < N ? od[128 + lane] : 0;
                read(now, i0, lane);
                read(after, i1, 64 + lane);
                uint64_t m = test(now, g[i0]), m2 = test(after, g[i1]);
                // The next sample that moves and its step; false at the end.
                int32_t it = 0;
                float d = 0.0f, an = 0.0f;
                auto next = [&]() {
                    for (;;) {
                        while (m == 0) {
                            s += 64;
                            if (s >= N) return false;
                            now = after;
                            m = m2;
                            const float gf = g[far];
                            read(after, far, s + 64 + lane);
                            far = s + 128 + lane < N ? od[s + 128 + lane] : 0;
                            m2 = test(after, gf);
                        }
                        // Every lane its own step, then the first one's.
                        const float al_new = fminf(fmaxf(now.al - now.G / now.q, 0.0f), C);
                        const int t = __builtin_ctzll(m);
                        const float dl = now.q > 0.0f ? (al_new - now.al) * now.y : 0.0f;
                        it = __builtin_amdgcn_readlane(now.i, t);
                        d = readlane_f(dl, t);
                        an = readlane_f(al_new, t);
                        max_pg = fmaxf(max_pg, fabsf(readlane_f(now.G, t)));
                        // Visited: t and the lanes below it.
                        const uint64_t open = t < 63 ? ~0ull << (t + 1) : 0;
                        now.lower &= open;
                        now.upper &= open;
                        now.inside &= open;
                        m &= open;
                        if (d != 0.0f) return true;
                    }
                };
                auto step = [&](gf4(&r)[kU], int32_t &id, gf4(&rb)[kU], int32_t &idb) {
                    if (id != it) {
                        load(it, r);
                        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
                    }
                    // The second sample that moves from here if this step changes
                    // little (the first one's row was asked for a step ago).
                    const uint64_t w = m & (m - 1);
                    const uint64_t w2 = w ? w : m ? m2 : m2 & (m2 - 1);
                    const int t2 = __builtin_ctzll(w2 | 1ull << 63);
                    idb = w ? __builtin_amdgcn_readlane(now.i, t2) : __builtin_amdgcn_readlane(after.i, t2);
                    load(idb, rb);
                    id = -1;
                    gf4 v[kU];
#pragma unroll
                    for (int u = 0; u < kU; u += 4)
                        if (kU % 4 == 0 && u + 4 <= whole)  // uniform
                            lds_read4<1024 * kS>((uint32_t)(uintptr_t)(g + col[u]), v[u],
                                                 v[min(u + 1, kU - 1)], v[min(u + 2, kU - 1)],
                                                 v[min(u + 3, kU - 1)]);
                        else
#pragma unroll
                            for (int t = u; t < min(u + 4, kU); ++t)
                                v[t] = *reinterpret_cast<const gf4 *>(g + col[t]);
#pragma unroll
                    for (int u = 0; u < kU; ++u)
#pragma unroll
                        for (int x = 0; x < 4; ++x) v[u][x] += d * r[u][x];
                    if constexpr (!kTwo && kS > 1) meet();
                    // Lanes past the end write what the last columns' lanes do, or,
                    // where those may have been ahead, nothing.
#pragma unroll
                    for (int u = 0; u < kU; ++u)
                        if (kTwo || kS == 1 || 256 * (kS * u + wave) + 4 * lane < N4)
                            *reinterpret_cast<gf4 *>(g_next + col[u]) = v[u];
                    if constexpr (kTwo) {
                        float *t = g;
                        g = g_next;
                        g_next = t;
                    }
                    if constexpr (kS > 1) meet();
                    // Not before every solver wave has taken the step: one that has
                    // not may yet read the old dual with a later block.
                    if (wave == 0 && lane == 0) al[it] = an;
                    c += d;
                    const float ga = g[now.i], gb = g[after.i];
                    m = test(now, ga);
                    m2 = test(after, gb);
                };
                for (;;) {
                    if (!next()) break;
                    step(r0, id0, r2, id2);
                    if (!next()) break;
                    step(r1, id1, r0, id0);
                    if (!next()) break;
                    step(r2, id2, r1, id1);
                }
                if (tid == 0) done[e & 1] = max_pg < a.eps;
            }
        } else {
            // The epoch f in [e + 1, e + W] with f = w (mod W), at its segment
            // e - f + W.
            const int w = wave - kS;
            const int32_t f = e + 1 + (((w - (e + 1)) % W) + W) % W;
            if (f >= 0 && f < a.max_epochs)
                gram_order(ord + (size_t)(f % B) * N4, N, state0, f, (int)(e - f + W), W, lane);
        }
        __syncthreads();
        if (e >= 0 && done[e & 1] != 0) {  // uniform
            epoch = e + 1;
            break;
        }
    }
    for (int32_t i = tid; i < N; i += (int32_t)blockDim.x) a.alpha[(size_t)k * N + i] = al[i];
    if (tid == 0) {
        a.b[k] = c;
        if (a.epochs) a.epochs[k] = epoch;
    }
}

// W_k = s2 sum_i alpha_ki y_ki x_i (samples in index order, zero duals
// skipped); thread t of workgroup (k, p) owns coordinates 2048 p + t + 256 j. The
// samples with a dual are listed first, so that four of them are in flight at a
// time (one at a time, all coordinates of a class in one workgroup: 1250 us at 256
// classes x 5120 samples x 7552, 89 us so).
__global__ __launch_bounds__(256) void k_gram_weights(const float *__restrict__ X,
                                                      const int32_t *__restrict__ labels,
                                                      int32_t N, int32_t D,
                                                      const float *__restrict__ alpha,
                                                      const float *__restrict__ sigma,
                                                      float *__restrict__ W) {
    constexpr int kJ = 8, kList = 1024;
    __shared__ float coef[kList];
    __shared__ int32_t index[kList];
    __shared__ int32_t listed[4];  // by each wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t k = blockIdx.x;
    int32_t d[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) d[j] = 2048 * (int32_t)blockIdx.y + tid + 256 * j;
    float acc[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) acc[j] = 0.0f;
    for (int32_t i0 = 0; i0 < N; i0 += kList) {
        // Wave w lists samples i0 + 256 w .. + 255, in order, from entry 256 w on.
        __syncthreads();
        int32_t n = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int32_t i = i0 + 256 * wave + 64 * q + lane;
            const float av = i < N ? alpha[(size_t)k * N + i] : 0.0f;
            const uint64_t m = __ballot(av != 0.0f);
            if (av != 0.0f) {
                const int e = 256 * wave + n + __builtin_popcountll(m & ((1ull << lane) - 1));
                coef[e] = labels[i] == k ? av : -av;
                index[e] = i;
            }
            n += __builtin_popcountll(m);
        }
        if (lane == 0) listed[wave] = n;
        __syncthreads();
        for (int w = 0; w < 4; ++w) {
            const int end = 256 * w + listed[w];
            for (int t = 256 * w; t < end; t += 4) {
                float x[4][kJ];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float *row = X + (size_t)index[min(t + u, end - 1)] * D;
#pragma unroll
                    for (int j = 0; j < kJ; ++j) x[u][j] = row[min(d[j], D - 1)];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (t + u >= end) break;  // uniform
                    const float cf = coef[t + u];
#pragma unroll
                    for (int j = 0; j < kJ; ++j) acc[j] += cf * x[u][j];
                }
            }
        }
    }
    const float sg = *sigma, s2 = sg * sg;
#pragma unroll
    for (int j = 0; j < kJ; ++j)
        if (d[j] < D) W[(size_t)k * D + d[j]] = s2 * acc[j];
}

}  // namespace

size_t train_gram_workspace_bytes(int32_t N, int32_t K) {
    const size_t n = (size_t)N, kn = (size_t)K * N;
    return sizeof(float) * (n * n + 2 * n + 64 + 3 * kn);
}

hipError_t launch_train_gram(const float *X, const int32_t *labels, int32_t N, int32_t D,
                             int32_t K, float C, float eps, int32_t max_epochs, uint64_t seed,
                             float *alpha, int32_t warm, float *W, float *b, int32_t *epochs,
                             void *workspace, hipStream_t s) {
    const size_t n = (size_t)N, kn = (size_t)K * N;
    float *G = static_cast<float *>(workspace);
    float *norms = G + n * n;
    float *zeros = norms + n;
    float *sigma = zeros + n;
    float *A = sigma + 64;
    float *G0 = A + kn;
    float *al = alpha ? alpha : G0 + kn;
    const dim3 blk(256), rows((N + 255) / 256);
    hipLaunchKernelGGL(k_gram_zero, rows, blk, 0, s, zeros, N);
    hipError_t e = launch_score_f32(X, N, X, zeros, N, D, G, nullptr, s, 1, nullptr, nullptr, true);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gram_diag, rows, blk, 0, s, G, N, norms);
    hipLaunchKernelGGL(k_gram_sigma, dim3((N + 15) / 16), blk, 0, s, norms, N, sigma);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const bool w = warm && alpha;
    if (w) {
        hipLaunchKernelGGL(k_gram_alpha_y, dim3((unsigned)((kn + 255) / 256)), blk, 0, s, alpha,
                           labels, N, K, A);
        if ((e = launch_score_f32(A, K, G, zeros, N, N, G0, nullptr, s, 1, nullptr, nullptr,
                                  true)) != hipSuccess)
            return e;
    }
    GramArgs a{G, labels, sigma, w ? G0 : nullptr, N, K, C, eps, max_epochs, seed, al, b, epochs};
    // Bytes of LDS a sample, less the orders' 2 (W + 1): two copies of g where more
    // than one wave solves and they fit beside two orders. As many order waves (at
    // most 4) as there is room for, one at least.
    const size_t n4 = (n + 3) & ~(size_t)3;
    const bool two = N > 1024 && n4 * (17 + 4) <= kGramLds;
    const size_t bytes = two ? 17 : 13;
    const int nw = (int)std::min<size_t>(4, (kGramLds / n4 - bytes) / 2 - 1);
    const size_t lds = (bytes + 2 * ((size_t)nw + 1)) * n4;
    auto solve = [&](auto kern, int solvers) {
        if ((e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds)) != hipSuccess)
            return;
        hipLaunchKernelGGL(kern, dim3(K), dim3(64 * (solvers + nw)), lds, s, a);
        e = hipGetLastError();
    };
    if (N <= 256) solve(k_train_gram<1, 1, false>, 1);
    else if (N <= 1024) solve(k_train_gram<1, 4, false>, 1);
    else if (!two) solve(k_train_gram<4, 8, false>, 4);
    else if (N <= 2048) solve(k_train_gram<2, 4, true>, 2);
    else if (N <= 4096) solve(k_train_gram<4, 4, true>, 4);
    else if (N <= 5120) solve(k_train_gram<4, 5, true>, 4);
    else solve(k_train_gram<4, 8, true>, 4);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gram_weights, dim3(K, (D + 2047) / 2048), blk, 0, s, X, labels, N, D, al,
                       sigma, W);
    return hipGetLastError();
}

size_t train_workspace_bytes(int32_t N) { return ((size_t)2 * N + 1) * sizeof(double); }

hipError_t launch_train(const float *X, const int32_t *labels, int32_t N, int32_t D, int32_t K,
                        double C, double eps, int32_t max_epochs, uint64_t seed, double *alpha,
                        int32_t warm, float *W, float *b, double *W64, double *b64,
                        int32_t *epochs, void *workspace, hipStream_t s) {
    double *norms = static_cast<double *>(workspace);
    double *qii = norms + N;
    double *sigma = qii + N;
    const dim3 rows((N + kWaves - 1) / kWaves);
    hipLaunchKernelGGL(k_row_norms, rows, dim3(kThreads), 0, s, X, N, D, nullptr, norms);
    hipLaunchKernelGGL(k_sigma, dim3(1), dim3(kThreads), 0, s, norms, N, sigma);
    hipLaunchKernelGGL(k_row_norms, rows, dim3(kThreads), 0, s, X, N, D, sigma, qii);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    TrainArgs a{X, labels, sigma, qii, N, D, K, C, eps, max_epochs, seed, warm, alpha,
                W, b, W64, b64, epochs};
    if (D <= 4 * kThreads) return launch_train_j<4>(a, s);
    if (D <= 8 * kThreads) return launch_train_j<8>(a, s);
    if (D <= 16 * kThreads) return launch_train_j<16>(a, s);
    return launch_train_j<32>(a, s);
}

}  // namespace lbpf
