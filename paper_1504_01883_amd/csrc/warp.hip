// Warped face crops (Sec. 2.1, Eq. 1: p' = x u + y v + t, the affine frame
// that turns the mapped face region into a rectangle; Sec. 3: the face is
// resized to 200 x 200 before its features are taken).
//
// Crop pixel (x, y) reads the source pixel
//   sx = floor((ux x + vx y + tx) / 2^16),  sy = floor((uy x + vy y + ty) / 2^16)
// (16.16 fixed point, exact in 64-bit integers, nearest sample). The host has
// checked that the four corner samples, and so by linearity every sample,
// lie inside the plane; the kernel clamps anyway so that no frame can send a
// load outside the plane.
//
// One workgroup per crop, or (few crops) per range of its rows. A lane makes 4
// adjacent output pixels of a row at a time, stored as one 4-byte and one 8-byte
// word; a wave holds as many rows side by side as fit its 64 lanes. Positions
// are kept in 32 bits where the planes' sides are below 2^15: every sample lies
// inside its plane, so the wrapped sums are exact.
//
// An axis-parallel frame (a resize: u_y = v_x = 0) with steps of at most 2
// source pixels reads a lane's 4 samples with one 8-byte (grey) and one 16-byte
// (depth) load: they lie within 8 pixels, at distances that are the same in
// every row, so the byte permutations that pick them are set up once per lane.
// 2048 boxes of 48-256 px to 200 x 200: 135 us (64-bit positions, one sample a
// load and a byte a store: 357), bound by the address processing of its gathered
// loads, 3 TB/s of samples and crops; rows in flight and workgroups change nothing.
#include "lbpf_internal.h"

#include <algorithm>

namespace lbpf {

namespace {

constexpr int kThreads = 256;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Unaligned addresses are fine on gfx950.
template <typename T>
__device__ __forceinline__ T ld(const void *p) {
    T v;
    __builtin_memcpy(&v, p, sizeof v);
    return v;
}
template <typename T>
__device__ __forceinline__ void st(void *p, T v) {
    __builtin_memcpy(p, &v, sizeof v);
}

template <typename P>
__device__ __forceinline__ int32_t sample(P a, int32_t lim) {
    const P q = a >> 16;  // arithmetic shift: floor division by 2^16
    return (int32_t)min<P>(max<P>(q, 0), (P)lim - 1);
}

// Four packed samples of a crop row: grey bytes, depth u16 pairs.
struct Quad {
    uint32_t g;
    u32x2 z;
};

// Any frame, pixel by pixel. U: the unsigned type positions are summed in (wraps
// are exact, see above), S: its signed twin.
template <typename U, typename S>
__device__ __forceinline__ Quad quad_any(const WarpDesc &d, int x0, int y) {
    auto at = [&](const int32_t *f, int i) {
        return (U)(S)f[i] * (U)x0 + (U)(S)f[2 + i] * (U)y + (U)(S)f[4 + i];
    };
    Quad q{0u, u32x2{0u, 0u}};
    U zx = at(d.df, 0), zy = at(d.df, 1), gx = at(d.gf, 0), gy = at(d.gf, 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const size_t zi = (size_t)sample<S>((S)zy, d.src_h) * d.d_pitch + sample<S>((S)zx, d.src_w);
        q.z[k >> 1] |= (uint32_t)d.d_src[zi] << (16 * (k & 1));
        if (d.g_src) {
            const size_t gi = (size_t)sample<S>((S)gy, d.src_h) * d.g_pitch + sample<S>((S)gx, d.src_w);
            q.g |= (uint32_t)d.g_src[gi] << (8 * k);
        }
        zx += (U)(S)d.df[0];
        zy += (U)(S)d.df[1];
        gx += (U)(S)d.gf[0];
        gy += (U)(S)d.gf[1];
    }
    return q;
}

// The four sample columns of output columns x0 .. x0 + 3 of an axis-parallel
// frame: the column `at` their load starts at, and each one's distance from it
// (0 .. 7).
struct Columns {
    int32_t at, off[4];
};
__device__ __forceinline__ Columns columns(const int32_t *f, int x0, int32_t src_w) {
    Columns c;
    uint32_t p = (uint32_t)f[0] * (uint32_t)x0 + (uint32_t)f[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c.off[k] = sample<int32_t>((int32_t)p, src_w);
        p += (uint32_t)f[0];
    }
    c.at = min(c.off[0], src_w - 8);
#pragma unroll
    for (int k = 0; k < 4; ++k) c.off[k] -= c.at;
    return c;
}

__device__ __forceinline__ bool resize_frame(const int32_t *f) {
    return f[1] == 0 && f[2] == 0 && f[0] >= 0 && f[0] <= 2 << 16;
}

__global__ __launch_bounds__(kThreads) void k_warp(const WarpDesc *__restrict__ descs) {
    const WarpDesc d = descs[blockIdx.x];  // a copy: not re-read after every store
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int w = d.w, h = d.h;
    const int ya = (int)((int64_t)h * blockIdx.y / gridDim.y);
    const int yb = (int)((int64_t)h * (blockIdx.y + 1) / gridDim.y);
    const bool narrow = d.src_w < 32768 && d.src_h < 32768;
    if (w < 4) {
        for (int y = ya + threadIdx.x; y < yb; y += kThreads) {
            const Quad q = quad_any<uint64_t, int64_t>(d, 0, y);  // w >= 3; the fourth sample is clamped, not kept
            for (int x = 0; x < w; ++x) {
                d.d_dst[y * w + x] = (uint16_t)(q.z[x >> 1] >> (16 * (x & 1)));
                if (d.g_src) d.g_dst[y * w + x] = (uint8_t)(q.g >> (8 * x));
            }
        }
        return;
    }
    const int groups = (w + 3) >> 2;                        // of 4 columns
    const int gw = min(groups, 64), rpw = 64 / gw;          // side by side in a wave
    const int sub = lane / gw, rows = kThreads / 64 * rpw;  // rows at a time
    if (sub >= rpw) return;
    const bool axis = narrow && d.src_w >= 8 && resize_frame(d.df) && (!d.g_src || resize_frame(d.gf));
    for (int g = lane - sub * gw; g < groups; g += gw) {
        // The last group starts at column w - 4: it may repeat columns of the
        // one before it, with the same values.
        const int x0 = min(4 * g, w - 4);
        auto put = [&](int y, const Quad &q) {
            st(d.d_dst + (size_t)y * w + x0, q.z);
            if (d.g_src) st(d.g_dst + (size_t)y * w + x0, q.g);
        };
        const int y0 = ya + wave * rpw + sub;
        if (axis) {
            const Columns cz = columns(d.df, x0, d.src_w), cg = columns(d.gf, x0, d.src_w);
            // perm(hi, lo, sel): bytes 0-3 are lo's, 4-7 hi's, 0x0C is 0. A depth
            // sample comes from the first four pixels of its load (zl) or the
            // last four (zh).
            uint32_t sg = 0, zl[2] = {0u, 0u}, zh[2] = {0u, 0u};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sg |= (uint32_t)cg.off[k] << (8 * k);
                const uint32_t o = 2u * (uint32_t)(cz.off[k] & 3), s = (o | (o + 1) << 8);
                zl[k >> 1] |= (cz.off[k] < 4 ? s : 0x0C0Cu) << (16 * (k & 1));
                zh[k >> 1] |= (cz.off[k] < 4 ? 0x0C0Cu : s) << (16 * (k & 1));
            }
#pragma unroll 2
            for (int y = y0; y < yb; y += rows) {
                const int32_t zy = sample<int32_t>((int32_t)((uint32_t)d.df[3] * (uint32_t)y + (uint32_t)d.df[5]), d.src_h);
                const u32x4 z = ld<u32x4>(d.d_src + (size_t)zy * d.d_pitch + cz.at);
                Quad q;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    q.z[i] = __builtin_amdgcn_perm(z.y, z.x, zl[i]) | __builtin_amdgcn_perm(z.w, z.z, zh[i]);
                if (d.g_src) {
                    const int32_t gy = sample<int32_t>((int32_t)((uint32_t)d.gf[3] * (uint32_t)y + (uint32_t)d.gf[5]), d.src_h);
                    const u32x2 v = ld<u32x2>(d.g_src + (size_t)gy * d.g_pitch + cg.at);
                    q.g = __builtin_amdgcn_perm(v.y, v.x, sg);
                }
                put(y, q);
            }
        } else if (narrow) {
            for (int y = y0; y < yb; y += rows) put(y, quad_any<uint32_t, int32_t>(d, x0, y));
        } else {
            for (int y = y0; y < yb; y += rows) put(y, quad_any<uint64_t, int64_t>(d, x0, y));
        }
    }
}

}  // namespace

hipError_t launch_warp(const WarpDesc *d, int32_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    // 8192 workgroups, at most 16 a crop: short ones level the crops' ends (2048
    // boxes to 200 x 200: 135 us with 4 a crop, 145 with one).
    const int parts = std::max(1, std::min(16, 8192 / n));
    hipLaunchKernelGGL(k_warp, dim3(n, parts), dim3(kThreads), 0, s, d);
    return hipGetLastError();
}

}  // namespace lbpf
