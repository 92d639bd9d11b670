// k_ray.hip -- ray-direction encoding added to the input views' feature maps
// (Sec. 3.2.1 and "Encode Input Images" of Sec. 3.2.2): the ray of a pixel
// of view m is cut by the planes z = near and z = far of the novel camera's
// frustum, both points are projected by the novel camera, and their
// difference (far minus near, in normalised device coordinates) goes
// through tanh, 8 octaves of sinusoids and a linear map to C channels.
//
// With o view m's centre and d the pixel's ray direction, both in the novel
// frame, the ray meets the plane z at P = o + (z - o_z)/d_z d, so
//   P_x / z = d_x / d_z + (o_x - o_z d_x / d_z) / z
// and the difference of P_x / z between the far and the near plane is
// (1/far - 1/near)(o_x - o_z d_x / d_z), likewise for y; the NDC
// difference applies the first two rows of the novel K (on its own grid,
// NDC = 2 (u, v) / (W_n, H_n) up to a constant that cancels).
//
// Two forms.  Per pixel: every map pixel evaluates its own encoding.  Low
// resolution, as the paper does it (k_ray_encoding into a workspace, then
// k_ray_upsample_add): the projected encoding is evaluated once per pixel of a
// coarse grid, then every map pixel adds its bilinear upsampling -- projection
// and bilinear interpolation are both linear, so projecting first gives the
// same values and leaves C channels, not 32, to interpolate; the second pass
// is bound by the feature maps' HBM traffic.
//
// The encoding runs in double up to the sinusoids (the top octave scales
// its argument by 128 pi): sin(pi t) and cos(pi t) from their Taylor
// series on a quarter period after an exact quadrant reduction, then each
// higher octave by the double-angle identities sin 2a = 2 sin a cos a,
// cos 2a = (cos a - sin a)(cos a + sin a) -- the angle error doubles per
// octave, about 1e-14 at the top.  The projection, in float, accumulates on top
// of the feature, which is rounded once at the store.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "uf_params.h"

namespace qk {
namespace {

// pi^n / n!, for the Taylor coefficients
__host__ __device__ constexpr double pi_pow_over_fact(int n) {
    double r = 1.0;
    for (int i = 1; i <= n; ++i) r *= 3.141592653589793 / (double)i;
    return r;
}

// sin(pi x) and cos(pi x) for |x| <= 1/4 (|pi x| <= 0.79): Taylor series to
// x^17 and x^16, the first omitted terms below 1e-17
__device__ inline void sincospi_quarter(double x, double &s, double &c) {
    constexpr double P1 = pi_pow_over_fact(1), P2 = pi_pow_over_fact(2),
                     P3 = pi_pow_over_fact(3), P4 = pi_pow_over_fact(4),
                     P5 = pi_pow_over_fact(5), P6 = pi_pow_over_fact(6),
                     P7 = pi_pow_over_fact(7), P8 = pi_pow_over_fact(8),
                     P9 = pi_pow_over_fact(9), P10 = pi_pow_over_fact(10),
                     P11 = pi_pow_over_fact(11), P12 = pi_pow_over_fact(12),
                     P13 = pi_pow_over_fact(13), P14 = pi_pow_over_fact(14),
                     P15 = pi_pow_over_fact(15), P16 = pi_pow_over_fact(16),
                     P17 = pi_pow_over_fact(17);
    const double z = x * x;
    double ps = fma(P17, z, -P15);
    ps = fma(ps, z, P13);
    ps = fma(ps, z, -P11);
    ps = fma(ps, z, P9);
    ps = fma(ps, z, -P7);
    ps = fma(ps, z, P5);
    ps = fma(ps, z, -P3);
    ps = fma(ps, z, P1);
    s = ps * x;
    double pc = fma(P16, z, -P14);
    pc = fma(pc, z, P12);
    pc = fma(pc, z, -P10);
    pc = fma(pc, z, P8);
    pc = fma(pc, z, -P6);
    pc = fma(pc, z, P4);
    pc = fma(pc, z, -P2);
    c = fma(pc, z, 1.0);
}

// sin(pi t), cos(pi t) for |t| <= 1: t = f + q/2 with q = rint(2t) and
// |f| <= 1/4 (both exact), then a rotation by q quarter turns
__device__ inline void sincospi_unit(double t, double &s, double &c) {
    const double q = rint(2.0 * t);
    double sf, cf;
    sincospi_quarter(fma(-0.5, q, t), sf, cf);
    const int qi = ((int)q) & 3;
    s = qi == 0 ? sf : qi == 1 ? cf : qi == 2 ? -sf : -cf;
    c = qi == 0 ? cf : qi == 1 ? -sf : qi == 2 ? -cf : sf;
}

// 1 / n!
__host__ __device__ constexpr double inv_fact(int n) {
    double r = 1.0;
    for (int i = 2; i <= n; ++i) r /= (double)i;
    return r;
}

// tanh(x) = 1 - 2 / (e^(2x) + 1), to an absolute error near 1e-16 (the
// octaves need absolute accuracy in t, so the cancellation near x = 0 costs
// nothing): e^y = 2^n e^r with n = rint(y / ln 2), r = y - n ln 2,
// |r| <= 0.35, e^r by its Taylor series to r^14; y is clamped to [-40, 40],
// where tanh is +-1 to double precision; the quotient by a reciprocal and
// two Newton steps.
__device__ inline double tanh_abs(double x) {
    constexpr double kLn2 = 0.6931471805599453, kLog2e = 1.4426950408889634;
    const double y = fmin(fmax(2.0 * x, -40.0), 40.0);
    const double n = rint(y * kLog2e);
    const double r = fma(-n, kLn2, y);
    double p = inv_fact(14);
#pragma unroll
    for (int k = 13; k >= 0; --k) p = fma(p, r, inv_fact(k));
    const double d = ldexp(p, (int)n) + 1.0;
    double q = __builtin_amdgcn_rcp(d);
    q = fma(q, fma(-d, q, 1.0), q);
    q = fma(q, fma(-d, q, 1.0), q);
    return fma(-2.0, q, 1.0);
}

__device__ inline float bf2f(uint16_t h) { return __uint_as_float((unsigned)h << 16); }

__device__ inline uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// The two angles' arguments (before tanh) of pixel (x, y) of view m's grid (the grid
// the composed D[m] was made for).
__device__ __forceinline__ void ray_difference(const RayParams &p, int m, int x, int y, double &ax, double &ay) {
    const double u = (double)x + 0.5, v = (double)y + 0.5;
    const double *D = p.D[m], *o = p.o[m];
    const double dx = fma(D[0], u, fma(D[1], v, D[2]));
    const double dy = fma(D[3], u, fma(D[4], v, D[5]));
    const double dz = fma(D[6], u, fma(D[7], v, D[8]));
    const double rz = o[2] / dz;
    ax = p.inv_band * fma(-rz, dx, o[0]);
    ay = p.inv_band * fma(-rz, dy, o[1]);
}

// the next octave: sin 2a, cos 2a
__device__ __forceinline__ void next_octave(double &s, double &c) {
    const double s2 = 2.0 * s * c, c2 = (c - s) * (c + s);
    s = s2;
    c = c2;
}

// 16 of the 32 sinusoids of a pixel: sine and cosine of one angle (x's, or y's) in 8
// octaves.
__device__ __forceinline__ void ray_sinusoids(const RayParams &p, int m, int x, int y, bool second, float fs[8],
                                              float fc[8]) {
    double ax, ay, s, c;
    ray_difference(p, m, x, y, ax, ay);
    sincospi_unit(tanh_abs(second ? fma(p.ky0, ax, p.ky1 * ay) : fma(p.kx0, ax, p.kx1 * ay)), s, c);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        fs[k] = (float)s;
        fc[k] = (float)c;
        if (k < 7) next_octave(s, c);
    }
}

// All 32, the two angles' chains side by side.
__device__ __forceinline__ void ray_sinusoids(const RayParams &p, int m, int x, int y, float e[32]) {
    double ax, ay, sx, cx, sy, cy;
    ray_difference(p, m, x, y, ax, ay);
    const double tx = tanh_abs(fma(p.kx0, ax, p.kx1 * ay)), ty = tanh_abs(fma(p.ky0, ax, p.ky1 * ay));
    sincospi_unit(tx, sx, cx);
    sincospi_unit(ty, sy, cy);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        e[4 * k] = (float)sx;
        e[4 * k + 1] = (float)cx;
        e[4 * k + 2] = (float)sy;
        e[4 * k + 3] = (float)cy;
        if (k < 7) {
            next_octave(sx, cx);
            next_octave(sy, cy);
        }
    }
}

// 8 channels of a feature pixel as float, and back (rounded once)
template <bool BF16>
__device__ inline void load8(const void *base, int64_t off, float a[8]) {
    if constexpr (BF16) {
        const uint4 r = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(base) + off);
        const unsigned wd[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a[2 * j] = bf2f((uint16_t)(wd[j] & 0xffffu));
            a[2 * j + 1] = bf2f((uint16_t)(wd[j] >> 16));
        }
    } else {
        const float4 *ptr = reinterpret_cast<const float4 *>(static_cast<const float *>(base) + off);
        const float4 r0 = ptr[0], r1 = ptr[1];
        a[0] = r0.x; a[1] = r0.y; a[2] = r0.z; a[3] = r0.w;
        a[4] = r1.x; a[5] = r1.y; a[6] = r1.z; a[7] = r1.w;
    }
}

template <bool BF16>
__device__ inline void store8(void *base, int64_t off, const float a[8]) {
    if constexpr (BF16) {
        uint4 r;
        r.x = f2bf(a[0]) | ((unsigned)f2bf(a[1]) << 16);
        r.y = f2bf(a[2]) | ((unsigned)f2bf(a[3]) << 16);
        r.z = f2bf(a[4]) | ((unsigned)f2bf(a[5]) << 16);
        r.w = f2bf(a[6]) | ((unsigned)f2bf(a[7]) << 16);
        *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(base) + off) = r;
    } else {
        float4 *ptr = reinterpret_cast<float4 *>(static_cast<float *>(base) + off);
        ptr[0] = make_float4(a[0], a[1], a[2], a[3]);
        ptr[1] = make_float4(a[4], a[5], a[6], a[7]);
    }
}

// N consecutive channels as float, and back (rounded once); N = 2 or a multiple of 4
template <int N, bool BF16>
__device__ __forceinline__ void load_n(const void *base, int64_t off, float a[N]) {
    if constexpr (N % 8 == 0) {
#pragma unroll
        for (int j = 0; j < N; j += 8) load8<BF16>(base, off + j, a + j);
    } else if constexpr (BF16) {
        const unsigned *w = reinterpret_cast<const unsigned *>(static_cast<const uint16_t *>(base) + off);
        unsigned r[N / 2];
        if constexpr (N == 4) {
            const uint2 v = *reinterpret_cast<const uint2 *>(w);
            r[0] = v.x;
            r[1] = v.y;
        } else {
            r[0] = w[0];
        }
#pragma unroll
        for (int j = 0; j < N / 2; ++j) {
            a[2 * j] = bf2f((uint16_t)(r[j] & 0xffffu));
            a[2 * j + 1] = bf2f((uint16_t)(r[j] >> 16));
        }
    } else {
        typedef float vec __attribute__((ext_vector_type(N)));
        const vec v = *reinterpret_cast<const vec *>(static_cast<const float *>(base) + off);
#pragma unroll
        for (int j = 0; j < N; ++j) a[j] = v[j];
    }
}

template <int N, bool BF16>
__device__ __forceinline__ void store_n(void *base, int64_t off, const float a[N]) {
    if constexpr (N % 8 == 0) {
#pragma unroll
        for (int j = 0; j < N; j += 8) store8<BF16>(base, off + j, a + j);
    } else if constexpr (BF16) {
        typedef unsigned vec __attribute__((ext_vector_type(N / 2)));
        vec v;
#pragma unroll
        for (int j = 0; j < N / 2; ++j) v[j] = f2bf(a[2 * j]) | ((unsigned)f2bf(a[2 * j + 1]) << 16);
        *reinterpret_cast<vec *>(static_cast<uint16_t *>(base) + off) = v;
    } else {
        typedef float vec __attribute__((ext_vector_type(N)));
        vec v;
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] = a[j];
        *reinterpret_cast<vec *>(static_cast<float *>(base) + off) = v;
    }
}

// The projected encoding e Wr of every pixel of a grid: LOW, of the (lH, lW)
// grid, float32, into the workspace [V][lH][lW][C]; otherwise of every map,
// added to its features (the per-pixel form).
//
// A wave takes 32 pixels at a time: lane 32 h + 16 a + n evaluates angle a of
// pixel 16 h + n, one evaluation per pixel and angle.  The product runs on the
// matrix cores in float, 16x16x4, with the k index of step t at 4 t + g for the
// lanes of group g = lane / 16: those are the encoding's components of octave
// t, and two swaps of lane groups turn the sines and cosines of an octave into
// the operands of both halves' 16 pixels.  The weights' channels are the rows,
// row 4 g + i of block b being channel (C / 4) g + 4 b + i, so that a lane ends
// with C / 4 consecutive channels of its pixel (C = 8: 2, rows 2 and 3 of each
// group empty).  A wave keeps the weights in registers over its pixels.
//
// The low-resolution grid of a 1080p pyramid (8 views, 240 x 135) took 24 and 15 us
// at 32 and 16 channels and 43 us added to its own map at 64, one thread per pixel
// with the weights as LDS broadcasts or scalars (LDS reads bound the first, few
// and long waves the rest); now 17, 12 and 25.  The chain of double operations, of
// which 4 waves per SIMD overlap, bounds it: held to 80 registers for 6 waves it
// spills (33, 23, 28 us).  A frame's small grids took 12 us a launch, now 5.
template <int C, bool LOW, bool BF16>
__global__ void __launch_bounds__(256) k_ray_encoding(const RayParams p) {
    constexpr int NB = C < 16 ? 1 : C / 16, NCH = C / 4;
    typedef float f4 __attribute__((ext_vector_type(4)));
    const int m = blockIdx.y;
    const int fw = LOW ? p.lW : p.fW[m];
    const int64_t np = (int64_t)(LOW ? p.lH : p.fH[m]) * fw;
    const int lane = threadIdx.x & 63, g = lane >> 4, n = lane & 15;
    const int64_t step = (int64_t)gridDim.x * 128;
    int64_t q0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32;
    if (q0 >= np) return;
    float w[NB][8];
    {
        const bool row = C >= 16 || (n & 3) < 2;
        const int ch = C < 16 ? 2 * (n >> 2) + (n & 1) : NCH * (n >> 2) + (n & 3);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float v = p.Wr[(4 * k + g) * C + ch + 4 * b];
                w[b][k] = row ? v : 0.0f;
            }
    }
    double rw = __builtin_amdgcn_rcp((double)fw);
    rw = fma(rw, fma(-(double)fw, rw, 1.0), rw);
    rw = fma(rw, fma(-(double)fw, rw, 1.0), rw);
    for (; q0 < np; q0 += step) {
        float e[2][8];
        {
            const int64_t qe = q0 + 16 * (lane >> 5) + n, q = qe < np ? qe : np - 1;
            // exact: the quotient is 1 / (2 fw) or more from the next integer
            const int y = (int)(((double)q + 0.5) * rw), x = (int)(q - (int64_t)y * fw);
            ray_sinusoids(p, m, x, y, (lane >> 4) & 1, e[0], e[1]);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            // s = (s0 s1 s2 s3), c alike by lane group: then (s0 c0 s2 c2) and
            // (s1 c1 s3 c3), then (s0 c0 s1 c1) and (s2 c2 s3 c3)
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(e[0][k]), __float_as_uint(e[1][k]), false, false);
            const auto t = __builtin_amdgcn_permlane32_swap(r[0], r[1], false, false);
            e[0][k] = __uint_as_float(t[0]);
            e[1][k] = __uint_as_float(t[1]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t q = q0 + 16 * h + n;
            const bool live = q < np;
            float a[NCH];
            if constexpr (!LOW) load_n<NCH, BF16>(p.src[m], (live ? q : np - 1) * C + NCH * g, a);
            f4 acc[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[b][i] = (LOW || 4 * b + i >= NCH) ? 0.0f : a[4 * b + i];
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[b][k], e[h][k], acc[b], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NCH; ++j) a[j] = acc[j / 4][j % 4];
            if (live) {
                if constexpr (LOW) store_n<NCH, false>(p.P, ((int64_t)m * np + q) * C + NCH * g, a);
                else store_n<NCH, BF16>(p.feat[m], q * C + NCH * g, a);
            }
        }
    }
}

// The same with a pixel per thread and the weights as scalars, for few channels: a
// pixel's ray and its division are worked out once for both angles, and 8 channels
// leave half of the matrix cores' rows empty.  The products' order differs, so the
// last bits may.
template <int C, bool LOW, bool BF16>
__global__ void __launch_bounds__(256) k_ray_pixels(const RayParams p) {
    const int m = blockIdx.y;
    const int fw = LOW ? p.lW : p.fW[m];
    const int64_t np = (int64_t)(LOW ? p.lH : p.fH[m]) * fw;
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= np) return;
    const int y = (int)(q / fw), x = (int)(q - (int64_t)y * fw);
    float e[32];
    ray_sinusoids(p, m, x, y, e);
    // all of the pixel's channels are read before any is written: the source may be
    // the map itself
    float a[C];
#pragma unroll
    for (int j = 0; j < C; ++j) a[j] = 0.0f;
    if constexpr (!LOW) load_n<C, BF16>(p.src[m], q * C, a);
    typedef const __attribute__((address_space(4))) float *scalars;   // uniform reads: scalar loads
    const scalars w = (scalars)p.Wr;
#pragma unroll
    for (int i = 0; i < 32; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) a[j] = fmaf(e[i], w[i * C + j], a[j]);
    if constexpr (LOW) store_n<C, false>(p.P, ((int64_t)m * np + q) * C, a);
    else store_n<C, BF16>(p.feat[m], q * C, a);
}

// Low-resolution form, second pass, for a low-resolution grid no finer than
// the map (lH <= fH, lW <= fW): a workgroup takes a segment of 256 / (C/8)
// pixels of one map row, one thread per (pixel, 8 channels).  Bilinear
// interpolation is separable: the workgroup first blends the two low-res
// rows its map row falls between into LDS (the segment spans at most
// 256 / (C/8) + 2 low-res columns), then every thread interpolates between
// two LDS columns and adds the result to its feature.  P is a few MB and
// stays in L2; the feature maps are read and written once.
template <int C, bool BF16>
__global__ void __launch_bounds__(256) k_ray_upsample_add(const RayParams p) {
    constexpr int NC = C / 8, SEG = 256 / NC, MAXCOL = SEG + 3;
    __shared__ float4 rowb[MAXCOL * C / 4];      // blended low-res row segment [col][C]
    const int m = blockIdx.z;
    const int fw = p.fW[m], fh = p.fH[m];
    const int y = blockIdx.y, xs = blockIdx.x * SEG;
    if (y >= fh || xs >= fw) return;             // uniform over the workgroup
    const int lh = p.lH, lw = p.lW;
    const float ry = (float)lh / (float)fh, rx = (float)lw / (float)fw;
    const float sy = fmaxf(((float)y + 0.5f) * ry - 0.5f, 0.0f);
    const int y0 = min((int)sy, lh - 1), y1 = min(y0 + 1, lh - 1);
    const float ly = sy - (float)y0;
    const int xe = min(xs + SEG, fw) - 1;
    const int cx_lo = min((int)fmaxf(((float)xs + 0.5f) * rx - 0.5f, 0.0f), lw - 1);
    const int cx_hi = min(min((int)fmaxf(((float)xe + 0.5f) * rx - 0.5f, 0.0f), lw - 1) + 1, lw - 1);
    const int ncol = cx_hi - cx_lo + 1;          // <= SEG + 2 when lW <= fW
    const float4 *P0 = reinterpret_cast<const float4 *>(p.P + (((int64_t)m * lh + y0) * lw + cx_lo) * C);
    const float4 *P1 = reinterpret_cast<const float4 *>(p.P + (((int64_t)m * lh + y1) * lw + cx_lo) * C);
    for (int k = threadIdx.x; k < ncol * (C / 4); k += 256) {
        const float4 a = P0[k], b = P1[k];
        rowb[k] = make_float4(fmaf(ly, b.x - a.x, a.x), fmaf(ly, b.y - a.y, a.y),
                              fmaf(ly, b.z - a.z, a.z), fmaf(ly, b.w - a.w, a.w));
    }
    __syncthreads();
    const int x = xs + threadIdx.x / NC, c0 = 8 * (threadIdx.x % NC);
    if (x > xe) return;
    const float sx = fmaxf(((float)x + 0.5f) * rx - 0.5f, 0.0f);
    const int x0 = min((int)sx, lw - 1), x1 = min(x0 + 1, lw - 1);
    const float lx = sx - (float)x0;
    const float *R = reinterpret_cast<const float *>(rowb);
    float t0[8], t1[8], a[8];
    load8<false>(R, (x0 - cx_lo) * C + c0, t0);
    load8<false>(R, (x1 - cx_lo) * C + c0, t1);
    const int64_t q = (int64_t)y * fw + x;
    load8<BF16>(p.src[m], q * C + c0, a);
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] += fmaf(lx, t1[j] - t0[j], t0[j]);
    store8<BF16>(p.feat[m], q * C + c0, a);
}

// The same for any low-resolution grid (also one finer than the map): one
// thread per (map pixel, 8 channels) reads the four taps of P directly.
template <int C, bool BF16>
__global__ void __launch_bounds__(256) k_ray_upsample_add_any(const RayParams p) {
    constexpr int NC = C / 8;
    const int m = blockIdx.y;
    const int fw = p.fW[m], fh = p.fH[m];
    const int64_t np = (int64_t)fh * fw;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= np * NC) return;
    const int64_t q = i / NC;
    const int c0 = 8 * (int)(i - q * NC);
    const int y = (int)(q / fw), x = (int)(q - (int64_t)y * fw);
    const int lh = p.lH, lw = p.lW;
    const float sy = fmaxf(((float)y + 0.5f) * ((float)lh / (float)fh) - 0.5f, 0.0f);
    const float sx = fmaxf(((float)x + 0.5f) * ((float)lw / (float)fw) - 0.5f, 0.0f);
    const int y0 = min((int)sy, lh - 1), x0 = min((int)sx, lw - 1);
    const int y1 = min(y0 + 1, lh - 1), x1 = min(x0 + 1, lw - 1);
    const float ly = sy - (float)y0, lx = sx - (float)x0;
    const float *Pm = p.P + (int64_t)m * lh * lw * C + c0;
    float t00[8], t10[8], t01[8], t11[8], a[8];
    load8<false>(Pm, ((int64_t)y0 * lw + x0) * C, t00);
    load8<false>(Pm, ((int64_t)y0 * lw + x1) * C, t10);
    load8<false>(Pm, ((int64_t)y1 * lw + x0) * C, t01);
    load8<false>(Pm, ((int64_t)y1 * lw + x1) * C, t11);
    load8<BF16>(p.src[m], q * C + c0, a);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float top = fmaf(lx, t10[j] - t00[j], t00[j]);
        const float bot = fmaf(lx, t11[j] - t01[j], t01[j]);
        a[j] += fmaf(ly, bot - top, top);
    }
    store8<BF16>(p.feat[m], q * C + c0, a);
}

// Blocks of k_ray_encoding per view: 128 pixels each, up to 8 waves per SIMD in
// all, then more pixels per wave
inline unsigned encoding_blocks(int64_t pixels, unsigned V) {
    const int64_t all = (pixels + 127) / 128, most = (2048 + V - 1) / V;
    return (unsigned)(all < most ? all : most);
}

// The encoding of a grid of `pixels` in each view.  8 channels, and 16 of a bfloat16
// map, take a pixel per thread from where that is the faster, us against the matrix
// cores: 8 views of 90x160, 135x240, 360x640 and 1080x1920, 8 channels: 4.8 / 5.9, 6.7
// / 9.8, 31 / 49, 228 / 400 (a low-resolution grid of 90x120 8.6 / 8.6, 135x240 16.3 /
// 18.3); 16 in bfloat16: 6.3 / 6.1, 9.3 / 9.9, 41 / 49, 348 / 448.  2 views of 90x160: 4.4 /
// 3.5 and 5.8 / 3.4.  16 in float32 never: 506 / 478 at the largest, 5.6 / 3.5 there.
template <int C, bool LOW, bool BF16>
void launch_encoding(const RayParams &p, int64_t pixels, unsigned V, hipStream_t s) {
    if constexpr (C == 8 || (C == 16 && BF16)) {
        constexpr int64_t kFrom = C == 16 ? 200000 : LOW ? 86000 : 75000;
        if (pixels * V >= kFrom) {
            hipLaunchKernelGGL((k_ray_pixels<C, LOW, BF16>), dim3((unsigned)((pixels + 255) / 256), V), dim3(256), 0, s, p);
            return;
        }
    }
    hipLaunchKernelGGL((k_ray_encoding<C, LOW, BF16>), dim3(encoding_blocks(pixels, V), V), dim3(256), 0, s, p);
}

template <int C>
hipError_t launch_c(const RayParams &p, hipStream_t s) {
    const unsigned V = (unsigned)p.V;
    bool same = p.lH > 0;                        // low grid == every map grid: nothing to upsample
    for (int m = 0; m < p.V; ++m) same = same && p.lH == p.fH[m] && p.lW == p.fW[m];
    if (p.lH > 0 && !same) {
        launch_encoding<C, true, false>(p, (int64_t)p.lH * p.lW, V, s);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        bool coarse = true;                      // the grid is no finer than any map
        int maxh = 0, maxw = 0;
        for (int m = 0; m < p.V; ++m) {
            coarse = coarse && p.lH <= p.fH[m] && p.lW <= p.fW[m];
            maxh = p.fH[m] > maxh ? p.fH[m] : maxh;
            maxw = p.fW[m] > maxw ? p.fW[m] : maxw;
        }
        if (coarse) {
            constexpr int SEG = 256 / (C / 8);
            const dim3 g((unsigned)((maxw + SEG - 1) / SEG), (unsigned)maxh, V);
            if (p.bf16)
                hipLaunchKernelGGL((k_ray_upsample_add<C, true>), g, dim3(256), 0, s, p);
            else
                hipLaunchKernelGGL((k_ray_upsample_add<C, false>), g, dim3(256), 0, s, p);
        } else {
            const dim3 g((unsigned)((p.max_pixels * (C / 8) + 255) / 256), V);
            if (p.bf16)
                hipLaunchKernelGGL((k_ray_upsample_add_any<C, true>), g, dim3(256), 0, s, p);
            else
                hipLaunchKernelGGL((k_ray_upsample_add_any<C, false>), g, dim3(256), 0, s, p);
        }
        return hipGetLastError();
    }
    if (p.bf16) launch_encoding<C, false, true>(p, p.max_pixels, V, s);
    else launch_encoding<C, false, false>(p, p.max_pixels, V, s);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ray_encoding(const RayParams &p, hipStream_t s) {
    switch (p.C) {
        case 8: return launch_c<8>(p, s);
        case 16: return launch_c<16>(p, s);
        case 32: return launch_c<32>(p, s);
        case 64: return launch_c<64>(p, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qk
