// k_backward.hip -- adjoint of the float32 Update & Fuse step and of the
// front-to-back composite (gfx950).
//
// The paper trains through generic differentiable rendering and prints no
// adjoint; this one is derived by the chain rule from the forward of
// Sec. 3.1-3.3 (reprojection, bilinear back-projection, attention across
// views, decode heads, over composite).  Nothing is taped: each layer-pixel
// re-gathers its samples and recomputes its attention, so the extra memory
// is 16 bytes per layer-pixel, per-workgroup weight-gradient partials and, for
// the sorted scatter, the samples' gradients.
//
// On the caller's stream:
//   k_zero_maps         clear the feature-map gradients (atomics' targets; the
//                       sorted scatter writes every pixel)
//   k_composite_adjoint one thread per pixel: for every layer, the gradient
//                       of rgb with respect to its colour and alpha
//                       (dc = g T a, da = g . T (c - B_behind))
//   k_uf_backward<C>    256 / C layer-pixels per wave, persistent workgroups:
//                       forward recompute with the key folded into the query
//                       (a_m = (scale W_k q) . s_m) and the value folded out
//                       (o = (sum_m p_m s_m) W_v), then the adjoint of
//                       decode, residual, W_o, W_v, softmax, W_k, W_q and
//                       RMSNorm; a second pass over the views forms every
//                       sample's gradient ds and differentiates the sample
//                       position with respect to depth.  ds goes to the maps
//                       by float atomics (small problems) or to memory, from
//                       where records sorted by map tile are summed without
//                       atomics (k_scatter.hip).  Products and weight gradients
//                       (sums over layer-pixels of outer products) run on the
//                       matrix cores (v_mfma_f32_16x16x4_f32); each workgroup
//                       writes one partial.
//   k_reduce_wgrad      sums the partials in a fixed order (deterministic).
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "uf_params.h"
#include "vbin.h"
#include "view_order.h"

namespace qk {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

__device__ inline float sigm(float x) { return 1.0f / (1.0f + __expf(-x)); }

// ---------------------------------------------------------------------------
// Feature-map gradients start at zero: blockIdx.y is the view.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_zero_maps(const BwdParams p) {
    const int m = blockIdx.y;
    const int64_t n4 = (int64_t)p.fH[m] * p.fW[m] * p.C / 4;
    float4 *d = reinterpret_cast<float4 *>(p.dfeat[m]);
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n4;
         i += (int64_t)gridDim.x * kBlock)
        d[i] = z;
}

// ---------------------------------------------------------------------------
// Composite adjoint, one thread per pixel.  rgb = sum_l T_l a_l c_l with
// T_l = prod_{j<l} (1 - a_j).  With B_l the composite of layers l..L-1 on
// their own, d rgb / d c_l = T_l a_l and d rgb / d a_l = T_l (c_l - B_{l+1}).
// The front-to-back pass stores (c_l, T_l); the back-to-front pass replaces
// them by (g T_l a_l, g . T_l (c_l - B_{l+1})).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_composite_adjoint(const BwdParams p) {
    const int64_t npix = (int64_t)p.H * p.W;
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= npix) return;
    const int C = p.C;
    float T = 1.0f;
    for (int l = 0; l < p.L; ++l) {
        const int64_t e = (int64_t)l * npix + q;
        const float4 *f = reinterpret_cast<const float4 *>(p.F_out + e * C);
        float x0 = 0.f, x1 = 0.f, x2 = 0.f;
        for (int c4 = 0; c4 < C / 4; ++c4) {
            const float4 v = f[c4];
            const float fv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float *wc = p.W_color + (4 * c4 + i) * 3;
                x0 = fmaf(fv[i], wc[0], x0);
                x1 = fmaf(fv[i], wc[1], x1);
                x2 = fmaf(fv[i], wc[2], x2);
            }
        }
        reinterpret_cast<float4 *>(p.comp)[e] = make_float4(sigm(x0), sigm(x1), sigm(x2), T);
        T *= 1.0f - p.alpha_out[e];
    }
    const float g0 = p.d_rgb[q * 3 + 0], g1 = p.d_rgb[q * 3 + 1], g2 = p.d_rgb[q * 3 + 2];
    float B0 = 0.f, B1 = 0.f, B2 = 0.f;
    for (int l = p.L - 1; l >= 0; --l) {
        const int64_t e = (int64_t)l * npix + q;
        const float4 ct = reinterpret_cast<const float4 *>(p.comp)[e];
        const float a = p.alpha_out[e];
        const float Ta = ct.w * a;
        const float da = ct.w * (g0 * (ct.x - B0) + g1 * (ct.y - B1) + g2 * (ct.z - B2));
        reinterpret_cast<float4 *>(p.comp)[e] = make_float4(g0 * Ta, g1 * Ta, g2 * Ta, da);
        B0 = fmaf(a, ct.x - B0, B0);
        B1 = fmaf(a, ct.y - B1, B1);
        B2 = fmaf(a, ct.z - B2, B2);
    }
}

// ---------------------------------------------------------------------------
// Standalone composite adjoint (the operator O on its own), one thread per
// pixel: d rgb / d c_l = T_l a_l, d rgb / d a_l = T_l (c_l - B_{l+1}) and
// d acc / d a_l = T_l P_{l+1}, with B_{l+1} the composite of the layers
// behind l and P_{l+1} the product of their (1 - a).  The front-to-back
// pass parks T_l in d_alpha (each thread touches only its own pixel); the
// back-to-front pass accumulates B and P and overwrites it.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_composite_backward(const CompBwdParams p) {
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= p.npix) return;
    float T = 1.0f;
    for (int l = 0; l < p.L; ++l) {
        const int64_t e = (int64_t)l * p.npix + q;
        p.d_alpha[e] = T;
        T *= 1.0f - p.alpha[e];
    }
    const float g0 = p.d_rgb[q * 3 + 0], g1 = p.d_rgb[q * 3 + 1], g2 = p.d_rgb[q * 3 + 2];
    const float gA = p.d_acc != nullptr ? p.d_acc[q] : 0.0f;
    float B0 = 0.f, B1 = 0.f, B2 = 0.f, P = 1.0f;
    for (int l = p.L - 1; l >= 0; --l) {
        const int64_t e = (int64_t)l * p.npix + q;
        const float Tl = p.d_alpha[e];
        const float a = p.alpha[e];
        const float c0 = p.color[e * 3 + 0], c1 = p.color[e * 3 + 1], c2 = p.color[e * 3 + 2];
        if (p.d_color != nullptr) {
            const float Ta = Tl * a;
            p.d_color[e * 3 + 0] = g0 * Ta;
            p.d_color[e * 3 + 1] = g1 * Ta;
            p.d_color[e * 3 + 2] = g2 * Ta;
        }
        p.d_alpha[e] = Tl * (g0 * (c0 - B0) + g1 * (c1 - B1) + g2 * (c2 - B2) + gA * P);
        B0 = fmaf(a, c0 - B0, B0);
        B1 = fmaf(a, c1 - B1, B1);
        B2 = fmaf(a, c2 - B2, B2);
        P *= 1.0f - a;
    }
}

// ---------------------------------------------------------------------------
// The per-layer-pixel kernel.  A wave takes PPT = 256 / C layer-pixels of one
// layer at a time and holds their C-vectors in one of two layouts, four floats
// per lane (C = 8: per lane and tile) each:
//
//   matrix layout   tile t of 16 pixels, lane (n, g) = (l % 16, l / 16): channels
//                   4g .. 4g+3 of pixel 16 t + n -- the result rows of
//                   v_mfma_f32_16x16x4_f32.  With the K slots taken in the
//                   order 4g + s at step s it is the B operand as well, so
//                   products chain without moving data (the weights, the A
//                   operand, are read to match).  C = 8 leaves the lanes of
//                   channels 8..15 at zero.
//   load layout     LPP = C / 4 adjacent lanes per pixel: 16-byte chunks of a
//                   tap's channels, which the texture path serves together.
//                   A pixel's dot products are sums over its lanes (DPP);
//                   each lane projects the pixel into a view of its own, LPP
//                   views at a time.
//
// Vectors cross between the two (and to one lane per pixel, for the decode)
// through the wave's own LDS rows; no barrier is needed for a slice that one
// wave writes and reads in order.
// ---------------------------------------------------------------------------
// 1 / x in double to its last bits: recip_d and a second Newton step
__device__ inline double recip2_d(double x) {
    const double r = recip_d(x);
    return fma(r, fma(-x, r, 1.0), r);
}
// 1 / x and 1 / sqrt(x) to within a hair of half a unit in the last place: the
// hardware estimate and a Newton step, for x of ordinary size.  (The estimates
// alone, about 1 ulp each, showed in the gradients' errors.)
__device__ inline float rcp1(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}
__device__ inline float rsq1(float x) {
    const float r = __builtin_amdgcn_rsqf(x);
    return fmaf(0.5f * r, fmaf(-x * r, r, 1.0f), r);
}
// sigma'(x) = sigma(x) sigma(-x): no cancellation when sigma(x) is near one.  (As e /
// (1 + e)^2 with one exponential its error showed in dLoss/dF.)  Beyond 80, where
// it is below 2e-35, held there: the estimates' step takes no infinity.
__device__ inline float dsigm(float x) {
    const float y = fabsf(x) > 80.0f ? 80.0f : x;
    return rcp1(1.0f + __expf(-y)) * rcp1(1.0f + __expf(y));
}

constexpr int kTapOob = (int)0x80000000; // past any map under 2 GiB

template <int CTRL>
__device__ inline float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// value of lane K of the pixel's LPP lanes
template <int LPP, int K>
__device__ inline int pix_bcast(int v) {
    constexpr int ctrl = LPP == 4 ? K * 0x55 : (K == 0 ? 0xA0 : 0xF5);
    return __builtin_amdgcn_update_dpp(0, v, ctrl, 0xf, 0xf, true);
}
template <int LPP, int K>
__device__ inline float pix_bcast(float v) {
    return __int_as_float(pix_bcast<LPP, K>(__float_as_int(v)));
}
// sum over the pixel's lanes
template <int LPP>
__device__ inline float pix_sum(float v) {
    v += dpp_f<0xB1>(v);                          // lanes 1, 0, 3, 2
    if constexpr (LPP == 4) v += dpp_f<0x4E>(v);  // lanes 2, 3, 0, 1
    return v;
}
// sum over a pixel's rows in the matrix layout (all four lane rows; for C = 8
// the upper two hold zeros)
__device__ inline float row_sum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float p = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(p), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// One layer-pixel in one view: the four taps' byte offsets in the map (in
// 16-byte units in the WIDE form), kTapOob (-1) where outside it, their
// bilinear weights, the fractions and d(position) / d(depth).
struct ViewProj {
    int o[4];
    float fx, fy, dx, dy;
};

template <int C, bool WIDE>
__device__ __forceinline__ void project(const double *A, int fw, int fh, double uc, double vc, double invd,
                               bool live, ViewProj &P) {
    constexpr int U = WIDE ? C / 4 : C * 4;       // one pixel of the map
    constexpr int OUT = WIDE ? -1 : kTapOob;
    const double pz = fma(A[6], uc, fma(A[7], vc, fma(A[11], invd, A[8])));
    const double qx = fma(A[0], uc, fma(A[1], vc, fma(A[9], invd, A[2])));
    const double qy = fma(A[3], uc, fma(A[4], vc, fma(A[10], invd, A[5])));
    const double rz = recip2_d(pz);
    const double X = qx * rz - 0.5, Y = qy * rz - 0.5;
    const bool ok = live && (pz > 1e-6) && (fabs(X) < 1e7) && (fabs(Y) < 1e7);
    // d p / d d = -b / d^2;  d(q / pz) / d d = (dq pz - q dpz) / pz^2
    const double k = ok ? invd * invd * rz * rz : 0.0;
    P.dx = ok ? (float)((qx * A[11] - A[9] * pz) * k) : 0.0f;
    P.dy = ok ? (float)((qy * A[11] - A[10] * pz) * k) : 0.0f;
    const double xf = floor(X), yf = floor(Y);
    P.fx = ok ? (float)(X - xf) : 0.0f;
    P.fy = ok ? (float)(Y - yf) : 0.0f;
    const int ix = ok ? (int)xf : -4, iy = ok ? (int)yf : -4;
    const bool vx0 = (unsigned)ix < (unsigned)fw, vx1 = (unsigned)(ix + 1) < (unsigned)fw;
    const bool vy0 = (unsigned)iy < (unsigned)fh, vy1 = (unsigned)(iy + 1) < (unsigned)fh;
    const int o = (iy * fw + ix) * U;
    P.o[0] = (vx0 && vy0) ? o : OUT;
    P.o[1] = (vx1 && vy0) ? o + U : OUT;
    P.o[2] = (vx0 && vy1) ? o + fw * U : OUT;
    P.o[3] = (vx1 && vy1) ? o + fw * U + U : OUT;
}

// One view's taps of the lane's channels, as loaded, and the projection.
struct Taps {
    float4 t[4];
    ViewProj p;
};

template <int C, bool WIDE, int K>
__device__ __forceinline__ void issue_taps(const BwdParams &p, int m, const ViewProj &mine, int chunk, Taps &T) {
    constexpr int LPP = C / 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) T.p.o[j] = pix_bcast<LPP, K>(mine.o[j]);
    T.p.fx = pix_bcast<LPP, K>(mine.fx);
    T.p.fy = pix_bcast<LPP, K>(mine.fy);
    T.p.dx = pix_bcast<LPP, K>(mine.dx);
    T.p.dy = pix_bcast<LPP, K>(mine.dy);
    if constexpr (WIDE) {
        const float4 *f = reinterpret_cast<const float4 *>(p.feat[m]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            T.t[j] = T.p.o[j] >= 0 ? f[T.p.o[j] + chunk] : make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        // a load past the map's bytes returns zeros
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(p.feat[m]), 0, p.fH[m] * p.fW[m] * C * 4, 0x00020000);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const auto a = __builtin_amdgcn_raw_buffer_load_b128(r, T.p.o[j] + 16 * chunk, 0, 0);
            T.t[j] = make_float4(__uint_as_float(a[0]), __uint_as_float(a[1]), __uint_as_float(a[2]),
                                 __uint_as_float(a[3]));
        }
    }
}

__device__ inline float4 blend(const Taps &T) {
    const float fx = T.p.fx, fy = T.p.fy;
    const float w00 = (1.f - fx) * (1.f - fy), w10 = fx * (1.f - fy);
    const float w01 = (1.f - fx) * fy, w11 = fx * fy;
    float4 s;
    s.x = fmaf(w00, T.t[0].x, fmaf(w10, T.t[1].x, fmaf(w01, T.t[2].x, w11 * T.t[3].x)));
    s.y = fmaf(w00, T.t[0].y, fmaf(w10, T.t[1].y, fmaf(w01, T.t[2].y, w11 * T.t[3].y)));
    s.z = fmaf(w00, T.t[0].z, fmaf(w10, T.t[1].z, fmaf(w01, T.t[2].z, w11 * T.t[3].z)));
    s.w = fmaf(w00, T.t[0].w, fmaf(w10, T.t[1].w, fmaf(w01, T.t[2].w, w11 * T.t[3].w)));
    return s;
}

__device__ inline float dot4(const float4 &a, const float4 &b) {
    return fmaf(a.x, b.x, fmaf(a.y, b.y, fmaf(a.z, b.z, a.w * b.w)));
}

// The weight matrices in LDS, each 16 x 16 row-major, zero beyond C; H the
// decode heads' (sigma, depth, r, g, b).  As the A operand of a product lane
// (m, g) takes elements [4g .. 4g+3][m] (y = x W) or, transposed, [m][4g ..
// 4g+3] (y = W x).
enum { kMatQ, kMatK, kMatV, kMatO, kMatH, kNumMat };

template <int C>
__device__ __forceinline__ float mat_element(const BwdParams &p, int w, int in, int out) {
    if (in >= C) return 0.0f;
    if (w == kMatH)
        return out == 0 ? p.w_sigma[in] : out == 1 ? p.w_depth[in]
             : out < 5 ? p.W_color[in * 3 + out - 2] : 0.0f;
    if (out >= C) return 0.0f;
    const float *W = w == kMatQ ? p.Wq : w == kMatK ? p.Wk : w == kMatV ? p.Wv : p.Wo;
    return W[in * C + out];
}

// y += x W, or y += W x when TRANS, for the wave's vectors (matrix layout)
template <bool TRANS, int MT>
__device__ __forceinline__ void product(const float *W, int n, int g, const f32x4 (&x)[MT], f32x4 (&y)[MT]) {
    f32x4 a;
    if constexpr (TRANS) a = *reinterpret_cast<const f32x4 *>(W + 16 * n + 4 * g);
    else
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = W[16 * (4 * g + i) + n];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < MT; ++t) y[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], x[t][i], y[t], 0, 0, 0);
}

template <int MT>
__device__ __forceinline__ void zero4(f32x4 (&y)[MT]) {
#pragma unroll
    for (int t = 0; t < MT; ++t) y[t] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Orders the wave's LDS accesses before and after it (no instruction: a wave's
// LDS accesses complete in order)
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// A wave's pixel rows in LDS: C channels, then four scalars (d depth so far,
// softmax reference, 1 / normaliser, ob . dob).
template <int C>
constexpr int kRow = C + 4;

// matrix layout <-> rows (lanes of channels past C: not stored, zero)
template <int C, int MT>
__device__ __forceinline__ void rows_store(float *rows, int n, int g, const f32x4 (&x)[MT]) {
    if (C < 16 && 4 * g >= C) return;
#pragma unroll
    for (int t = 0; t < MT; ++t) *reinterpret_cast<f32x4 *>(rows + (16 * t + n) * kRow<C> + 4 * g) = x[t];
}
template <int C, int MT>
__device__ __forceinline__ void rows_load(const float *rows, int n, int g, f32x4 (&x)[MT]) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        x[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (C == 16 || 4 * g < C) x[t] = *reinterpret_cast<const f32x4 *>(rows + (16 * t + n) * kRow<C> + 4 * g);
    }
}

// acc += sum over the wave's pixels of a (x) b, from their rows (pixels along
// K: lane (c, k) feeds element c of pixel 4 s + k at step s; for C = 8
// elements 8..15 hold what lies there and reach only entries never read)
template <int C>
__device__ __forceinline__ void outer_rows(const float *a, const float *b, int n, int g, f32x4 &acc) {
    const int c = C < 16 ? n & (C - 1) : n;
#pragma unroll
    for (int s = 0; s < 64 / C; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[(4 * s + g) * kRow<C> + c],
                                                   b[(4 * s + g) * kRow<C> + c], acc, 0, 0, 0);
}

// How the samples' gradients reach the maps: float atomics (32-bit byte
// offsets, or for maps of 2 GiB and more 64-bit addresses), or rows of ds in
// memory for the sorted scatter -- with up to kKeep views the taps of the first
// pass are kept in registers for the second.
enum { kNarrow, kWide, kSort, kSortKeep };
constexpr int kKeep = kBwdKeep;

// What bounds it (960x540, L = 8, C = 16, V = 4, i.i.d. depths).  The float
// atomics alone take 3.5 ms: they execute at the memory side, ~19 rows of C
// floats per ns however they are grouped, so from kScatterMin on the gradients
// go through the sort (0.69 ms with its binning, k_scatter.hip).  What is left
// was, with a pixel per lane, 2.1 ms of 64-line gathers, LDS reads of the weights
// and 4700 vector instructions per 64 pixels; quads of lanes per tap row, the
// products on the matrix cores and 16 pixels at a time (few enough registers to
// keep the taps of four views for the second pass, at two waves per SIMD) leave
// 0.96 ms: the texture data path is busy 77 % of it, the vector units 45 and the
// matrix cores 21, and two waves hide no more (gathering again at three 1.10 ms,
// four waves spill).  The whole adjoint 4.0 -> 1.77 ms.
template <int C, int MODE>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(MODE == kSortKeep ? kBwdWavesKeep : kBwdWaves)))
k_uf_backward(const BwdParams p) {
    static_assert(C == 8 || C == 16, "the backward kernel holds C <= 16 channels per pixel");
    constexpr bool WIDE = MODE == kWide, SORT = MODE >= kSort, KEEP = MODE == kSortKeep;
    constexpr int LPP = C / 4;                    // lanes per pixel in the load layout
    constexpr int PPT = 64 / LPP;                 // pixels of a wave
    constexpr int MT = PPT / 16;                  // their tiles in the matrix layout
    constexpr int ROW = kRow<C>;
    __shared__ __attribute__((aligned(16))) float s_a[kWaves][PPT * ROW > 256 ? PPT * ROW : 256];
    __shared__ __attribute__((aligned(16))) float s_b[kWaves][PPT * ROW];
    __shared__ int2 s_ow[SORT ? 1 : kWaves][SORT ? 1 : PPT * 4];   // one view's tap offsets and weights
    __shared__ __attribute__((aligned(16))) float s_w[kNumMat][256];
    __shared__ double s_cam[kMaxViews * 12];
    __shared__ int2 s_wh[kMaxViews];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;       // matrix layout
    const int chunk = lane % LPP, lp = lane / LPP;   // load layout
    float *A = s_a[wave], *B = s_b[wave];
    int2 *Sow = s_ow[SORT ? 0 : wave];

    for (int i = threadIdx.x; i < kNumMat * 256; i += kBlock)
        s_w[i >> 8][i & 255] = mat_element<C>(p, i >> 8, (i >> 4) & 15, i & 15);
    for (int i = threadIdx.x; i < p.V * 12; i += kBlock) s_cam[i] = p.camd[i / 12][i % 12];
    for (int i = threadIdx.x; i < p.V; i += kBlock) s_wh[i] = make_int2(p.fW[i], p.fH[i]);
    __syncthreads();

    f32x4 gQ = {0.f, 0.f, 0.f, 0.f}, gK = gQ, gV = gQ, gO = gQ, gH = gQ;
    const float half_l = 0.5f / (float)p.L;
    const float band = p.inv_near - p.inv_far;
    const float kap = half_l * band;
    const bool has_ch = 4 * g < C;                // this lane's channels exist

    // A wave's pixels lie in one layer; the items run through the layers of
    // PPT pixels before the next PPT, and each XCD (workgroups are dispatched
    // round-robin over the 8) takes one contiguous range of them, so the rows of
    // the maps that a band of pixels samples stay in its L2.
    const int32_t npix = p.H * p.W, items = p.L * ((npix + PPT - 1) / PPT);
    const int nr = min(8, (int)gridDim.x), r = (int)blockIdx.x % nr;
    const int32_t item_end = (int32_t)((int64_t)items * (r + 1) / nr);
    const int32_t item_step = ((int)gridDim.x - r + nr - 1) / nr * kWaves;
    const int32_t item_first = (int32_t)((int64_t)items * r / nr), item_half = item_first + (item_end - item_first) / 2;
    const int32_t item0 = item_first + (int)blockIdx.x / nr * kWaves + wave;
    // the depth of this lane's pixel (load layout) of an item, read one item
    // ahead: the projections wait on it, and the taps on them
    auto item_depth = [&](int32_t item) {
        const int32_t q0 = (int32_t)fast_div((uint32_t)item, p.div_l), li = item - q0 * p.L;
        return p.depth_in[min(li * npix + q0 * PPT + lp, (li + 1) * npix - 1)];
    };
    float depth_next = item0 < item_end ? item_depth(item0) : 1.0f;
    int32_t item = item0;
#pragma unroll 1
    for (int part = 0; part < p.parts; ++part) {
    const int32_t part_end = part + 1 < p.parts ? item_half : item_end;
    for (; item < part_end; item += item_step) {
        const float depth_ld = depth_next;
        if (item + item_step < item_end) depth_next = item_depth(item + item_step);
        const int32_t q0 = (int32_t)fast_div((uint32_t)item, p.div_l), li = item - q0 * p.L;
        const int32_t base = li * npix + q0 * PPT, N = (li + 1) * npix;
        const bool full = N - base >= PPT;        // no pixel past the layer's end
        // vectors of this wave's pixels in memory (matrix layout); pixels past
        // the layer's end read its last one and count as zero
        auto load_vec = [&](const float *src, f32x4 (&x)[MT]) {
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const int32_t e = min(base + 16 * t + n, N - 1);
                x[t] = has_ch ? *reinterpret_cast<const f32x4 *>(src + (int64_t)e * C + 4 * g)
                              : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        };
        // rows of a vector, zero for pixels past the end
        auto rows_live = [&](float *rows, f32x4 (&x)[MT]) {
            if (!full) {
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    if (base + 16 * t + n >= N) x[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            rows_store<C>(rows, n, g, x);
        };

        // ---- the pixel of this lane in the load layout, and its first views'
        //      projections
        const int32_t e_ld = base + lp;
        const bool live_ld = e_ld < N;
        const uint32_t ec_ld = (uint32_t)(live_ld ? e_ld : N - 1);
        const uint32_t rem = ec_ld - (uint32_t)(li * npix), yy = fast_div(rem, p.div_w);
        const double uc = (double)(rem - yy * p.div_w.d) + 0.5, vc = (double)yy + 0.5;
        const double invd = recip2_d((double)depth_ld);
        ViewProj mine;
        auto proj = [&](int m0) {
            const int m = min(m0 + chunk, p.V - 1);
            const int2 wh = s_wh[m];
            project<C, WIDE>(s_cam + 12 * m, wh.x, wh.y, uc, vc, invd, live_ld, mine);
        };
        // the views in order: all in flight and kept (up to kKeep), or the taps
        // of the next view in flight behind the current one
        Taps kept[KEEP ? kKeep : 1];
        if constexpr (KEEP) {
            static_for<0, kKeep>([&](auto kk) {
                constexpr int k = decltype(kk)::value;
                if (k < p.V) {
                    if constexpr (k % LPP == 0) proj(k);
                    issue_taps<C, WIDE, k % LPP>(p, k, mine, chunk, kept[k]);
                }
            });
        }
        auto run_views = [&](auto &&step) {
            if constexpr (KEEP) {
                static_for<0, kKeep>([&](auto kk) {
                    constexpr int k = decltype(kk)::value;
                    if (k < p.V) step(kept[k], k);
                });
            } else {
                Taps buf[2];
                views_in_order<LPP>(
                    p.V, proj,
                    [&](auto kk, int m, auto slot) {
                        issue_taps<C, WIDE, decltype(kk)::value>(p, m, mine, chunk, buf[decltype(slot)::value]);
                    },
                    [&](int m, auto slot) {
                        __builtin_amdgcn_sched_barrier(0);
                        step(buf[decltype(slot)::value], m);
                        __builtin_amdgcn_sched_barrier(0);
                    });
            }
        };

        // ---- query folded with the key: q~ = scale W_k (N(F) W_q)
        f32x4 f[MT], q[MT];
        float ir[MT];                             // 1 / RMS
        load_vec(p.F_in, f);
        // what the decode will need (one lane per pixel), read now
        const int32_t e_px = base + lane, ec_px = min(e_px, N - 1);
        float4 cg = make_float4(0.f, 0.f, 0.f, 0.f);          // dLoss/d(colour, alpha)
        float ddn = 0.f, d_px = 1.f, a_px = 0.5f;
        if (lane < PPT) {
            if (p.comp) cg = reinterpret_cast<const float4 *>(p.comp)[ec_px];
            if (p.d_alpha_out) cg.w += p.d_alpha_out[ec_px];
            if (p.d_depth_out) ddn = p.d_depth_out[ec_px];
            d_px = p.depth_in[ec_px];
            a_px = p.alpha_in[ec_px];
        }
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const float ss = row_sum(fmaf(f[t][0], f[t][0], fmaf(f[t][1], f[t][1],
                                     fmaf(f[t][2], f[t][2], f[t][3] * f[t][3]))));
            ir[t] = rsq1(ss * (1.0f / (float)C) + 1e-6f);
        }
        auto normalised = [&](f32x4 (&x)[MT]) {
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) x[t][i] = f[t][i] * ir[t];
        };
        {
            f32x4 x[MT], y[MT];
            normalised(x);
            zero4(q);
            product<false>(s_w[kMatQ], n, g, x, q);
            zero4(y);
            product<true>(s_w[kMatK], n, g, q, y);
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) y[t][i] *= p.scale;
            wave_order();
            rows_store<C>(B, n, g, y);
            wave_order();
        }
        float *row_ld = A + lp * ROW;
        const float4 qv = *reinterpret_cast<const float4 *>(B + lp * ROW + 4 * chunk);

        // ---- pass 1 over the views: online softmax of a_m = q~ . s_m and
        //      ob = sum_m p_m s_m.  The weights are exp(a_m - mx) for a
        //      reference mx moved only when a logit passes it by more than 8
        //      (always at the first view), as in the forward kernel; pass 2
        //      uses the same reference.
        float mx = -1e30f, iz, logit[KEEP ? kKeep : 1];
        {
            float z = 0.f;
            float4 ob = make_float4(0.f, 0.f, 0.f, 0.f);
            run_views([&](const Taps &T, int m) {
                const float4 s = blend(T);
                const float a = pix_sum<LPP>(dot4(qv, s));
                if constexpr (KEEP) logit[m] = a;
                float diff = a - mx;
                if (diff > 8.0f) {
                    const float rr = __expf(-diff);
                    z *= rr;
                    ob.x *= rr; ob.y *= rr; ob.z *= rr; ob.w *= rr;
                    mx = a;
                    diff = 0.0f;
                }
                const float pw = __expf(diff);
                z += pw;
                ob.x = fmaf(pw, s.x, ob.x);
                ob.y = fmaf(pw, s.y, ob.y);
                ob.z = fmaf(pw, s.z, ob.z);
                ob.w = fmaf(pw, s.w, ob.w);
            });
            iz = rcp1(z);
            *reinterpret_cast<float4 *>(row_ld + 4 * chunk) = make_float4(ob.x * iz, ob.y * iz, ob.z * iz, ob.w * iz);
            wave_order();
        }

        // ---- o = ob W_v; F' = F + o W_o; decode and its adjoint; back
        //      through W_o and W_v to dob = W_v W_o^T dF'
        f32x4 dfp[MT];
        {
            f32x4 ob[MT], o[MT], fp[MT], x[MT];
            rows_load<C>(A, n, g, ob);
            zero4(o);
            product<false>(s_w[kMatV], n, g, ob, o);
            zero4(fp);                            // summed before f joins: fewer roundings at its size
            product<false>(s_w[kMatO], n, g, o, fp);
#pragma unroll
            for (int t = 0; t < MT; ++t) fp[t] += f[t];
            zero4(x);
            product<false>(s_w[kMatH], n, g, fp, x);
            wave_order();
            rows_store<C>(A, n, g, x);            // columns 0..4: the heads
            wave_order();
            if (lane < PPT) {
                // one lane per pixel
                const bool live = e_px < N;
                float *row = A + lane * ROW;
                const float4 x4 = *reinterpret_cast<const float4 *>(row);
                const float xs = x4.x, xd = x4.y, xc[3] = {x4.z, x4.w, row[4]};
                const float dco[3] = {cg.x, cg.y, cg.z}, dal = cg.w;
                float dd_in = 0.f, da_in = 0.f;
                float h[5];                       // d x_sigma, d x_depth, d x_color
#pragma unroll
                for (int j = 0; j < 3; ++j) h[2 + j] = dco[j] * dsigm(xc[j]);
                const float th = tanhf(xd), dth = fmaf(-th, th, 1.0f);
                if (p.mode == 0) {
                    const float a_in = a_px, ac = fminf(fmaxf(a_in, 1e-6f), 1.0f - 1e-6f);
                    h[0] = dal * dsigm(logf(ac / (1.0f - ac)) + xs);
                    if (a_in > 1e-6f && a_in < 1.0f - 1e-6f) da_in = h[0] / (a_in * (1.0f - a_in));
                    const float disp = fmaf(kap, th, 1.0f / d_px);
                    h[1] = 0.f;
                    if (disp > p.inv_far && disp < p.inv_near) {
                        const float dn = rcp1(disp);
                        const float ddisp = -ddn * dn * dn;
                        dd_in = -ddisp / (d_px * d_px);
                        h[1] = ddisp * kap * dth;
                    }
                } else {
                    h[0] = dal * dsigm(xs);
                    const float delta = ((float)(p.L - li) - 0.5f) / (float)p.L;
                    const float dn = rcp1(fmaf(delta + half_l * th, band, p.inv_far));
                    h[1] = -ddn * dn * dn * kap * dth;
                }
                if (live) p.d_alpha[e_px] = da_in;
                const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
                float4 *r4 = reinterpret_cast<float4 *>(row);
                r4[0] = live ? make_float4(h[0], h[1], h[2], h[3]) : z4;
                r4[1] = live ? make_float4(h[4], 0.f, 0.f, 0.f) : z4;
                if constexpr (C == 16) r4[2] = r4[3] = z4;
                row[C] = dd_in;
            }
            rows_live(B, fp);
            wave_order();
            outer_rows<C>(B, A, n, g, gH);
            rows_load<C>(A, n, g, x);             // h
            zero4(dfp);
            product<true>(s_w[kMatH], n, g, x, dfp);
            if (p.dF_out) {
                load_vec(p.dF_out, x);
#pragma unroll
                for (int t = 0; t < MT; ++t) dfp[t] += x[t];
            }
            f32x4 dov[MT], dob[MT];
            zero4(dov);
            product<true>(s_w[kMatO], n, g, dfp, dov);
            wave_order();
            rows_live(A, o);
            rows_live(B, dfp);
            wave_order();
            outer_rows<C>(A, B, n, g, gO);
            zero4(dob);
            product<true>(s_w[kMatV], n, g, dov, dob);
            float delta[MT];
#pragma unroll
            for (int t = 0; t < MT; ++t)
                delta[t] = row_sum(fmaf(ob[t][0], dob[t][0], fmaf(ob[t][1], dob[t][1],
                                   fmaf(ob[t][2], dob[t][2], ob[t][3] * dob[t][3]))));
            wave_order();
            rows_live(A, ob);
            rows_live(B, dov);
            wave_order();
            outer_rows<C>(A, B, n, g, gV);
            wave_order();
            rows_store<C>(A, n, g, dob);
            if (g == 0) {
#pragma unroll
                for (int t = 0; t < MT; ++t) A[(16 * t + n) * ROW + C + 1] = delta[t];
            }
            wave_order();
        }

        // ---- pass 2 over the views: softmax adjoint, dI scatter, depth
        //      through the sample position.  ds_m = p_m dob + da_m q~
        {
            const float4 dob = *reinterpret_cast<const float4 *>(row_ld + 4 * chunk);
            const float dd0 = row_ld[C], delta = row_ld[C + 1];
            float ddv = 0.f;
            float4 sh = make_float4(0.f, 0.f, 0.f, 0.f);    // sum_m da_m s_m
            run_views([&](const Taps &T, int m) {
                const float4 s = blend(T);
                const float a = KEEP ? logit[KEEP ? m : 0] : pix_sum<LPP>(dot4(qv, s));
                const float sd = pix_sum<LPP>(dot4(s, dob));
                const float pm = __expf(a - mx) * iz;
                const float da = pm * (sd - delta);
                sh.x = fmaf(da, s.x, sh.x);
                sh.y = fmaf(da, s.y, sh.y);
                sh.z = fmaf(da, s.z, sh.z);
                sh.w = fmaf(da, s.w, sh.w);
                const float4 ds = make_float4(fmaf(pm, dob.x, da * qv.x), fmaf(pm, dob.y, da * qv.y),
                                              fmaf(pm, dob.z, da * qv.z), fmaf(pm, dob.w, da * qv.w));
                const float fx = T.p.fx, fy = T.p.fy, ex = 1.f - fx, ey = 1.f - fy;
                // along x: ds . ((1 - fy)(t10 - t00) + fy (t11 - t01)), along y
                // alike.  The taps are differenced before the products: what
                // neighbouring texels have in common, nearly all of a smooth
                // map, would cancel only after it had been rounded.
                const float gX = fmaf(ey, dot4(ds, T.t[1] - T.t[0]), fy * dot4(ds, T.t[3] - T.t[2]));
                const float gY = fmaf(ex, dot4(ds, T.t[2] - T.t[0]), fx * dot4(ds, T.t[3] - T.t[1]));
                ddv = fmaf(gX, T.p.dx, fmaf(gY, T.p.dy, ddv));
                if constexpr (SORT) {                        // scattered afterwards
                    if (live_ld)
                        __builtin_nontemporal_store(f32x4{ds.x, ds.y, ds.z, ds.w}, reinterpret_cast<f32x4 *>(
                            p.ds + ((int64_t)m * p.N + e_ld) * C + 4 * chunk));
                    return;
                }
                // dI scatter: the ds rows and tap offsets to LDS, then every
                // atomic instruction covers whole rows of C floats, a pixel's
                // two taps of a row side by side
                wave_order();
                reinterpret_cast<float4 *>(B)[lane] = ds;
                if (chunk == 0) {
                    int4 *ow = reinterpret_cast<int4 *>(Sow + 4 * lp);
                    ow[0] = make_int4(T.p.o[0], __float_as_int(ex * ey), T.p.o[1], __float_as_int(fx * ey));
                    ow[1] = make_int4(T.p.o[2], __float_as_int(ex * fy), T.p.o[3], __float_as_int(fx * fy));
                }
                wave_order();
                constexpr int PPI = 64 / (2 * C);            // pixels per instruction (one tap row)
                const int c = lane % C, tx = (lane / C) & 1, pi = lane / (2 * C);
#pragma unroll
                for (int j = 0; j < PPT / PPI; ++j) {
                    const int px = PPI * j + pi;
                    const float d1 = B[px * C + c];
#pragma unroll
                    for (int ty = 0; ty < 2; ++ty) {
                        const int2 ow = Sow[4 * px + 2 * ty + tx];
                        const float val = __int_as_float(ow.y) * d1;
                        if constexpr (WIDE) {
                            if (ow.x >= 0) unsafeAtomicAdd(p.dfeat[m] + (int64_t)ow.x * 4 + c, val);
                        } else {
                            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                                p.dfeat[m], 0, p.fH[m] * p.fW[m] * C * 4, 0x00020000);
                            __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(val, rs, ow.x + 4 * c, 0, 0);
                        }
                    }
                }
            });
            wave_order();
            *reinterpret_cast<float4 *>(B + lp * ROW + 4 * chunk) = sh;
            wave_order();
            ddv = pix_sum<LPP>(ddv);
            if (chunk == 0 && live_ld) p.d_depth[e_ld] = dd0 + ddv;
        }

        // ---- dq = scale W_k^T sh; key and query weight gradients; RMSNorm
        //      adjoint dF += (dxn - xn (xn . dxn) / C) / r
        {
            f32x4 sh[MT], x[MT], dq[MT], dx[MT];
            rows_load<C>(B, n, g, sh);
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) sh[t][i] *= p.scale;
            normalised(x);
            zero4(dq);
            product<false>(s_w[kMatK], n, g, sh, dq);
            wave_order();
            rows_live(A, sh);
            rows_live(B, q);
            wave_order();
            outer_rows<C>(A, B, n, g, gK);
            zero4(dx);
            product<true>(s_w[kMatQ], n, g, dq, dx);
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const float k = row_sum(fmaf(x[t][0], dx[t][0], fmaf(x[t][1], dx[t][1],
                                        fmaf(x[t][2], dx[t][2], x[t][3] * dx[t][3])))) * (1.0f / (float)C);
#pragma unroll
                for (int i = 0; i < 4; ++i) dfp[t][i] += (dx[t][i] - x[t][i] * k) * ir[t];
                const int32_t e = base + 16 * t + n;
                if (has_ch && e < N)
                    __builtin_nontemporal_store(dfp[t], reinterpret_cast<f32x4 *>(p.dF + (int64_t)e * C + 4 * g));
            }
            wave_order();
            rows_live(A, x);
            rows_live(B, dq);
            wave_order();
            outer_rows<C>(A, B, n, g, gQ);
            wave_order();
        }
    }

    // ---- workgroup partial of every weight-gradient tile, where the items are many
    //      after each half of them: a wave's sums are float, and their roundings
    //      grow with their length.  The D layout of a 16 x 16 tile: lane l holds column l % 16, rows
    //      4 (l / 16) + i.
    __syncthreads();
    float *red = &s_a[0][0];                            // kWaves x 256 floats used
    f32x4 *acc[kGradTiles] = {&gQ, &gK, &gV, &gO, &gH};
    float *out = p.partials + ((size_t)blockIdx.x * p.parts + part) * kGradTiles * kGradTileElems;
#pragma unroll
    for (int t = 0; t < kGradTiles; ++t) {
        const int col = lane & 15, row0 = 4 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wave * 256 + (row0 + i) * 16 + col] = (*acc[t])[i];
        *acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
        {
            const int idx = threadIdx.x;               // 256 entries, one per thread
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) s += red[w * 256 + idx];
            out[t * kGradTileElems + idx] = s;
        }
        __syncthreads();
    }
    }
}

// Deterministic sum of the workgroup partials into the weight gradients.
// A block takes 16 consecutive entries of one tile; its 16 lanes per entry
// sum interleaved partials, then one lane combines the 16 sums in order.
__global__ void __launch_bounds__(kBlock) k_reduce_wgrad(const BwdParams p) {
    __shared__ double red[16][17];
    const int e16 = threadIdx.x & 15, part = threadIdx.x >> 4;
    const int gid = blockIdx.x * 16 + e16;                 // entry in [0, 5 * 256)
    const int t = gid / kGradTileElems, rc = gid % kGradTileElems;
    // eight partials asked for before the first is added (one at a time each was
    // a wait: 739 partials took 15.2 us, now 5.7), added in order
    const float *at = p.partials + (size_t)t * kGradTileElems + rc;
    constexpr size_t kStep = (size_t)kGradTiles * kGradTileElems;
    const int n = p.blocks * p.parts;
    double s = 0.0;
    int b = part;
    for (; b + 7 * 16 < n; b += 8 * 16) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = at[(b + 16 * i) * kStep];
#pragma unroll
        for (int i = 0; i < 8; ++i) s += (double)v[i];
    }
    for (; b < n; b += 16) s += (double)at[b * kStep];
    red[e16][part] = s;
    __syncthreads();
    if (part != 0) return;
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) tot += red[e16][k];
    const int row = rc / 16, col = rc % 16;
    const int C = p.C;
    float *dst = nullptr;
    switch (t) {
        case 0: if (row < C && col < C) dst = p.dWq + row * C + col; break;
        case 1: if (row < C && col < C) dst = p.dWk + row * C + col; break;
        case 2: if (row < C && col < C) dst = p.dWv + row * C + col; break;
        case 3: if (row < C && col < C) dst = p.dWo + row * C + col; break;
        default:
            if (row < C) {
                if (col == 0) dst = p.dw_sigma + row;
                else if (col == 1) dst = p.dw_depth + row;
                else if (col < 5) dst = p.dW_color + row * 3 + (col - 2);
            }
            break;
    }
    if (dst != nullptr) *dst = (float)tot;
}

}  // namespace

hipError_t launch_composite_backward(const CompBwdParams &p, hipStream_t s) {
    const int64_t blocks = (p.npix + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_composite_backward, dim3((unsigned)blocks), dim3(kBlock), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_scatter(const ViewsParams &p, const ScatterParams &sp, int C, hipStream_t s);

// The maps' tiles, the cameras and the workspace of the sorted scatter.
static void scatter_params(const BwdParams &p, ViewsParams &v, ScatterParams &sp) {
    v.V = p.V;
    v.L = p.L;
    v.H = p.H;
    v.W = p.W;
    v.N = p.N;
    v.depth = p.depth_in;
    v.tw = 1 << kVbLog2Tw;
    v.th = kScatterTh;
    while ((1 << v.log2_th) < v.th) ++v.log2_th;
    for (int m = 0; m < p.V; ++m) {
        for (int k = 0; k < 12; ++k) v.cam[m][k] = p.camd[m][k];
        v.vH[m] = p.fH[m];
        v.vW[m] = p.fW[m];
        v.ntx[m] = (p.fW[m] + v.tw - 1) / v.tw;
        v.nty[m] = (p.fH[m] + v.th - 1) / v.th;
        v.tbase[m + 1] = v.tbase[m] + v.ntx[m] * v.nty[m];
        sp.dfeat[m] = p.dfeat[m];
    }
    const int tiles = v.tbase[p.V];
    v.nbins = 4 * tiles;
    v.cursor = p.bins;
    v.total = p.bins + v.nbins;
    v.start = v.total + 4;
    v.rec = reinterpret_cast<int32_t *>(v.start + ((tiles + 3) & ~3));
    v.div_hw = make_fast_div((uint32_t)(p.H * p.W));
    v.div_w = make_fast_div((uint32_t)p.W);
    sp.ds = p.ds;
    const int64_t records = p.V * p.N;
    sp.listed = v.total + 1;
    sp.list = reinterpret_cast<uint2 *>(p.bins + scatter_list_at(tiles, records));
    sp.list_cap = (uint32_t)scatter_list_cap(records);
}

hipError_t launch_update_fuse_backward(const BwdParams &p, hipStream_t s) {
    if (p.C != 8 && p.C != 16) return hipErrorInvalidValue;
    hipError_t e;
    if (p.ds == nullptr) {
        int64_t zero_blocks = 1;
        for (int m = 0; m < p.V; ++m) {
            const int64_t n4 = (int64_t)p.fH[m] * p.fW[m] * p.C / 4;
            zero_blocks = std::max<int64_t>(zero_blocks, std::min<int64_t>(1024, (n4 + kBlock - 1) / kBlock));
        }
        hipLaunchKernelGGL(k_zero_maps, dim3((unsigned)zero_blocks, (unsigned)p.V), dim3(kBlock), 0, s, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (p.comp != nullptr) {
        const int64_t npix = (int64_t)p.H * p.W;
        hipLaunchKernelGGL(k_composite_adjoint, dim3((unsigned)((npix + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, s, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const dim3 g((unsigned)p.blocks), b(kBlock);
    auto main_pass = [&](auto c) {
        constexpr int C = decltype(c)::value;
        if (p.ds != nullptr && p.V <= kKeep) hipLaunchKernelGGL((k_uf_backward<C, kSortKeep>), g, b, 0, s, p);
        else if (p.ds != nullptr) hipLaunchKernelGGL((k_uf_backward<C, kSort>), g, b, 0, s, p);
        else if (p.wide) hipLaunchKernelGGL((k_uf_backward<C, kWide>), g, b, 0, s, p);
        else hipLaunchKernelGGL((k_uf_backward<C, kNarrow>), g, b, 0, s, p);
    };
    if (p.C == 8) main_pass(std::integral_constant<int, 8>{});
    else main_pass(std::integral_constant<int, 16>{});
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.ds != nullptr) {
        ViewsParams v{};
        ScatterParams sp{};
        scatter_params(p, v, sp);
        if ((e = launch_vbin(v, s)) != hipSuccess) return e;
        if ((e = launch_scatter(v, sp, p.C, s)) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_reduce_wgrad, dim3(kGradTiles * kGradTileElems / 16), dim3(kBlock), 0, s, p);
    return hipGetLastError();
}

}  // namespace qk
