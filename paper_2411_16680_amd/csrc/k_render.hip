// k_render.hip -- the final render of an LDM (Sec. 3.1, Eq. 1, and
// Sec. 3.2.3 "Upsampling & Activation"): bilinear upsampling of the
// unactivated depth, density and blend-weight logits to the output grid,
// activation after the upsampling, back-projection of every input image onto
// every layer through the decoded depth, blending of the images with the
// blend weights and the front-to-back over composite.
//
// One thread per output pixel, 16 x 16 pixel tiles (a wave covers 16 x 4), so
// the neighbouring threads that share low-resolution logit taps and, at
// similar depths, image taps sit in the same wave.  With a view count known at
// compile time each layer first reads the four taps' V blend logits in
// vectors, upsamples all of them and takes their maximum, so the per-view code
// only exponentiates; other view counts run the softmax online (running
// maximum, rescaled sums).  Neither the weights nor the per-view samples are
// stored.
//
// The vector unit bounds it (71 % busy): about 50 instructions per pixel, layer and
// view and 140 more per pixel and layer, a third of them double (a position needs
// that: a disparity is worth up to ~1e3 px), at three waves per SIMD.  So the
// layers share what does not depend on the disparity (A (u, v, 1), three
// doubles a view in registers: without it 382 us against 311), the projection
// takes positions from the image's centre on (one comparison per axis), a wave
// inside the image masks nothing, and texels enter the blend as halves
// (add_sample).  1080p from 512 x 288, 6 layers, repeated: 8 views 382 us before,
// 241 now; 5 views, which ran online, 321 and 217.  Did not help (under the profiler,
// 296 us): the logit taps in LDS (296; fewer loads, as many more instructions), a
// layer's logits read ahead (305), 128 registers for a fourth wave (305, spills), 64 x
// 4 and 32 x 8 tiles (294); beyond 8 views a loop over groups of four (12 views 333
// repeated, 361).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "uf_params.h"

namespace qk {
namespace {

// RGBA8 images are read as buffer resources: a load at a byte offset outside
// the image reads zero.  A tap outside the image is sent to kTapOOB, far past
// the end (images are under 1 GiB), never to a negative offset: the compiler
// may merge the loads of neighbouring taps or fold a constant into the
// instruction's immediate offset, and a negative register offset would then
// take a valid tap out of range with it.
constexpr int kTapOOB = 0x40000000;

// What a layer needs of a view, in the 64 bytes of one scalar load: the
// disparity's column of the projection, the image's centre hx, hy =
// floor((size - 1) / 2), its width, the image, its bytes and a row's.
struct RenderView {
    double b[3];
    double hx, hy, wd;
    const void *img;
    int bytes, pitch;
};

// The kernel's arguments (under 4 KiB): the views, with their projections taken
// to texel positions counted from the image's centre (A: the columns of x, y
// and 1) and the centre's byte offset, and the rest of RenderParams.
struct RenderArgs {
    RenderView v[kMaxViews];
    int centre[kMaxViews];
    double A[kMaxViews][9];
    const float *depth_logit, *sigma_logit, *blend_logit;
    float *rgb, *acc, *depth;
    int V, L, h, w, H, W, rows;           // rows: of a workgroup's tile
    double rx, ry, band, inv_far;
};
static_assert(sizeof(RenderArgs) < 4096, "kernel arguments");

__device__ inline __amdgpu_buffer_rsrc_t layer_rsrc(const float *p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, (int)min(bytes, (int64_t)0x7fffffff), 0x00020000);
}

__device__ inline unsigned load_texel(__amdgpu_buffer_rsrc_t r, int byte_off) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0);
}

__device__ inline float sigmoid_(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

// One view's four texels (00, 10, 01, 11) and the position between them.
struct Tex {
    unsigned a[4];
    float wx, wy;
};

// The texels around position (cx, cy), counted from the centre, of a view's
// image; texels outside it, and all of them where pz says the point is behind
// the camera, read zero.  Where the whole wave lies inside -- nearly always --
// the two texels of a row come with one load.  |cx| < hx is inside (of an image
// of even width the last column goes the general way too), and a position that
// is not a number is not; wx and wy are clamped, so that such a position's are
// numbers too (the clamp is a modifier of the conversion).
__device__ __forceinline__ void issue_texels(const RenderView &v, int centre, double cx, double cy, double pz, Tex &t) {
    const double xf = floor(cx), yf = floor(cy);
    t.wx = __builtin_amdgcn_fmed3f((float)(cx - xf), 0.0f, 1.0f);
    t.wy = __builtin_amdgcn_fmed3f((float)(cy - yf), 0.0f, 1.0f);
    asm("" : "+v"(t.wx), "+v"(t.wy));                // (now: later would hold four doubles)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(v.img), 0, v.bytes, 0x00020000);
    const bool in = pz > 1e-6 && fabs(cx) < v.hx && fabs(cy) < v.hy;
    int o = (int)((unsigned)(int)fma(yf, v.wd, xf) * 4u + (unsigned)centre);
    asm("" : "+v"(o));                               // (no branch around it)
    o = in ? o : kTapOOB;
    const auto r0 = __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0);
    const auto r1 = __builtin_amdgcn_raw_buffer_load_b64(rs, o, v.pitch, 0);
    t.a[0] = r0[0];
    t.a[1] = r0[1];
    t.a[2] = r1[0];
    t.a[3] = r1[1];
    const unsigned long long all = __builtin_amdgcn_ballot_w64(pz > 1e-6) & __builtin_amdgcn_ballot_w64(fabs(cx) < v.hx) &
                                   __builtin_amdgcn_ballot_w64(fabs(cy) < v.hy);
    if (__builtin_expect(all != __builtin_amdgcn_ballot_w64(true), 0)) {
        const double fx = cx + v.hx, fy = cy + v.hy;
        const int iw = v.pitch >> 2, ih = v.bytes / v.pitch;
        const bool ok = pz > 1e-6 && fx > -2.0 && fx < (double)(iw + 1) && fy > -2.0 && fy < (double)(ih + 1);
        const int ix = ok ? (int)(xf + v.hx) : -4, iy = ok ? (int)(yf + v.hy) : -4;
        const bool vx0 = (unsigned)ix < (unsigned)iw, vx1 = (unsigned)(ix + 1) < (unsigned)iw;
        const bool vy0 = (unsigned)iy < (unsigned)ih, vy1 = (unsigned)(iy + 1) < (unsigned)ih;
        const int q = (int)(((unsigned)iy * (unsigned)iw + (unsigned)ix) * 4u);
        t.a[0] = load_texel(rs, (vx0 && vy0) ? q : kTapOOB);
        t.a[1] = load_texel(rs, (vx1 && vy0) ? q + 4 : kTapOOB);
        t.a[2] = load_texel(rs, (vx0 && vy1) ? q + v.pitch : kTapOOB);
        t.a[3] = load_texel(rs, (vx1 && vy1) ? q + v.pitch + 4 : kTapOOB);
    }
}

// Adds e times the bilinear sample to c, in units of 2^24.  A byte b in the
// low end of a half is the number b 2^-24, exactly, and the mixed fma takes
// halves and floats: one mask gives a texel's red and blue, one byte
// permutation the green of two, where a conversion per channel took three.  The
// sample is summed by itself: its texels added to c one by one, with e in the
// weights, saved two instructions a view and rounded four times at c's size.
__device__ __forceinline__ void add_sample(const Tex &t, float e, float &c0, float &c1, float &c2) {
    typedef _Float16 half2 __attribute__((ext_vector_type(2)));
    const float g = 1.0f - t.wy;
    const float w1 = t.wx * g, w3 = t.wx * t.wy;
    const float w[4] = {g - w1, w1, t.wy - w3, w3};
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        const half2 rb0 = __builtin_bit_cast(half2, t.a[r] & 0x00ff00ffu);
        const half2 rb1 = __builtin_bit_cast(half2, t.a[r + 1] & 0x00ff00ffu);
        const half2 gg = __builtin_bit_cast(half2, __builtin_amdgcn_perm(t.a[r + 1], t.a[r], 0x0c050c01u));
        s0 = fmaf(w[r], (float)rb0[0], s0);
        s1 = fmaf(w[r], (float)gg[0], s1);
        s2 = fmaf(w[r], (float)rb0[1], s2);
        s0 = fmaf(w[r + 1], (float)rb1[0], s0);
        s1 = fmaf(w[r + 1], (float)gg[1], s1);
        s2 = fmaf(w[r + 1], (float)rb1[1], s2);
    }
    c0 = fmaf(e, s0, c0);
    c1 = fmaf(e, s1, c1);
    c2 = fmaf(e, s2, c2);
}

// NV views known at compile time (0: p.V, the softmax online).  Up to 8 views a
// pixel's A (u, v, 1) of every view is kept over the layers (HOIST).
template <int NV>
__global__ void __launch_bounds__(256) k_render_ibr(const RenderArgs p) {
    constexpr bool HOIST = NV > 0 && NV <= 8;
    // XCD-aware tile order: workgroups are dispatched round-robin over the
    // 8 XCDs, so workgroup i is given tile (i % 8) * per + i / 8 and each XCD
    // walks one contiguous band of 16-row tiles; with horizontal-ish
    // baselines the band's samples fall in a band of image rows that stays
    // in the XCD's L2
    const int tiles_x = (p.W + 15) >> 4;
    const int n = gridDim.x;
    int tile;
    {
        const int i = blockIdx.x, xcd = i & 7, loc = i >> 3, q = n >> 3, rem = n & 7;
        tile = (xcd < rem) ? xcd * (q + 1) + loc : rem * (q + 1) + (xcd - rem) * q + loc;
    }
    const int x = (tile % tiles_x) * 16 + (threadIdx.x & 15);
    const int y = (tile / tiles_x) * p.rows + (threadIdx.x >> 4);
    if (x >= p.W || y >= p.H) return;              // no barriers below

    // upsampling taps: source coordinate (x + 0.5) w / W - 0.5, clamped
    // below at 0; the second tap clamped to the last column / row
    double sx = ((double)x + 0.5) * p.rx - 0.5, sy = ((double)y + 0.5) * p.ry - 0.5;
    sx = sx < 0.0 ? 0.0 : sx;
    sy = sy < 0.0 ? 0.0 : sy;
    int x0 = (int)sx, y0 = (int)sy;                 // sx, sy >= 0: truncation is floor
    x0 = x0 < p.w - 1 ? x0 : p.w - 1;
    y0 = y0 < p.h - 1 ? y0 : p.h - 1;
    const int x1 = x0 + 1 < p.w ? x0 + 1 : p.w - 1, y1 = y0 + 1 < p.h ? y0 + 1 : p.h - 1;
    const double lxd = sx - x0, lyd = sy - y0;
    const float lx = (float)lxd, ly = (float)lyd;
    const int64_t hw = (int64_t)p.h * p.w;
    // Offsets count from the tile's first row of logits, in 32 bits where NV > 0 (the
    // launcher sees to it that a tile's rows are that close; a layer's need not be)
    int first_row = 0;
    if constexpr (NV > 0) {
        const double s0 = ((double)(tile / tiles_x * p.rows) + 0.5) * p.ry - 0.5;
        first_row = __builtin_amdgcn_readfirstlane(min(max((int)s0, 0), p.h - 1));
    }
    const int64_t row_at = (int64_t)first_row * p.w, left = hw - row_at;
    using idx = std::conditional_t<(NV > 0), int, int64_t>;
    const idx t00 = (idx)(y0 - first_row) * p.w + x0, t10 = (idx)(y0 - first_row) * p.w + x1;
    const idx t01 = (idx)(y1 - first_row) * p.w + x0, t11 = (idx)(y1 - first_row) * p.w + x1;
    auto at = [&](const float *q, idx i) {
        if constexpr (NV > 0) return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(layer_rsrc(q, 4 * left), 4 * i, 0, 0));
        else return q[i];
    };
    auto lerp_f = [&](float a00, float a10, float a01, float a11) {
        return (1.0f - ly) * ((1.0f - lx) * a00 + lx * a10) + ly * ((1.0f - lx) * a01 + lx * a11);
    };

    const double u = (double)x + 0.5, vv = (double)y + 0.5;
    const int V = NV > 0 ? NV : p.V, L = p.L;
    const double rL = 1.0 / (double)L;
    double base[HOIST ? 3 * NV : 1];               // A (u, v, 1)
    if constexpr (HOIST) {
#pragma unroll
        for (int m = 0; m < NV; ++m)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                base[3 * m + i] = fma(p.A[m][3 * i], u, fma(p.A[m][3 * i + 1], vv, p.A[m][3 * i + 2]));
    }
    float Tr = 1.0f, out0 = 0.0f, out1 = 0.0f, out2 = 0.0f, dmap = 0.0f;

    for (int li = 0; li < L; ++li) {
        const float *D = p.depth_logit + li * hw + row_at, *S = p.sigma_logit + li * hw + row_at;
        const float alpha = sigmoid_(lerp_f(at(S, t00), at(S, t10), at(S, t01), at(S, t11)));
        // depth: the logit is interpolated in double, since an error in it is
        // magnified by the parallax (up to ~1e3 px per unit of disparity)
        const double xd = (1.0 - lyd) * ((1.0 - lxd) * (double)at(D, t00) + lxd * (double)at(D, t10)) +
                          lyd * ((1.0 - lxd) * (double)at(D, t01) + lxd * (double)at(D, t11));
        const double delta = ((double)(L - li) - 0.5) * rL;
        const double disp = fma(fma(0.5 * rL, (double)tanhf((float)xd), delta), p.band, p.inv_far);
        double rd = __builtin_amdgcn_rcp(disp);         // refined as 1 / pz below
        rd = fma(rd, fma(-disp, rd, 1.0), rd);
        const float depth = disp != 0.0 ? (float)rd : __builtin_inff();

        // one view's image, back-projected through this layer's depth: the
        // four texels' loads are issued here and blended later (blend_view),
        // so the next view's loads are in flight while this one is blended
        auto issue_view = [&](int m, const RenderView &v, int centre, const double (&A)[9], Tex &t) {
            double pz, qx, qy;
            if constexpr (HOIST) {
                qx = fma(v.b[0], disp, base[3 * m]);
                qy = fma(v.b[1], disp, base[3 * m + 1]);
                pz = fma(v.b[2], disp, base[3 * m + 2]);
            } else {
                pz = fma(A[6], u, fma(A[7], vv, fma(v.b[2], disp, A[8])));
                qx = fma(A[0], u, fma(A[1], vv, fma(v.b[0], disp, A[2])));
                qy = fma(A[3], u, fma(A[4], vv, fma(v.b[1], disp, A[5])));
            }
            // 1/pz: the hardware reciprocal refined by one Newton step (the
            // relative error squares, far below what the coordinates need)
            double rz = __builtin_amdgcn_rcp(pz);
            rz = fma(rz, fma(-pz, rz, 1.0), rz);
            issue_texels(v, centre, qx * rz, qy * rz, pz, t);
        };
        // a view's record, read a view before it is used
        struct View {
            RenderView v;
            int centre;
            double A[9];                             // not where HOIST took it
        };
        auto view = [&](int m) {
            View r;
            r.v = p.v[m];
            r.centre = p.centre[m];
            if constexpr (!HOIST)
                for (int i = 0; i < 9; ++i) r.A[i] = p.A[m][i];
            return r;
        };
        // blend: softmax over the views of the upsampled logits
        const float *B = p.blend_logit + (li * hw + row_at) * V;
        float z = 0.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
        if constexpr (NV > 0) {
            // all views' logits first (in the widest loads that V floats per
            // tap stay aligned to), then their maximum, then the views
            constexpr int VW = NV % 4 == 0 ? 4 : NV % 2 == 0 ? 2 : 1;
            typedef float vec __attribute__((ext_vector_type(VW)));
            const __amdgpu_buffer_rsrc_t brs = layer_rsrc(B, 4 * left * NV);
            auto tap = [&](int i, int c) {
                const int o = i * (4 * NV), k = c * (int)sizeof(vec);
                if constexpr (VW == 4) return __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(brs, o, k, 0));
                else if constexpr (VW == 2) return __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(brs, o, k, 0));
                else return __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b32(brs, o, k, 0));
            };
            float xb[NV];
#pragma unroll
            for (int c = 0; c < NV / VW; ++c) {
                const vec a = tap(t00, c), b = tap(t10, c), d = tap(t01, c), e = tap(t11, c);
#pragma unroll
                for (int i = 0; i < VW; ++i) xb[VW * c + i] = lerp_f(a[i], b[i], d[i], e[i]);
            }
            float mx = xb[0];
#pragma unroll
            for (int m = 1; m < NV; ++m) mx = fmaxf(mx, xb[m]);
            // two texel buffers in turn: the loads of the next view are issued
            // before this one is blended
            Tex t[2];
            int first = 0;          // hidden: the views' records are read again in each
            asm volatile("" : "+s"(first));     // layer, all at once they would take the scalar registers
            View next = view(first);
            issue_view(0, next.v, next.centre, next.A, t[0]);
            next = view(first + (NV > 1 ? 1 : 0));
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                if (m + 1 < NV) issue_view(m + 1, next.v, next.centre, next.A, t[(m + 1) & 1]);
                if (m + 2 < NV) next = view(first + m + 2);
                const float e = __expf(xb[m] - mx);
                add_sample(t[m & 1], e, c0, c1, c2);
                z += e;
                // each view blended before the next but one is issued: all
                // views' texels at once would take the register file
                asm volatile("" : "+v"(c0), "+v"(c1), "+v"(c2));
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // online: running maximum, sums rescaled when it moves
            float mx = -3.0e38f;
            View next = view(0);
            for (int m = 0; m < V; ++m) {
                const View now = next;
                next = view(m + 1 < V ? m + 1 : 0);
                const float xb = lerp_f(B[t00 * V + m], B[t10 * V + m], B[t01 * V + m], B[t11 * V + m]);
                if (xb > mx) {                       // move the reference
                    const float r = __expf(mx - xb);
                    z *= r; c0 *= r; c1 *= r; c2 *= r;
                    mx = xb;
                }
                const float e = __expf(xb - mx);
                Tex t;
                issue_view(m, now.v, now.centre, now.A, t);
                add_sample(t, e, c0, c1, c2);
                z += e;
            }
        }
        // beta = e / z; texels v / 255, summed in units of 2^24
        const float k = Tr * alpha * (16777216.0f / 255.0f) / z;
        out0 = fmaf(k, c0, out0);
        out1 = fmaf(k, c1, out1);
        out2 = fmaf(k, c2, out2);
        dmap = fmaf(Tr * alpha, depth, dmap);
        Tr *= 1.0f - alpha;
    }
    const int64_t q = (int64_t)y * p.W + x;
    p.rgb[q * 3 + 0] = out0;
    p.rgb[q * 3 + 1] = out1;
    p.rgb[q * 3 + 2] = out2;
    if (p.acc != nullptr) p.acc[q] = 1.0f - Tr;
    if (p.depth != nullptr) p.depth[q] = dmap;
}

}  // namespace

hipError_t launch_render_ibr(const RenderParams &p, hipStream_t s) {
    // Tiles of 16 x 16, or where that is 64 workgroups at most 16 x 4: a wave to a
    // compute unit instead of four to a quarter of them (9 views to 160 x 90: 22.9
    // -> 21.7 us, 16 views 29.9 -> 28.6; at 320 x 180, 240 of them, 8 views would
    // take 16.4 for 15.5).
    const int tiles_x = (p.W + 15) / 16;
    RenderArgs a = {};
    a.rows = (int64_t)tiles_x * ((p.H + 15) / 16) <= 64 ? 4 : 16;
    const dim3 g(tiles_x * ((p.H + a.rows - 1) / a.rows)), b(16 * a.rows);
    for (int m = 0; m < p.V; ++m) {
        RenderView &v = a.v[m];
        const double *c = p.cam[m];
        v.hx = (p.iW[m] - 1) / 2;
        v.hy = (p.iH[m] - 1) / 2;
        a.centre[m] = 4 * ((p.iH[m] - 1) / 2 * p.iW[m] + (p.iW[m] - 1) / 2);
        for (int i = 0; i < 3; ++i) {
            a.A[m][i] = c[i] - (v.hx + 0.5) * c[6 + i];
            a.A[m][3 + i] = c[3 + i] - (v.hy + 0.5) * c[6 + i];
            a.A[m][6 + i] = c[6 + i];
        }
        v.b[0] = c[9] - (v.hx + 0.5) * c[11];
        v.b[1] = c[10] - (v.hy + 0.5) * c[11];
        v.b[2] = c[11];
        v.wd = p.iW[m];
        v.img = p.img[m];
        v.pitch = 4 * p.iW[m];
        v.bytes = p.iH[m] * v.pitch;
    }
    a.depth_logit = p.depth_logit;
    a.sigma_logit = p.sigma_logit;
    a.blend_logit = p.blend_logit;
    a.rgb = p.rgb;
    a.acc = p.acc;
    a.depth = p.depth;
    a.V = p.V; a.L = p.L; a.h = p.h; a.w = p.w; a.H = p.H; a.W = p.W;
    a.rx = p.rx; a.ry = p.ry; a.band = p.band; a.inv_far = p.inv_far;
    const bool vec = render_vectors(p.V, p.h, p.w, p.H, a.rows, reinterpret_cast<uintptr_t>(p.blend_logit));
#define QK_RENDER(NV) case NV: hipLaunchKernelGGL((k_render_ibr<NV>), g, b, 0, s, a); break
    switch (vec ? p.V : 0) {
    QK_RENDER(1); QK_RENDER(2); QK_RENDER(3); QK_RENDER(4); QK_RENDER(5); QK_RENDER(6); QK_RENDER(7); QK_RENDER(8);
    QK_RENDER(12); QK_RENDER(16);
    default: hipLaunchKernelGGL((k_render_ibr<0>), g, b, 0, s, a); break;
    }
#undef QK_RENDER
    return hipGetLastError();
}

}  // namespace qk
