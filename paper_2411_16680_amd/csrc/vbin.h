// vbin.h -- records of layer-pixels binned by the view tile their bilinear
// footprint falls in (k_views.hip: the render to the input views; k_scatter.hip:
// the feature-map gradients).
#pragma once
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "uf_params.h"

namespace qk {

constexpr int kVbLog2Tw = 5;                    // tiles are 32 view pixels wide

// 1 / x in double: the hardware reciprocal refined by one Newton step (its
// relative error squares, far below what the coordinates need).  The binned
// passes all reproject through it, so they agree bit for bit.
__device__ inline double recip_d(double x) {
#pragma clang fp contract(on)
    const double r = __builtin_amdgcn_rcp(x);
    return fma(r, fma(-x, r, 1.0), r);
}

// The footprint of layer-pixel q in view m: its layer, the view pixel
// (ix, iy) of its top left tap and the fractions; false when no tap lies in
// the view.  The reprojection of k_splat (reciprocals as above); a sample
// with fxc <= -1 or fxc >= vW (likewise y) has no tap inside.  Every binned
// pass calls it: the tile pass recomputes a record's footprint from the
// layer-pixel index the write pass stored.  All three passes are bound by
// VALU instructions, so the index divisions are multiplications.
// (The binned form runs only while V L H W < 2^31, so a layer-pixel index
// and its divisions fit 32 bits.)
__device__ inline uint32_t fast_div(uint32_t n, const FastDiv &f) {
    const uint32_t q = __umulhi(n, f.mul) >> f.shift;
    return f.d == 1u ? n : q;
}

__device__ inline bool vbin_footprint(const ViewsParams &p, int m, int q, float depth, float &fx,
                                      float &fy, int &ix, int &iy, int &l) {
#pragma clang fp contract(on)
    const uint32_t uq = (uint32_t)q, ul = fast_div(uq, p.div_hw);
    const uint32_t r = uq - ul * p.div_hw.d, uy = fast_div(r, p.div_w);
    l = (int)ul;
    const int y = (int)uy, x = (int)(r - uy * p.div_w.d);
    const double u = (double)x + 0.5, v = (double)y + 0.5;
    const double invd = recip_d((double)depth);
    const double *A = p.cam[m];
    const int vw = p.vW[m], vh = p.vH[m];
    const double pz = fma(A[6], u, fma(A[7], v, fma(A[11], invd, A[8])));
    const double qx = fma(A[0], u, fma(A[1], v, fma(A[9], invd, A[2])));
    const double qy = fma(A[3], u, fma(A[4], v, fma(A[10], invd, A[5])));
    const double rz = recip_d(pz);
    const double fxc = qx * rz - 0.5, fyc = qy * rz - 0.5;
    const bool ok = (pz > 1e-6) && (fxc > -1.0) && (fxc < (double)vw) && (fyc > -1.0) &&
                    (fyc < (double)vh);
    const double xf = floor(fxc), yf = floor(fyc);
    fx = (float)(fxc - xf);
    fy = (float)(fyc - yf);
    ix = ok ? (int)xf : 0;
    iy = ok ? (int)yf : 0;
    return ok;
}

// The bin of a footprint (the tile sides are powers of two).
__device__ inline int vbin_bin(const ViewsParams &p, int m, int ix, int iy) {
    const int tx = min((ix + 1) >> kVbLog2Tw, p.ntx[m] - 1);
    const int ty = min((iy + 1) >> p.log2_th, p.nty[m] - 1);
    const int cls = (ix == (tx << kVbLog2Tw) - 1 ? 1 : 0) | (iy == (ty << p.log2_th) - 1 ? 2 : 0);
    return 4 * (p.tbase[m] + ty * p.ntx[m] + tx) + cls;
}

// XCD-aware order: workgroups are dispatched round-robin over the 8 XCDs;
// workgroup i takes item (i % 8) * per + i / 8, so each XCD walks one
// contiguous range.
__device__ inline int xcd_order(int i, int n) {
    const int xcd = i & 7, loc = i >> 3, q8 = n >> 3, rem = n & 7;
    return (xcd < rem) ? xcd * (q8 + 1) + loc : rem * (q8 + 1) + (xcd - rem) * q8 + loc;
}

// Tile t's records: those in its own four bins, then the crossing bins of the
// tiles to the right (left-crossing), below (top-crossing) and below right
// (both), as one index space of cum[5] records, record k at rec[o + k] with o
// from its range.  A tile's bins lie one after the other, and the write pass has
// left every cursor at its bin's end.
struct VbinRanges {
    uint32_t rs[5], cum[6];
    __device__ inline uint32_t at(uint32_t k) const {
        uint32_t o = rs[0];
#pragma unroll
        for (int j = 1; j < 5; ++j) o = (k >= cum[j]) ? rs[j] - cum[j] : o;
        return o + k;
    }
};
__device__ inline VbinRanges vbin_ranges(const ViewsParams &p, int t, int tx, int ty, int ntx, int nty) {
    VbinRanges r;
    uint32_t re[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) r.rs[j] = re[j] = 0u;
    auto range = [&](int j, int tile, int first, int last) {
        r.rs[j] = first == 0 ? p.start[tile] : p.cursor[4 * tile + first - 1];
        re[j] = p.cursor[4 * tile + last];
    };
    const int right = tx + 1 < ntx ? 1 : 0, below = ty + 1 < nty ? ntx : 0;
    range(0, t, 0, 3);
    if (right) {
        range(1, t + 1, 1, 1);
        range(2, t + 1, 3, 3);
    }
    if (below) range(3, t + ntx, 2, 3);
    if (right && below) range(4, t + ntx + 1, 3, 3);
    r.cum[0] = 0u;
#pragma unroll
    for (int j = 0; j < 5; ++j) r.cum[j + 1] = r.cum[j] + (re[j] - r.rs[j]);
    return r;
}

// Clears the bin counts, counts, hands out the tiles' runs and writes the
// records (k_views.hip).
hipError_t launch_vbin(const ViewsParams &p, hipStream_t s);

}  // namespace qk
