// k_scatter.hip -- feature-map gradients of the backward pass by sorting: the
// per-layer-pixel kernel has stored every sample's gradient ds (a row of C
// floats per view and layer-pixel), the records are binned by the tile of the
// map their bilinear footprint falls in (k_views.hip's passes), and one
// workgroup per tile writes each of its pixels once,
//   dI(x, y) = sum over the records of the four cells around it of w_tap ds.
// No atomics on the maps, and nothing is cleared first.  A tile's workgroup takes
// its first kScatterOwn records; where more crowd there (a map much smaller than
// the level, a view that sees it from afar) it lists the rest in pieces as large,
// which a second launch spreads over the chip and adds.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "uf_params.h"
#include "vbin.h"

namespace qk {
namespace {

constexpr int kTh = kScatterTh, kTw = 1 << kVbLog2Tw;
constexpr int kCw = kTw + 1, kCh = kTh + 1, kCells = kCw * kCh;   // cells whose taps reach the tile
constexpr int kThreads = 256;
constexpr int kBatch = 1280, kPer = kBatch / kThreads;            // records sorted at a time

struct ScatterLds {
    int cnt[kCells + 1];                 // counts, then a cell's first record
    int sum[kThreads / 64];
    float4 w[kBatch];                    // tap weights 00, 10, 01, 11
    uint32_t q[kBatch];                  // byte offset of the row of ds
};

// A tile of a view's map, its place and records.
struct Tile {
    int m, x0, y0;
    VbinRanges ranges;
    __device__ Tile(const ViewsParams &p, int t) {
        m = 0;
        for (int i = 1; i < p.V; ++i) m = (t >= p.tbase[i]) ? i : m;
        const int ntx = p.ntx[m], lt = t - p.tbase[m];
        const int ty = lt / ntx, tx = lt - ty * ntx;
        x0 = tx * kTw;
        y0 = ty * kTh;
        ranges = vbin_ranges(p, t, tx, ty, ntx, p.nty[m]);
    }
};

// A workgroup sorts records first .. last - 1 of a tile by cell (top left tap) in
// LDS, a batch at a time; then C lanes, one per channel, own two pixel columns and
// walk down the rows of the three columns of cells that reach them, summing in
// registers.  A record's row of ds is read one and a half times on average.  The
// first batch of a tile writes its pixels and later ones add to them; ADD: other
// workgroups add to the same pixels.
// 16.6 M records of 64 bytes (960x540, L = 8, C = 16, V = 4): 0.50 ms, 2.1 TB/s
// of rows, bound by the latency of the short lists (8 records a cell there).
// Tiles are 4 rows high so that such a tile is one batch at six workgroups per
// CU: 8 rows in two batches took 0.55 ms, in one batch of 2560 0.68 ms; with a
// pixel's own four lists per C lanes, every row read four times, 1.07 ms.
template <int C, bool ADD>
__device__ __forceinline__ void scatter_records(const ViewsParams &p, const ScatterParams &sp, const Tile &tile,
                                                uint32_t first, uint32_t last, ScatterLds &lds) {
    constexpr int RG = kThreads / C / (kTw / 2); // groups of rows
    constexpr int RH = kTh / RG;                 // pixel rows of a group
    auto &s_cnt = lds.cnt;
    auto &s_sum = lds.sum;
    auto &s_w = lds.w;
    auto &s_q = lds.q;
    const int m = tile.m, x0 = tile.x0, y0 = tile.y0;
    const VbinRanges &ranges = tile.ranges;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ch = tid % C, col = tid / C % (kTw / 2), row0 = tid / C / (kTw / 2) * RH;
    const __amdgpu_buffer_rsrc_t ds = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(sp.ds + (int64_t)m * p.N * C), 0, (int)(uint32_t)(p.N * C * 4), 0x00020000);
    const int vw = p.vW[m], vh = p.vH[m];
    float *out = sp.dfeat[m];

    // (a tile without records is one empty batch: its pixels are zero)
    for (uint32_t b0 = first; b0 == 0 || b0 < last; b0 += kBatch) {
        for (int i = tid; i <= kCells; i += kThreads) s_cnt[i] = 0;
        __syncthreads();
        int cell[kPer], rank[kPer], q[kPer];
        float2 f[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const uint32_t i = b0 + k * kThreads + tid;
            cell[k] = -1;
            q[k] = i < last ? p.rec[ranges.at(i)] : -1;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            rank[k] = 0;
            f[k] = make_float2(0.0f, 0.0f);
            if ((unsigned)q[k] >= (unsigned)p.N) continue;
            int ix, iy, l;
            if (!vbin_footprint(p, m, q[k], p.depth[q[k]], f[k].x, f[k].y, ix, iy, l)) continue;
            const int cx = ix - x0 + 1, cy = iy - y0 + 1;
            if ((unsigned)cx >= (unsigned)kCw || (unsigned)cy >= (unsigned)kCh) continue;
            cell[k] = cy * kCw + cx;
            rank[k] = atomicAdd(&s_cnt[cell[k]], 1);
        }
        __syncthreads();
        // exclusive scan of the counts, two cells per thread
        static_assert(kCells <= 2 * kThreads, "two cells per thread");
        const int c0 = 2 * tid < kCells ? s_cnt[2 * tid] : 0;
        const int c1 = 2 * tid + 1 < kCells ? s_cnt[2 * tid + 1] : 0;
        int inc = c0 + c1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(inc, off);
            if (lane >= off) inc += v;
        }
        if (lane == 63) s_sum[wave] = inc;
        __syncthreads();
        int run = inc - c0 - c1;
#pragma unroll
        for (int w = 0; w < kThreads / 64 - 1; ++w) run += w < wave ? s_sum[w] : 0;
        if (2 * tid <= kCells) s_cnt[2 * tid] = run;
        if (2 * tid + 1 <= kCells) s_cnt[2 * tid + 1] = run + c0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (cell[k] < 0) continue;
            const int at = s_cnt[cell[k]] + rank[k];
            const float fx = f[k].x, fy = f[k].y;
            s_w[at] = make_float4((1.0f - fx) * (1.0f - fy), fx * (1.0f - fy), (1.0f - fx) * fy, fx * fy);
            s_q[at] = (uint32_t)q[k] * (uint32_t)(C * 4);
        }
        __syncthreads();
        // cell row r holds the records whose lower taps lie in pixel row r
        float a0 = 0.0f, b0v = 0.0f, a1 = 0.0f, b1 = 0.0f;   // columns a, b of rows r - 1, r
#pragma unroll 1
        for (int r = row0; r <= row0 + RH; ++r) {
            const int c = r * kCw + 2 * col;
            // f(w, d) over the records of one cell, four rows of ds in flight
            auto walk = [&](int k0, int k1, auto &&add) {
#pragma unroll 1
                for (int k = k0; k < k1; k += 4) {
                    float d[4];
                    float4 w[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int kk = min(k + u, k1 - 1);
                        w[u] = s_w[kk];
                        d[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ds, (int)(s_q[kk] + 4 * ch), 0, 0));
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) add(w[u], k + u < k1 ? d[u] : 0.0f);
                }
            };
            const int e0 = s_cnt[c], e1 = s_cnt[c + 1], e2 = s_cnt[c + 2], e3 = s_cnt[c + 3];
            walk(e0, e1, [&](const float4 &w, float d) {
                a0 = fmaf(w.y, d, a0);
                a1 = fmaf(w.w, d, a1);
            });
            walk(e1, e2, [&](const float4 &w, float d) {
                a0 = fmaf(w.x, d, a0);
                a1 = fmaf(w.z, d, a1);
                b0v = fmaf(w.y, d, b0v);
                b1 = fmaf(w.w, d, b1);
            });
            walk(e2, e3, [&](const float4 &w, float d) {
                b0v = fmaf(w.x, d, b0v);
                b1 = fmaf(w.z, d, b1);
            });
            const int x = x0 + 2 * col, y = y0 + r - 1;
            if (r > row0 && y < vh) {            // row r - 1 is complete for this batch
                float *dst = out + ((int64_t)y * vw + x) * C + ch;
                if constexpr (ADD) {
                    if (x < vw && a0 != 0.0f) unsafeAtomicAdd(dst, a0);
                    if (x + 1 < vw && b0v != 0.0f) unsafeAtomicAdd(dst + C, b0v);
                } else {
                    if (x < vw) dst[0] = b0 == 0 ? a0 : dst[0] + a0;
                    if (x + 1 < vw) dst[C] = b0 == 0 ? b0v : dst[C] + b0v;
                }
            }
            a0 = a1;
            b0v = b1;
            a1 = b1 = 0.0f;
        }
        __syncthreads();
    }
}

template <int C>
__global__ void __launch_bounds__(kThreads) k_scatter_tiles(const ViewsParams p, const ScatterParams sp) {
    __shared__ ScatterLds lds;
    __shared__ uint32_t s_at;
    const int t = xcd_order(blockIdx.x, gridDim.x);
    const Tile tile(p, t);
    const uint32_t total = tile.ranges.cum[5];
    if (total > kScatterOwn) {                   // list what is left
        const uint32_t n = (total - 1) / kScatterOwn;
        if (threadIdx.x == 0) s_at = atomicAdd(sp.listed, n);
        __syncthreads();
        const uint32_t at = s_at;
        for (uint32_t i = threadIdx.x; i < n; i += kThreads)
            if (at + i < sp.list_cap) sp.list[at + i] = make_uint2((uint32_t)t, (i + 1) * kScatterOwn);
    }
    scatter_records<C, false>(p, sp, tile, 0, min(total, (uint32_t)kScatterOwn), lds);
}

// The pieces that k_scatter_tiles listed.  4 views of 131x251, 8 layers, C = 16 (the
// whole adjoint): maps of 4 x 32 5.91 -> 0.57 ms (float atomics 0.69), focal lengths
// a hundredth 31 -> 0.79 (9 to 12); the launch takes 3 us where no tile is crowded.
// Pieces of 5120 records: 0.77 and 1.35 ms.
template <int C>
__global__ void __launch_bounds__(kThreads) k_scatter_rest(const ViewsParams p, const ScatterParams sp) {
    __shared__ ScatterLds lds;
    const uint32_t n = min(*sp.listed, sp.list_cap);
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
        const uint2 piece = sp.list[i];
        const Tile tile(p, (int)piece.x);
        scatter_records<C, true>(p, sp, tile, piece.y, min(tile.ranges.cum[5], piece.y + kScatterOwn), lds);
    }
}

}  // namespace

hipError_t launch_scatter(const ViewsParams &p, const ScatterParams &sp, int C, hipStream_t s) {
    const dim3 g((unsigned)p.tbase[p.V]), r(std::min<uint32_t>(sp.list_cap, 6 * 256)), b(kThreads);
    if (C == 8) hipLaunchKernelGGL(k_scatter_tiles<8>, g, b, 0, s, p, sp);
    else hipLaunchKernelGGL(k_scatter_tiles<16>, g, b, 0, s, p, sp);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (C == 8) hipLaunchKernelGGL(k_scatter_rest<8>, r, b, 0, s, p, sp);
    else hipLaunchKernelGGL(k_scatter_rest<16>, r, b, 0, s, p, sp);
    return hipGetLastError();
}

}  // namespace qk
