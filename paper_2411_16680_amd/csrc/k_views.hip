// k_views.hip -- render of a decoded intermediate LDM into every input view
// (Sec. 3.2.2 "Decoding and rendering the intermediate LDM", Eq. 2): the
// projection operator, the transpose of the bilinear back-projection, splats
// each layer-pixel's colour and density into the four view pixels around its
// reprojection (per layer, per view, unnormalised), then each view composites
// its projected layers front to back.
//
// Two forms.  The binned form (up to 128 layers) never writes the projected
// layers: every (view, layer-pixel) becomes a record in the bin of the view
// tile its taps reach, and one workgroup per tile adds its records into LDS
// and composites the tile (see "Binned form" below).  The planes form, for
// more layers: a fill kernel clears the projected layers (no
// hipMemsetAsync, so the call can be captured in a graph); k_splat, one
// thread per (view, layer-pixel), scatters with float atomics regrouped
// through LDS so that eight adjacent lanes add the four channels of a tap
// and of its right neighbour (32 contiguous bytes) instead of 64 lanes
// hitting 64 scattered words; k_views_composite, one thread per view pixel.
// Both forms form the same products of tap weight and payload and the same
// composite; only the order of the float additions into a view pixel
// differs.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "uf_params.h"
#include "vbin.h"

// multiply-adds fused within an expression only: the binned form's counting
// and writing passes evaluate the same reprojection and must round it alike
#pragma clang fp contract(on)

namespace qk {
namespace {

__global__ void __launch_bounds__(256) k_views_zero(const ViewsParams p) {
    const int64_t n4 = p.ws_floats >> 2;
    float4 *w = reinterpret_cast<float4 *>(p.ws);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256)
        w[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// Per wave: 64 layer-pixels x 2 tap rows = 128 entries -- the float index
// in ws of the row's left and right taps (-1 = dropped) and their weights --
// and the 64 payloads (r, g, b, alpha).  A row's two taps are neighbours in
// the plane, so one entry is 32 contiguous bytes.
struct SplatSlice {
    int4 e[128];         // dst_left, dst_right, weight bits left, right
    float4 val[64];
};

__global__ void __launch_bounds__(256) k_splat(const ViewsParams p) {
    __shared__ SplatSlice sl[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    SplatSlice &s = sl[wave];
    // one (view, 256 layer-pixels) chunk per workgroup, views slowest, in an
    // XCD-aware order (workgroups are dispatched round-robin over the 8 XCDs:
    // workgroup i takes chunk (i % 8) * per + i / 8), so each XCD scatters
    // the rows of one layer into one view at a time and the band of the
    // view's plane those rows reach stays in its L2
    const int64_t bpv = (p.N + 255) / 256, n = bpv * p.V;
    int64_t chunk;
    {
        const int64_t i = blockIdx.x, xcd = i & 7, loc = i >> 3, q8 = n >> 3, rem = n & 7;
        chunk = (xcd < rem) ? xcd * (q8 + 1) + loc : rem * (q8 + 1) + (xcd - rem) * q8 + loc;
    }
    const int m = (int)(chunk / bpv);
    const int64_t q = (chunk - (int64_t)m * bpv) * 256 + threadIdx.x;   // layer-pixel
    const bool live = q < p.N;
    const int64_t hw = (int64_t)p.H * p.W;
    const int l = live ? (int)(q / hw) : 0;
    const int64_t r = live ? q - (int64_t)l * hw : 0;
    const int y = (int)(r / p.W), x = (int)(r - (int64_t)y * p.W);
    const double u = (double)x + 0.5, v = (double)y + 0.5;
    int4 row0 = make_int4(-1, -1, 0, 0), row1 = make_int4(-1, -1, 0, 0);
    if (live) {
        s.val[lane] = make_float4(p.color[q * 3 + 0], p.color[q * 3 + 1], p.color[q * 3 + 2],
                                  p.alpha[q]);
        const double invd = 1.0 / (double)p.depth[q];
        const double *A = p.cam[m];
        const int vw = p.vW[m], vh = p.vH[m];
        const double pz = fma(A[6], u, fma(A[7], v, fma(A[11], invd, A[8])));
        const double qx = fma(A[0], u, fma(A[1], v, fma(A[9], invd, A[2])));
        const double qy = fma(A[3], u, fma(A[4], v, fma(A[10], invd, A[5])));
        const double rz = 1.0 / pz;
        const double fxc = qx * rz - 0.5, fyc = qy * rz - 0.5;
        if ((pz > 1e-6) && (fxc > -2.0) && (fxc < (double)(vw + 1)) && (fyc > -2.0) &&
            (fyc < (double)(vh + 1))) {
            const double xf = floor(fxc), yf = floor(fyc);
            const float fx = (float)(fxc - xf), fy = (float)(fyc - yf);
            const int ix = (int)xf, iy = (int)yf;
            const int64_t base = p.sbase[m] + (int64_t)l * vh * vw * 4;
            const bool vx0 = (unsigned)ix < (unsigned)vw, vx1 = (unsigned)(ix + 1) < (unsigned)vw;
            const bool vy0 = (unsigned)iy < (unsigned)vh, vy1 = (unsigned)(iy + 1) < (unsigned)vh;
            const int64_t o0 = base + ((int64_t)iy * vw + ix) * 4, o1 = o0 + (int64_t)vw * 4;
            row0 = make_int4((vx0 && vy0) ? (int)o0 : -1, (vx1 && vy0) ? (int)o0 + 4 : -1,
                             __float_as_int((1.0f - fx) * (1.0f - fy)),
                             __float_as_int(fx * (1.0f - fy)));
            row1 = make_int4((vx0 && vy1) ? (int)o1 : -1, (vx1 && vy1) ? (int)o1 + 4 : -1,
                             __float_as_int((1.0f - fx) * fy), __float_as_int(fx * fy));
        }
    }
    s.e[2 * lane] = row0;
    s.e[2 * lane + 1] = row1;
    __syncthreads();
    // lanes 8k..8k+7 add entry 8 j + k: the left tap's four channels, then
    // the right tap's
    const int c = lane & 3, right = (lane >> 2) & 1;
#pragma unroll 4
    for (int j = 0; j < 16; ++j) {
        const int en = 8 * j + (lane >> 3);
        const int4 ent = s.e[en];
        const int d = right ? ent.y : ent.x;
        if (d >= 0) {
            const float4 pv = s.val[en >> 1];
            const float val = c == 0 ? pv.x : c == 1 ? pv.y : c == 2 ? pv.z : pv.w;
            unsafeAtomicAdd(p.ws + d + c, __int_as_float(right ? ent.w : ent.z) * val);
        }
    }
}

__global__ void __launch_bounds__(256) k_views_composite(const ViewsParams p) {
    const int m = blockIdx.y;
    const int64_t np = (int64_t)p.vH[m] * p.vW[m];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= np) return;
    const float4 *S = reinterpret_cast<const float4 *>(p.ws + p.sbase[m]);
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    for (int l = 0; l < p.L; ++l) {
        const float4 s = S[(int64_t)l * np + i];
        const float w = T * s.w;
        c0 = fmaf(w, s.x, c0);
        c1 = fmaf(w, s.y, c1);
        c2 = fmaf(w, s.z, c2);
        T *= 1.0f - s.w;
    }
    float *rgb = p.rgb[m];
    rgb[i * 3 + 0] = c0;
    rgb[i * 3 + 1] = c1;
    rgb[i * 3 + 2] = c2;
    if (p.acc[m] != nullptr) p.acc[m][i] = 1.0f - T;
}


// ---------------------------------------------------------------------------
// Binned form.
//
//   k_vbin_zero    clears the bin counts
//   k_vbin_count   a workgroup takes up to 8192 layer-pixels of one view:
//                  their records' bins, counted in an LDS hash table, then
//                  one global add per distinct bin
//   k_vbin_scan    each tile's run of records; its bins' counts become their
//                  write cursors
//   k_vbin_write   the same records; per distinct bin of the workgroup one
//                  global add on the bin's cursor reserves a run of slots,
//                  a record's slot is that base plus its rank in the bin
//   k_vbin_tile    one workgroup per (view, tile): adds the taps of its
//                  records that fall inside the tile into LDS (all layers of
//                  the tile) and composites each pixel front to back
//
// The tile sums are 64-bit fixed point (2^-32 units) added with integer LDS
// atomics: on this chip a float atomic add in LDS costs several times an
// integer one, and integer sums are exact, so the result does not depend on
// the order in which records arrive (the render is bitwise reproducible).
// Each contribution (tap weight times payload, rounded to float as in the
// planes form) is rounded to the nearest 2^-32; a sum stays below 2^31 in
// magnitude unless more than 2^31 records reach one view pixel of a layer.
//
// A record is binned by the tile holding (ix + 1, iy + 1), the right column
// and bottom row of its taps; its left column (ix) may then lie in the tile
// to the left and its top row (iy) in the tile above.  Each tile has four
// bins by which of the two its records cross (bit 0 left, bit 1 top), so a
// tile's workgroup reads its own four bins and only the crossing bins of
// the tiles to its right, below and below right: every record is stored
// once and read by at most four workgroups.
// ---------------------------------------------------------------------------

constexpr int kVbThreads = 512;                 // counting and writing workgroups
constexpr int kVbHashBits = 11;
constexpr int kVbHash = 1 << kVbHashBits;       // LDS hash slots
constexpr int kVbProbes = 16;                   // a key that finds no slot goes to global memory
constexpr int kVbTileThreads = 512;
constexpr float kVbFix = 4294967296.0f;         // fixed-point scale of the tile sums, 2^32
constexpr float kVbUnfix = 2.3283064365386963e-10f;   // 2^-32

// Slot of key b in the workgroup's hash table (linear probing), or -1 when
// its first kVbProbes slots hold other keys: such a record is counted (and
// later placed) by a global add of its own.  A chunk is up to 8192
// neighbouring layer-pixels of one view, whose bins lie in a band of tiles.
__device__ inline int vbin_slot(int *hkey, int b) {
    int h = (int)(((uint32_t)b * 2654435761u) >> (32 - kVbHashBits));
    for (int probe = 0; probe < kVbProbes; ++probe) {
        const int old = atomicCAS(&hkey[h], -1, b);
        if (old == -1 || old == b) return h;
        h = (h + 1) & (kVbHash - 1);
    }
    return -1;
}

// The workgroup's view and first layer-pixel, views slowest.  The chunks in
// flight together add to the same bins' counters; dispatched round-robin,
// each XCD's share of them is spread over a whole layer.  (In an XCD-aware
// order, or with the views fastest, an XCD's chunks fall on a few counter
// lines and both passes take 1.8 times as long.)
template <int KPT>
__device__ inline void vbin_chunk(const ViewsParams &p, int &m, int64_t &q0) {
    constexpr int chunk = KPT * kVbThreads;
    const int cpv = (int)((p.N + chunk - 1) / chunk);
    m = (int)blockIdx.x / cpv;
    q0 = (int64_t)((int)blockIdx.x - m * cpv) * chunk;
}

__global__ void __launch_bounds__(256) k_vbin_zero(const ViewsParams p) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    // cursor[nbins] is the records' total, then the scatter's count of listed pieces
    // (nbins is a multiple of 4, so the last block reaches both)
    if (i < p.nbins + 4) p.cursor[i] = 0u;
}

// KPT layer-pixels per thread.  What bounds both passes is the rate of global
// adds, ~25 per ns whatever their locality, one per distinct bin of a chunk:
// at 1080p chunks of 8192 make a third of the adds that chunks of 1024 do.
template <int KPT>
__global__ void __launch_bounds__(kVbThreads) k_vbin_count(const ViewsParams p) {
    __shared__ int hkey[kVbHash];
    __shared__ uint32_t hcnt[kVbHash];
    for (int i = threadIdx.x; i < kVbHash; i += kVbThreads) {
        hkey[i] = -1;
        hcnt[i] = 0u;
    }
    __syncthreads();
    int m;
    int64_t q0;
    vbin_chunk<KPT>(p, m, q0);
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
        const int64_t q = q0 + k * kVbThreads + threadIdx.x;
        if (q >= p.N) break;
        float fx, fy;
        int ix, iy, l;
        if (vbin_footprint(p, m, (int)q, p.depth[q], fx, fy, ix, iy, l)) {
            const int b = vbin_bin(p, m, ix, iy), sl = vbin_slot(hkey, b);
            atomicAdd(sl >= 0 ? &hcnt[sl] : &p.cursor[b], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kVbHash; i += kVbThreads)
        if (hkey[i] >= 0) atomicAdd(&p.cursor[hkey[i]], hcnt[i]);
}

// A tile's records lie in one run, its four bins in order; which run is of no
// matter (the tile sums do not depend on it), so a workgroup sums its 256
// tiles' counts, takes that many slots off the running total with one add and
// scans the tiles inside.  (Ordered prefix sums by a single workgroup took
// 80 us for the 65 280 bins of eight 1080p views, this takes 6 us.)
__global__ void __launch_bounds__(256) k_vbin_scan(const ViewsParams p) {
    __shared__ uint32_t wave_sum[4], base;
    const int t = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool live = 4 * t < p.nbins;
    const uint4 c = live ? reinterpret_cast<const uint4 *>(p.cursor)[t] : make_uint4(0u, 0u, 0u, 0u);
    const uint32_t s = c.x + c.y + c.z + c.w;
    uint32_t inc = s;                            // inclusive scan over the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = __shfl_up(inc, off);
        if (lane >= off) inc += v;
    }
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    if (threadIdx.x == 0) base = atomicAdd(p.total, wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3]);
    __syncthreads();
    uint32_t run = base + inc - s;
#pragma unroll
    for (int w = 0; w < 3; ++w) run += (w < wave) ? wave_sum[w] : 0u;
    if (!live) return;
    p.start[t] = run;
    reinterpret_cast<uint4 *>(p.cursor)[t] = make_uint4(run, run + c.x, run + c.x + c.y, run + c.x + c.y + c.z);
}

template <int KPT>
__global__ void __launch_bounds__(kVbThreads) k_vbin_write(const ViewsParams p) {
    __shared__ int hkey[kVbHash];
    __shared__ uint32_t hcnt[kVbHash];
    __shared__ uint32_t hbase[kVbHash];
    for (int i = threadIdx.x; i < kVbHash; i += kVbThreads) {
        hkey[i] = -1;
        hcnt[i] = 0u;
    }
    __syncthreads();
    int m;
    int64_t q0;
    vbin_chunk<KPT>(p, m, q0);
    const uint32_t cap = (uint32_t)(p.V * p.N);      // both passes bin alike: never reached
    uint32_t at[KPT];                                // hash slot and rank in its bin
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
        at[k] = ~0u;
        const int64_t q = q0 + k * kVbThreads + threadIdx.x;
        if (q >= p.N) continue;
        float fx, fy;
        int ix, iy, l;
        if (!vbin_footprint(p, m, (int)q, p.depth[q], fx, fy, ix, iy, l)) continue;
        const int b = vbin_bin(p, m, ix, iy), sl = vbin_slot(hkey, b);
        if (sl >= 0) {
            at[k] = ((uint32_t)sl << 16) | atomicAdd(&hcnt[sl], 1u);
        } else {
            const uint32_t slot = atomicAdd(&p.cursor[b], 1u);
            if (slot < cap) p.rec[slot] = (int)q;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kVbHash; i += kVbThreads)
        if (hkey[i] >= 0) hbase[i] = atomicAdd(&p.cursor[hkey[i]], hcnt[i]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KPT; ++k) {
        if (at[k] == ~0u) continue;
        const uint32_t slot = hbase[at[k] >> 16] + (at[k] & 0xffffu);
        if (slot < cap) p.rec[slot] = (int)(q0 + k * kVbThreads + threadIdx.x);
    }
}

// A contribution in 2^-32 units, rounded to the nearest (ties to even).  For
// |c| < 2^19 (QUICK) by one double fma: adding 1.5 * 2^52 leaves the integer
// in the low 51 bits (the constant's low word is zero, so taking its bits out
// is one 32-bit subtraction), three instructions where the general conversion
// of a float to 64 bits takes over ten; the same integer either way.
template <bool QUICK>
__device__ inline unsigned long long vbin_fixed(float c) {
    if constexpr (QUICK) {
        const double d = fma((double)c, 4294967296.0, 6755399441055744.0);
        return __builtin_bit_cast(unsigned long long, d) - 0x4338000000000000ull;
    } else {
        return (unsigned long long)__float2ll_rn(c * kVbFix);
    }
}

// What bounds it: VALU instructions (the footprint in double and 16
// conversions per record, ~60 % of the time) beside the LDS adds, with the
// gathers hidden only by waves in flight: 32 KiB of sums and 512 threads, so
// four workgroups fill a CU's wave slots (64 KiB tiles, with 6 % fewer
// records read twice, ran at half the waves and 14 % longer; 256 or 1024
// threads and two or four records at a time were slower too).  Eight 1080p
// views of a 1080p LDM of 4 layers, under the profiler: 1.43 -> 0.73 ms, the
// counting and writing passes 0.37 -> 0.22 and 0.47 -> 0.26; the whole call 2.34 ->
// 1.17 ms without it.
// PL: the distance of the channels' planes where the tile fits it (the adds'
// offsets are then immediates), 0: as the layers ask.
template <int PL>
__global__ void __launch_bounds__(kVbTileThreads) k_vbin_tile(const ViewsParams p) {
    // four planes of [L][th][tw] (r, g, b, alpha) sums, 2^-32: one per channel, so
    // the lanes of one add, at scattered pixels, spread over all LDS banks
    // (with a pixel's four sums adjacent each add reached a quarter of them)
    extern __shared__ unsigned long long tacc[];
    // XCD-aware order: each XCD walks one band of tile rows, whose records
    // come from a band of LDM rows that stays in its L2
    const int t = xcd_order(blockIdx.x, gridDim.x);
    int m = 0;
    for (int i = 1; i < p.V; ++i) m = (t >= p.tbase[i]) ? i : m;
    const int ntx = p.ntx[m], nty = p.nty[m];
    const int lt = t - p.tbase[m];
    const int tx = lt % ntx, ty = lt / ntx;
    const int tw = 1 << kVbLog2Tw, th = p.th, tpix = tw * th;
    const int plane = PL > 0 ? PL : p.L * tpix;
    const int x0 = tx * tw, y0 = ty * th;
    const int vw = p.vW[m], vh = p.vH[m];
    const unsigned xlim = (unsigned)min(tw, vw - x0), ylim = (unsigned)min(th, vh - y0);
    {
        for (int i = threadIdx.x; i < p.L * tpix; i += kVbTileThreads)
#pragma unroll
            for (int c = 0; c < 4; ++c) tacc[c * plane + i] = 0ull;
    }
    __syncthreads();
    const VbinRanges ranges = vbin_ranges(p, t, tx, ty, ntx, nty);
    const uint32_t total = ranges.cum[5];
    for (uint32_t k = threadIdx.x; k < total; k += (uint32_t)kVbTileThreads) {
        // the record is the layer-pixel's index: its footprint is recomputed
        // by the same function the binning passes ran (so it is the one they
        // binned) and its payload read from the LDM; an index out of range is
        // only a record never written
        const int q = p.rec[ranges.at(k)];
        if ((unsigned)q >= (unsigned)p.N) continue;
        const float d = p.depth[q];
        const float *c = p.color + (int64_t)q * 3;
        const float4 v = make_float4(c[0], c[1], c[2], p.alpha[q]);
        float fx, fy;
        int ix, iy, l;
        if (!vbin_footprint(p, m, q, d, fx, fy, ix, iy, l)) continue;
        const float w[4] = {(1.0f - fx) * (1.0f - fy), fx * (1.0f - fy), (1.0f - fx) * fy, fx * fy};
        const int lx = ix - x0, ly = iy - y0;
        const bool inx[2] = {(unsigned)lx < xlim, (unsigned)(lx + 1) < xlim};
        const bool iny[2] = {(unsigned)ly < ylim, (unsigned)(ly + 1) < ylim};
        unsigned long long *d0 = tacc + ((l * th + ly) * tw + lx);
        auto add = [&](auto quick) {
            constexpr bool Q = decltype(quick)::value;
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4) {
                if (!(inx[t4 & 1] && iny[t4 >> 1])) continue;
                unsigned long long *dst = d0 + (t4 >> 1) * tw + (t4 & 1);
                atomicAdd(dst, vbin_fixed<Q>(w[t4] * v.x));
                atomicAdd(dst + plane, vbin_fixed<Q>(w[t4] * v.y));
                atomicAdd(dst + 2 * plane, vbin_fixed<Q>(w[t4] * v.z));
                atomicAdd(dst + 3 * plane, vbin_fixed<Q>(w[t4] * v.w));
            }
        };
        // payloads under 2^18 (and finite) convert by a double add
        const float big = fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)));
        const bool quick = big < 262144.0f && !__builtin_isnan(v.x + v.y + v.z + v.w);
        if (__all(quick)) add(std::true_type{});
        else add(std::false_type{});
    }
    __syncthreads();
    for (int i = threadIdx.x; i < tpix; i += kVbTileThreads) {
        const int lx = i % tw, ly = i / tw;
        const int x = x0 + lx, y = y0 + ly;
        if (x >= vw || y >= vh) continue;
        float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
        for (int l = 0; l < p.L; ++l) {
            const unsigned long long *e = &tacc[(l * th + ly) * tw + lx];
            const float4 s = make_float4((float)(long long)e[0] * kVbUnfix,
                                         (float)(long long)e[plane] * kVbUnfix,
                                         (float)(long long)e[2 * plane] * kVbUnfix,
                                         (float)(long long)e[3 * plane] * kVbUnfix);
            const float w = T * s.w;
            c0 = fmaf(w, s.x, c0);
            c1 = fmaf(w, s.y, c1);
            c2 = fmaf(w, s.z, c2);
            T *= 1.0f - s.w;
        }
        const int64_t o = (int64_t)y * vw + x;
        float *rgb = p.rgb[m];
        rgb[o * 3 + 0] = c0;
        rgb[o * 3 + 1] = c1;
        rgb[o * 3 + 2] = c2;
        if (p.acc[m] != nullptr) p.acc[m][o] = 1.0f - T;
    }
}

}  // namespace

hipError_t launch_vbin(const ViewsParams &p, hipStream_t s) {
    hipLaunchKernelGGL(k_vbin_zero, dim3(p.nbins / 256 + 1), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // layer-pixels per thread: as many as leave ~8 workgroups per CU
    const int64_t per = p.N * p.V / ((int64_t)kVbThreads * 2048);
    auto passes = [&](auto kpt) {
        constexpr int K = decltype(kpt)::value;
        const int64_t cpv = (p.N + K * kVbThreads - 1) / (K * kVbThreads);
        const dim3 g((unsigned)(cpv * p.V)), b(kVbThreads);
        hipLaunchKernelGGL(k_vbin_count<K>, g, b, 0, s, p);
        hipError_t pe = hipGetLastError();
        if (pe != hipSuccess) return pe;
        hipLaunchKernelGGL(k_vbin_scan, dim3((p.nbins / 4 + 255) / 256), dim3(256), 0, s, p);
        if ((pe = hipGetLastError()) != hipSuccess) return pe;
        hipLaunchKernelGGL(k_vbin_write<K>, g, b, 0, s, p);
        return hipGetLastError();
    };
    e = per >= 16 ? passes(std::integral_constant<int, 16>{})
      : per >= 4 ? passes(std::integral_constant<int, 4>{}) : passes(std::integral_constant<int, 1>{});
    return e;
}

hipError_t launch_render_to_views(const ViewsParams &p, hipStream_t s) {
    if (p.binned) {
        hipError_t e = launch_vbin(p, s);
        if (e != hipSuccess) return e;
        // the distance of the sums' planes, fixed where it can be
        const int tile_sums = p.L * p.th * p.tw;
        const dim3 tg((unsigned)p.tbase[p.V]), tb(kVbTileThreads);
        auto tile = [&](auto pl) {
            constexpr int PL = decltype(pl)::value;
            const size_t lds = ((size_t)3 * (PL > 0 ? PL : tile_sums) + tile_sums) * 8;
            hipLaunchKernelGGL(k_vbin_tile<PL>, tg, tb, lds, s, p);
        };
        if (tile_sums <= 1024) tile(std::integral_constant<int, 1024>{});
        else tile(std::integral_constant<int, 0>{});
        return hipGetLastError();
    }
    const int64_t n4 = p.ws_floats / 4;
    const int zb = (int)((n4 + 255) / 256 < 8192 ? (n4 + 255) / 256 : 8192);
    hipLaunchKernelGGL(k_views_zero, dim3(zb > 0 ? zb : 1), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_splat, dim3((unsigned)(((p.N + 255) / 256) * p.V)), dim3(256), 0, s, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_views_composite, dim3((unsigned)((p.max_view_pixels + 255) / 256), p.V),
                       dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace qk
