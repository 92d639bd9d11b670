// k_conv.hip -- residual CNN block of a fusion block (Sec. 3.3: the
// one-to-many attention is interleaved with residual 3x3 convolutional
// blocks, mirroring a Transformer's MLP block): per layer,
// F_out = F + W2 * gelu(W1 * N(F)) with N the per-pixel RMS normalisation
// over the channels (unit gain, eps 1e-6, as the attention's pre-norm),
// 3x3 kernels and zero padding, gelu(x) = x Phi(x) (erf by Hastings'
// approximation, 1.5e-7), C = 32 channels,
// bfloat16 storage and MFMA operands, float32 accumulation.
//
// An implicit GEMM on v_mfma_f32_16x16x32_bf16: for each of the 9 taps, the
// A operand is the tap's W^T (16 output channels x 32 input channels, one
// fragment per half of the outputs) and the B operand 16 pixels x 32 input
// channels -- one 16-byte LDS read per lane, since pixels are channel-last.
//
// A persistent workgroup of four waves walks tiles of 30 x TY outputs.  It
// stages the 34 x (TY + 4) input region normalised (2-pixel halo, zeros outside
// the image; a quad of lanes holds one pixel's four 8-channel chunks and sums its
// squares with two lane exchanges), computes the first convolution on the 32 x
// (TY + 2) region the second one needs (two column blocks of 16; GELU, zeros
// outside the image -- the second convolution pads with zeros too -- rounded to
// bfloat16 as its operand), then the second convolution, adds the un-normalised
// input and stores bfloat16.  A wave takes one column block and half of the rows
// with the kernel's 18 fragments in registers, and walks down the rows: the
// three shifted operands of an input row serve the three output rows it reaches,
// 18 products per three LDS reads, each sum still taken tap by tap in order.
//
// What bounds it: with the fragments in LDS every product read 1.5 operands and
// the LDS pipe was busy throughout; now it is vector work (GELU, normalisation,
// 51 % busy) beside the matrix cores (24 %).  16 layers of 480x270: 193 -> 134 us
// (570 TFLOP/s), the same bits.  The tile's height is chosen per call
// (conv_tile_rows).  Both kernels' fragments in registers (144) spilled and took 298
// us; the next tile's input read ahead changed nothing, two workgroups per CU overlap
// each other's staging; eight waves on a tile where there is one per unit changed
// nothing either.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "uf_params.h"

namespace qk {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kC = 32, TX = kConvTileCols, MX = TX + 2, IX = TX + 4;
constexpr int NFRAG = 2 * 9 * 2 * 64;            // [conv][tap][half of C_out][lane]

// Place of 16-byte chunk q of column c in an LDS row (64 bytes a pixel): the
// chunks are permuted so that the 16-byte reads of 16 neighbouring columns spread
// over all banks; by the column alone, so a walk down the rows adds constants.
__device__ inline int chunk_at(int c, int q) { return c * 4 + (q ^ ((c >> 2) & 3)); }

__device__ inline f32x4 mma(const uint4 &a, const uint4 &b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ inline float bf2f(uint16_t h) { return __uint_as_float((unsigned)h << 16); }

// the value of lane (l ^ D) of the quad
template <int D>
__device__ inline float quad_xor(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), D == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true));
}

// gelu(x) = x Phi(x) = x (1 + erf(x / sqrt 2)) / 2, with erf from Hastings'
// rational approximation (Abramowitz and Stegun 7.1.26): for z >= 0,
// erf z = 1 - t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) e^{-z^2},
// t = 1 / (1 + p z), |error| <= 1.5e-7 -- far below the bfloat16 rounding the
// result gets as an operand; odd in z.
__device__ inline float gelu(float x) {
    const float z = fabsf(x) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
    float poly = fmaf(1.061405429f, t, -1.453152027f);
    poly = fmaf(poly, t, 1.421413741f);
    poly = fmaf(poly, t, -0.284496736f);
    poly = fmaf(poly, t, 0.254829592f);
    const float e = 1.0f - poly * t * __expf(-z * z);      // erf |x| / sqrt 2
    return 0.5f * x * (1.0f + copysignf(e, x));
}

// Weight fragments: lane (c, g) of fragment (conv, tap, half) holds
// W[tap][8g .. 8g+7][16 half + c] (input channels along K).
__global__ void __launch_bounds__(256) k_conv_frag(const ConvParams p) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= NFRAG) return;
    const int lane = i & 63, half = (i >> 6) & 1, tap = (i >> 7) % 9, conv = (i >> 7) / 9;
    const float *Wm = conv ? p.W2 : p.W1;
    const int c = lane & 15, g = lane >> 4;
    bf16x8 v;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = (__bf16)Wm[(tap * kC + 8 * g + k) * kC + 16 * half + c];
    p.frag[i] = __builtin_bit_cast(uint4, v);
}

// A wave's 3x3 convolution of ROWS rows of one column block of 16 pixels, from
// LDS rows of PITCH pixels: lane (n, g) holds output channels 4g .. 4g+3 and 16
// + 4g .. of pixel n.  row(ro) is called as the first input row of output row
// ro arrives, emit(ro, a0, a1) when its sum is complete; taps are added in
// order.
template <int ROWS, int PITCH, typename Row, typename Emit>
__device__ __forceinline__ void conv_rows(const uint4 *src, int col, int g, const uint4 (&w)[9][2],
                                          Row &&row, Emit &&emit) {
    f32x4 acc[3][2];
    const uint4 *at[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) at[dx] = src + chunk_at(col + dx, g);
#pragma unroll
    for (int i = 0; i < ROWS + 2; ++i) {
        uint4 b[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) b[dx] = at[dx][i * PITCH * 4];
        if (i < ROWS) {
            row(i);
            acc[i % 3][0] = acc[i % 3][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const int ro = i - dy;
                if (ro < 0 || ro >= ROWS) continue;
                acc[ro % 3][0] = mma(w[3 * dy + dx][0], b[dx], acc[ro % 3][0]);
                acc[ro % 3][1] = mma(w[3 * dy + dx][1], b[dx], acc[ro % 3][1]);
            }
        if (i >= 2) emit(i - 2, acc[(i - 2) % 3][0], acc[(i - 2) % 3][1]);
    }
}

// four floats to bfloat16, a pair per conversion
__device__ inline uint2 pack4(float a, float b, float c, float d) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return make_uint2(__builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{a, b}), bf16x2)),
                      __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{c, d}), bf16x2)));
}

template <int TY>
__global__ void __launch_bounds__(256, 2) k_residual_conv(const ConvParams p) {
    constexpr int MY = TY + 2, IY = TY + 4;
    __shared__ uint4 s_in[IY * IX * 4];          // normalised input
    // GELU of the first convolution (the last two columns' operands run 2 pixels
    // over; their results are not used)
    __shared__ uint4 s_mid[(MY * MX + 2) * 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int cb = wave & 1, rh = wave >> 1;     // this wave's column block and half of the rows
    // a kernel's fragments in registers, read (from L1) for each tile: both at
    // once would take 144 registers and spill
    auto load_frags = [&](int conv, uint4 (&w)[9][2]) {
        const uint4 *f = p.frag + conv * 9 * 2 * 64;
        asm volatile("" : "+s"(f));              // not hoisted out of the tile loop
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) w[t][h] = f[(t * 2 + h) * 64 + lane];
    };
    const int per_layer = p.tiles_x * p.tiles_y;
    uint2 *mid2 = reinterpret_cast<uint2 *>(s_mid);

    // each XCD (workgroups are dispatched round-robin over the 8) takes one
    // contiguous range of tiles, as many as its share of the workgroups: neighbours
    // share their halos in its L2, and no workgroup has a tile more than it must
    const int nb = (int)gridDim.x, r = (int)blockIdx.x & 7, q8 = nb >> 3, rem = nb & 7;
    const int before = r * q8 + min(r, rem), mine = q8 + (r < rem);
    const int64_t t_end = p.n_tiles * (before + mine) / nb;
    for (int64_t t = p.n_tiles * before / nb + ((int)blockIdx.x >> 3); t < t_end; t += mine) {
        const int l = (int)(t / per_layer);
        const int rem = (int)(t - (int64_t)l * per_layer);
        const int ty = rem / p.tiles_x, tx = rem - ty * p.tiles_x;
        const int x0 = tx * TX, y0 = ty * TY;
        const uint16_t *Fl = p.F + (int64_t)l * p.H * p.W * kC;
        uint16_t *Ol = p.F_out + (int64_t)l * p.H * p.W * kC;

        // the 4 lanes of a quad hold one pixel (256 and the last pass's cut are
        // multiples of 4, so quads stay whole)
        constexpr int NCH = IY * IX * 4, NSTAGE = (NCH + 255) / 256;
        uint4 v[NSTAGE];
#pragma unroll
        for (int k = 0; k < NSTAGE; ++k) {
            const int i = tid + 256 * k;
            const int pix = i >> 2, q = i & 3;
            const int rr = pix / IX, c = pix - rr * IX;
            const int y = y0 - 2 + rr, x = x0 - 2 + c;
            v[k] = make_uint4(0u, 0u, 0u, 0u);
            if (i < NCH && y >= 0 && y < p.H && x >= 0 && x < p.W)
                v[k] = *reinterpret_cast<const uint4 *>(Fl + ((int64_t)y * p.W + x) * kC + 8 * q);
        }
        __syncthreads();                         // the previous tile's reads are done
#pragma unroll
        for (int k = 0; k < NSTAGE; ++k) {
            const int i = tid + 256 * k;
            const unsigned wd[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
            float f[8], ss = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f[2 * j] = bf2f((uint16_t)(wd[j] & 0xffffu));
                f[2 * j + 1] = bf2f((uint16_t)(wd[j] >> 16));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) ss = fmaf(f[j], f[j], ss);
            ss += quad_xor<1>(ss);
            ss += quad_xor<2>(ss);
            const float rn = rsqrtf(ss * (1.0f / kC) + 1e-6f);   // outside: 0 * rn = 0
            const uint2 lo = pack4(f[0] * rn, f[1] * rn, f[2] * rn, f[3] * rn);
            const uint2 hi = pack4(f[4] * rn, f[5] * rn, f[6] * rn, f[7] * rn);
            const int rr = (i >> 2) / IX, c = (i >> 2) - rr * IX;
            if (i < NCH) s_in[rr * IX * 4 + chunk_at(c, i & 3)] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
        __syncthreads();

        // first convolution, rows rh MY / 2 .. of the middle region
        {
            const int m0 = rh * (MY / 2), mc = 16 * cb + n;
            const int x = x0 - 1 + mc;
            const bool in_x = x >= 0 && x < p.W;
            uint2 *mid_lo = mid2 + m0 * MX * 8 + 2 * chunk_at(mc, g >> 1) + (g & 1);
            uint2 *mid_hi = mid2 + m0 * MX * 8 + 2 * chunk_at(mc, 2 + (g >> 1)) + (g & 1);
            uint4 w[9][2];
            load_frags(0, w);
            conv_rows<MY / 2, IX>(s_in + m0 * IX * 4, mc, g, w, [](int) {},
                                  [&](int ro, const f32x4 &a0, const f32x4 &a1) {
                const int y = y0 - 1 + m0 + ro;
                uint2 o0 = make_uint2(0u, 0u), o1 = o0;
                if (in_x && y >= 0 && y < p.H) {
                    o0 = pack4(gelu(a0[0]), gelu(a0[1]), gelu(a0[2]), gelu(a0[3]));
                    o1 = pack4(gelu(a1[0]), gelu(a1[1]), gelu(a1[2]), gelu(a1[3]));
                }
                mid_lo[ro * MX * 8] = o0;
                mid_hi[ro * MX * 8] = o1;
            });
        }
        __syncthreads();

        // second convolution, residual, store: rows rh TY / 2 .. of the tile
        {
            const int r0 = rh * (TY / 2), c = 16 * cb + n, x = x0 + c;
            const bool in_x = c < TX && x < p.W;
            uint2 res[3][2];                     // the un-normalised input, two rows ahead of its use
            uint4 w[9][2];
            load_frags(1, w);
            conv_rows<TY / 2, MX>(s_mid + r0 * MX * 4, c, g, w,
                                  [&](int ro) {
                const int y = y0 + r0 + ro;
                res[ro % 3][0] = res[ro % 3][1] = make_uint2(0u, 0u);
                if (in_x && y < p.H) {
                    const uint16_t *src = Fl + ((int64_t)y * p.W + x) * kC + 4 * g;
                    res[ro % 3][0] = *reinterpret_cast<const uint2 *>(src);
                    res[ro % 3][1] = *reinterpret_cast<const uint2 *>(src + 16);
                }
            },
                                  [&](int ro, const f32x4 &a0, const f32x4 &a1) {
                const int y = y0 + r0 + ro;
                if (in_x && y < p.H) {
                    uint16_t *dst = Ol + ((int64_t)y * p.W + x) * kC + 4 * g;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const f32x4 &a = h ? a1 : a0;
                        const uint2 u = res[ro % 3][h];
                        *reinterpret_cast<uint2 *>(dst + 16 * h) =
                            pack4(a[0] + bf2f((uint16_t)(u.x & 0xffffu)), a[1] + bf2f((uint16_t)(u.x >> 16)),
                                  a[2] + bf2f((uint16_t)(u.y & 0xffffu)), a[3] + bf2f((uint16_t)(u.y >> 16)));
                    }
                }
            });
        }
    }
}

}  // namespace

hipError_t launch_residual_conv(const ConvParams &pin, int num_cu, bool frag_ready, hipStream_t s) {
    ConvParams p = pin;
    p.tiles_x = (p.W + TX - 1) / TX;
    const int64_t slots = 2 * (int64_t)(num_cu > 0 ? num_cu : 256);
    const int ty = conv_tile_rows(p.L, p.H, p.W, num_cu > 0 ? num_cu : 256);
    p.tiles_y = (p.H + ty - 1) / ty;
    p.n_tiles = (int64_t)p.L * p.tiles_x * p.tiles_y;
    hipError_t e;
    if (!frag_ready) {                           // else p.frag already holds them
        hipLaunchKernelGGL(k_conv_frag, dim3((NFRAG + 255) / 256), dim3(256), 0, s, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const unsigned blocks = (unsigned)(slots < p.n_tiles ? slots : p.n_tiles);
    const dim3 gr(blocks), bl(256);
    switch (ty) {
    case 2: hipLaunchKernelGGL(k_residual_conv<2>, gr, bl, 0, s, p); break;
    case 4: hipLaunchKernelGGL(k_residual_conv<4>, gr, bl, 0, s, p); break;
    case 6: hipLaunchKernelGGL(k_residual_conv<6>, gr, bl, 0, s, p); break;
    case 8: hipLaunchKernelGGL(k_residual_conv<8>, gr, bl, 0, s, p); break;
    case 10: hipLaunchKernelGGL(k_residual_conv<10>, gr, bl, 0, s, p); break;
    case 12: hipLaunchKernelGGL(k_residual_conv<12>, gr, bl, 0, s, p); break;
    default: hipLaunchKernelGGL(k_residual_conv<16>, gr, bl, 0, s, p); break;
    }
    return hipGetLastError();
}

}  // namespace qk
