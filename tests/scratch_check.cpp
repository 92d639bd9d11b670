// The C-ABI's workspaces against a stand-in for the HIP runtime with a fixed
// amount of device memory: what a call allocates, frees and waits for, and which
// way the backward takes.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "quark.h"
#include "uf_params.h"

static size_t g_memory = (size_t)1 << 40, g_live = 0;
static std::map<void *, size_t> g_blocks;
static int g_allocs = 0, g_frees = 0, g_syncs = 0;
static bool g_capturing = false;
static qk::BwdParams g_bwd;
static int fails = 0;

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipMalloc(void **p, size_t n) {
    ++g_allocs;
    if (g_live + n > g_memory) return hipErrorOutOfMemory;
    *p = std::malloc(1);
    g_blocks[*p] = n;
    g_live += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    ++g_frees;
    g_live -= g_blocks.at(p);
    g_blocks.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { ++g_syncs; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++g_syncs; return g_capturing ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
}

namespace qk {
hipError_t launch_update_fuse(const UFParams &, int, int, int, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_update_fuse_batch(const UFParams *, const UFBatch &, int, int, int, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_fp8_scales(const F8Params &, hipStream_t) { return hipSuccess; }
hipError_t launch_fold_weights(const FoldParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_composite(const CompParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_composite_backward(const CompBwdParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_update_fuse_backward(const BwdParams &p, hipStream_t) { g_bwd = p; return hipSuccess; }
hipError_t launch_ldm_init(const InitParams &, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_render_ibr(const RenderParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_render_to_views(const ViewsParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_residual_conv(const ConvParams &, int, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_layer_collapse(const CollapseParams &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_ray_encoding(const RayParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_upsample2x(const Up2Params &, hipStream_t) { return hipSuccess; }
hipError_t launch_ldm_decode(const DecodeParams &, hipStream_t) { return hipSuccess; }
hipError_t scratch_address(int, float **out) { static float s[16]; *out = s; return hipSuccess; }
}  // namespace qk

#define P(a) ((float *)(uintptr_t)(a))
#define CHECK(c) do { if (!(c)) { std::printf("line %d: " #c " (%s)\n", __LINE__, qk_last_error()); ++fails; } } while (0)

static qk_camera camera(double tx, int w, int h) {
    qk_camera c;
    std::memset(&c, 0, sizeof(c));
    c.K[0] = c.K[4] = 50.0;
    c.K[2] = 0.5 * w;
    c.K[5] = 0.5 * h;
    c.K[8] = 1.0;
    for (int i = 0; i < 4; ++i) c.E[5 * i] = 1.0;
    c.E[3] = -tx;
    c.width = w;
    c.height = h;
    return c;
}

// One backward of V views, L layers of 128 x 256, 16 channels; calls made of the
// allocator and waits are counted afresh.
static qk_status backward(qk_context *ctx, int V, int L, int map_w = 256, int map_h = 128) {
    const int H = 128, W = 256, C = 16;
    qk_camera cams[16], nov = camera(0.05, W, H);
    qk_feature_map fm[16];
    float *df[16];
    for (int m = 0; m < V; ++m) {
        cams[m] = camera(0.1 * m, W, H);
        fm[m] = {P(0x100000000 + 0x10000000 * (uintptr_t)m), QK_F32, map_h, map_w, C};
        df[m] = P(0x200000000 + 0x10000000 * (uintptr_t)m);
    }
    qk_weights w = {P(0x1000), P(0x2000), P(0x3000), P(0x4000), P(0x5000), P(0x6000), P(0x7000), C, C, 1, C};
    qk_weight_grads dw = {P(0x8000), P(0x9000), P(0xa000), P(0xb000), P(0xc000), P(0xd000), P(0xe000)};
    qk_ldm in = {P(0x300000000), P(0x400000000), P(0x500000000), L, H, W, C, QK_F32};
    qk_ldm out = {P(0x310000000), P(0x410000000), P(0x510000000), L, H, W, C, QK_F32};
    qk_ldm din = {P(0x320000000), P(0x420000000), P(0x520000000), L, H, W, C, QK_F32};
    g_allocs = g_frees = g_syncs = 0;
    return qk_update_fuse_backward(ctx, nullptr, V, cams, fm, &nov, 0.5f, 20.0f, &w, QK_UPDATE_RESIDUAL, &in, &out,
                                   P(0x600000000), nullptr, &din, df, &dw);
}

static qk_status views(qk_context *ctx, int L, int H, int W) {
    qk_camera cam = camera(0.1, W, H), nov = camera(0.05, W, H);
    qk_ldm_decoded ld = {P(0x300000000), P(0x400000000), P(0x500000000), L, H, W};
    qk_view_image vo;
    std::memset(&vo, 0, sizeof(vo));
    vo.rgb = P(0x600000000);
    vo.H = H;
    vo.W = W;
    g_allocs = g_frees = g_syncs = 0;
    return qk_render_to_views(ctx, nullptr, 1, &cam, &nov, &ld, &vo);
}

int main() {
    qk_context *ctx = nullptr;
    const int V = 4, L = 8;                     // 16.8 M sample-gradient floats
    const size_t rows = (size_t)4 * 16 * V * L * 128 * 256;

    // room for all: sorted, and nothing more on later calls
    CHECK(qk_context_create(0, 0, &ctx) == QK_OK);
    CHECK(backward(ctx, V, L) == QK_OK);
    CHECK(g_bwd.ds != nullptr);
    const int blocks = g_bwd.blocks;
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds != nullptr);
    CHECK(g_allocs == 0 && g_frees == 0 && g_syncs == 0);
    // under capture a larger problem than ever takes the way that needs no allocation
    CHECK(backward(ctx, 2, 2 * L) == QK_OK);
    g_capturing = true;
    CHECK(backward(ctx, 6, 2 * L) == QK_OK);
    CHECK(g_bwd.ds == nullptr && g_allocs == 0 && g_frees == 0 && g_syncs == 0);
    g_capturing = false;
    CHECK(backward(ctx, 6, 2 * L) == QK_OK && g_bwd.ds != nullptr);
    CHECK(qk_context_destroy(ctx) == QK_OK);
    CHECK(g_live == 0);

    // memory for the small workspace alone: refused once, then neither asked for
    // nor waited for; the same workgroups, so the same weight gradients
    g_memory = rows;
    CHECK(qk_context_create(0, 0, &ctx) == QK_OK);
    CHECK(backward(ctx, V, L) == QK_OK);
    CHECK(g_bwd.ds == nullptr && g_bwd.blocks == blocks);
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds == nullptr);
    CHECK(g_allocs == 0 && g_frees == 0 && g_syncs == 0);
    g_capturing = true;
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds == nullptr);
    g_capturing = false;
    CHECK(qk_context_destroy(ctx) == QK_OK);
    CHECK(g_live == 0);
    g_memory = (size_t)1 << 40;

    // a cap that leaves room for the sorted scatter: a later call that has to have
    // the room gets it, and the backward goes on without
    CHECK(qk_context_create(0, rows + ((size_t)48 << 20), &ctx) == QK_OK);
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds != nullptr);
    CHECK(views(ctx, 8, 1024, 2048) == QK_OK);  // 64 MiB of records
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds == nullptr && g_bwd.blocks == blocks);
    CHECK(g_allocs == 0 && g_frees == 0 && g_syncs == 0);
    CHECK(views(ctx, 8, 1024, 2048) == QK_OK && g_allocs == 0);
    CHECK(views(ctx, 16, 2048, 4096) == QK_ENOMEM);      // 512 MiB: past the cap in any case
    CHECK(qk_context_destroy(ctx) == QK_OK);
    CHECK(g_live == 0);

    // the same after a captured backward: its graph holds the workspace, which stays
    CHECK(qk_context_create(0, rows + ((size_t)48 << 20), &ctx) == QK_OK);
    CHECK(backward(ctx, V, L) == QK_OK);
    g_capturing = true;
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds != nullptr && g_allocs == 0 && g_syncs == 0);
    g_capturing = false;
    const float *held = g_bwd.ds;
    CHECK(views(ctx, 8, 1024, 2048) == QK_ENOMEM);
    CHECK(backward(ctx, V + 2, L) == QK_OK && g_bwd.ds == nullptr && g_frees == 0);
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds == held && g_frees == 0);
    CHECK(qk_context_destroy(ctx) == QK_OK);
    CHECK(g_live == 0);

    // the same where the device's memory is what ends
    g_memory = rows + ((size_t)48 << 20);
    CHECK(qk_context_create(0, 0, &ctx) == QK_OK);
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds != nullptr);
    CHECK(views(ctx, 8, 1024, 2048) == QK_OK);
    CHECK(backward(ctx, V, L) == QK_OK && g_bwd.ds == nullptr);
    CHECK(backward(ctx, V, L) == QK_OK && g_allocs == 0 && g_frees == 0 && g_syncs == 0);
    CHECK(qk_context_destroy(ctx) == QK_OK);
    CHECK(g_live == 0);

    // long sums of the weight gradients are written in two parts, whatever memory is
    // left, and the workspace holds them for any number of views
    CHECK(qk_context_create(0, 0, &ctx) == QK_OK);
    CHECK(backward(ctx, V, 31) == QK_OK && g_bwd.parts == 1);      // 31 items a wave
    CHECK(backward(ctx, V, 32) == QK_OK && g_bwd.parts == 2 && g_bwd.blocks == blocks);
    CHECK(backward(ctx, V + 2, 47) == QK_OK && g_bwd.parts == 1);  // 768 workgroups
    CHECK(backward(ctx, V + 2, 48) == QK_OK && g_bwd.parts == 2);
    CHECK(g_bwd.comp - g_bwd.partials == (ptrdiff_t)2 * g_bwd.blocks * qk::kGradTiles * qk::kGradTileElems);
    CHECK(qk_context_destroy(ctx) == QK_OK);

    // samples count up to 10^7 texels from a map's corner: the binning knows no such
    // limit, so larger maps take the atomics
    g_memory = (size_t)1 << 40;
    CHECK(qk_context_create(0, 0, &ctx) == QK_OK);
    CHECK(backward(ctx, V, L, 10000000, 1) == QK_OK && g_bwd.ds != nullptr && !g_bwd.wide);
    CHECK(backward(ctx, V, L, 10000001, 1) == QK_OK && g_bwd.ds == nullptr && !g_bwd.wide);
    CHECK(backward(ctx, V, L, 1, 10000001) == QK_OK && g_bwd.ds == nullptr && !g_bwd.wide);
    CHECK(qk_context_destroy(ctx) == QK_OK);

    std::printf("%d failures\n", fails);
    return fails != 0;
}
