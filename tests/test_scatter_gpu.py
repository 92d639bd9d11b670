"""The backward's feature-map gradients by sorting (large problems), at its
edges: views kept in registers and gathered again (V up to 4, more), maps of
another grid than the LDM, ragged tiles, crowded cells (several sorting
batches), tiles no sample reaches, a context whose cap forces the float
atomics, and maps of 2 GiB (64-bit addresses).

Bars: test_backward_gpu's against the FP64 oracle.  Sorted against atomics, and
64-bit against 32-bit addresses: the same float32 terms summed in another
order; sums of up to a few hundred terms, so 1e-5 of the largest element."""

import numpy as np
import pytest

import test_backward_gpu as tb
from paper_2411_16680_amd import lib, runner, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return lib.Context(0)


# (C, V, H, W, L, feat_hw): at least 16 M sample-gradient floats each
CASES = {
    "C16-V4": (16, 4, 131, 251, 8, None),
    "C16-V4-coarse-maps-crowded": (16, 4, 131, 251, 8, (17, 35)),
    "C16-V5-gathered-again": (16, 5, 125, 203, 8, (125, 190)),
    "C16-V1": (16, 1, 331, 509, 6, (301, 477)),
    "C8-V3": (8, 3, 243, 401, 7, None),
    "C8-V6-gathered-again": (8, 6, 190, 301, 6, (95, 151)),
    "C8-V2-fine-maps": (8, 2, 243, 601, 7, (486, 1201)),
}


def _scene(name):
    C, V, H, W, L, fhw = CASES[name]
    assert C * V * H * W * L >= 16000000
    return synth.make_custom(V=V, H=H, W=W, C=C, L=L, feat_hw=fhw, seed=70 + C + V)


@pytest.mark.parametrize("name", list(CASES))
def test_sorted_against_oracle(ctx, name):
    sc = _scene(name)
    lvl = sc.levels[0]
    tb._say("sorted", name)
    ups = tb._upstream(lvl, 5)
    gpu = tb._run_backward(ctx, sc, lvl, mode="residual", **ups)
    ref = tb._oracle(sc, lvl, ups, 0)
    tb._assert_close(tb._errors(gpu, ref), name)


def test_cap_falls_back_to_atomics(ctx):
    name = "C16-V4"
    sc = _scene(name)
    lvl = sc.levels[0]
    tb._say("capped", name)
    N = lvl.L * lvl.H * lvl.W
    small = lib.Context(0, workspace_bytes=16 * N + (8 << 20))     # no room for the samples' rows
    ups = tb._upstream(lvl, 6, ldm=False)
    a = tb._run_backward(ctx, sc, lvl, mode="paper", **ups)
    b = tb._run_backward(small, sc, lvl, mode="paper", **ups)
    for x, y in zip(a["feats"], b["feats"]):
        assert np.max(np.abs(x - y)) <= 1e-5 * np.max(np.abs(x))


def test_samples_outside_leave_zeros(ctx):
    """Every map pixel is written, also those of tiles no sample reaches."""
    sc = synth.make_custom(V=2, H=256, W=512, C=16, L=4, arc=3.0, radius=1.0, seed=77)
    lvl = sc.levels[0]
    tb._say("wide arc")
    ups = tb._upstream(lvl, 7, ldm=False)
    gpu = tb._run_backward(ctx, sc, lvl, mode="residual", **ups)
    ref = tb._oracle(sc, lvl, ups, 0)
    for g, r in zip(gpu["feats"], ref["feats"]):
        tb._say("untouched", int(np.sum(r == 0)), "of", r.size)
        assert np.all(g[r == 0] == 0)
        assert np.max(np.abs(g - r)) <= 2e-3 * np.max(np.abs(r))


def test_maps_of_two_gib(ctx):
    """64-bit addresses against the same call on the maps' corner: a camera
    given on a grid in that grid's pixels samples the same texels of both."""
    sc = synth.make_custom(V=2, H=24, W=40, C=16, L=3, feat_hw=(48, 64), seed=78)
    lvl = sc.levels[0]
    tb._say("2 GiB maps")
    big_hw = (4096, 8256)                                       # 2.02 GiB of float32 x 16
    dl = runner.level_to_device(lvl)
    g = torch.Generator().manual_seed(9)
    d_rgb = torch.randn((lvl.H, lvl.W, 3), generator=g).cuda()

    def cams(h, w):
        out = []
        for c in sc.in_cams:
            K = np.diag([64 / c.width, 48 / c.height, 1.0]) @ c.K      # on the corner's pixels
            out.append(synth.Camera(K, c.E, w, h))
        return out

    def run(feats, in_cams):
        lib.update_fuse(ctx, in_cams, feats, sc.novel, sc.near, sc.far, dl.weights,
                        (dl.F, dl.depth, dl.alpha), (dl.F_out, dl.depth_out, dl.alpha_out),
                        precision="fp32", rgb_out=dl.rgb)
        dfe = [torch.full_like(f, 7.0) for f in feats]
        d_in = tuple(torch.empty_like(t) for t in (dl.F, dl.depth, dl.alpha))
        dW = {k: torch.empty_like(v) for k, v in dl.weights.items()}
        lib.update_fuse_backward(ctx, in_cams, feats, sc.novel, sc.near, sc.far, dl.weights,
                                 (dl.F, dl.depth, dl.alpha), (dl.F_out, dl.depth_out, dl.alpha_out),
                                 d_in, dfe, dW, d_rgb=d_rgb)
        torch.cuda.synchronize()
        return dfe

    small = [torch.zeros((96, 160, 16), device="cuda") for _ in range(2)]
    for s, f in zip(small, dl.feats):
        s[:48, :64] = f
    a = run(small, cams(96, 160))
    # the forward takes maps under 1 GiB, so its outputs are kept from above
    fwd = (dl.F_out.clone(), dl.alpha_out.clone())
    big = []
    for f in dl.feats:
        b = torch.zeros(big_hw + (16,), device="cuda")
        b[:48, :64] = f
        big.append(b)
    dfe = [torch.full_like(f, 7.0) for f in big]
    d_in = tuple(torch.empty_like(t) for t in (dl.F, dl.depth, dl.alpha))
    dW = {k: torch.empty_like(v) for k, v in dl.weights.items()}
    lib.update_fuse_backward(ctx, cams(*big_hw), big, sc.novel, sc.near, sc.far, dl.weights,
                             (dl.F, dl.depth, dl.alpha), (fwd[0], dl.depth_out, fwd[1]),
                             d_in, dfe, dW, d_rgb=d_rgb)
    torch.cuda.synchronize()
    for x, y in zip(a, dfe):
        top = float(x.abs().max())
        assert top > 0
        # samples past the small corner's edge land on zeros of either map
        assert float((x[:95, :159] - y[:95, :159]).abs().max()) <= 1e-5 * top
