"""A composited step of a small level, whose layers are split over the waves of
a workgroup: layer counts that leave the last waves a layer short or without
any, widths around a wave's pixels, each channel count, head count and
precision, without the accumulated alpha, in place, and at the largest level
that is split and one past it.

Bars: test_parity_gpu's for the step (the colours of a wave's layers are summed
before the next wave's, in float, the same number of roundings).  In place and
not, the results are the same bits."""

import numpy as np
import pytest

import oracle
import test_parity_gpu as tp
from paper_2411_16680_amd import lib, runner, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return lib.Context(0)


def _scene(C, V, H, W, L, heads, dtype, seed):
    return synth.make_custom(V=V, H=H, W=W, C=C, L=L, seed=seed, heads=heads,
                             head_dim=C // heads, dtype=dtype)


# (C, heads, V, H, W, L)
CASES = [(8, 1, 2, 3, 63, 2), (8, 1, 3, 5, 65, 5), (8, 1, 1, 2, 129, 13),
         (16, 1, 2, 4, 31, 3), (16, 1, 3, 5, 33, 6), (32, 1, 2, 3, 15, 4), (32, 1, 3, 5, 17, 7),
         (32, 2, 2, 3, 49, 9), (32, 4, 2, 5, 16, 5), (64, 1, 2, 3, 17, 2), (64, 2, 3, 2, 31, 5),
         (64, 4, 2, 3, 48, 3)]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "C%d-h%d-V%d-%dx%d-L%d" % c)
def test_split_step(ctx, case, prec):
    C, heads, V, H, W, L = case
    tp._say("split", case, prec)
    sc = _scene(C, V, H, W, L, heads, "bf16" if prec == "bf16" else "f32", 70 + C + L)
    lvl = sc.levels[0]
    dl = runner.level_to_device(lvl)
    wts = lib.make_weights(dl.weights, heads=heads)
    for form in ("standard", "folded") if heads == 1 else ("standard",):
        lib.update_fuse(ctx, sc.in_cams, dl.feats, sc.novel, sc.near, sc.far, wts,
                        (dl.F, dl.depth, dl.alpha), (dl.F_out, dl.depth_out, dl.alpha_out),
                        precision=prec, attn_form=form, rgb_out=dl.rgb, acc_out=dl.acc)
        gpu = runner.level_outputs_numpy(dl)
        tp.compare(gpu, oracle.run_level(sc, lvl), prec, sc, lvl, label=f"split {case} {prec} {form}")
        # in place, without the accumulated alpha
        F, d, a = dl.F.clone(), dl.depth.clone(), dl.alpha.clone()
        rgb = torch.full_like(dl.rgb, float("nan"))
        lib.update_fuse(ctx, sc.in_cams, dl.feats, sc.novel, sc.near, sc.far, wts, (F, d, a), (F, d, a),
                        precision=prec, attn_form=form, rgb_out=rgb)
        torch.cuda.synchronize()
        for x, y in ((F, dl.F_out), (d, dl.depth_out), (a, dl.alpha_out), (rgb, dl.rgb)):
            assert torch.equal(x, y)


@pytest.mark.parametrize("H", [256, 257])
def test_last_level_that_is_split(ctx, H):
    """2 layers, C = 32, float32: 512 tiles of 16 pixels and one row more."""
    sc = _scene(32, 2, H, 32, 2, 1, "f32", 90)
    lvl = sc.levels[0]
    dl = runner.level_to_device(lvl)
    lib.update_fuse(ctx, sc.in_cams, dl.feats, sc.novel, sc.near, sc.far, dl.weights,
                    (dl.F, dl.depth, dl.alpha), (dl.F_out, dl.depth_out, dl.alpha_out),
                    precision="fp32", rgb_out=dl.rgb, acc_out=dl.acc)
    tp.compare(runner.level_outputs_numpy(dl), oracle.run_level(sc, lvl), "fp32", sc, lvl,
               label=f"split at {H} rows")
