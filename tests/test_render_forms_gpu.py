"""The final render's forms: each view count that has a kernel of its own and
one that has none, with images that samples leave on every side (the lanes
inside and the masked ones in one wave), images of one and two columns or rows,
of even and odd size, and logits that are only 4-byte aligned; against the
FP64 oracle.

Bar: that of the render's parity (RGB 1e-4, alpha 1e-5, depth 1e-5 relative):
the arithmetic is the same, a sample's position in double, its weights, the
softmax and the blend in float."""

import numpy as np
import pytest

import oracle
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"rgb": 1e-4, "acc": 1e-5, "depth": 1e-5}


def _check(rs, shift=0):
    ctx = lib.Context(0)
    imgs = [torch.from_numpy(im).cuda() for im in rs.images]
    lg = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda() for a in rs.logits]
    if shift:
        buf = torch.empty(lg[2].numel() + shift, device="cuda")
        off = buf[shift:].view(lg[2].shape)
        off.copy_(lg[2])
        lg[2] = off
    rgb = torch.full((rs.H, rs.W, 3), float("nan"), device="cuda")
    acc = torch.full((rs.H, rs.W), float("nan"), device="cuda")
    dep = torch.full((rs.H, rs.W), float("nan"), device="cuda")
    lib.render_ibr(ctx, rs.in_cams, imgs, rs.novel, rs.near, rs.far, tuple(lg), rgb,
                   acc_out=acc, depth_out=dep)
    torch.cuda.synchronize()
    ref = oracle.render_ibr(rs.in_cams, rs.images, rs.novel, rs.near, rs.far, *rs.logits, rs.H, rs.W)
    got = {"rgb": rgb, "acc": acc, "depth": dep}
    for k, tol in TOL.items():
        g = got[k].cpu().numpy()
        assert np.all(np.isfinite(g)), k
        d = np.abs(g - ref[k])
        if k == "depth":
            d = d / np.maximum(np.abs(ref[k]), 1e-30)
        assert float(d.max()) <= tol, (k, float(d.max()))


@pytest.mark.parametrize("V", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 16])
def test_view_counts(V):
    _check(synth.make_render(V=V, W=53, H=37, L=3, lowres_hw=(13, 18), img_hw=(41, 62), seed=100 + V))


@pytest.mark.parametrize("img_hw", [(1, 1), (1, 40), (40, 1), (2, 2), (2, 31), (30, 3), (24, 40), (25, 41)])
@pytest.mark.parametrize("V", [6, 9])
def test_image_sizes(img_hw, V):
    _check(synth.make_render(V=V, W=70, H=34, s=2, L=2, img_hw=img_hw, seed=7))


@pytest.mark.parametrize("V,shift", [(8, 1), (8, 2), (6, 1), (6, 2), (5, 1), (4, 3), (16, 2)])
def test_logits_aligned_to_4_bytes(V, shift):
    _check(synth.make_render(V=V, W=50, H=30, s=2, L=3, seed=20), shift=shift)


def test_output_smaller_than_the_logits():
    _check(synth.make_render(V=8, W=33, H=20, L=3, lowres_hw=(61, 97), img_hw=(60, 90), seed=21))
