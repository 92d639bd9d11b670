"""The depth gradient on smooth feature maps: texels of a large common value and
small differences between neighbours, which alone carry it.

With W_q = 0 the softmax is uniform, with only dLoss/dF' given the sample's
gradient is a V-th of W_v W_o^T dF', and the depth gradient is its product with
the taps' differences.  Those two products and the sum over C are chains of 16
float32 terms at most, the differences, weights and positions a rounding each;
taken as independent, under 10 roundings of 2^-24 reach a result relative to the
terms it sums, whose norm is at most sqrt(C) / 2 = 2 times the sum's: 1e-6 of the
norm, whatever the texels have in common.  (Differences taken after the products
lose that common part's roundings: 4e-5 at 10 and 0.01.)  Compared where every
view's sample is inside its map: at its edge the difference to the zeros outside
is the common value itself, and would drown the others."""

import numpy as np
import pytest

import test_backward_gpu as tb
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return lib.Context(0)


def _inside(sc, lvl):
    """Layer-pixels whose four taps lie inside the map in every view."""
    hw = [f.shape[:2] for f in lvl.feats]
    u, v = np.meshgrid(np.arange(lvl.W) + 0.5, np.arange(lvl.H) + 0.5)
    ok = np.ones(lvl.depth.shape, bool)
    for t, (h, w) in zip(lib.camera_tables(sc.in_cams, hw, sc.novel, lvl.H, lvl.W), hw):
        ray = np.tensordot(t[:9].reshape(3, 3), np.stack([u, v, np.ones_like(u)]), 1)
        p = ray[:, None] + t[9:, None, None, None] / lvl.depth.astype(np.float64)
        x, y = p[0] / p[2] - 0.5, p[1] / p[2] - 0.5
        ok &= (p[2] > 1e-6) & (x >= 0) & (x < w - 1) & (y >= 0) & (y < h - 1)
    return ok


# C, V, H, W, L: atomics with one view and with views gathered again, the sorted
# scatter with its taps kept and gathered again
SIZES = [(16, 1, 40, 56, 4), (8, 1, 40, 56, 4), (16, 5, 40, 56, 4), (8, 3, 40, 56, 4),
         (16, 4, 131, 251, 8), (16, 5, 125, 203, 8), (8, 3, 243, 401, 7)]


@pytest.mark.parametrize("common,diff", [(0.0, 1.0), (1.0, 0.01), (10.0, 0.01)])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "C%d-V%d-%dx%d-L%d" % s)
def test_depth_gradient(ctx, size, common, diff):
    C, V, H, W, L = size
    sc = synth.make_custom(V=V, H=H, W=W, C=C, L=L, seed=50 + C + V)
    lvl = sc.levels[0]
    r = np.random.default_rng(4)
    sign = np.where(r.random(C) < 0.5, -1.0, 1.0)
    lvl.feats = [(common * sign + diff * r.standard_normal(f.shape)).astype(np.float32) for f in lvl.feats]
    lvl.weights["Wq"] = np.zeros_like(lvl.weights["Wq"])
    ups = tb._upstream(lvl, 5, rgb=False)
    ups["dd_out"] = ups["da_out"] = None
    tb._say("smooth", size, common, diff)
    gpu = tb._run_backward(ctx, sc, lvl, mode="residual", **ups)
    ref = tb._oracle(sc, lvl, ups, 0)
    inside = _inside(sc, lvl)
    assert np.mean(inside) > 0.25
    err = np.linalg.norm((gpu["depth"] - ref["depth"])[inside]) / np.linalg.norm(ref["depth"][inside])
    tb._say(f"depth gradient {err:.2e}")
    assert err <= 1e-6
