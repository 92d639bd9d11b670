"""Render to the input views at the edges of its binned form: layer counts
around the tile heights 8, 1 and the largest (a tile's sums at a fixed
distance up to 32 layers, then as the layers ask), the counting passes with
one, four and sixteen layer-pixels per thread, and payloads on both sides of
the fixed-point conversions' limit.  Bar and oracle as in test_views_gpu."""

import numpy as np
import pytest

import test_views_gpu as tv
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return lib.Context(0)


CASES = {
    "tile-height-8": dict(V=2, W=65, H=33, L=4, seed=31),
    "tile-height-1-L32": dict(V=2, W=37, H=9, L=32, seed=32),
    "tile-height-1-L33": dict(V=2, W=37, H=9, L=33, seed=33),
    "L65": dict(V=2, W=21, H=7, L=65, seed=34),
    "most-layers-L128": dict(V=2, W=33, H=6, L=128, seed=35),
    "four-per-thread": dict(V=4, W=640, H=480, L=4, seed=36),
    "sixteen-per-thread": dict(V=8, W=1024, H=530, L=4, view_hw=(265, 512), seed=37),
    # many layer-pixels in few view pixels: long runs in one bin
    "crowded": dict(V=2, W=256, H=192, L=4, view_hw=(5, 7), seed=38),
}


@pytest.mark.parametrize("name", list(CASES))
def test_binned_edges(ctx, name):
    vs = synth.make_views(**CASES[name])
    tv._say("case", name, f"V={vs.V} ldm {vs.depth.shape} views {vs.view_hw[0]}")
    a, _ = tv._compare(name, ctx, vs)
    b, _ = tv._gpu(ctx, vs)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("scale", [2.0 ** 17, 2.0 ** 18, 2.0 ** 24])
def test_large_payloads(ctx, scale):
    vs = synth.make_views(V=2, W=48, H=32, L=3, seed=39)
    vs.color = (vs.color * np.float32(scale)).astype(np.float32)
    vs.color[:, ::3] *= np.float32(-1.0)
    tv._compare(f"payload-{scale:g}", ctx, vs)
