"""The backward's optional workspace on the device: a context capped so that a
render to the input views has to have the room it took, the backward with it and
without it.  Bars: test_scatter_gpu's (map gradients, another order of the same
sums); the render is bitwise reproducible."""

import numpy as np
import pytest

import test_backward_gpu as tb
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def level():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sc = synth.make_custom(V=4, H=131, W=251, C=16, L=8, seed=90)
    return sc, tb._upstream(sc.levels[0], 6, ldm=False)


def test_workspace_is_given_up_under_a_cap(level):
    sc, ups = level
    lvl = sc.levels[0]
    rows = 4 * 16 * 4 * lvl.L * lvl.H * lvl.W
    capped, free = lib.Context(0, workspace_bytes=rows + (48 << 20)), lib.Context(0)
    v = synth.make_views(V=8, W=960, H=540, L=5, seed=3)

    def views(ctx):                       # 83 MB of records
        dev = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
               for a in (v.depth, v.alpha, v.color)]
        out = [torch.zeros((c.height, c.width, 3), device="cuda") for c in v.in_cams]
        lib.render_to_views(ctx, v.in_cams, v.novel, *dev, out)
        torch.cuda.synchronize()
        return out

    tb._say("capped")
    a = tb._run_backward(capped, sc, lvl, mode="residual", **ups)
    shown = views(capped)
    b = tb._run_backward(capped, sc, lvl, mode="residual", **ups)
    c = tb._run_backward(free, sc, lvl, mode="residual", **ups)
    for x, y in zip(shown, views(free)):
        assert torch.equal(x, y)
    for g in (a, b):
        for x, y in zip(g["feats"], c["feats"]):
            assert np.max(np.abs(x - y)) <= 1e-5 * np.max(np.abs(y))


@pytest.mark.parametrize("C,V,H,W,L", [(16, 4, 131, 251, 8), (16, 5, 125, 203, 8), (8, 3, 243, 401, 7),
                                       (8, 6, 190, 301, 6)])
def test_weight_gradients_whatever_memory_is_left(C, V, H, W, L):
    """Each is a sum in a fixed order, also where the maps' gradients take the
    other way: the same bits."""
    sc = synth.make_custom(V=V, H=H, W=W, C=C, L=L, seed=91)
    lvl = sc.levels[0]
    ups = tb._upstream(lvl, 7)
    tb._say("weights", C, V)
    small = lib.Context(0, workspace_bytes=16 * L * H * W + (8 << 20))
    a = tb._run_backward(lib.Context(0), sc, lvl, mode="residual", **ups)
    b = tb._run_backward(small, sc, lvl, mode="residual", **ups)
    for k in tb.NAMES:
        assert np.array_equal(a[k], b[k]), k
