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
