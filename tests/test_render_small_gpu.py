"""The final render to small images, whose workgroups take tiles of 16 x 4 pixels, and
just past them (16 x 16): cut tiles in both directions, view counts known at
compile time, among them those that read a view's projection per layer, and not.
Bar and oracle as in test_render_gpu."""

import pytest

import test_render_gpu as tr
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return lib.Context(0)


@pytest.mark.parametrize("V", [1, 4, 7, 9, 12, 16])
@pytest.mark.parametrize("H,W", [(1, 1), (5, 33), (127, 128), (128, 127), (129, 128), (128, 129), (17, 900)])
def test_small(ctx, H, W, V):
    rs = synth.make_render(V=V, W=W, H=H, L=3, lowres_hw=(max(1, H // 3), max(1, W // 2)), img_hw=(45, 67),
                           seed=H + W + V)
    tr._compare(f"{H}x{W} V{V}", tr._gpu_render(ctx, rs), tr._oracle(rs))
