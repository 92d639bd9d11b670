"""Residual CNN block at the edges of its tiles (30 x 8 and 30 x 16 outputs, the
16-row ones where their rounds are fewer).  Bar and oracle as in
test_conv_gpu."""

import numpy as np
import pytest

import oracle
import test_conv_gpu as tc
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return lib.Context(0)


@pytest.mark.parametrize("W", [28, 29, 30, 31, 32, 61])
@pytest.mark.parametrize("H", [7, 8, 9])
def test_small_tiles(ctx, H, W):
    F, W1, W2 = synth.make_conv_block(L=2, H=H, W=W, seed=100 * H + W)
    tc._compare(f"{H}x{W}", tc._gpu(ctx, F, W1, W2), oracle.residual_conv(F, W1, W2))


@pytest.mark.parametrize("L,H,W", [(150, 16, 31), (300, 16, 30), (140, 17, 59), (90, 33, 29)])
def test_many_layers_large_tiles(ctx, L, H, W):
    F, W1, W2 = synth.make_conv_block(L=L, H=H, W=W, seed=L + H + W)
    got = tc._gpu(ctx, F, W1, W2)
    assert np.all(np.isfinite(got))
    for l in (0, L // 2, L - 1):
        tc._compare(f"L{L}-{H}x{W}-layer{l}", got[l:l + 1], oracle.residual_conv(F[l:l + 1], W1, W2))
