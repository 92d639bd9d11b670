"""Residual CNN block at each height of its tiles (2, 4, 8, 10, 12 and 16 rows on
256 compute units, in this order), with a last tile row that is cut.  Bar and
oracle as in test_conv_gpu."""

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


@pytest.mark.parametrize("L,H,W", [(2, 41, 64), (5, 39, 61), (16, 37, 61), (60, 37, 31), (100, 33, 31),
                                   (8, 147, 253)])
def test_tile_heights(ctx, L, H, W):
    F, W1, W2 = synth.make_conv_block(L=L, H=H, W=W, seed=L + H + W)
    got = tc._gpu(ctx, F, W1, W2)
    assert np.all(np.isfinite(got))
    for l in sorted({0, L // 2, L - 1}):
        tc._compare(f"L{L}-{H}x{W}-layer{l}", got[l:l + 1], oracle.residual_conv(F[l:l + 1], W1, W2))
