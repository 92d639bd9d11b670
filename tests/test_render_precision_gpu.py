"""The final render's blend in full float32, against the FP64 oracle: images of one
colour each, one opaque layer and equal blend logits, so that the sums over texels
and views make the error (the constant 1 / 255, whose float is 5.9e-8 off, is
taken as the float it is).

A rounding is 2.4e-8 of its value in the root mean square (up to 2^-24, over
mantissas spread evenly).  A view's sample has about 8 (four weights, four
products), independent from view to view; the sum over V views rounds V times at
sizes that grow to the result's, V / 3 at its size; the quotient, its product with
the sum and with the constant 3 times: 2.4e-8 sqrt(8 / V + V / 3 + 3).  (With each
texel added to the views' sum by itself there are 4 V of those roundings: 1.2e-7
at 16 views.)"""

import numpy as np
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


@pytest.mark.parametrize("V", [4, 5, 8, 9, 16])
def test_blend(ctx, V):
    err = []
    for seed in range(8):
        rs = synth.make_render(V=V, W=128, H=72, s=2, L=1, seed=20 + 100 * seed + V, arc=0.2)
        for im in rs.images:
            im[..., :3] = im[0, 0, :3] // 2 + 128
        rs.depth_logit[:] = -30.0                # the far plane
        rs.sigma_logit[:] = 30.0
        rs.blend_logit[:] = 0.0
        inside = (slice(18, 54), slice(32, 96))  # of every image
        got = tr._gpu_render(ctx, rs)["rgb"][inside].astype(np.float64)
        ref = tr._oracle(rs)["rgb"][inside] * (255.0 * float(np.float32(1.0 / 255.0)))
        assert np.min(ref) > 0.5
        err.append(np.mean(((got - ref) / ref) ** 2))
    err, bound = np.sqrt(np.mean(err)), 2.4e-8 * np.sqrt(8 / V + V / 3 + 3)
    tr._say("blend", V, f"{err:.2e} of {bound:.2e}")
    assert err <= bound
