"""Parity of the float32 standard form with one head (its projections applied
to the query and to the weighted sum of the samples) at the edges of its
tiles, for one view upwards and for both numbers of rows a workgroup takes at
C = 64, with and without the composite and with the blend-weight logits.

Bars: test_parity_gpu's float32 bounds for the step.  Logits: a sum of C
products of a query and a sample, each of about unit size with C-term sums
behind them, so absolute error 1e-4 (C = 64: 64 * 64 * 2^-24 * a few)."""

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


# (C, V, H, W, L): widths around the 64 G pixels of a workgroup, odd heights;
# C = 64 with one row per workgroup (few tiles) and two (the last row alone)
CASES = [(8, 1, 3, 257, 2), (8, 3, 5, 31, 3), (16, 2, 7, 129, 3), (16, 5, 2, 128, 1),
         (32, 1, 4, 65, 2), (32, 6, 5, 63, 3), (64, 1, 3, 65, 2), (64, 3, 5, 64, 3),
         (64, 2, 257, 130, 2), (64, 4, 515, 60, 1)]


@pytest.mark.parametrize("logits", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "C%d-V%d-%dx%d-L%d" % c)
def test_reassociated_form(ctx, case, logits):
    C, V, H, W, L = case
    tp._say("reassociated", case, logits)
    sc = synth.make_custom(V=V, H=H, W=W, C=C, L=L, seed=50 + C + V)
    lvl = sc.levels[0]
    dl = runner.level_to_device(lvl)
    blend = torch.full((L, H, W, V), float("nan"), device="cuda") if logits else None
    lib.update_fuse(ctx, sc.in_cams, dl.feats, sc.novel, sc.near, sc.far, dl.weights,
                    (dl.F, dl.depth, dl.alpha), (dl.F_out, dl.depth_out, dl.alpha_out),
                    precision="fp32", attn_form="standard", rgb_out=dl.rgb, acc_out=dl.acc,
                    blend_logit_out=blend)
    gpu = runner.level_outputs_numpy(dl)
    ref = oracle.run_level(sc, lvl)
    tp.compare(gpu, ref, "fp32", sc, lvl, label=f"reassociated {case} logits={logits}")
    if logits:
        want = oracle.update_fuse(sc.in_cams, sc.novel, sc.near, sc.far, lvl, want_logits=True)
        err = np.max(np.abs(blend.cpu().numpy() - want["blend_logit"]))
        tp._say("logits max-abs", f"{err:.3g}")
        assert err <= 1e-4
