"""A composited step of a small level, its layers split over a workgroup's waves, against
the same rows inside a level too large for that: cameras given on the level's own
grid see the same pixels, so every output has the same bits."""

import numpy as np
import pytest

import test_parity_gpu as tp
from paper_2411_16680_amd import lib, runner, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return lib.Context(0)


# C, heads, V, W, L, rows of the split level, rows of the other (past twice the
# workgroups that split)
CASES = [(8, 1, 3, 65, 5, 3, 600), (8, 1, 2, 64, 2, 4, 1600), (16, 1, 2, 33, 13, 5, 900), (32, 1, 3, 50, 7, 4, 500),
         (32, 4, 3, 49, 9, 4, 500), (32, 2, 2, 16, 2, 6, 1600), (64, 1, 3, 33, 6, 5, 300), (64, 4, 2, 20, 4, 5, 400)]


@pytest.mark.parametrize("prec,form", [("fp32", "standard"), ("fp32", "folded"), ("bf16", "standard"),
                                       ("bf16", "folded")])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "C%d-h%d-V%d-W%d-L%d" % c[:5])
def test_same_bits_as_unsplit(ctx, case, prec, form):
    C, heads, V, W, L, rows, many = case
    if form == "folded" and heads > 1:
        pytest.skip("one head")
    tp._say("split bits", case, prec, form)
    sc = synth.make_custom(V=V, H=many, W=W, C=C, L=L, seed=60 + C + L, heads=heads, head_dim=C // heads,
                           feat_hw=(40, 60), dtype="bf16" if prec == "bf16" else "f32")
    lvl = sc.levels[0]
    dl = runner.level_to_device(lvl)
    wts = lib.make_weights(dl.weights, heads=heads)
    novel = lambda h: synth.Camera(np.array([[W, 0, W / 2], [0, W, rows / 2], [0, 0, 1.0]]), sc.novel.E, W, h)

    def run(h):
        cut = [t[:, :h].contiguous() for t in (dl.F, dl.depth, dl.alpha)]
        out = [torch.empty_like(t) for t in cut]
        rgb, acc = torch.empty((h, W, 3), device="cuda"), torch.empty((h, W), device="cuda")
        lib.update_fuse(ctx, sc.in_cams, dl.feats, novel(h), sc.near, sc.far, wts, cut, out, precision=prec,
                        attn_form=form, rgb_out=rgb, acc_out=acc)
        torch.cuda.synchronize()
        return [t[:, :rows] for t in out] + [rgb[:rows], acc[:rows]]

    for a, b in zip(run(rows), run(many)):
        assert torch.equal(a, b)
