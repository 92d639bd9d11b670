"""The final render of layers whose logits take 2 GiB and more, which keeps the view
counts' own kernels (offsets count from a tile's first row).

The logits' grid is an odd multiple of the output's, so every output pixel reads
one element exactly, and the logits there are those of a small render on the
output's grid; all others are large random numbers.  Both renders do the same
arithmetic on the same numbers: the same bits."""

import os
import shutil
import subprocess

import numpy as np
import pytest

import test_render_gpu as tr
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RULE = """
#include <cstdio>
#include <hip/hip_runtime.h>
#include "uf_params.h"
int main() {
    int V, h, w, H, rows;
    unsigned long at;
    while (std::scanf("%d %d %d %d %d %lu", &V, &h, &w, &H, &rows, &at) == 6)
        std::printf("%d", (int)qk::render_vectors(V, h, w, H, rows, at));
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rule(tmp_path):
    """Which calls read vectors: by alignment, and by what a tile spans."""
    (tmp_path / "rule.cpp").write_text(RULE)
    exe = str(tmp_path / "rule")
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                        os.path.join(ROOT, "paper_2411_16680_amd", "csrc"), str(tmp_path / "rule.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    cases = [((8, 288, 512, 1080, 16, 4096), 1), ((8, 288, 512, 1080, 16, 4104), 0),
             ((6, 288, 512, 1080, 16, 4104), 1), ((6, 288, 512, 1080, 16, 4100), 0),
             ((5, 288, 512, 1080, 16, 4100), 1), ((8, 8192, 8192, 1080, 16, 4096), 1),
             ((16, 40000, 40000, 1080, 16, 4096), 1), ((16, 40000, 40000, 40, 16, 4096), 0),
             ((8, 8192, 8192, 16, 16, 4096), 0), ((8, 8192, 8191, 16, 16, 4096), 1),
             ((1, 1, (1 << 29) - 1, 1, 4, 4096), 1), ((1, 1, 1 << 29, 1, 4, 4096), 0)]
    r = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c, _ in cases), capture_output=True,
                       text=True, timeout=60)
    assert r.stdout == "".join(str(v) for _, v in cases)


@pytest.mark.gpu
@pytest.mark.parametrize("V", [8, 5])
def test_same_bits_as_a_small_render(V):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = lib.Context(0)
    H, W, ky, kx = 90, 160, 97, 81
    h, w = H * ky, W * kx
    assert h * w * V >= 1 << 29
    rs = synth.make_render(V=V, W=W, H=H, L=1, lowres_hw=(H, W), img_hw=(120, 200), seed=31)
    small = tr._gpu_render(ctx, rs)
    imgs, lg = tr._device(rs)
    big = []
    for t in lg:
        b = torch.full((1, h, w) + tuple(t.shape[3:]), 50.0, device="cuda").uniform_(-50.0, 50.0)
        b[:, ky // 2::ky, kx // 2::kx] = t
        big.append(b)
    out = [torch.full((H, W, 3), float("nan"), device="cuda")] + [torch.full((H, W), float("nan"), device="cuda")
                                                                  for _ in range(2)]
    tr._say("large logits", V, h, w)
    lib.render_ibr(ctx, rs.in_cams, imgs, rs.novel, rs.near, rs.far, tuple(big), out[0], acc_out=out[1],
                   depth_out=out[2])
    torch.cuda.synchronize()
    for k, t in zip(("rgb", "acc", "depth"), out):
        assert np.array_equal(small[k], t.cpu().numpy()), k
