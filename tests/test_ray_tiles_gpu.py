"""The ray encoding where its 32-pixel pieces end: maps and low-resolution
grids of one pixel, one short of a half piece and of a piece, of one and one
past, and one larger than all the waves of a launch take at once; every
channel count and type, added to the map and through the low-resolution grid;
against the FP64 oracle.

Bar, derived as for the encoding's parity: with S = |f| + sum_i |Wr[i][c]|,
1e-6 + 4e-6 S for float32 maps, and 2^-8 of the value more for bfloat16."""

import numpy as np
import pytest

import oracle
from paper_2411_16680_amd import lib, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(V, C, dtype, hws, low=None):
    rs = synth.make_ray(V=V, W=64, H=36, levels=((1, C),), seed=C + V)
    Wr = rs.Wr[0]
    rng = np.random.default_rng(3 * C + V)
    dev, exact = [], []
    for h, w in hws:
        f = torch.from_numpy(rng.standard_normal((h, w, C)).astype(np.float32))
        f = f.to(torch.bfloat16) if dtype == "bf16" else f
        exact.append(f.double().numpy())
        dev.append(f.cuda())
    lib.ray_encoding(lib.Context(0), rs.in_cams, rs.novel, rs.near, rs.far,
                     torch.from_numpy(Wr).cuda(), dev, low_hw=low)
    torch.cuda.synchronize()
    for m, (d, f) in enumerate(zip(dev, exact)):
        h, w = hws[m]
        enc = (oracle.ray_encoding(rs.in_cams[m], rs.novel, rs.near, rs.far, Wr, h, w) if low is None else
               oracle.ray_encoding_lowres(rs.in_cams[m], rs.novel, rs.near, rs.far, Wr, low, h, w))
        ref = f + enc
        tol = 1e-6 + 4e-6 * (np.abs(f) + np.sum(np.abs(Wr.astype(np.float64)), axis=0))
        if dtype == "bf16":
            tol = tol + 2.0 ** -8 * (np.abs(ref) + tol)
        assert np.all(np.abs(d.double().cpu().numpy() - ref) <= tol), (m, h, w)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C", [8, 16, 32, 64])
def test_map_edges(C, dtype):
    _check(7, C, dtype, [(1, 1), (3, 5), (1, 16), (17, 1), (1, 31), (4, 8), (3, 11)])


@pytest.mark.parametrize("low", [(1, 1), (3, 5), (4, 4), (1, 17), (4, 8), (3, 11), (8, 16), (7, 19)])
@pytest.mark.parametrize("C", [8, 16, 32, 64])
def test_low_grid_edges(C, low):
    _check(2, C, "f32", [(9, 20), (8, 19)], low=low)


def test_more_pixels_than_the_launch_takes_at_once():
    _check(1, 8, "bf16", [(520, 513)])
