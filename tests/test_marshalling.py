"""Cameras, feature maps and levels as the C structures hold them, from arrays
of other types, orders and strides."""

import ctypes
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2411_16680_amd import lib


def _cam(K, E, w=640, h=480):
    return SimpleNamespace(K=K, E=E, width=w, height=h)


K = np.arange(9, dtype=np.float64).reshape(3, 3) + 0.1
E = np.arange(16, dtype=np.float64).reshape(4, 4) - 0.7


@pytest.mark.parametrize("K_,E_", [
    (K, E),
    (np.asfortranarray(K), np.asfortranarray(E)),
    (np.repeat(K, 2, axis=1)[:, ::2], np.flip(np.flip(E, 0).copy(), 0)),
    (K.astype(">f8"), E.astype(">f8")),
    (K.tolist(), E.tolist()),
])
def test_camera_bytes(K_, E_):
    cams = lib._cameras([_cam(K_, E_), _cam(K_, E_, -1, 2 ** 31)])
    for c in (lib.make_camera(_cam(K_, E_)), cams[0], cams[1]):
        assert list(c.K) == K.reshape(-1).tolist()
        assert list(c.E) == E.reshape(-1).tolist()
    assert (cams[0].width, cams[0].height) == (640, 480)
    assert (cams[1].width, cams[1].height) == (-1, -2 ** 31)
    assert ctypes.sizeof(cams) == 2 * ctypes.sizeof(lib.qk_camera)


def test_camera_types_and_sizes():
    c = lib.make_camera(_cam(K.astype(np.float32), np.arange(16).reshape(4, 4)))
    assert list(c.K) == K.astype(np.float32).astype(np.float64).reshape(-1).tolist()
    assert list(c.E) == [float(i) for i in range(16)]
    assert len(lib._cameras([])) == 0
    with pytest.raises(ValueError):
        lib.make_camera(_cam(np.zeros((3, 4)), E))
    with pytest.raises(ValueError):
        lib.make_camera(_cam(K, np.zeros((3, 4))))


def test_maps_and_levels():
    torch = pytest.importorskip("torch")
    for dt, code in ((torch.float32, lib.QK_F32), (torch.bfloat16, lib.QK_BF16), (torch.float16, 99)):
        f = torch.zeros(5, 7, 8, dtype=dt)
        m = lib._fmap(f)
        assert (m.data, m.dtype, m.H, m.W, m.C) == (f.data_ptr(), code, 5, 7, 8)
    assert lib._fmap(torch.zeros(5, 7)).C == 0
    F, d, a = torch.zeros(2, 3, 4, 8), torch.zeros(2, 3, 4), torch.zeros(2, 3, 4)
    for args, C in (((F, d, a), 8), ((None, d, None), 0), ((F, None, a), 8), ((F, None, None), 8)):
        l = lib.make_ldm(*args)
        assert (l.L, l.H, l.W, l.C, l.dtype) == (2, 3, 4, C, lib.QK_F32)
        assert [l.F, l.depth, l.alpha] == [None if t is None else t.data_ptr() for t in args]
    with pytest.raises(ValueError):
        lib.make_ldm(F, torch.zeros(3, 4), None)
