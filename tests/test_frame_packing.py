"""The packed frame arrays of the entry points against the field-by-field
builders (CPU): the same bytes for every kind of value they accept, the same
exceptions for what they refuse."""
import ctypes as C
import dataclasses

import numpy as np
import pytest
import torch

from paper_2503_01074_amd import _lib, api


def _geom(**over):
    g = api.SonarGeometry(r_min=0.5, r_max=20.0, n_range=512, n_azimuth=256, fov_az=2.2689, fov_el=0.349, fan_h=512,
                          fan_w=1024, seed_lo=7, seed_hi=9, frame_id=3, param_row=2, range_norm=1)
    return dataclasses.replace(g, **over)


def _hits(n=5):
    f = lambda: torch.zeros(n)
    return api.DeviceHits(f(), f(), f(), f(), f(), f(), torch.zeros(n, dtype=torch.int32))


def _either(fn):
    """The result's bytes, or the exception's type."""
    try:
        return bytes(fn())
    except Exception as e:   # noqa: BLE001
        return type(e)


@pytest.mark.parametrize("over", [
    {}, dict(r_max=np.float32(12.5), n_range=np.int64(77), gamma_k=np.int32(3)), dict(r_max=1e300), dict(r_min=-np.inf),
    dict(fov_az=float("nan")), dict(n_range=2 ** 40 + 5), dict(n_azimuth=-3), dict(seed_lo=-1, seed_hi=2 ** 70 + 4),
    dict(frame_id=2 ** 32 + 11), dict(speckle_mode=True), dict(n_range=3.5), dict(r_max="far"), dict(r_max=2),
    dict(path_factor=np.float64(1.0)), dict(range_norm=True), dict(range_norm=2.9), dict(param_row=None)])
def test_sonar_frames(over):
    g, h = _geom(**over), _hits()
    t = [torch.zeros(4) for _ in range(7)]
    for ptrs in ([None] * 7, t, [t[0], None, t[2], None, t[4], None, t[6]]):
        def packed():
            arr = (_lib.SonarFrame * 3)()
            api._pack_sonar(arr, 1, g, h, *ptrs)
            assert bytes(arr[0]) == bytes(arr[2]) == b"\0" * C.sizeof(_lib.SonarFrame)
            return arr[1]
        assert _either(packed) == _either(lambda: api._sonar_struct(g, h, *ptrs))


def test_sonar_frames_without_some_returns():
    h = _hits(0)
    h.ny = None
    arr = (_lib.SonarFrame * 1)()
    api._pack_sonar(arr, 0, _geom(), h)
    assert bytes(arr[0]) == bytes(api._sonar_struct(_geom(), h))


@pytest.mark.parametrize("row", [0, 3, np.int64(2), -1, 2 ** 33 + 1, 1.5, None])
def test_camera_frames(row):
    J, d, o = torch.zeros(3, 5, 7), torch.zeros(5, 7), torch.zeros(3, 5, 7)
    for extra in ([None] * 3, [J, o, d]):
        def packed():
            arr = (_lib.UwFrame * 1)()
            api._pack_uw(arr, 0, J, d, o, row, *extra)
            return arr[0]
        assert _either(packed) == _either(lambda: api._uw_struct(J, d, o, row, *extra))


@pytest.mark.parametrize("intr", [(1.0, 2.0, 3.0, 4.0), np.array([9.5, 8.5, 1.0, 2.0], np.float32), (1, 2, 3, 4),
                                  (1e300, 1.0, 1.0, 1.0), ("1", "2", "3", "4"), (1.0, 2.0, 3.0), (1.0, None, 2.0, 3.0),
                                  torch.tensor([3.0, 4.0, 5.0, 6.0])])
def test_conditioning_frames(intr):
    srgb, z = torch.zeros(6, 10, 4, dtype=torch.uint8), torch.zeros(6, 10)
    for args in ((srgb, z, z, z), (None, z, None, z), (srgb, None, z, None), (None, None, None, None, z, z)):
        def packed():
            arr = (_lib.CamFrame * 1)()
            api._pack_cam(arr, 0, 6, 10, intr, *args)
            return arr[0]
        assert _either(packed) == _either(lambda: api._cam_struct(6, 10, intr, *args))


@pytest.mark.parametrize("cls", [_lib.SonarFrame, _lib.UwFrame, _lib.CamFrame, _lib.CamOutFrame, _lib.RayFrame])
def test_frame_arrays_pass_unchanged(cls):
    arr = (cls * 3)()
    ptr, n, keep = _lib._frames(arr, cls)
    assert ptr is arr and n == 3 and keep is arr
