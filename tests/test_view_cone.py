"""The bounding cone that the binning drops Gaussians by (csrc/hp_cone.h),
compiled for the host and compared with the oracle's tiles: every active tile
of every kind of camera, with its cap radius on top, lies inside the cone."""
import ctypes as C
import math
import os
import subprocess

import numpy as np
import pytest

import oracle as O
from paper_2606_29794_amd import _abi as A
from paper_2606_29794_amd import scenes as SC

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2606_29794_amd", "csrc")


@pytest.fixture(scope="module")
def cone(tmp_path_factory):
    d = tmp_path_factory.mktemp("cone")
    src = d / "cone.cpp"
    src.write_text('#include "hp_cone.h"\nextern "C" void cone(const hp_view* v, int kt, float* o) '
                   '{ HpCone c = hp_view_cone(v, kt); o[0] = c.sr; o[1] = c.cr; }\n')
    so = str(d / "cone.so")
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", so], check=True)
    L = C.CDLL(so)

    def f(cam, kt):
        v = A.hp_view()
        v.cam_type, v.fov_x, v.fov_y, v.order = cam["cam_type"], cam["fov_x"], cam["fov_y"], cam["order"]
        out = (C.c_float * 2)()
        L.cone(C.byref(v), kt, out)
        return float(out[0]), float(out[1])
    return f


CAMS = [(SC.CAM_FULL, 360, 180), (SC.CAM_FISHEYE, 60, 60), (SC.CAM_FISHEYE, 180, 100), (SC.CAM_FISHEYE, 220, 220),
        (SC.CAM_FISHEYE, 360, 360), (SC.CAM_PINHOLE, 10, 6), (SC.CAM_PINHOLE, 60, 36), (SC.CAM_PINHOLE, 90, 120),
        (SC.CAM_PINHOLE, 179, 3)]


@pytest.mark.parametrize("kind,fx,fy", CAMS)
@pytest.mark.parametrize("order", [2, 4, 5, 6, 8])
def test_cone_holds_every_active_tile(cone, kind, fx, fy, order):
    cam = dict(SC.make_camera(np.random.default_rng(1), order, kind, fov_x=math.radians(fx), fov_y=math.radians(fy)))
    kt = O.tile_order(order)
    sr, cr = cone(cam, kt)
    assert abs(sr * sr + cr * cr - 1.0) < 1e-6
    cam["fov_x"], cam["fov_y"] = float(np.float32(cam["fov_x"])), float(np.float32(cam["fov_y"]))
    act = O.tile_active(order, O.mask(cam)).astype(bool)
    c, r = O.tile_caps(order)
    half = math.atan2(sr, cr)
    if half >= 0.5 * math.pi - 1e-6:
        return  # the whole sphere: nothing is dropped
    axis_angle = np.arccos(np.clip(c[act] @ np.array([0.0, 0.0, 1.0]), -1, 1))
    assert (axis_angle + r[act]).max(initial=0.0) < 2.0 * half


def test_cone_is_narrow_where_the_view_is(cone):
    """A 60-degree pinhole at Nside 2048 keeps the directions within 36
    degrees of its axis: the corner of the frustum and two tile radii."""
    fx = math.radians(60.0)
    cam = SC.make_camera(np.random.default_rng(1), 11, SC.CAM_PINHOLE, fov_x=fx, fov_y=SC.pinhole_fov_y(fx))
    assert math.degrees(2 * math.atan2(*cone(cam, 7))) < 36.0
