"""The node-order task list at its capacity (16 P + 2^20 tasks): whole-sphere
Gaussians on a full sphere at order 11 make a task at each of the 3,072 nodes
of the split level, so 343 of them just fit and 400 do not.  Nearly all of
these tasks pass through the part of the list that its workgroups share."""
import ctypes as C

import numpy as np
import pytest

from paper_2606_29794_amd import _abi as A

pytestmark = pytest.mark.gpu

NODES = 3072


@pytest.fixture(scope="module")
def setting():
    from paper_2606_29794_amd.raster import Camera, Rasterizer
    cam = Camera(np.eye(3, dtype=np.float32), np.zeros(3, np.float32), np.zeros(3, np.float32), A.HP_CAM_FULL,
                 2 * np.pi, np.pi, 11)
    return Rasterizer(), cam


def _project(R, cam, P):
    import torch
    from paper_2606_29794_amd.raster import Gaussians
    from tests.test_gpu_async_bin import _whole_sphere_scene
    g = Gaussians(*[torch.as_tensor(a, device="cuda") for a in _whole_sphere_scene(P)])
    proj = R.preprocess(g, cam)
    assert float(R.projected_arrays(proj, P)[2].min()) >= 3.14
    return proj


def test_tasks_past_the_capacity(setting):
    import torch
    from paper_2606_29794_amd.raster import _p, _stream
    R, cam = setting
    P = 400
    assert NODES * P > 16 * P + 2 ** 20
    print("task overflow at order 11, P", P, flush=True)
    proj, m, v = _project(R, cam, P), R.mask(cam), cam.view()
    ws_n = A.lib().hp_bin_sorted_workspace_bytes(P, 11, R.prm.tile_log2)
    ws = torch.empty(ws_n, dtype=torch.uint8, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    cap = 1 << 20
    vals = torch.full((cap,), -7, dtype=torch.int32, device="cuda")
    ranges = torch.full((m.n_tiles, 2), 9, dtype=torch.int32, device="cuda")
    A.call("hp_bin_sorted", A.HP_BIN_ALL, _p(proj), P, C.byref(v), C.byref(R.prm), _p(R.grid(11)), _p(m.buf),
           _p(vals), _p(ranges), m.n_tiles, cap, _p(cnt), _p(ws), ws_n, _stream())
    got = C.c_int64(0)
    assert A.lib().hp_check_count(_p(cnt), cap, C.byref(got), _stream()) == A.HP_ERR_CAPACITY
    assert got.value == np.iinfo(np.int64).max
    assert int((vals != -7).sum()) == 0 and int(ranges.abs().sum()) == 0


def test_tasks_just_below_the_capacity(setting):
    R, cam = setting
    P = 343
    assert NODES * P <= 16 * P + 2 ** 20 < NODES * (P + 1) - 16
    print("task capacity at order 11, P", P, flush=True)
    proj, m = _project(R, cam, P), R.mask(cam)
    vals, ranges, n = R.bin_sorted(proj, P, cam)
    assert n == P * m.n_tiles
    r = ranges[: m.n_tiles].long()
    assert bool((r[:, 1] - r[:, 0] == P).all()) and int(r[0, 0]) == 0 and bool((r[1:, 0] == r[:-1, 1]).all())
    # every tile's list is the Gaussians by depth, ties by id
    depth = R.projected_arrays(proj, P)[1].cpu().numpy()
    order = np.lexsort((np.arange(P), depth)).astype(np.int32)
    import torch
    want = torch.as_tensor(order, device="cuda")
    assert bool((vals[:n].view(m.n_tiles, P) == want).all())
