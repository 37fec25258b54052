"""hp_bin_sorted against hp_bin + hp_sort, bit for bit, over every route of
the sorted binning: Gaussians dropped by the mask's cone before the depth
sort, split levels of 12 to 12,288 nodes, workgroups with few and with many
tasks, and the smallest scenes."""
import math

import numpy as np
import pytest

from paper_2606_29794_amd import scenes as SC

pytestmark = pytest.mark.gpu

CAMS = {"full": (SC.CAM_FULL, 360, 180), "fisheye": (SC.CAM_FISHEYE, 200, 150), "narrow": (SC.CAM_FISHEYE, 50, 40),
        "pinhole": (SC.CAM_PINHOLE, 75, 50), "slit": (SC.CAM_PINHOLE, 8, 5)}


@pytest.fixture(scope="module")
def R():
    import torch
    from paper_2606_29794_amd import raster
    assert torch.cuda.is_available()
    return raster.Rasterizer()


def _lists(R, g, cam, mask_cam=None):
    """(vals, ranges) of hp_bin_sorted and of hp_bin + hp_sort."""
    proj = R.preprocess(g, cam)
    if mask_cam is not None:  # a mask of another field of view than the view's
        R._masks[cam.mask_key(R.prm.tile_log2)] = R.mask(mask_cam)
        R._created(("mask",) + cam.mask_key(R.prm.tile_log2))
    m = R.mask(cam)
    vals, ranges, n = R.bin_sorted(proj, g.P, cam)
    keys, v2, n2 = R.bin(proj, g.P, cam)
    r2 = R.sort(keys, v2, n2, m.n_tiles)
    assert n == n2
    return (vals[:n].cpu().numpy(), ranges.cpu().numpy()[:m.n_tiles]), (v2[:n2].cpu().numpy(),
                                                                       r2.cpu().numpy()[:m.n_tiles])


def _same(got, want):
    (v, r), (v2, r2) = got, want
    assert np.array_equal(v, v2)
    size = r[:, 1].astype(np.int64) - r[:, 0]
    assert np.array_equal(size, r2[:, 1].astype(np.int64) - r2[:, 0])
    assert np.array_equal(r[size > 0], r2[size > 0])  # an empty tile's start is free


@pytest.mark.parametrize("P", [1, 2, 63, 255, 256, 257, 6000])
@pytest.mark.parametrize("kind", sorted(CAMS))
@pytest.mark.parametrize("order", [3, 5, 6, 7, 8, 10, 11, 12])
def test_sorted_binning_equals_pairs_and_sort(R, order, kind, P):
    from paper_2606_29794_amd.raster import Camera, Gaussians
    if order == 12 and (kind in ("full", "fisheye") or P not in (2, 6000)):
        pytest.skip("201M-pixel masks: one narrow camera of each kind is enough")
    if order == 11 and kind == "full" and P != 257:
        pytest.skip("one full sphere at Nside 2048 is enough")
    t, fx, fy = CAMS[kind]
    rng = np.random.default_rng(100 * order + P)
    sc = SC.make_scene(P, 0, "log", 1.0, 20.0, 5 + P, log_scale_mu=-2.5, rng=rng)
    cam = Camera.from_dict(SC.make_camera(rng, order, t, fov_x=math.radians(fx), fov_y=math.radians(fy),
                                          center_radius=0.5))
    _same(*_lists(R, Gaussians.from_scene(sc), cam))


@pytest.mark.parametrize("order", [8, 11])
def test_large_discs(R, order):
    """Discs of 0.3 to pi radians: every workgroup has far more tasks than
    Gaussians, at both split levels of the node-order task list."""
    from paper_2606_29794_amd.raster import Camera, Gaussians
    rng = np.random.default_rng(order)
    sc = SC.make_scene(700, 0, "volume", 2.0, 6.0, 3, log_scale_mu=-0.3, rng=rng)
    cam = Camera.from_dict(SC.make_camera(rng, order, SC.CAM_FISHEYE, fov_x=math.radians(120), fov_y=math.radians(120)))
    _same(*_lists(R, Gaussians.from_scene(sc), cam))


def test_cone_comes_from_the_mask(R):
    """The lists follow the mask, also when the view names a narrower field of
    view than the mask was made for."""
    from paper_2606_29794_amd.raster import Camera, Gaussians
    rng = np.random.default_rng(11)
    sc = SC.make_scene(5000, 0, "log", 1.0, 20.0, 4, rng=rng)
    d = SC.make_camera(rng, 8, SC.CAM_PINHOLE, fov_x=math.radians(100), fov_y=math.radians(100))
    wide, narrow = Camera.from_dict(d), Camera.from_dict(dict(d, fov_x=math.radians(21.0), fov_y=math.radians(21.0)))
    g = Gaussians.from_scene(sc)
    got, want = _lists(R, g, narrow, mask_cam=wide)
    _same(got, want)
    assert got[0].size == _lists(R, g, wide)[0][0].size


@pytest.mark.parametrize("kind", ["full", "pinhole"])
@pytest.mark.parametrize("P", [1, 63, 64, 65, 1023, 1024, 1025, 2048, 8191, 8192, 8193])
def test_lists_in_depth_order(R, P, kind):
    """Every tile's list by increasing depth and, among equal depths, by id,
    at the edges of the one-workgroup depth sort (waves, rounds, its largest
    scene and the first beyond), with a third of the depths shared."""
    from paper_2606_29794_amd.raster import Camera, Gaussians
    t, fx, fy = CAMS[kind]
    rng = np.random.default_rng(P)
    sc = SC.make_scene(P, 0, "log", 1.0, 20.0, 5 + P, log_scale_mu=-2.5, rng=rng)
    twin = rng.integers(0, P, P // 3)
    sc.mean[:, rng.choice(P, P // 3, replace=False)] = sc.mean[:, twin]
    cam = Camera.from_dict(SC.make_camera(rng, 6, t, fov_x=math.radians(fx), fov_y=math.radians(fy)))
    g = Gaussians.from_scene(sc)
    proj = R.preprocess(g, cam)
    depth = R.projected_arrays(proj, P)[1].cpu().numpy()
    vals, ranges, n = R.bin_sorted(proj, P, cam)
    v, r = vals[:n].cpu().numpy().astype(np.int64), ranges.cpu().numpy()[:R.mask(cam).n_tiles].astype(np.int64)
    tile = np.full(n, -1)
    for k, (a, b) in enumerate(r):
        tile[a:b] = k
    assert n == 0 or tile.min() >= 0
    key = list(zip(tile.tolist(), depth[v].tolist(), v.tolist()))
    assert all(a < b for a, b in zip(key, key[1:]) if a[0] == b[0])
