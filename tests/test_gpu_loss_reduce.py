"""The loss's sums over the tiles' partials: one workgroup, or pieces of 1,024
first, on both sides of that rule and with lengths that fill the last piece or
do not.  Tiles of one pixel give as many partials as pixels at little cost."""
import math

import numpy as np
import pytest

from paper_2606_29794_amd import scenes as SC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fov,n", [(3.0, None), (141.0, 16356), (142.0, 16592), (146.0, 17408), (200.0, 28814),
                                   (360.0, 49152)])
def test_sums_over_the_tiles(fov, n):
    import torch
    from paper_2606_29794_amd.raster import Camera, Rasterizer
    kind = SC.CAM_FULL if fov == 360.0 else SC.CAM_FISHEYE
    rng = np.random.default_rng(3)
    cam = Camera.from_dict(SC.make_camera(rng, 6, kind, fov_x=math.radians(fov), fov_y=math.radians(fov)))
    R = Rasterizer(tile_log2=0)
    m = R.mask(cam)
    assert m.n_tiles == m.n_active and n in (None, m.n_tiles)
    img, ref = (torch.as_tensor(rng.random((3, m.n_active)).astype(np.float32), device="cuda") for _ in range(2))
    out, smap, _ = R.ssim_loss(img, ref, cam, want_map=True)
    saved, _, _ = R.ssim_forward_saved(img, ref, cam)
    want = [smap.double().mean().item(), (img - ref).abs().double().mean().item()]
    # each partial sums three floats in float32, the rest is in 64 bits: 4 u of a
    # partial's absolute sum, and u of the rounded result
    tol = 5 * 2.0 ** -24
    assert abs(out[0].item() - want[0]) <= tol * smap.abs().double().mean().item()
    assert abs(out[1].item() - want[1]) <= tol * want[1]
    assert torch.equal(out, saved)
