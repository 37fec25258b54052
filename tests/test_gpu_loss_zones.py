"""The polar windows of fine grids (order 8 on): the short series of the window
weight on the CPU, and the loss with it against the oracle."""
import math

import numpy as np
import pytest

import oracle as O
from paper_2606_29794_amd import scenes as SC
from tests import parity as PT


def test_series_holds_over_a_window():
    """Every window of order >= 8 stays within s^2 < 1e-3 (ten steps between
    neighbouring centres under 1.6 / nside each), and there the exponent from
    1/2 - u.v / 2 and the three-term series is that of the great-circle
    distance to half a float ulp."""
    rng = np.random.default_rng(3)
    for order in (3, 5, 8, 12):
        N = 1 << order
        for k in range(400):
            f = int(rng.choice((0, 1, 2, 3, 8, 9, 10, 11)))
            # corners, edges and the inside of the cap faces
            x, y = (int(v) for v in (rng.integers(0, N, 2) if k % 2 else rng.choice((0, 1, N - 2, N - 1), 2)))
            u = O.pix_vec(order, O.chart_pixel(order, f, x, y))
            for dx, dy in ((1, 0), (-1, 0), (0, 1), (0, -1)):
                q = O.chart_pixel(order, f, x + dx, y + dy)
                if q < 0:
                    continue
                v = O.pix_vec(order, q)
                chord = float(np.linalg.norm(u - v))
                assert 2 * math.asin(chord / 2) * N < 1.6, (order, f, x, y)
    assert (math.sin(5 * 1.6 / 256)) ** 2 < 1e-3
    s2 = np.linspace(0, 1e-3, 1001)[1:]
    k = (np.arcsin(np.sqrt(s2))) ** 2 / s2
    assert np.abs((1 + s2 * (1 / 3 + s2 * 8 / 45)) / k - 1).max() < 1.3e-10


@pytest.mark.gpu
@pytest.mark.parametrize("sigma", [1.5, 1e-6])
@pytest.mark.parametrize("order,masked", [(8, False), (8, True)])
def test_loss_with_polar_windows(order, masked, sigma):
    """Tiles wholly polar, mixed and cut by the mask's edge, at the first order
    of the short series, with the tolerances of the loss's other tests; a
    window far narrower than a pixel takes the general path and leaves only
    its own pixel."""
    import torch
    from paper_2606_29794_amd import _abi as A
    from paper_2606_29794_amd.raster import Camera, Rasterizer
    R = Rasterizer()
    rng = np.random.default_rng(order + masked)
    cam = (SC.make_camera(rng, order, SC.CAM_FISHEYE, fov_x=math.radians(200), fov_y=math.radians(160)) if masked
           else SC.make_camera(rng, order, SC.CAM_FULL))
    act = O.mask(cam)
    img = rng.random((3, act.size)).astype(np.float32)
    ref = (0.6 * img + 0.4 * rng.random((3, act.size))).astype(np.float32)
    up = torch.tensor([1.7], dtype=torch.float32, device="cuda")
    sp = A.default_ssim_params(zones=1, sigma=sigma)
    out, smap, dimg = R.ssim_loss(torch.as_tensor(img, device="cuda"), torch.as_tensor(ref, device="cuda"),
                                  Camera.from_dict(cam), sp=sp, dL_dloss=up, want_map=True)
    torch.cuda.synchronize()
    out, smap, dimg = out.cpu().numpy(), smap.cpu().numpy(), dimg.cpu().numpy()
    if sigma < 1:
        # the window is the pixel: the variances vanish and SSIM is its luminance term
        c1 = float(np.float32(sp.C1))
        x, y = img.astype(np.float64), ref.astype(np.float64)
        assert np.abs(smap - (2 * x * y + c1) / (x * x + y * y + c1)).max() < 2e-3
        assert np.isfinite(dimg).all()
        return
    s_o, map_o, _ = O.hssim(order, act, img, ref, want_map=True, zones=True)
    L_o, gL_o = O.loss(order, act, img, ref, want_grad=True, zones=True)
    assert abs(out[0] - s_o) < 2e-6 and abs(out[2] - L_o) < 2e-6
    assert np.abs(smap - map_o).max() < 2e-5
    PT.grad_compare("loss gradient with polar windows", dimg, 1.7 * gL_o)
