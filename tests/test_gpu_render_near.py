"""The forward render where entries are near all, some or none of a wave's
pixels (the series for k2, both forms, the general one), against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2606_29794_amd import scenes as SC
from tests import parity as PT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    from paper_2606_29794_amd import raster
    assert torch.cuda.is_available()
    return raster.Rasterizer()


def _scene(seed):
    """Discs of 5 to 60 degrees: their edges cross the limit of the series (14.5
    degrees) and of the wave test (13.8 degrees less the wave's extent)."""
    rng = np.random.default_rng(seed)
    return SC.make_scene(150, 0, "volume", 2.0, 6.0, seed, log_scale_mu=-0.9, log_scale_sigma=0.5, rgb_dc=True, rng=rng), rng


@pytest.mark.parametrize("order", [2, 4, 5, 6, 7])
def test_near_and_far_entries(R, order):
    """Waves from 64 pixels across most of a face, where no entry is near, to
    some two degrees; images, exact hit counts away from fragile decisions."""
    sc, rng = _scene(order)
    cam = SC.make_camera(rng, order, SC.CAM_FULL)
    g, c, st = PT.gpu_forward(R, sc, cam)
    act = O.mask(cam)
    rgb_o, T_o, nu, frag = O.render(sc, cam, O.preprocess(sc, cam), act, **PT.BANDS)
    PT.compare_render(st.rgb.cpu().numpy().astype(np.float64), st.T.cpu().numpy().astype(np.float64), rgb_o, T_o, frag)
    nu_g = R.render_fwd(st.projected, g.P, st.vals, st.ranges, c, want_used=True)[3].cpu().numpy()
    assert np.array_equal(nu_g[frag == 0], nu[frag == 0])


def test_colour_that_is_not_finite_stays_in_its_pixels(R):
    """A Gaussian of infinite colour changes the pixels that composite it and no
    other pixel of their waves."""
    sc, rng = _scene(9)
    cam = SC.make_camera(rng, 6, SC.CAM_FULL)
    images = []
    for value in (0.25, 0.75, np.inf):
        sc.sh[0, :, 40] = value
        images.append(PT.gpu_forward(R, sc, cam)[2].rgb.cpu().numpy())
    hit = (images[0] != images[1]).any(axis=0)
    assert hit.any() and not hit.all()
    assert np.isfinite(images[2][:, ~hit]).all() and np.array_equal(images[2][:, ~hit], images[0][:, ~hit])
