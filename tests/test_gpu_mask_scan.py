"""The visibility mask's tile tables (offsets, compact ids, active tiles)
against the oracle's pixels, at tile counts of one step of the scan (up to 4,096
tiles), of a partly filled step and of several steps.  Whole numbers: equal."""
import math

import numpy as np
import pytest

import oracle as O
from paper_2606_29794_amd import scenes as SC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["full", "pinhole"])
@pytest.mark.parametrize("order", [0, 4, 8, 9, 10])
def test_mask_tile_tables(order, kind):
    from paper_2606_29794_amd import raster
    from paper_2606_29794_amd.raster import Camera
    rng = np.random.default_rng(order)
    fx = math.radians(75)
    cam = (SC.make_camera(rng, order, SC.CAM_FULL) if kind == "full" else
           SC.make_camera(rng, order, SC.CAM_PINHOLE, fov_x=fx, fov_y=SC.pinhole_fov_y(fx)))
    m = raster.Rasterizer().mask(Camera.from_dict(cam))
    pix = O.mask(cam)
    kt = O.tile_order(order)
    n = 12 * 4 ** kt
    count = np.bincount(pix >> (2 * (order - kt)), minlength=n)
    active = np.flatnonzero(count)
    compact = np.full(n, -1)
    compact[active] = np.arange(active.size)
    # the mask's layout: a 256-byte header, then four tables of n int32, each padded to 256 bytes
    row = (4 * n + 255) // 256 * 256
    tables = m.buf[256:256 + 4 * row].cpu().numpy().reshape(4, row).view(np.int32)
    start, cnt, cmp_, tiles = (t[:n] for t in tables)
    assert (m.n_active, m.n_tiles) == (pix.size, active.size)
    assert np.array_equal(cnt, count)
    assert np.array_equal(start, np.cumsum(count) - count)
    assert np.array_equal(cmp_, compact)
    assert np.array_equal(tiles[:active.size], active)
    assert np.array_equal(m.active_pix.cpu().numpy(), pix)
