"""Tile queries over lists of up to thousands of entries on few tiles, where
the waves of a workgroup filter one list together: list lengths at the edges
of a wave's batch (256 entries) and of the workgroup's step (1,024), against
the oracle's brackets."""
import numpy as np
import pytest

from paper_2606_29794_amd import scenes as SC
from tests.test_gpu_query import R, _check_bracket  # noqa: F401 (R is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,f", [("ring", 1), ("ring", 4), ("nested", 1), ("nested", 4)])
@pytest.mark.parametrize("P", [255, 257, 1023, 1025, 3001])
def test_long_lists_on_few_tiles(R, P, mode, f):  # noqa: F811
    rng = np.random.default_rng(P)
    sc = SC.make_scene(P, 0, "volume", 2.0, 6.0, P, log_scale_mu=0.3, rng=rng)  # discs of a quarter radian to pi
    cam = SC.make_camera(rng, 5, SC.CAM_FULL)
    n = _check_bracket(R, sc, cam, mode, f, "long")
    assert n > 12 * P  # of 48 tiles
