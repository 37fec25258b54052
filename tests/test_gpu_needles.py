"""Gradients of needle-like Gaussians (one scale far above the others) under a
dense random upstream gradient, against the oracle's 64-bit ones.

The gradient of a footprint's covariance is formed by the conic Q, whose
entries reach aspect^2 times the smallest.  Carried as dL/dQ, the last bits of
its sums over the pixels come back multiplied by Q on both sides: a relative
error of some u aspect^2 (u = 2^-24), where sums over Q d of every pixel leave
some u aspect.  The tolerance on the scale gradient, 10 u aspect, has 10 for
the roundings of a term and the depth of a sum; the rotation gradient, in which
the conic's own rounding enters every pixel's weight, gets twice that.
"""
import ctypes as C

import numpy as np
import pytest

import oracle as O
from paper_2606_29794_amd import _abi as A
from paper_2606_29794_amd import scenes as SC
from tests import parity as PT

pytestmark = pytest.mark.gpu

KEYS = ("mean", "scale", "rot", "opacity", "sh")
U = 2.0 ** -24


def _needles(P, aspect, seed):
    """Needles 0.15 rad long (one sigma), seen from the origin at distances
    from 3 to 6, so that the order in depth is not one of rounding."""
    rng = np.random.default_rng(seed)
    sc = SC.make_scene(P, 0, "volume", 3.0, 6.0, seed, rgb_dc=True)
    r = np.linalg.norm(sc.mean, axis=0)
    sc.scale[:] = (0.15 * r / aspect).astype(np.float32)
    sc.scale[rng.integers(0, 3, P), np.arange(P)] = (0.15 * r).astype(np.float32)
    sc.opacity[:] = rng.uniform(0.3, 0.8, P).astype(np.float32)
    cam = SC.make_camera(rng, 8, SC.CAM_FULL)
    return sc, cam, rng


@pytest.mark.parametrize("route,aspect", [("fused", 48), ("noalloc", 48), ("split", 6), ("fused", 6)])
def test_needle_gradients_match_the_oracle(route, aspect):
    import torch
    from paper_2606_29794_amd.raster import Camera, Gaussians, Rasterizer, _p, _stream
    sc, camd, rng = _needles(48, aspect, 31)
    R = Rasterizer()
    cam = Camera.from_dict(camd)
    g = Gaussians.from_scene(sc)
    st = R.forward(g, cam)
    act = O.mask(camd)
    pr = O.preprocess(sc, camd)
    frag = O.render(sc, camd, pr, act, **PT.BANDS)[3]
    dC = rng.normal(size=(3, act.size))
    dC[:, frag != 0] = 0.0
    dC = dC.astype(np.float32)
    ref = O.render_bwd(sc, camd, pr, act, dC.astype(np.float64))
    up = torch.as_tensor(dC, device="cuda")
    z = torch.zeros_like
    gr = Gaussians(z(g.mean), z(g.scale), z(g.rot), z(g.opacity), z(g.sh))
    if route == "fused":
        R.backward(g, st, up, None, gr)
    elif route == "noalloc":
        v, gs = cam.view(), g.struct()
        gg = A.hp_gaussians_grad(*(getattr(gr, k).data_ptr() for k in KEYS))
        A.call("hp_render_bwd_noalloc", C.byref(gs), _p(st.projected), _p(st.vals), _p(st.ranges), st.mask.n_tiles,
               C.byref(v), C.byref(R.prm), _p(st.mask.buf), st.mask.n_active, _p(st.T), _p(st.n_contrib), _p(up), None,
               None, C.byref(gg), _stream())
    else:
        acc = torch.zeros((10, g.P), dtype=torch.float32, device="cuda")
        R.backward_pixels(st, up, None, acc)
        R.backward_preprocess(g, cam, acc, gr)
    torch.cuda.synchronize()
    err = {k: PT.grad_compare(k, getattr(gr, k).cpu().numpy(), getattr(ref, k)) for k in KEYS}
    print(route, aspect, {k: "%.1e" % e for k, e in err.items()})
    assert err["scale"] <= 10 * U * aspect, err
    assert err["rot"] <= 20 * U * aspect, err
