"""Gaussians so small that the reciprocal of their covariance's determinant
overflows (the determinant is subnormal): they are listed, their conic is not
finite, no pixel composites them, and their gradients are zero."""
import ctypes as C

import numpy as np
import pytest

from paper_2606_29794_amd import _abi as A
from paper_2606_29794_amd import scenes as SC

pytestmark = pytest.mark.gpu

KEYS = ("mean", "scale", "rot", "opacity", "sh")


@pytest.mark.parametrize("depth", [False, True])
@pytest.mark.parametrize("route", ["fused", "noalloc", "split"])
def test_tiny_footprints_get_zero_gradients(route, depth):
    import torch
    from paper_2606_29794_amd.raster import Camera, Gaussians, Rasterizer, _p, _stream
    wl = SC.config1(P=3000, order=6)
    sc = wl.scene
    tiny = np.arange(0, 3000, 100)
    r = np.linalg.norm(sc.mean[:, tiny], axis=0)
    sc.scale[:, tiny] = (1e-10 * r).astype(np.float32)                    # round: det 1e-40
    sc.scale[:, tiny[::2]] = (np.array([[0.1], [1e-19], [1e-19]]) * r[::2]).astype(np.float32)  # needles: the same det
    R = Rasterizer()
    cam = Camera.from_dict(wl.cameras[0])
    g = Gaussians.from_scene(sc)
    st = R.forward(g, cam, want_depth=depth)
    conic = R.projected_arrays(st.projected, g.P)[0].reshape(g.P, 16)[:, 9:12].cpu().numpy()
    bad = tiny[~np.isfinite(conic[tiny]).all(axis=1)]
    listed = set(st.vals[: st.n_pairs].tolist())
    assert sum(int(i) in listed for i in bad) >= 5 and np.isfinite(np.delete(conic, tiny, axis=0)).all()
    n = st.mask.n_active
    rng = np.random.default_rng(4)
    dC = torch.as_tensor(rng.normal(size=(3, n)).astype(np.float32), device="cuda")
    dD = torch.as_tensor(rng.normal(size=n).astype(np.float32), device="cuda") if depth else None
    z = torch.zeros_like
    gr = Gaussians(z(g.mean), z(g.scale), z(g.rot), z(g.opacity), z(g.sh))
    if route == "fused":
        R.backward(g, st, dC, None, gr, dL_dinv_depth=dD)
    elif route == "noalloc":
        v, gs = cam.view(), g.struct()
        gg = A.hp_gaussians_grad(*(getattr(gr, k).data_ptr() for k in KEYS))
        A.call("hp_render_bwd_noalloc", C.byref(gs), _p(st.projected), _p(st.vals), _p(st.ranges), st.mask.n_tiles,
               C.byref(v), C.byref(R.prm), _p(st.mask.buf), n, _p(st.T), _p(st.n_contrib), _p(dC), None, _p(dD),
               C.byref(gg), _stream())
    else:
        acc = torch.zeros((10, g.P), dtype=torch.float32, device="cuda")
        R.backward_pixels(st, dC, None, acc, dL_dinv_depth=dD)
        assert bool(torch.isfinite(acc).all()) and int(acc[:, torch.as_tensor(bad, device="cuda")].count_nonzero()) == 0
        R.backward_preprocess(g, cam, acc, gr)
    torch.cuda.synchronize()
    for k in KEYS:
        t = getattr(gr, k).reshape(-1, g.P).cpu().numpy()
        assert np.isfinite(t).all(), k
        assert np.count_nonzero(t[:, bad]) == 0, k
        assert np.count_nonzero(t) > 0, k
