"""Pixels of a partial tile that lie outside the image take no part in the
backward pass: opaque splats centred just beyond the right or the bottom edge
cover only such pixels with a high alpha (40 records at the 0.99 clamp divide
a transmittance by 1e80), and a faint wide splat behind them is the last
contributor of pixels inside, so that every record of the tile is walked.  The
gradients stay finite and match the oracle at every tile shape and split."""
import numpy as np
import pytest

from oracle import preprocess as opp
from oracle import render as orender
from synth.scenes import make_scene, make_view

from _gpu_common import GRAD_BLOCKS, gpu_ready, gpu_render, grad_violations, log

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

W, H = 53, 37     # 16-wide tiles end at 64, 8-wide ones at 56; bands of 4 rows at 40


def _scene(edge, view):
    n = 41
    sc = make_scene(3, n, 5, dist="cfg0")
    p = sc.params.astype(np.float64)
    sl = opp.field_slices(3, 0)
    rng = np.random.default_rng(8)
    x, y = np.full(n, W + 2.5), rng.uniform(19.0, 21.0, n)
    if edge == "bottom":
        x, y = rng.uniform(19.0, 21.0, n), np.full(n, H + 2.5)
    x[-1], y[-1] = (W - 8.0, 20.0) if edge == "right" else (20.0, H - 8.0)
    z = np.linspace(3.0, 4.0, n)
    z[-1] = 6.0
    # camera space to world: p = R mu + t
    cam = np.stack([(x - view.cx) / view.fx * z, (y - view.cy) / view.fy * z, z])
    p[sl["mu_x"]] = np.asarray(view.R, np.float64).reshape(3, 3).T @ (
        cam - np.asarray(view.t, np.float64).reshape(3, 1))
    p[sl["rot"]] = np.array([1.0, 0.0, 0.0, 0.0])[:, None]
    sigma = np.full(n, 4.0)     # support radius in pixels
    sigma[-1] = 30.0
    p[sl["log_s_x"]] = np.log(sigma * z / view.fx)
    p[sl["b_x"]] = 0.0
    p[sl["o"]] = 0.999
    p[sl["o"], -1] = 0.3
    sc.params = p.astype(np.float32)
    return sc


@pytest.mark.parametrize("edge", ["right", "bottom"])
@pytest.mark.parametrize("tuning", [dict(), dict(batch_depth=128), dict(tile_w=32), dict(tile_h=8),
                                    dict(tile_w=8, tile_h=8), dict(batch_depth=256)])
def test_pixels_outside_the_image_leave_no_gradient(edge, tuning):
    from paper_2510_03312_amd import Tuning
    log(f"[outside] {edge} {tuning}")
    view = make_view(W, H)
    sc = _scene(edge, view)
    rng = np.random.default_rng(1)
    d_image, d_t = rng.normal(size=(H, W, 3)), rng.normal(size=(H, W))
    o = orender.render(sc.params, 3, 0, view, d_image=d_image, d_tfinal=d_t, record_f32=True)
    ok = o["flags"] == 0
    d_image, d_t = d_image * ok[..., None], d_t * ok
    o = orender.render(sc.params, 3, 0, view, d_image=d_image, d_tfinal=d_t, record_f32=True)
    g = gpu_render({"scenes": [sc], "views": [view]}, Tuning(**tuning), want_grad=True,
                   d_images=[d_image], d_tfinals=[d_t])["dparams"][0]
    assert ok.mean() > 0.9 and (o["ncontrib"] > 0).any() and np.abs(o["dparams"]).max() > 0
    assert np.isfinite(g).all()
    sl = opp.field_slices(3, 0)
    bad = {b: int(grad_violations(g[sl[b]], o["dparams"][sl[b]]).sum())
           for b in GRAD_BLOCKS if sl[b].stop > sl[b].start}
    assert not any(bad.values()), bad
