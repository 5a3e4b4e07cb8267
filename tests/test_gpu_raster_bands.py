"""Frames of few tiles share each 16x16 tile among two or four wavefronts (a
band of its rows each); a batch depth of 128 takes one wavefront per tile.
Both must composite the same image bit for bit, and the same gradients up to
the order of the float32 sums, at the tile counts around the limits and for
images that end inside a band."""
import numpy as np
import pytest
import torch

from synth import make_config

from _gpu_common import grad_violations, log, to_dev

pytestmark = pytest.mark.gpu

# (workload, primitives, width, height): one tile; ends inside a band; around
# 2048, 3072 and 4352 tiles; a dense scene whose pixels stop
SIZES = [("headline", 3000, 16, 16), ("headline", 20000, 61, 37), ("cfg0", 1, 40, 40),
         ("cfg0", 4000, 97, 131), ("headline", 60000, 1024, 512), ("headline", 60000, 1040, 512),
         ("cfg2", 60000, 1024, 768), ("cfg2", 60000, 1025, 769), ("cfg2", 60000, 1088, 1024),
         ("cfg2", 60000, 1089, 1024)]


@pytest.mark.parametrize("name,n,width,height", SIZES)
@pytest.mark.parametrize("with_t", [False, True])
def test_bands_match_whole_tiles(name, n, width, height, with_t):
    from paper_2510_03312_amd import Renderer, SceneRef, Tuning
    cfg = make_config(name, n=n, width=width, height=height)
    params = cfg["scenes"][0].params.copy()
    if name == "cfg0":
        params[-4] = 0.995    # opaque enough for the 0.99 clamp and early stops
    rng = np.random.default_rng(5)
    d_image = to_dev(rng.normal(size=(width * height, 3)).astype(np.float32))
    d_t = to_dev(rng.normal(size=width * height).astype(np.float32)) if with_t else None
    out = []
    for batch in (64, 128):
        r = Renderer(Tuning(batch_depth=batch))
        sc = SceneRef(to_dev(params), cfg["scenes"][0].dim, cfg["scenes"][0].rot)
        image, t = r.forward([sc], cfg["views"])
        n_con = r.ncontrib().clone()
        g = r.backward(d_image, d_t)[0]
        torch.cuda.synchronize()
        out.append((image, t, n_con, g.cpu().numpy()))
    (ia, ta, na, ga), (ib, tb, nb, gb) = out
    assert torch.equal(ia, ib) and torch.equal(ta, tb) and torch.equal(na, nb)
    bad = sum(int(grad_violations(ga[k], gb[k].astype(np.float64)).sum()) for k in range(ga.shape[0]))
    log(f"{name} {width}x{height} dt={with_t}: gradient entries over the bar {bad}")
    assert bad == 0
