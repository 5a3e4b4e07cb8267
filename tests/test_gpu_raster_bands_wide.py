"""32x16 tiles are shared by two wavefronts (eight rows each) at every batch
depth; 16x16 tiles with 128 records a batch take one.  Every pixel must meet
the same contributors, so the images agree bit for bit, and the gradients up
to the order of the float32 sums, for images that end inside a band, lists
longer than a batch, and tile counts around 3072 (where 256 records a batch
go back to one wavefront forward)."""
import numpy as np
import pytest
import torch

from synth import make_config

from _gpu_common import grad_violations, log, to_dev

pytestmark = pytest.mark.gpu

# (workload, primitives, width, height)
SIZES = [("headline", 3000, 32, 16), ("headline", 30000, 61, 37), ("cfg0", 1, 40, 40),
         ("cfg0", 4000, 97, 131), ("cfg2", 60000, 1536, 1024), ("cfg2", 60000, 1537, 1024)]


@pytest.mark.parametrize("name,n,width,height", SIZES)
@pytest.mark.parametrize("batch", [64, 128, 256])
def test_wide_tiles_match_square_ones(name, n, width, height, batch):
    from paper_2510_03312_amd import Renderer, SceneRef, Tuning
    cfg = make_config(name, n=n, width=width, height=height)
    params = cfg["scenes"][0].params.copy()
    if name == "cfg0":
        params[-4] = 0.995    # opaque enough for the 0.99 clamp and early stops
    rng = np.random.default_rng(7)
    d_image = to_dev(rng.normal(size=(width * height, 3)).astype(np.float32))
    out = []
    for tuning in (Tuning(tile_w=32, batch_depth=batch), Tuning(batch_depth=128)):
        r = Renderer(tuning)
        sc = SceneRef(to_dev(params), cfg["scenes"][0].dim, cfg["scenes"][0].rot)
        image, t = r.forward([sc], cfg["views"])
        g = r.backward(d_image)[0]
        torch.cuda.synchronize()
        out.append((image, t, g.cpu().numpy()))
    (ia, ta, ga), (ib, tb, gb) = out
    assert torch.equal(ia, ib) and torch.equal(ta, tb)
    bad = sum(int(grad_violations(ga[k], gb[k].astype(np.float64)).sum()) for k in range(ga.shape[0]))
    log(f"{name} {width}x{height} batch {batch}: gradient entries over the bar {bad}")
    assert bad == 0
