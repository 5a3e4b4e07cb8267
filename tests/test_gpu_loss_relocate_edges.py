"""Sizes at the edges of what a workgroup takes, against the oracles.

Loss: up to 300 tiles of 128 x 16 pixels a frame goes by tiles of 16 x 16, a
larger one by those of 128 x 16, two columns a lane; up to eight view
descriptors travel with the launches, more go through the workspace.  Bars as
in test_gpu_ssim: float32 statistics, 1e-3 of the largest entry.
Relocation: 4096 primitives per scan workgroup, 1024 per step of the row
pass; exact but for the cloned opacity (one float32 ulp)."""
import pytest

from _gpu_common import gpu_ready, log
from test_gpu_relocate import _compare, _scene
from test_gpu_ssim import _check

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.mark.parametrize("sizes", [
    [(15, 15)], [(16, 16)], [(17, 33)], [(1, 1)], [(1, 40)], [(300, 1)],
    [(129, 17), (3, 2)] * 4, [(129, 17), (3, 2), (40, 18)] * 3,         # eight, nine views
    [(1280, 480)], [(1281, 433)], [(1, 4801)],                          # 300, 308, 301 tiles
    [(129, 17)] * 76, [(127, 15)] * 301, [(128, 16), (133, 33)] * 44])  # 304, 301, 308
def test_loss_at_tile_edges(sizes):
    log(f"[ssim edges] {len(sizes)} views, {sizes[:3]}")
    _check(sizes, 11 + len(sizes), 0.3)


@pytest.mark.parametrize("n,dead", [(2, 0.5), (255, 0.3), (1023, 0.3), (1025, 0.3), (4095, 0.9),
                                    (4096, 0.02), (4097, 0.3), (3 * 4096 + 1, 0.3),
                                    (257 * 4096, 0.01)])
def test_relocation_at_tile_edges(n, dead):
    log(f"[relocate edges] n {n} dead {dead}")
    _compare(*_scene(6, 0, n, dead, n + 3), 6, 0)
