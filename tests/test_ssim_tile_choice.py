"""Which tiles the image loss walks: frames of narrow views (whose tiles of
128 x 16 pixels would be mostly empty) and small frames take tiles of 16 x 16,
others tiles of 128 x 16.  The workspace holds 16 bytes a tile, so its size
tells the choice without a GPU.  On the GPU: a workspace that holds only the
wide tiles' sums still serves a narrow frame, and the tiles of many views find
their view (64 probes a round: around 64, 128 and 4096 views), and frames at the
limits of 512 and 2304 small tiles agree with the oracle.  Bars as in
test_gpu_ssim."""
import numpy as np
import pytest

pytest.importorskip("paper_2510_03312_amd._lib")
from _gpu_common import gpu_ready, log, to_dev
from oracle import ssim as oss
from paper_2510_03312_amd import _lib

_align = lambda x: (x + 255) // 256 * 256  # noqa: E731


def _tiles(sizes, w):
    return sum(-(-a // w) * -(-b // 16) for a, b in sizes)


def _bytes(sizes, tiles):
    off = _align(_align(32 * len(sizes)) + 16 * tiles)
    return _align(off + 36 * sum(a * b for a, b in sizes))


NARROW = [[(64, 64)] * 100, [(1, 4801)], [(16, 16)] * 301, [(32, 32)] * 1024, [(16, 16384)],
          [(33, 16384)], [(70, 5000)], [(160, 120)] * 20, [(640, 480)], [(1, 1)]]
WIDE = [[(1920, 1080)], [(1280, 720)], [(1000, 700)], [(64, 16384)], [(64, 64)] * 1024,
        [(320, 240)] * 8, [(128, 128)] * 100]


@pytest.mark.parametrize("sizes,width", [(s, 16) for s in NARROW] + [(s, 128) for s in WIDE])
def test_tile_choice(sizes, width):
    need = _lib.ubs_ssim_loss(sizes, 0, 0, 0.2, 0, 0, 0, 0, 0)
    assert need == _bytes(sizes, _tiles(sizes, width))
    assert need <= _bytes(sizes, _tiles(sizes, 16))


def _run(sizes, ws_bytes, seed):
    import torch
    rng = np.random.default_rng(seed)
    imgs = [rng.uniform(size=(h, w, 3)).astype(np.float32) for w, h in sizes]
    tgts = [np.clip(x + 0.15 * rng.normal(size=x.shape), 0, 1).astype(np.float32) for x in imgs]
    flat = lambda xs: to_dev(np.concatenate([x.reshape(-1, 3) for x in xs]))  # noqa: E731
    x, y = flat(imgs), flat(tgts)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    d, loss = torch.empty_like(x), torch.zeros(1, dtype=torch.float64, device="cuda")
    _lib.ubs_ssim_loss(sizes, x.data_ptr(), y.data_ptr(), 0.3, d.data_ptr(), loss.data_ptr(),
                       ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ref_loss, ref_g = oss.loss_and_grad(imgs, tgts, 0.3)
    ref = np.concatenate([g.reshape(-1, 3) for g in ref_g])
    ties = np.concatenate([(a == b).reshape(-1, 3) for a, b in zip(imgs, tgts)])
    err = np.abs(d.cpu().numpy() - ref) * ~ties
    assert abs(float(loss[0]) - ref_loss) <= 1e-5 * abs(ref_loss) + 1e-9
    assert np.all(err <= 1e-3 * np.abs(ref).max() + 1e-3 * np.abs(ref))


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")
@pytest.mark.parametrize("sizes", [[(64, 64)] * 100, [(16, 16)] * 301, [(5, 7)] * 64, [(20, 3)] * 65,
                                   [(3, 17)] * 129, [(2, 2)] * 4096, [(130, 33)] * 300,
                                   [(256, 512)], [(255, 513)], [(768, 768)], [(768, 769)]])
def test_values_at_both_workspace_sizes(sizes):
    log(f"[ssim choice] {len(sizes)} views of {sizes[0]}")
    need = _lib.ubs_ssim_loss(sizes, 0, 0, 0.3, 0, 0, 0, 0, 0)
    for ws_bytes in {need, _bytes(sizes, _tiles(sizes, 128))}:
        _run(sizes, ws_bytes, 3)
