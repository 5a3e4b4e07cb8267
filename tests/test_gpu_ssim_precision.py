"""The image loss's gradient in float32 is no further from float64 than the
plain form is: five planes (x, y, x^2, y^2, x y) windowed tap after tap, rows
then columns, every operation rounded to float32 (fused multiply-adds), which is
evaluated here on the CPU.  Images as the loss meets them: smooth, with the noise
of a render late and early in training; each of the kernels' tile forms."""
import numpy as np
import pytest

from _gpu_common import gpu_ready, log, to_dev
from oracle import ssim as oss

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

f32 = np.float32
_TAPS = np.exp(-np.arange(-5, 6) ** 2 / 4.5)
TAPS = (_TAPS / _TAPS.sum()).astype(f32)


def _fma(a, b, c):
    return (a.astype(np.float64) * np.float64(b) + c.astype(np.float64)).astype(f32)


def _blur(z):
    for ax in (1, 0):
        n = z.shape[ax]
        pad = np.pad(z, [(5, 5) if a == ax else (0, 0) for a in range(z.ndim)])
        z = np.zeros_like(z)
        for k in range(11):
            z = _fma(np.take(pad, np.arange(k, k + n), axis=ax), TAPS[k], z)
    return z


def _plain_gradient(x, y, lam):
    mx, my, sxx, syy, sxy = (_blur(z) for z in (x, y, x * x, y * y, x * y))
    c1, c2, two = f32(1e-4), f32(9e-4), f32(2)
    a1, a2 = two * mx * my + c1, two * (sxy - mx * my) + c2
    b1, b2 = mx * mx + my * my + c1, (sxx - mx * mx) + (syy - my * my) + c2
    ib = f32(1) / (b1 * b2)
    S = a1 * a2 * ib
    scale = f32(-lam / x.size)
    d_m = scale * (two * my * (a2 - a1) * ib - two * mx * S * (f32(1) / b1 - f32(1) / b2))
    d_xx, d_xy = scale * (-S / b2), scale * (two * a1 * ib)
    sgn = np.sign(x - y).astype(f32) * f32((1.0 - lam) / x.size)
    return _blur(d_m) + two * x * _blur(d_xx) + y * _blur(d_xy) + sgn


@pytest.mark.parametrize("w,h", [(320, 180), (640, 400), (1300, 520)])
@pytest.mark.parametrize("noise", [0.01, 0.1])
def test_gradient_is_as_close_as_the_plain_form(w, h, noise):
    import torch
    from paper_2510_03312_amd.optim import ssim_loss

    class V:
        width, height = w, h
    g = torch.Generator()
    g.manual_seed(w)
    small = torch.rand((1, 3, 9, 13), generator=g)
    y = torch.nn.functional.interpolate(small, size=(h, w), mode="bilinear")[0].permute(1, 2, 0).numpy()
    y = np.ascontiguousarray(y, dtype=f32)
    x = np.clip(y + noise * np.random.default_rng(w).normal(size=y.shape), 0, 1).astype(f32)
    _, d = ssim_loss(to_dev(x.reshape(-1, 3)), to_dev(y.reshape(-1, 3)), [V], 0.2)
    _, (ref,) = oss.loss_and_grad([x], [y], 0.2)
    same = x == y
    err = lambda a: float(np.linalg.norm((a - ref) * ~same) / np.linalg.norm(ref))  # noqa: E731
    got, plain = err(d.cpu().numpy().reshape(y.shape).astype(np.float64)), err(_plain_gradient(x, y, 0.2))
    log(f"[ssim precision] {w}x{h} noise {noise}: {got:.2e}, plain form {plain:.2e}")
    assert got <= plain
