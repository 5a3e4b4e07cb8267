"""The size of a frame's workspace, byte for byte: a caller may have laid out
its memory for it, and a smaller buffer is refused.  (The sizes of the first
release of this ABI version; a layout that grows needs a new version.)"""
import dataclasses

import pytest

pytest.importorskip("paper_2510_03312_amd._lib")
from paper_2510_03312_amd import _lib  # noqa: E402
from synth import make_config  # noqa: E402

from test_abi_host import _frame  # noqa: E402


def _bytes(n_scenes, n_views, n):
    cfg = make_config("headline", n=n, width=64, height=64)
    view = cfg["views"][0]
    cfg["scenes"] = cfg["scenes"] * n_scenes
    cfg["views"] = [dataclasses.replace(view, scene=k % n_scenes) for k in range(n_views)]
    lay = _lib.UbsLayout()
    assert _lib.ubs_preprocess(_frame(cfg).c, 0, 0, lay, 0) == 0
    return lay.bytes


@pytest.mark.parametrize("n_scenes,n_views,n,expected", [
    (1, 1, 1, 27009536), (1, 1, 1000, 27113472), (1, 64, 10, 31231744), (1, 65, 10, 31300096),
    (1, 200, 300, 45980928), (3, 7, 1000, 34137088), (4, 4, 257, 36359424),
    (5, 128, 100, 48702720), (9, 20, 5000, 62444288)])
def test_frame_workspace_size(n_scenes, n_views, n, expected):
    assert _bytes(n_scenes, n_views, n) == expected
