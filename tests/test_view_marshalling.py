"""A view's matrices as they reach the C structs: every kind of array, tensor
or list gives the same float32 entries as its conversion through a float64
tensor, and what that conversion refuses stays refused."""
import numpy as np
import pytest
import torch

from paper_2510_03312_amd.renderer import _floats, _view_to_c

R = np.random.default_rng(3).normal(size=(3, 3))


class _View:
    scene, width, height = 0, 8, 4
    fx = fy = 5.0
    cx, cy, time = 4.0, 2.0, 0.25

    def __init__(self, R, t):
        self.R, self.t = R, t


@pytest.mark.parametrize("x", [R, R.astype(np.float32), R.astype(np.float16), R.T,
                               R.astype(np.float32).T, R[:, ::2], (R * 9).astype(np.int32),
                               torch.from_numpy(R), torch.from_numpy(R).float(), R.tolist(),
                               np.array([[np.nan, np.inf, -0.0]])],
                         ids=lambda x: type(x).__name__)
def test_entries_are_those_of_the_float64_tensor(x):
    want = torch.as_tensor(x, dtype=torch.float64).reshape(-1).numpy()
    np.testing.assert_array_equal(np.array(_floats(x)), want)
    assert all(type(e) is float for e in _floats(x))
    if want.size == 9:
        c = _view_to_c(_View(x, [1.0, 2.0, 3.0]))
        np.testing.assert_array_equal(np.array(c.R), want.astype(np.float32))


def test_what_was_refused_stays_refused():
    for bad in (R[::-1], R.astype(">f4"), np.array([["a"]])):
        with pytest.raises((TypeError, ValueError)):
            torch.as_tensor(bad, dtype=torch.float64)
        with pytest.raises((TypeError, ValueError)):
            _floats(bad)
    with pytest.raises(IndexError):
        _view_to_c(_View(np.zeros(10), np.zeros(3)))
