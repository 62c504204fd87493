"""The binding's short cuts for lists: the values numpy would make of them, the same refusals, and the current stream."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2605_13319_amd import nav


@pytest.mark.parametrize("a", [[0], [5, -1, 2 ** 31 - 1], [True, np.int64(7)], [1.0, 2.9], (3, 4), range(5), np.arange(4), [], [np.float32(2.0)]])
def test_integers(a):
    got, n = nav._ints(a)
    want = nav._i32(a)
    assert n == len(want) and [got[i] for i in range(n)] == want.tolist()


@pytest.mark.parametrize("a", [[2 ** 31], ["x"], [None], [[1], [2, 3]]])
def test_refused_integers(a):
    with pytest.raises(Exception) as want:
        nav._i32(a)
    with pytest.raises(type(want.value)):
        nav._ints(a)


@pytest.mark.parametrize("a", [[0.0, 0.1, 1.0 - 2.0 ** -24, 1e-40], [0, 1], [0.5, 1], (0.25,), np.float64([0.3]), [float("nan"), float("inf")]])
def test_floats(a):
    got, want = nav._floats(a), nav._f32(a)
    assert np.array_equal(np.array([got[i] for i in range(len(want))], dtype=np.float32), want, equal_nan=True)
    assert nav._floats(None) is None


class Scalar:
    """What has a value for Python but is not a plain number: with a device tensor's refusal of numpy."""
    def __index__(self):
        return 5

    def __float__(self):
        return 0.5

    def __array__(self, *args, **kwargs):
        raise TypeError("not for numpy")


@pytest.mark.parametrize("a", [[5, torch.tensor([6])], [torch.tensor([5]), 6], [5, Scalar()], [np.array([1, 2]), np.array([1, 2, 3])]])
def test_integers_that_numpy_refuses_stay_refused(a):
    with pytest.raises(Exception) as want:
        nav._i32(a)
    with pytest.raises(type(want.value)):
        nav._ints(a)


@pytest.mark.parametrize("a", [[0.5, np.array([0.3])], [0.5, torch.tensor([0.3])], [0.5, Scalar()], [0.5, [0.3]], [0.5, 2 + 0j]])
def test_floats_that_numpy_refuses_stay_refused(a):
    with pytest.raises(Exception) as want:
        nav._f32(a)
    with pytest.raises(type(want.value)):
        nav._floats(a)


@pytest.mark.gpu
def test_the_current_stream():
    assert nav._stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert nav._stream() == s.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert isinstance(nav._ints([1])[0], C.Array)
