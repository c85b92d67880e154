"""Argument marshalling of the ctypes binding, on the CPU: the lists and
matrices that the state calls take reach C as NumPy would convert them."""
import ctypes as C

import numpy as np
import pytest

from paper_2311_01512_amd import native as N


@pytest.mark.parametrize("xs", [(1, 2, 3), [7], (), range(4), np.array([5, 6]), [np.int64(4), np.uint8(9)], [True],
                                (x for x in (3, 1)), [1.0, 2.7], bytes([1, 2])])
def test_int_lists(xs):
    xs = list(xs) if not isinstance(xs, (list, tuple, range, np.ndarray, bytes)) else xs
    keep, address, n = N._int_list(xs)
    assert list((C.c_int * n).from_address(address) if n else []) == list(N.ints(xs)) and keep is not None


@pytest.mark.parametrize("xs", [[2 ** 31], [-2 ** 40], ["a"], [None], [float("nan")]])
def test_int_lists_refused(xs):
    with pytest.raises(Exception) as want:
        N.ints(xs)
    with pytest.raises(want.type):
        N._int_list(xs)


@pytest.mark.parametrize("m", [np.arange(16).reshape(4, 4), np.arange(16.).reshape(4, 4).T,
                               (np.arange(64) * 1j).reshape(8, 8)[::2, ::2], [[1, 2j], [3, 4]],
                               np.arange(4096).reshape(64, 64) + 1j, (np.arange(4096) * 1j).reshape(64, 64).T])
def test_matrices(m):
    keep, data = N._matrix(m)
    n = np.asarray(m).size
    raw = data if isinstance(data, bytes) else C.string_at(data, 16 * n)
    assert np.array_equal(np.frombuffer(raw, dtype=np.complex128), N.cmatrix(m).reshape(-1).view(np.complex128))
    assert keep.shape == np.shape(m)
