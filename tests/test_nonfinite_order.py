"""The order the SVD kernels sort their columns into is a permutation whatever the keys hold: the positions
index arrays in LDS and, in the reverse-sweep form of the kernel, in device memory."""

import ctypes
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NAN, INF = float("nan"), float("inf")


def _order(key):
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2309_15642_amd", "libgpeps_peaks.so"))
    k = np.ascontiguousarray(key, dtype=np.float64)
    out = np.full(len(k), -7, dtype=np.int32)
    fn = lib.gpeps_probe_falling_order
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    assert fn(k.ctypes.data, len(k), out.ctypes.data) == 0
    return out


@pytest.mark.parametrize("key", [[NAN], [NAN] * 5, [1.0, NAN, 2.0, NAN], [NAN, INF, 0.0, INF, NAN, 3.0], [INF, INF], [0.0] * 4,
                                 [-1.0, NAN, -1.0]])
def test_order_of_any_keys_is_a_permutation(key):
    assert sorted(_order(key)) == list(range(len(key)))


def test_numbers_fall_and_ties_keep_their_order():
    rng = np.random.default_rng(2)
    key = rng.integers(0, 9, 64).astype(float)
    assert np.array_equal(_order(key), np.argsort(-key, kind="stable"))
    key[[3, 40]] = NAN
    got = _order(key)
    assert list(got[-2:]) == [3, 40] and np.all(np.diff(key[got[:-2]]) <= 0)
