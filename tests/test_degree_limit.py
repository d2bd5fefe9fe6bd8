"""A weighted degree past the limit of 2^27 is refused as such, with a device and
without one."""
import ctypes
import os

import numpy as np
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1301_0955_amd", "liblcd.so")


def _star(leaves, w):
    rp = np.concatenate([[0, leaves], leaves + np.arange(1, leaves + 1)]).astype(np.int32)
    col = np.concatenate([np.arange(1, leaves + 1), np.zeros(leaves)]).astype(np.int32)
    return rp, col, np.full(2 * leaves, w, np.uint8)


def _upload(rp, col, w):
    lib = ctypes.CDLL(LIB)
    lib.lcd_last_error.restype = ctypes.c_char_p
    lib.lcd_graph_upload.argtypes = [ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
                                     ctypes.c_int32, ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
    lib.lcd_graph_free.argtypes = [ctypes.c_void_p]
    h = ctypes.c_void_p()
    st = lib.lcd_graph_upload(rp.size - 1, col.size, rp.ctypes.data_as(ctypes.c_void_p),
                              col.ctypes.data_as(ctypes.c_void_p), w.ctypes.data_as(ctypes.c_void_p), 0, None,
                              ctypes.byref(h))
    msg = lib.lcd_last_error().decode()
    if h:
        lib.lcd_graph_free(h)
    return st, msg


LEAVES = 2 ** 27 // 255 + 1      # 255 x this many is just past 2^27


def _check_refused():
    st, msg = _upload(*_star(LEAVES, 255))
    assert st == 1 and "weighted degree %d exceeds 2^27" % (255 * LEAVES) in msg
    rp, col, w = _star(LEAVES, 255)
    w[5] = 254                       # a broken rule comes first
    st, msg = _upload(rp, col, w)
    assert st == 1 and "edge 0-6 has unequal weights" in msg


def test_degree_past_the_limit_is_refused():
    _check_refused()


@pytest.mark.gpu
def test_degree_past_the_limit_is_refused_on_the_device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _check_refused()
    st, msg = _upload(*_star(LEAVES - 1, 255))
    assert st == 0, msg
