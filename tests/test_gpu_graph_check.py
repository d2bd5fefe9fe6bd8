"""The device check of an uploaded graph: every rule is reported with the first
entry that breaks one, whatever breaks later; sound graphs keep their degrees
and volume (weights to 255, empty rows, no edges)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd
    lcd.library()
    return lcd


# a path 0-1-2-3 and an isolated node 4
RP = [0, 1, 3, 5, 6, 6]
COL = [1, 0, 2, 1, 3, 2]
W = [5, 5, 255, 255, 1, 1]


@pytest.mark.parametrize("at,col,w,text", [
    (2, 5, None, "neighbour id 5 of node 1 out of range"),
    (3, -1, None, "edge 1-2 has no reverse entry"),      # before the id out of range, in row 2
    (0, -1, None, "neighbour id -1 of node 0 out of range"),
    (0, 0, None, "self-loop at node 0"),
    (2, 0, None, "row 1 is not strictly ascending"),
    (4, 4, None, "edge 2-4 has no reverse entry"),
    (1, None, 0, "edge 0-1 has unequal weights"),
    (0, None, 0, "zero weight on edge 0-1"),
    (3, None, 254, "edge 1-2 has unequal weights"),
])
def test_first_broken_rule_is_reported(L, at, col, w, text):
    c, ww = list(COL), list(W)
    if col is not None:
        c[at] = col
    if w is not None:
        ww[at] = w
    with pytest.raises(L.LcdError) as e:
        L.Graph.from_host(5, np.array(RP, np.int32), np.array(c, np.int32), np.array(ww, np.uint8))
    assert e.value.status == L.LCD_EINVAL and text in str(e.value)


@pytest.mark.parametrize("rp,col,w,maxk,vol", [
    (RP, COL, W, 260, 522), (RP, COL, None, 2, 6), ([0, 0, 0], [], None, 0, 0)])
def test_sound_graphs(L, rp, col, w, maxk, vol):
    import ctypes
    G = L.Graph.from_host(len(rp) - 1, np.array(rp, np.int32), np.array(col, np.int32),
                          None if w is None else np.array(w, np.uint8))
    n, nnz, k, v = ctypes.c_int32(), ctypes.c_int64(), ctypes.c_int64(), ctypes.c_int64()
    assert L.library().lcd_graph_info(G._h, ctypes.byref(n), ctypes.byref(nnz), ctypes.byref(k), ctypes.byref(v)) == 0
    assert (n.value, nnz.value, k.value, v.value) == (len(rp) - 1, len(col), maxk, vol)
