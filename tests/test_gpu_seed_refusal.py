"""A permutation that lcd_seeds refuses leaves the caller's seed count alone."""
import ctypes

import numpy as np
import pytest

from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", [1, 2])
@pytest.mark.parametrize("device", [False, True], ids=["host", "device"])
def test_refused_perm_leaves_the_count(rule, device):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd as L
    g = W.lfr_hierarchical(1000, 2.5, 12.0, 60, 1.5, 20, 100, mu=0.3, levels=2, seed=3)
    G = L.Graph.from_workload(g)
    perm = np.arange(g.n, dtype=np.int32)
    perm[17] = 3
    P = ctypes.c_void_p
    if device:
        d = torch.from_numpy(perm).cuda()
        out = torch.empty(g.n, dtype=torch.int32, device="cuda")
        pp, op = P(d.data_ptr()), P(out.data_ptr())
    else:
        out = np.empty(g.n, np.int32)
        pp, op = perm.ctypes.data_as(P), out.ctypes.data_as(P)
    count = ctypes.c_int32(77)
    st = L.library().lcd_seeds(G._h, rule, pp, int(device), None, op, ctypes.byref(count))
    assert st == L.LCD_EINVAL and count.value == 77
    if device:
        d[17] = 17
    else:
        perm[17] = 17
    torch.cuda.synchronize()
    assert L.library().lcd_seeds(G._h, rule, pp, int(device), None, op, ctypes.byref(count)) == L.LCD_OK
    assert 0 < count.value < g.n
