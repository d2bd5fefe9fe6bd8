"""A graph holds the global tables that its launches run on: one per resident
workgroup of the launch's width, more once a launch of narrower workgroups
comes, and none the fewer afterwards."""
import numpy as np
import pytest

from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu

N = 4 << 20
TABLE = 131072 * (32 + 4 + 4) + 4 * 2 * 131072      # records, scratch, queue; hash
WHOLE = 4 << 30                                     # the whole-graph tables' budget
SLACK = 256 << 20


def test_tables_follow_the_launch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd as L
    cus = L.lcd_device_info()["compute_units"]
    g = W.lfr_hierarchical(6000, 2.5, 24.0, 200, 1.5, 20, 600, mu=0.35, levels=3, seed=9)
    rp = np.concatenate([g.row_ptr, np.full(N - g.n, g.nnz, np.int32)]).astype(np.int32)
    sc = np.array([1.0, 0.7])

    def sweep(G, sets):
        res = L.lcd_sweep(G, sc, np.arange(sets + 1, dtype=np.int32), np.arange(sets, dtype=np.int32))
        out = [np.sort(res.membership(s)[1].cpu().numpy()) for s in range(2)]
        res.free()
        return out

    G = L.Graph.from_host(N, rp, g.col, g.w)
    many = sweep(G, 2000)          # whatever a first launch of the kernels takes
    G.free()
    torch.cuda.empty_cache()
    G = L.Graph.from_host(N, rp, g.col, g.w)
    free = torch.cuda.mem_get_info()[0]
    few = sweep(G, 50)
    held_few = free - torch.cuda.mem_get_info()[0]
    again = sweep(G, 2000)
    held_many = free - torch.cuda.mem_get_info()[0]
    few2 = sweep(G, 50)
    held_after = free - torch.cuda.mem_get_info()[0]
    print("held: %d, %d, %d" % (held_few, held_many, held_after), flush=True)
    # twelve waves a compute unit: three workgroups of four, four of three
    assert held_few <= 3 * cus * TABLE + WHOLE + SLACK
    assert held_many <= 4 * cus * TABLE + WHOLE + SLACK
    assert abs(held_after - held_many) <= SLACK
    for a, b in zip(many + few, again + few2):
        assert np.array_equal(a, b)
