"""A graph whose adjacency records would take more than an eighth of the free
memory goes without them, and every growth kernel gathers a row's fields
instead: the same records as the oracle.  The memory is held while the graph is
uploaded and given back before anything runs on it."""
import numpy as np
import pytest

import oracle
from _gpu_common import compare_results
from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu

RECORD = 24           # bytes per directed entry
LEAVE = 768 << 20     # free while the graph is uploaded, about


@pytest.fixture(scope="module", params=[True, False], ids=["weighted", "unweighted"])
def case(request):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd as L
    g = W.lfr_hierarchical_fast(500_000, 2.5, 20.0, 200, 1.5, 20, 300, mu=0.3, levels=3, weighted=request.param,
                                seed=5)
    torch.cuda.empty_cache()
    ballast = []
    while len(ballast) < 3 and torch.cuda.mem_get_info()[0] > 8 * RECORD * g.nnz:
        ballast.append(torch.empty(torch.cuda.mem_get_info()[0] - LEAVE, dtype=torch.uint8, device="cuda"))
    free = torch.cuda.mem_get_info()[0]
    assert LEAVE // 2 < free < 8 * RECORD * g.nnz
    G = L.Graph.from_host(g.n, g.row_ptr, g.col, g.w)
    held = free - torch.cuda.mem_get_info()[0]
    del ballast
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    full = L.Graph.from_host(g.n, g.row_ptr, g.col, g.w)
    held_full = free - torch.cuda.mem_get_info()[0]
    full.free()
    # without the records, and with them
    assert held < RECORD * g.nnz <= held_full
    sc = np.array([1.1, 0.9, 0.7, 0.55])
    sets = [[q] for q in range(0, g.n, 15919)] + [W.bfs_prefix(g, 17, 200), W.bfs_prefix(g, 4242, 40)]
    sp = np.concatenate([[0], np.cumsum([len(s) for s in sets])]).astype(np.int32)
    sn = np.concatenate(sets).astype(np.int32)
    return L, G, sc, sp, sn, oracle.Oracle.from_graph(g).run_sets(sp, sn, sc)


@pytest.mark.parametrize("kw", [dict(), dict(lds_capacity=64), dict(lds_capacity=64, team_capacity=2048),
                                dict(lds_capacity=64, spill_mode=1), dict(lds_capacity=64, spill_mode=2, mode=1),
                                dict(lds_capacity=64, output_mode=1, mode=1)],
                         ids=["default", "global", "lds", "waves", "loop", "delta"])
def test_rows_without_records(case, kw):
    L, G, sc, sp, sn, ref = case
    res = L.lcd_sweep(G, sc, sp, sn, **kw)
    compare_results(L.sweep_to_numpy(res), ref, label=str(kw))
    res.free()
