"""Small device budgets that a server has to take, under every number of hardware
queues (the variable decides the lanes; the server reads it when it is made):
the lanes' buffers and, for each lane behind tier 0, a table of the kind its
stage runs, at 40 bytes an entry (60 from 65,536 entries on).  Every query is
answered as by the oracle, also where the lanes are fewer for it."""
import numpy as np
import pytest

import oracle
from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu

LANE = 1024 * (8 + 4 + 4 + 4 * 3) + 65536 * 4 + 8 * (2 + 11 * 4) + 32 + 256 * 16


# lanes per number of queues: all, with a table of 16,384 entries (or of every
# node on smaller graphs), with a table of every node
LANES = {4: (4, 3, 3), 8: (6, 3, 1), 12: (8, 5, 1)}


@pytest.mark.parametrize("queues", [4, 8, 12])
@pytest.mark.parametrize("n", [3_000, 12_000, 20_000, 50_000])
def test_server_runs_on_a_small_budget(n, queues, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd as L
    monkeypatch.setenv("GPU_MAX_HW_QUEUES", str(queues))
    lanes, mid, whole = LANES[queues]
    cap = 1 << (n - 1).bit_length()
    if cap <= 16384:      # the graph has no larger tables: those lanes share one kind
        budget = lanes * LANE + (mid if queues == 4 else mid + 1) * 40 * cap
    else:
        budget = lanes * LANE + mid * 40 * 16384 + whole * (60 if cap >= 65536 else 40) * cap
    g = W.lfr_hierarchical(n, 2.5, 15.0, 100, 1.5, 20, 200, mu=0.25, levels=3, weighted=True, wmax=16, seed=5)
    G = L.Graph.from_workload(g)
    o = oracle.Oracle.from_graph(g)
    _, sets, alphas = W.query_stream(g, 40, 2000.0, max_size=256, seed=11)
    queries = [(W.bfs_prefix(g, 7, 256), 0.5)] + list(zip(sets, alphas))
    with L.Server(G, mem_budget=budget) as srv:
        assert srv.stats()["mem_held"] <= budget
        tickets = [srv.submit(s, a) for s, a in queries]
        for t, (s, a) in zip(tickets, queries):
            r = srv.result(t, 60_000)
            per, K, V, f, ctr, _ = o.run_set(s, np.array([a]))
            assert np.array_equal(r["members"], per[0]) and (r["K"], r["V"]) == (int(K[0]), int(V[0]))
            assert np.array_equal(r["ctr"], np.asarray(ctr[0], np.uint64))
    with pytest.raises(L.LcdError) as e:
        L.Server(G, mem_budget=budget // 3)
    assert e.value.status == L.LCD_ENOMEM
