"""The largest global tables of 16-bit indices, 32,768 entries (graphs of 16,385
to 32,768 nodes): communities that outgrow the 16,384-entry tier end there,
also by the whole range of ids, against the oracle."""
import numpy as np
import pytest

import oracle
from _gpu_common import compare_results
from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kw", [(32_768, dict()), (32_767, dict(team_waves=3, output_mode=1)),
                                  (16_385, dict(lds_capacity=64, mode=1))],
                         ids=["all-ids", "delta", "least"])
def test_largest_packed_tables(n, kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd as L
    g = W.lfr_hierarchical(n, 2.5, 8.0, 60, 1.5, 20, 300, mu=0.3, levels=3, weighted=True, wmax=16, seed=11)
    sc = np.array([0.9, 0.5, 0.2])
    sp = np.arange(7, dtype=np.int32)
    sn = (np.arange(6) * 2707 % n).astype(np.int32)
    ref = oracle.Oracle.from_graph(g).run_sets(sp, sn, sc)
    res = L.lcd_sweep(L.Graph.from_workload(g), sc, sp, sn, **kw)
    st = res.stats()
    last = st["tiers"] - 1
    assert (st["tier_kind"][last], st["tier_capacity"][last]) == (3, 32768)
    assert st["tier"][last]["sets_finished"] > 0
    compare_results(L.sweep_to_numpy(res), ref, label="n = %d" % n)
    res.free()
