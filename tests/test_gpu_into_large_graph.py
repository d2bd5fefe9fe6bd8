"""lcd_sweep_into on graphs of 4,194,304 nodes and more, where lcd_sweep plans
other tables: its limit of LCD_NOALLOC_TABLE_ENTRIES entries per community is
the same there.  The graph is a 6,000-node one on ids spread over the range
(ascending, so every tie falls the same way), the rest isolated nodes, and the
oracle runs on the small one."""
import numpy as np
import pytest

import oracle
from _gpu_common import compare_results
from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu

N = 4 << 20


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd
    lcd.library()
    return lcd


@pytest.fixture(scope="module")
def case():
    g = W.lfr_hierarchical(6000, 2.5, 24.0, 200, 1.5, 20, 600, mu=0.35, levels=3, weighted=True, wmax=255, seed=9)
    step = N // g.n
    rp = np.full(N + 1, g.nnz, np.int32)
    ends = np.arange(g.n, dtype=np.int64) * step
    rp[:1] = 0
    rp[1:] = np.asarray(g.row_ptr)[np.searchsorted(ends, np.arange(1, N + 1), side="left")]
    big = W.Graph(n=N, row_ptr=rp, col=(np.asarray(g.col) * step).astype(np.int32), w=g.w, meta={})
    sc = np.array([1.2, 1.0, 0.8, 0.65, 0.55])
    sp, sn = W.seed_rule1(g, 5)
    sp, sn, _ = W.subsample_sets(sp, sn, max(1, (sp.size - 1) // 40))
    ref = oracle.Oracle.from_graph(g).run_sets(sp, sn, sc)
    ref["members"] = np.asarray(ref["members"]) * step
    return big, step, sc, sp, sn, ref


@pytest.mark.parametrize("kw", [dict(), dict(lds_capacity=64, team_capacity=128), dict(team_waves=3)],
                         ids=["default", "lds", "waves"])
def test_into_holds_its_table_entries(L, case, kw):
    big, step, sc, sp, sn, ref = case
    G = L.Graph.from_workload(big)
    o = L.lcd_sweep_into(G, sc, sp, (sn * step).astype(np.int32), members_cap=4_000_000, **kw)
    R = (sp.size - 1) * sc.size
    got = dict(n_scales=sc.size, n_sets=sp.size - 1, off=o["rec_off"][:R].cpu().numpy(),
               cnt=o["rec_cnt"][:R].cpu().numpy(), K=o["rec_k"][:R].cpu().numpy(), V=o["rec_v"][:R].cpu().numpy(),
               f=o["rec_f"][:R].cpu().numpy(), members=o["members"].cpu().numpy(),
               ctr=o["rec_ctr"][:4 * R].cpu().numpy().reshape(-1, 4).astype(np.uint64))
    assert ref["cnt"].max() > 1024      # more entries than any LDS table of the default plan
    compare_results(got, ref, label="into, %s" % kw)
