"""Small workgroup tables in LDS whose initial community alone outnumbers them:
the rows of hubs bring in as many new ids at once as the workgroup has threads
(up to 256 beside the table's entries), and the community moves on to the next
tables."""
import numpy as np
import pytest

import oracle
from _gpu_common import compare_results
from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu


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
    # eight hubs, each linked to 120 leaves of its own in rings of ten
    n = 8 + 8 * 120
    leaf = np.arange(8, n)
    at = leaf - 8
    u = np.concatenate([at // 120, leaf])
    v = np.concatenate([leaf, 8 + at // 10 * 10 + (at + 1) % 10])
    g = W.csr_from_edges(n, u, v, np.random.default_rng(3).integers(1, 9, u.size))
    sets = [[0], list(range(8)), [0, 2, 4, 6], [1, 3, 400, 900], [77]]
    sp = np.concatenate([[0], np.cumsum([len(s) for s in sets])]).astype(np.int32)
    sn = np.concatenate(sets).astype(np.int32)
    sc = np.array([1.1, 0.9, 0.7])
    return g, sc, sp, sn, oracle.Oracle.from_graph(g).run_sets(sp, sn, sc)


@pytest.mark.parametrize("cap,waves", [(128, 0), (128, 4), (192, 0), (192, 8), (320, 4), (384, 4), (384, 8), (704, 8),
                                       (768, 4)])
def test_hubs_outgrow_a_small_table(L, case, cap, waves):
    g, sc, sp, sn, ref = case
    res = L.lcd_sweep(L.Graph.from_workload(g), sc, sp, sn, lds_capacity=64, team_capacity=cap, team_waves=waves)
    st = res.stats()
    assert st["tier_kind"][1] == 2 and st["tier_capacity"][1] == cap and st["n_spilled"] > 0
    compare_results(L.sweep_to_numpy(res), ref, label="LDS tables of %d, %d waves" % (cap, waves))
    res.free()
