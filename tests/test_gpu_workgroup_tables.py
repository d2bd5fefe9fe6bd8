"""Workgroup tables against the oracle where their layouts can go wrong: the
smallest LDS table, sizes beside a power of two (the hash's load), launches
of few and of many sets, global tables of 16-bit indices, resumed sets, removal passes, one wave to eight; heavy weights (d
and degree in the hundreds of thousands), ranks of both signs and far beyond
the bucket range.  Members, K, V and counters bit for bit, f within 1e-12."""
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
    g = W.lfr_hierarchical(6000, 2.5, 24.0, 200, 1.5, 20, 600, mu=0.35, levels=3, weighted=True, wmax=255, seed=9)
    # far from the usual scales at both ends: ranks down to -40 L(k) and up
    sc = np.array([40.0, 3.0, 1.2, 1.0, 0.9, 0.8, 0.7, 0.6, 0.55])
    sp, sn = W.seed_rule1(g, 5)
    sp, sn, _ = W.subsample_sets(sp, sn, max(1, (sp.size - 1) // 60))
    ref = oracle.Oracle.from_graph(g).run_sets(sp, sn, sc)
    return g, sc, sp, sn, ref


@pytest.mark.parametrize("kw", [
    dict(lds_capacity=64),
    dict(lds_capacity=64, team_capacity=128, team_waves=1),    # 16-bit global tables, resumed sets
    dict(lds_capacity=64, team_capacity=192, team_waves=8, output_mode=1),
    dict(lds_capacity=64, team_capacity=1088, team_waves=3),
    dict(lds_capacity=128, team_capacity=2048, team_waves=2, mode=1),
    dict(lds_capacity=64, team_capacity=128, team_waves=2, grow_calls=1, k_prune=1),
], ids=lambda kw: "-".join("%s%d" % (k[:6], v) for k, v in kw.items()))
def test_workgroup_tables_match_oracle(L, case, kw):
    g, sc, sp, sn, ref = case
    if "grow_calls" in kw:
        # one call and one pass per scale: against the one-wave tiers
        G = L.Graph.from_workload(g)
        a = L.sweep_to_numpy(L.lcd_sweep(G, sc, sp, sn, spill_mode=1, grow_calls=1, k_prune=1))
        b = L.sweep_to_numpy(L.lcd_sweep(G, sc, sp, sn, **kw))
        assert np.array_equal(a["ctr"], b["ctr"]) and np.array_equal(a["K"], b["K"]) and np.array_equal(a["V"], b["V"])
        for r in range(a["cnt"].size):
            assert np.array_equal(a["members"][a["off"][r]:a["off"][r] + a["cnt"][r]],
                                  b["members"][b["off"][r]:b["off"][r] + b["cnt"][r]]), r
        return
    G = L.Graph.from_workload(g)
    res = L.lcd_sweep(G, sc, sp, sn, **kw)
    st = res.stats()
    assert st["n_spilled"] > 0
    compare_results(L.sweep_to_numpy(res), ref, label=str(kw))
    res.free()


def test_many_sets_match_few(L, case):
    """The set count chooses the waves; the records of a set do not depend on it."""
    g, sc, sp, sn, ref = case
    n = sp.size - 1
    reps = 1 + 4 * 256 // n + 1
    sp2 = np.concatenate([[0]] + [sp[1:] + q * sp[-1] for q in range(reps)]).astype(np.int32)
    sn2 = np.tile(sn, reps).astype(np.int32)
    G = L.Graph.from_workload(g)
    res = L.lcd_sweep(G, sc, sp2, sn2)
    st = res.stats()
    assert sp2.size - 1 > 1024 and 2 not in st["tier_kind"][:st["tiers"]]
    got = res.sets_to_numpy(np.arange((reps - 1) * n, reps * n, dtype=np.int32))
    compare_results(got, ref, label="many sets")
    res.free()
