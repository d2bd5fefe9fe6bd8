"""Kernels that work in chunks and batches, at the edges of those: the offsets
scan around its chunk of 1,024 sets, the cover check around a wave's 64
members, the seed selection's check of perm, and the partner walk's batches of
64 and 8 members against the order that decides which partner is first."""
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


@pytest.mark.parametrize("n_sets", [1, 1023, 1024, 1025, 2049, 5000])
def test_offsets_over_chunks(L, n_sets):
    g = W.lfr_hierarchical(1000, 2.5, 12.0, 60, 1.5, 20, 100, mu=0.3, levels=2, seed=3)
    G = L.Graph.from_workload(g)
    sn = (np.arange(n_sets) % g.n).astype(np.int32)
    res = L.lcd_sweep(G, np.array([1.0, 0.8]), np.arange(n_sets + 1, dtype=np.int32), sn)
    full = L.sweep_to_numpy(res)
    for s in range(2):
        cp, m = [x.cpu().numpy() for x in res.membership(s)[:2]]
        cnt = full["cnt"].reshape(n_sets, 2)[:, s]
        assert np.array_equal(cp, np.concatenate([[0], np.cumsum(cnt)]))
        j = n_sets - 1
        r = 2 * j + s
        assert np.array_equal(m[cp[j]:cp[j + 1]], full["members"][full["off"][r]:full["off"][r] + full["cnt"][r]])
    assert res.counters()[0] == full["ctr"].reshape(-1, 4)[:, 0].sum()


@pytest.mark.parametrize("at", [0, 1, 63, 64, 65, 127, 128, 199])
def test_cover_check_sees_every_member(L, at):
    n = 400
    good = [np.arange(0, 200, dtype=np.int32), np.arange(150, 151, dtype=np.int32)]
    L.lcd_cover_nmi(n, good, good)
    for v in (-1, n, good[0][at - 1] if at else 1):       # out of range, or not ascending
        x = good[0].copy()
        x[at] = v
        with pytest.raises(L.LcdError) as e:
            L.lcd_cover_nmi(n, [x, good[1]], good)
        assert e.value.status == L.LCD_EINVAL


@pytest.mark.parametrize("bad", [{0: -1}, {7: 3000}, {2999: 5}, {3: 2, 9: 8}])
def test_perm_check_names_the_first_entry(L, bad):
    g = W.lfr_hierarchical(3000, 2.5, 12.0, 60, 1.5, 20, 100, mu=0.3, levels=2, seed=3)
    G = L.Graph.from_workload(g)
    perm = np.arange(g.n, dtype=np.int32)
    L.lcd_seeds(G, perm, rule=1)
    for i, v in bad.items():
        perm[i] = v
    seen, first = set(), None
    for i, v in enumerate(perm.tolist()):
        if v < 0 or v >= g.n or v in seen:
            first = i
            break
        seen.add(v)
    for rule in (1, 2):
        with pytest.raises(L.LcdError) as e:
            L.lcd_seeds(G, perm, rule=rule)
        assert e.value.status == L.LCD_EINVAL and "(entry %d)" % first in str(e.value)


@pytest.mark.parametrize("eta", [(1, 10), (1, 2), (9, 10)])
def test_merge_of_overlapping_seeds(L, eta):
    """Seed sets of 1 to 200 nodes that share nodes: partners are found within
    the first, a middle and no batch of members."""
    g = W.lfr_hierarchical(2000, 2.5, 14.0, 60, 1.5, 20, 200, mu=0.25, levels=2, weighted=True, wmax=8, seed=4)
    rng = np.random.default_rng(2)
    sets = []
    for size in (1, 7, 8, 9, 63, 64, 65, 72, 128, 200) * 3:
        base = W.bfs_prefix(g, int(rng.integers(g.n)), size)
        sets.append(np.sort(np.unique(base)).astype(np.int32))
    for x in list(sets[3:10]):
        sets.append(np.sort(np.unique(np.concatenate([x[: x.size // 2], W.bfs_prefix(g, int(rng.integers(g.n)), 20)])))
                    .astype(np.int32))
    sp = np.concatenate([[0], np.cumsum([x.size for x in sets])]).astype(np.int32)
    sn = np.concatenate(sets).astype(np.int32)
    sc = np.array([0.9, 0.7])
    res = L.lcd_sweep_merge(L.Graph.from_workload(g), sc, sp, sn, eta=eta)
    ref = oracle.Oracle.from_graph(g).run_merge(sp, sn, sc, eta=eta)
    compare_results(L.sweep_to_numpy(res), ref, label="merge")
    assert np.array_equal(L.merged_into(res), ref["into"])
    res.free()
