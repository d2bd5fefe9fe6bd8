"""The workgroup queue where it leaves its usual path, on each table layout
(LDS; global, 16-bit indices; global, 32-bit indices), against the oracle:
  hub    a hub joins whose row is longer than the fresh list: entries past the
         list's end are found by a rebuild
  ties   hundreds of entries of one rank rank above the ones that improve: one
         bucket wider than a step's window, and windows that grow
  runs   long runs of additions: the queue is rebuilt again and again
The layouts are told apart by the tiers' kinds and capacities, and that the
sets ended there by the tiers' counts."""
import numpy as np
import pytest

import oracle
from _gpu_common import compare_results
from paper_1301_0955_amd import workloads as W

pytestmark = pytest.mark.gpu

N_WIDE = 4 << 20      # from here on the first global tables have 131,072 entries

LAYOUTS = {
    "lds-2": (dict(lds_capacity=64, team_capacity=4096, team_waves=2), 2, 4096),
    "lds-1": (dict(lds_capacity=64, team_capacity=4096, team_waves=1), 2, 4096),
    "pack-1": (dict(lds_capacity=64, team_waves=1), 3, 4096),
    "pack-4": (dict(lds_capacity=64), 3, 4096),
    "pack-8": (dict(lds_capacity=64, team_waves=8), 3, 4096),
    "wide-2": (dict(lds_capacity=64, team_waves=2), 3, 131072),
    "wide-4": (dict(lds_capacity=64), 3, 131072),
}


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0955_amd import lcd
    lcd.library()
    return lcd


def _ring(ids):
    ids = np.asarray(ids)
    return ids, np.roll(ids, -1)


def _hub():
    # two cores of 12, heavily linked inside and to their hub; each hub has
    # 1,400 leaves of its own, in rings of seven
    u, v, w = [], [], []
    n = 2 * 13 + 2 * 1400
    for c in range(2):
        core = np.arange(12) + 13 * c
        hub, i = 12 + 13 * c, np.arange(1400)
        leaf = 26 + 1400 * c + i
        a, b = np.triu_indices(12, 1)
        u += [core[a], core, np.full(1400, hub), leaf]
        v += [core[b], np.full(12, hub), leaf, leaf - i + i // 7 * 7 + (i + 1) % 7]
        w += [np.full(a.size, 40), np.full(12, 255), np.ones(1400), np.ones(1400)]
    u.append(np.array([12]))
    v.append(np.array([25]))
    w.append(np.array([3]))
    sets = [[0], [13, 14, 15], list(range(6)), [5, 20]]
    return n, u, v, w, sets, np.array([1.0, 0.8, 0.6, 0.4])


def _ties():
    # a core whose members have 24 leaves of degree two each (600 of one
    # rank), and satellites with ten links into the core and one outside: at
    # alpha 1.8 the leaves rank above them and do not improve, they do
    core, leaf, sat, far = np.arange(25), 25 + np.arange(600), 625 + np.arange(40), 665 + np.arange(40)
    a, b = np.triu_indices(25, 1)
    u = [core[a], leaf % 25, leaf, np.repeat(sat, 10), sat, far]
    v = [core[b], leaf, 25 + ((leaf - 25) ^ 1), np.tile(np.arange(10), 40), far, np.roll(far, 1)]
    w = [np.full(x.size, 8 if i == 0 else 1) for i, x in enumerate(u)]
    sets = [list(range(25)), list(range(12)), [3], [625, 0, 1]]
    return 705, u, v, w, sets, np.array([2.0, 1.8, 1.7, 1.5, 1.1, 0.8])


def _runs():
    g = W.lfr_hierarchical(3000, 2.5, 24.0, 200, 1.5, 20, 600, mu=0.35, levels=3, weighted=True, wmax=255, seed=9)
    row = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    up = row < g.col
    return g.n, [row[up]], [g.col[up]], [g.w[up]], [[q] for q in range(0, g.n, 97)], np.array([1.3, 1.0, 0.7, 0.5])


CASES = {"hub": _hub, "ties": _ties, "runs": _runs}


@pytest.fixture(scope="module", params=list(CASES))
def case(request):
    n, u, v, w, sets, sc = CASES[request.param]()
    g = W.csr_from_edges(n, np.concatenate(u), np.concatenate(v), np.concatenate(w))
    sp = np.concatenate([[0], np.cumsum([len(s) for s in sets])]).astype(np.int32)
    sn = np.concatenate(sets).astype(np.int32)
    return g, sc, sp, sn, oracle.Oracle.from_graph(g).run_sets(sp, sn, sc)


@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_queue_branches_match_oracle(L, case, layout):
    g, sc, sp, sn, ref = case
    kw, kind, cap = LAYOUTS[layout]
    n, rp = g.n, g.row_ptr
    if cap >= 65536:
        n = N_WIDE
        rp = np.concatenate([rp, np.full(n - g.n, g.nnz)]).astype(np.int32)
    elif kind == 3:
        cap = min(cap, 1 << (n - 1).bit_length())      # one table kind: every node fits
    elif n <= cap:
        n, rp = cap + 1, np.concatenate([rp, np.full(cap + 1 - g.n, g.nnz)]).astype(np.int32)
    res = L.lcd_sweep(L.Graph.from_host(n, rp, g.col, g.w), sc, sp, sn, **kw)
    st = res.stats()
    assert (st["tier_kind"][1], st["tier_capacity"][1]) == (kind, cap)
    assert st["tier"][1]["sets_finished"] > 0 and st["n_spilled"] == st["tier"][1]["sets_finished"]
    compare_results(L.sweep_to_numpy(res), ref, label=layout)
    res.free()
