"""Set-up of a graph: the symmetry check and the reverse-entry map, both from
the stable order of the entries by column.  Asymmetric graphs of every kind
are refused when validated (and only lose the entry cache when not), symmetric
ones pass and give the oracle's result from cached sweeps, at vertex counts
around the sort's digits."""
import numpy as np
import pytest

import graphgen
import oracle
import paper_2507_06471_amd as lvp

pytestmark = pytest.mark.gpu

ASYMMETRIC = 3


def random_graph(n, m, seed, loops=True):
    rng = np.random.default_rng(seed)
    u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    if not loops:
        u, v = u[u != v], v[u != v]
    return graphgen.from_edges(n, u, v, rng.integers(1, 9, len(u)))


def status(g):
    try:
        with lvp.Graph.from_csr(g, validate=True):
            return 0
    except lvp.LvError as e:
        return e.status


@pytest.mark.parametrize("n", [1, 2, 3, 255, 256, 257, 2047, 65535, 65536, 65537, 70000])
def test_symmetric_graphs_pass_and_cache(n):
    g = random_graph(n, 4 * n + 3, n)
    assert status(g) == 0
    want = oracle.louvain(g)
    for keep_order in (False, True):
        with lvp.Graph.from_csr(g, keep_order=keep_order) as dg:
            got = lvp.louvain(dg, tuning={"cache_pct": 100})
            off, idx, w = dg.csr()
        assert np.array_equal(off, g.offsets) and np.array_equal(idx, g.indices) and np.array_equal(w, g.weights)
        assert np.array_equal(got.final_labels, want.final_labels) and got.q_int == want.q_int
        if got.levels[0].info["sweeps"] > 2:
            assert got.levels[0].info["cached_sweeps"] == got.levels[0].info["sweeps"] - 2


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("kind", ["missing", "moved", "weight", "one_way_rows"])
def test_asymmetric_graphs_are_refused(kind, seed):
    n = [40, 300, 5000][seed % 3]
    g = random_graph(n, 5 * n, 100 + seed, loops=seed % 2 == 0)
    row = np.repeat(np.arange(n), np.diff(g.offsets))
    off, idx, w = g.offsets.copy(), g.indices.copy(), g.weights.copy()
    cand = np.flatnonzero(row != idx)
    e = int(cand[(seed * 7919) % len(cand)])
    if kind == "weight":
        w[e] += 1
    elif kind == "missing":
        idx, w = np.delete(idx, e), np.delete(w, e)
        off[row[e] + 1:] -= 1
    elif kind == "moved":  # (r, c) -> (r, c') with c' not yet in the row: equal counts, no partner
        r = row[e]
        have = set(idx[off[r]:off[r + 1]].tolist())
        c = next(x for x in range(n) if x not in have and x != r)
        seg = np.arange(off[r], off[r + 1])
        idx[e] = c
        o = np.argsort(idx[seg], kind="stable")
        idx[seg], w[seg] = idx[seg][o], w[seg][o]
    else:  # two rows trade an entry's target: in- and out-degrees stay what they were
        e2 = next(int(x) for x in cand[::-1]
                  if row[x] != row[e] and idx[x] != idx[e] and row[x] != idx[e] and row[e] != idx[x]
                  and idx[x] not in idx[off[row[e]]:off[row[e] + 1]]
                  and idx[e] not in idx[off[row[x]]:off[row[x] + 1]])
        idx[e], idx[e2] = idx[e2], idx[e]
        for r in (row[e], row[e2]):
            seg = np.arange(off[r], off[r + 1])
            o = np.argsort(idx[seg], kind="stable")
            idx[seg], w[seg] = idx[seg][o], w[seg][o]
    bad = graphgen.CSR(n, off.astype(np.int32), idx.astype(np.int32), w.astype(np.int32))
    assert status(bad) == ASYMMETRIC
    with lvp.Graph.from_csr(bad, validate=False) as dg:  # taken unchecked, without the cache unless only a weight differs
        got = lvp.louvain(dg, tuning={"cache_pct": 100}, max_sweeps=6)
    assert (got.levels[0].info["cached_sweeps"] > 0) <= (kind == "weight")


def test_validation_with_the_cache_left_out():
    g = random_graph(3000, 20000, 9)
    with lvp.Graph.from_csr(g, validate=True, entry_cache=False) as dg:
        got = lvp.louvain(dg)
    assert np.array_equal(got.final_labels, oracle.louvain(g).final_labels)


# Runs of equal keys are merged per 64-lane wavefront and per tile of 2048
# keys: run lengths around both, one run over several tiles, nothing left after
# the loops are dropped, and each way of counting (weights, listings, once).
@pytest.mark.parametrize("runs", [[1], [2048], [4097], [63, 1, 64, 65], [2047, 1, 2048, 2], [1, 2049, 5000, 3],
                                  [1] * 2047, [1] * 2049, [3] * 1366])
@pytest.mark.parametrize("how", ["weights", "listings", "once", "loops_dropped"])
def test_runs_of_equal_edges(runs, how):
    n = len(runs) + 1
    which = np.repeat(np.arange(len(runs), dtype=np.int32), runs)
    rng = np.random.default_rng(len(runs) + runs[0])
    rng.shuffle(which)
    src, dst = which, (which if how == "loops_dropped" else which + 1).astype(np.int32)
    w = rng.integers(1, 9, len(which)).astype(np.int32) if how == "weights" else None
    flags = {"simple": how == "once", "drop_loops": how == "loops_dropped"}
    want = oracle.graph_from_edges(n, src, dst, w, **flags)
    with lvp.Graph.from_edges(n, src, dst, w, **flags) as g:
        got = g.csr()
    assert all(np.array_equal(a, b) for a, b in zip(got, want))


# The sort works in wavefronts of 1024 keys, tiles of 4096 and groups of eight
# tiles: an edge list is two keys an edge, so edge counts around half of each,
# with and without weights moved along, and digits from one value to all.
@pytest.mark.parametrize("m", [1, 511, 512, 513, 2047, 2048, 2049, 16383, 16384, 16385, 18433])
@pytest.mark.parametrize("n", [2, 700, 70000])
def test_sort_sizes(m, n):
    rng = np.random.default_rng(m + n)
    src, dst = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
    for w in (None, rng.integers(1, 9, m).astype(np.int32)):
        want = oracle.graph_from_edges(n, src, dst, w)
        with lvp.Graph.from_edges(n, src, dst, w) as g:
            got = g.csr()
        assert all(np.array_equal(a, b) for a, b in zip(got, want)), w is None
