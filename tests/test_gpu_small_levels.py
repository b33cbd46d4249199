"""Small levels: two launches a sweep (every class in one launch whose movers
are committed in place, then the pair refresh).  Sizes at the edges of the
classes and of the workgroups' row blocks, hubs, packed graphs that stop at
different sweeps, few and many movers per workgroup, and the size at which a
level leaves the path, against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle
import paper_2507_06471_amd as lvp
from test_gpu_parity import compare_louvain, compare_lpa

pytestmark = pytest.mark.gpu


def stars(degrees, extra, seed):
    """Vertices of the given degrees over a common pool, plus `extra` random edges; random weights."""
    rng = np.random.default_rng(seed)
    pool = max(degrees) + 7
    n = len(degrees) + pool
    u = [np.full(d, i) for i, d in enumerate(degrees)]
    v = [len(degrees) + rng.choice(pool, size=d, replace=False) for d in degrees]
    u.append(rng.integers(0, n, extra))
    v.append(rng.integers(0, n, extra))
    u, v = np.concatenate(u), np.concatenate(v)
    return graphgen.from_edges(n, u, v, rng.integers(1, 6, len(u)))


# every class bound and its neighbours; 8193 is a hub
EDGES = [1, 3, 4, 5, 8, 9, 32, 33, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 3072, 3073, 8191]


@pytest.mark.parametrize("extra", [0, 20000])
@pytest.mark.parametrize("hub", [False, True])
def test_class_edges(extra, hub):
    g = stars(EDGES + ([8193, 12000] if hub else []), extra, 5)
    g.name = f"stars extra={extra} hub={hub}"
    compare_louvain(g, keep_graphs=True)
    compare_lpa(g)


@pytest.mark.parametrize("rows", [127, 128, 129, 255, 256, 257, 1023, 1024, 1025])
def test_row_blocks(rows):
    # rows of 2 (ring) and of 6 entries around one workgroup's block of rows
    ring = np.arange(rows)
    g = graphgen.from_edges(rows, ring, (ring + 1) % rows)
    g.name = f"ring {rows}"
    compare_louvain(g)
    compare_lpa(g)
    u = np.tile(ring, 3)
    v = np.concatenate([(ring + k) % rows for k in (1, 2, 3)])
    h = graphgen.from_edges(rows, u, v, 1 + (u * 7 + v) % 5)
    h.name = f"band {rows}"
    compare_louvain(h)
    compare_lpa(h)


@pytest.mark.parametrize("sweeps", [1, 2, 3, 4, 5, 20, 41])
def test_sweep_limits(sweeps):
    # fewer, as many and more sweeps than the host runs ahead
    g = graphgen.sbm(3000, 125, 0.06, 0.001, seed=sweeps)
    want = oracle.louvain(g, max_sweeps=sweeps)
    with lvp.Graph.from_csr(g) as dg:
        got = lvp.louvain(dg, max_sweeps=sweeps)
        lp = lvp.lpa(dg, max_sweeps=sweeps)
    assert [lv.moves for lv in got.levels] == [[int(x) for x in lv.moves] for lv in want.levels]
    assert np.array_equal(got.final_labels, want.final_labels) and got.q_int == want.q_int
    wl = oracle.lpa(g, max_sweeps=sweeps)
    assert np.array_equal(lp.labels, wl.labels) and lp.moves == [int(x) for x in wl.moves]


def test_many_movers_into_few_communities():
    # complete bipartite-like crowding: thousands of rows join a handful of communities in one sweep
    rng = np.random.default_rng(9)
    n, hubs = 9000, 6
    u = np.repeat(np.arange(hubs, n), 2)
    v = rng.integers(0, hubs, len(u))
    g = graphgen.from_edges(n, u, v, rng.integers(1, 4, len(u)))
    g.name = "crowd"
    compare_louvain(g)
    compare_lpa(g)


def test_packed_graphs_of_unequal_length():
    gs = [graphgen.sbm(700, 100, 0.1, 0.001, seed=1), graphgen.rmat(9, seed=2),
          graphgen.from_edges(2, [0], [1]), graphgen.rmat(13, seed=3),
          graphgen.from_edges(5, [], []), stars([8193, 40], 100, 6)]
    with lvp.Graph.batch(gs) as bg:
        got = lvp.louvain(bg)
        lp = lvp.lpa(bg)
    for i, g in enumerate(gs):
        want = oracle.louvain(g)
        assert np.array_equal(got[i].final_labels, want.final_labels), i
        assert [lv.moves for lv in got[i].levels] == [[int(x) for x in lv.moves] for lv in want.levels], i
        wl = oracle.lpa(g)
        assert np.array_equal(lp[i].labels, wl.labels) and lp[i].moves == [int(x) for x in wl.moves], i


@pytest.mark.parametrize("drop", [1, 0])
def test_both_sides_of_the_size_rule(drop):
    # 2^22 - 2 entries (the last small size) and 2^22: a weighted circulant of degree 64
    n = 1 << 16
    u = np.tile(np.arange(n), 32)
    v = (u + np.repeat(np.arange(1, 33), n)) % n
    w = 1 + (u * 2654435761 % 4294967296 >> 13) % 7
    keep = len(u) - drop
    g = graphgen.from_edges(n, u[:keep], v[:keep], w[:keep])
    assert g.nnz == (1 << 22) - 2 * drop
    g.name = f"size rule {g.nnz}"
    compare_louvain(g)
    compare_lpa(g)


@pytest.mark.parametrize("tuning", [None, {"agg_sort": 1}])
@pytest.mark.parametrize("gap", [1, 63, 2047, 2048, 4097, 9001])
def test_runs_of_empty_rows(gap, tuning):
    # entries between runs of isolated vertices, so that a tile of rows holds none, one or a few
    at = np.arange(40) * (gap + 1) + gap // 2
    u = np.concatenate([at[:-1], at[:-3], [at[-1]]])
    v = np.concatenate([at[1:], at[3:], [at[-1]]])
    g = graphgen.from_edges(int(at[-1]) + 1 + gap, u, v, 1 + np.arange(len(u)) % 3)
    g.name = f"gap {gap}"
    compare_louvain(g, tuning=tuning, keep_graphs=True)
    compare_louvain(g, tuning=tuning, keep_order=True)
    compare_lpa(g)
    with lvp.Graph.from_csr(g) as dg:
        off, idx, w = dg.csr()
    assert np.array_equal(off, g.offsets) and np.array_equal(idx, g.indices) and np.array_equal(w, g.weights)


@pytest.mark.parametrize("n", [1, 2, 1023, 8191, 8192, 8193, 16385, 64 * 8192 + 1, 130 * 8192 + 77])
def test_scan_tiles(n):
    # vertex counts around the tiles of the renumbering scan, up to several look-back windows;
    # a few communities spread over the whole range of ids and both ends
    rng = np.random.default_rng(n)
    at = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 300)]))
    u = at[rng.integers(0, len(at), 900)]
    v = at[rng.integers(0, len(at), 900)]
    g = graphgen.from_edges(n, u, v, rng.integers(1, 5, 900))
    g.name = f"scan n={n}"
    compare_louvain(g, keep_graphs=True)
    compare_louvain(g, keep_order=True)
    compare_lpa(g)


def test_packed_graphs_with_empty_ones():
    empty = graphgen.from_edges(0, [], [])
    lone = graphgen.from_edges(3, [], [])
    gs = [empty, lone, graphgen.sbm(500, 50, 0.2, 0.002, seed=4), empty, graphgen.from_edges(2, [0, 0], [1, 0]), lone,
          empty]
    with lvp.Graph.batch(gs) as bg:
        got = lvp.louvain(bg)
    for i, g in enumerate(gs):
        want = oracle.louvain(g)
        assert np.array_equal(got[i].final_labels, want.final_labels), i
        assert got[i].q_int == want.q_int


@pytest.mark.parametrize("drop", [1, 0, -1])
def test_both_sides_of_the_hashing_rule(drop):
    # 2^20 - 2, 2^20 (the last to be hashed) and 2^20 + 2 entries
    n = 1 << 15
    u = np.tile(np.arange(n), 16)
    v = (u + np.repeat(np.arange(1, 17), n)) % n
    keep = len(u) - max(drop, 0)
    u, v = u[:keep], v[:keep]
    if drop < 0:
        u, v = np.append(u, 0), np.append(v, n // 2)
    g = graphgen.from_edges(n, u, v, 1 + (u * 48271 + v * 7) % 6)
    assert g.nnz == (1 << 20) - 2 * drop
    g.name = f"hash rule {g.nnz}"
    compare_louvain(g, keep_graphs=True)


@pytest.mark.parametrize("n", [1, 5, 256, 1023, 4097, 300000])
@pytest.mark.parametrize("kind", ["one", "own", "few", "random"])
def test_modularity_of_labels(n, kind):
    # one community, every vertex its own, a handful, and more than a workgroup's table holds
    rng = np.random.default_rng(n)
    m = 3 * n
    g = graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(1, 9, m))
    lab = {"one": np.full(n, n - 1), "own": rng.permutation(n), "few": rng.integers(0, min(n, 5), n),
           "random": rng.integers(0, n, n)}[kind].astype(np.int32)
    row = np.repeat(np.arange(n), np.diff(g.offsets))
    a = g.weights.astype(np.int64) * np.where(row == g.indices, 2, 1)
    k = np.bincount(row, weights=a, minlength=n).astype(np.int64)
    vol = np.zeros(n, dtype=np.int64)
    np.add.at(vol, lab, k)
    M = int(k.sum())
    want = M * int(a[lab[row] == lab[g.indices]].sum()) - int((vol * vol).sum())
    bad = lab.copy()
    bad[n // 2] = n if n % 2 else -1
    for keep_order in (False, True):
        with lvp.Graph.from_csr(g, keep_order=keep_order) as dg:
            assert lvp.modularity(dg, lab)[:2] == (want, M)
            with pytest.raises(lvp.LvError):
                lvp.modularity(dg, bad)
            assert lvp.modularity(dg, lab)[:2] == (want, M)
