"""Device memory that an idle handle holds: the stored graph and its reverse
map (4 bytes an entry each for columns, weights and map), what little set-up
leaves for the first call, and no more."""
import functools

import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2507_06471_amd as lvp

pytestmark = pytest.mark.gpu

HANDLES = 4
SLACK = 16 << 20  # 8 MiB that set-up may leave, and slabs in whole MiB


@functools.lru_cache(maxsize=None)
def graph(weighted):
    g = graphgen.rmat(18, 16, seed=3)
    if weighted:
        g = graphgen.CSR(g.n, g.offsets, g.indices, graphgen.pair_weights(g, 1, 8, 1))
    return g, oracle.lpa(g).labels


def per_handle(make):
    """(bytes of device memory that each of a few handles holds, one of the handles)"""
    make().close()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    hs = [make() for _ in range(HANDLES)]
    held = (before - torch.cuda.mem_get_info()[0]) / HANDLES
    for h in hs[1:]:
        h.close()
    return held, hs[0]


@pytest.mark.parametrize("options", [{}, {"keep_order": True}, {"entry_cache": False}, {"validate": False}])
@pytest.mark.parametrize("weighted", [False, True])
def test_handle_of_a_csr(weighted, options):
    g, labels = graph(weighted)
    held, h = per_handle(lambda: lvp.Graph.from_csr(g, **options))
    stored = g.nnz * (4 + 4 * weighted + 4 * options.get("entry_cache", True)) + 24 * g.n
    print(f"nnz={g.nnz} stored {stored >> 20} MiB, held {held / 2**20:.1f} MiB", flush=True)
    assert held <= stored + SLACK
    with h:  # and the handle is whole
        off, idx, w = h.csr()
        got = lvp.lpa(h)
    assert np.array_equal(off, g.offsets) and np.array_equal(idx, g.indices) and np.array_equal(w, g.weights_or_ones())
    assert np.array_equal(got.labels, labels)


@pytest.mark.parametrize("keep_order", [False, True])
@pytest.mark.parametrize("kind", ["simple", "counted", "weighted"])
def test_handle_of_an_edge_list(kind, keep_order):
    rng = np.random.default_rng(8)
    n, m = 200000, 3000000
    u, v = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
    w = rng.integers(1, 9, m).astype(np.int32) if kind == "weighted" else None
    held, h = per_handle(lambda: lvp.Graph.from_edges(n, u, v, w, simple=kind == "simple", keep_order=keep_order))
    # weights in each of the three: the list has loops.  Counted by listings: repeats are found late.
    stored = 2 * m * 12 + 24 * n
    print(f"nnz={h.nnz} stored {stored >> 20} MiB, held {held / 2**20:.1f} MiB", flush=True)
    assert held <= stored + SLACK
    with h:
        off, idx, ww = h.csr()
    o, i, x = oracle.graph_from_edges(n, u, v, w, simple=kind == "simple")
    assert np.array_equal(off, o) and np.array_equal(idx, i) and np.array_equal(ww, x)
