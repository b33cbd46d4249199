"""Levels of 2^22 entries or more, which do not take the small levels' launches:
a sweep is captured and replayed, launched one by one or timed kernel by
kernel, with the classes that cannot fill the chip merged into one launch
(all but the timed ones), with and without the entry cache, for one graph and
for packed ones, against the oracle."""
import functools

import numpy as np
import pytest

import graphgen
import oracle
import paper_2507_06471_amd as lvp

pytestmark = pytest.mark.gpu

LARGE = 1 << 22


@functools.lru_cache(maxsize=None)
def one():
    g = graphgen.rmat(18, 16, seed=3)
    assert g.nnz >= LARGE
    return g, oracle.louvain(g), oracle.lpa(g)


@functools.lru_cache(maxsize=None)
def packed():
    gs = [graphgen.rmat(17, 16, seed=4), graphgen.from_edges(3, [0], [2]), graphgen.lfr(50000, seed=5)[0],
          graphgen.from_edges(40, [], []), graphgen.sbm(6000, 100, 0.3, 0.001, seed=6), graphgen.rmat(12, 16, seed=7)]
    assert sum(g.nnz for g in gs) >= LARGE
    return gs, [oracle.louvain(g) for g in gs], [oracle.lpa(g) for g in gs]


def same_louvain(got, want, what):
    assert [lv.moves for lv in got.levels] == [[int(x) for x in lv.moves] for lv in want.levels], what
    assert np.array_equal(got.final_labels, want.final_labels) and got.q_int == want.q_int, what


def same_lpa(got, want, what):
    assert np.array_equal(got.labels, want.labels) and got.moves == [int(x) for x in want.moves], what


@pytest.mark.parametrize("cache", [True, False])
@pytest.mark.parametrize("driver", ["captured", "eager", "timed"])
def test_one_graph(driver, cache):
    g, lou, lpa = one()
    kw = dict(timing=driver == "timed", hipgraph=driver == "captured", cache=cache)
    with lvp.Graph.from_csr(g) as dg:
        for rep in range(2):
            got = lvp.louvain(dg, **kw)
            same_louvain(got, lou, (driver, cache, rep))
            same_lpa(lvp.lpa(dg, **kw), lpa, (driver, cache, rep))
            if not cache:
                assert got.levels[0].info["cached_sweeps"] == 0


@pytest.mark.parametrize("cache", [True, False])
@pytest.mark.parametrize("driver", ["captured", "eager"])
def test_packed_graphs(driver, cache):
    gs, lou, lpa = packed()
    kw = dict(hipgraph=driver == "captured", cache=cache)
    with lvp.Graph.batch(gs) as bg:
        for rep in range(2):
            for i, r in enumerate(lvp.louvain(bg, **kw)):
                same_louvain(r, lou[i], (driver, cache, rep, i))
            for i, r in enumerate(lvp.lpa_batch(bg, **kw)):
                same_lpa(r, lpa[i], (driver, cache, rep, i))


@pytest.mark.parametrize("tuning", [{"block_max": 64, "part_keys": 48, "part_slots": 64}, {"fused": 1}, {"hub_mode": 1},
                                    {"sub_max": 8, "wave_max": 8, "block_max": 2000}])
def test_other_schedules(tuning):
    g, lou, lpa = one()
    with lvp.Graph.from_csr(g) as dg:
        same_louvain(lvp.louvain(dg, tuning=tuning), lou, tuning)
        same_lpa(lvp.lpa(dg, tuning=tuning), lpa, tuning)
