"""Out-of-memory in a later, larger call on a handle that has run before.

The walk of test_gpu_faults uses a fresh handle for every allocation point, so
no buffer holds anything yet when one fails.  Here the handle has completed a
run whose largest hashed level is small; the next run's is larger, so the
aggregation's table grows, and every allocation of that run is made to fail in
turn.  The handle must then give the oracle's result: a table that grew before
the failure holds arbitrary memory and has to be cleared before it is used."""
import os

import numpy as np
import pytest

import graphgen
import oracle
import paper_2507_06471_amd as lvp
from test_gpu_faults import LV_E_NOMEM, fault_env, free_bytes, say  # noqa: F401

pytestmark = pytest.mark.gpu

HASHED = 1 << 20  # levels of at most this many entries are aggregated in the table


def _table(run):
    """Slots of the hash table that the run's largest hashed level asks for."""
    e = max(lv.nnz for lv in run.levels if 0 < lv.nnz <= HASHED)
    return 1 << (max(1024, 2 * e) - 1).bit_length()


def test_table_that_grew_before_the_failure_is_cleared(fault_env):  # noqa: F811
    g = graphgen.rmat(16, 16, seed=13)
    first, then = oracle.louvain(g), oracle.louvain(g, max_sweeps=1)
    assert g.nnz > HASHED and _table(then) > _table(first)
    with lvp.Graph.from_csr(g) as h:  # the first kernel of a process loads the library's module (152 MiB)
        lvp.louvain(h)
    base = free_bytes()
    failed = 0
    for k in range(1, 200):
        with lvp.Graph.from_csr(g) as h:
            assert np.array_equal(lvp.louvain(h).final_labels, first.final_labels)
            os.environ["LV_FAULT_ALLOC_AT"] = str(k)
            try:
                lvp.louvain(h, max_sweeps=1)
                survived = True
            except lvp.LvError as e:
                assert e.status == LV_E_NOMEM, f"k={k}: {e}"
                survived = False
            finally:
                os.environ.pop("LV_FAULT_ALLOC_AT", None)
            for want, sweeps in ((then, 1), (first, 20)):
                got = lvp.louvain(h, max_sweeps=sweeps)
                assert np.array_equal(got.final_labels, want.final_labels) and got.q_int == want.q_int, f"k={k}"
        if survived:
            break
        failed += 1
    say(f"grown run: {failed} allocation points forced to fail, each recovered")
    assert survived and failed >= 2  # the table's keys and its sums at least
    assert abs(free_bytes() - base) < (32 << 20)
