"""The model-wide selection where a unit's rows (layers x KV heads) end inside a trip of four or of two rows for each of the 16 lane
groups, or leave some groups without a row: page lists against the oracle, bit for bit."""
from __future__ import annotations

import pytest

import workload
from helpers import plan_of
from test_gpu_shared_scope import assert_lists_equal, layers_of, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cluster", [0, 2])
@pytest.mark.parametrize("heads,n_layers", [(1, 15), (1, 17), (3, 11), (3, 21), (2, 32), (5, 13), (16, 5), (17, 4), (8, 12), (7, 14), (3, 43)])
def test_rows_around_a_trip(heads, n_layers, cluster):
    lens = [1500, 700, 100]
    sp = workload.WorkloadSpec("rows", 3, (0, 1500), heads, heads, 16, ("fixed", 96), (1, 1), 1, 2, budget_bp=800,
                               pages_per_chunk=4, chunks_per_grid=4)
    ids, nsel, _, oids, onsel, _, lib, *_ = run_both(sp, layers_of(sp, range(70, 70 + n_layers), lens), plan_of(sp), cluster,
                                                     max_sel=sp.max_pages)
    assert_lists_equal(ids, nsel, oids, onsel, heads)
    lib.close()


@pytest.mark.parametrize("heads,n_layers", [(1, 15), (1, 17), (8, 4), (8, 7), (7, 14), (3, 43)])
def test_infinite_components_keep_their_sign(heads, n_layers):
    """One row of two pages holds an infinity of either sign: their scores, and those of their chunks and grids, are infinite and not NaN,
    also where the last trip over the rows has fewer than the others."""
    lens = [1500, 700]
    sp = workload.WorkloadSpec("inf", 2, (0, 1500), heads, heads, 16, ("fixed", 96), (1, 1), 1, 2, budget_bp=800,
                               pages_per_chunk=4, chunks_per_grid=4)
    wls = layers_of(sp, range(90, 90 + n_layers), lens)
    for page, value in ((18, float("inf")), (34, float("-inf"))):      # in a grid each
        wls[0].k_pool[wls[0].block_table[:, page].long(), 0, 3, 5] = value
    ids, nsel, _, oids, onsel, _, lib, *_ = run_both(sp, wls, plan_of(sp), max_sel=sp.max_pages)
    assert_lists_equal(ids, nsel, oids, onsel, heads)
    lib.close()
