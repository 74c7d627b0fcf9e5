"""The model-wide selection where a unit's rows (layers x KV heads) end inside a trip of four rows for each of the 16 lane
groups, or leave some groups without a row: page lists against the oracle, bit for bit."""
from __future__ import annotations

import pytest

import workload
from helpers import plan_of
from test_gpu_shared_scope import assert_lists_equal, layers_of, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cluster", [0, 2])
@pytest.mark.parametrize("heads,n_layers", [(1, 15), (1, 17), (3, 21), (2, 32), (5, 13), (16, 5), (17, 4), (3, 43)])
def test_rows_around_a_trip(heads, n_layers, cluster):
    lens = [1500, 700, 100]
    sp = workload.WorkloadSpec("rows", 3, (0, 1500), heads, heads, 16, ("fixed", 96), (1, 1), 1, 2, budget_bp=800,
                               pages_per_chunk=4, chunks_per_grid=4)
    ids, nsel, _, oids, onsel, _, lib, *_ = run_both(sp, layers_of(sp, range(70, 70 + n_layers), lens), plan_of(sp), cluster,
                                                     max_sel=sp.max_pages)
    assert_lists_equal(ids, nsel, oids, onsel, heads)
    lib.close()
