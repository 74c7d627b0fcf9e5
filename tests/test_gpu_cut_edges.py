"""The cuts of a selection level at the sizes where one way of cutting hands over to the next (64 and 256 slots) and
where a search by value has the least to go by: all keys but one equal, one key far above the rest, k of 1 and of all
but one.  Page lists are compared with the oracle's exactly: both sides score in fp64 and rank by (score, index)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import workload
from helpers import plan_of
from test_gpu_parity import check_all

pytestmark = pytest.mark.gpu

SINK, WINDOW = 1, 2


def spec_of(pages):
    # (chunks of one page and grids of one chunk: every level has as many slots as there are pages)
    return workload.WorkloadSpec("edges", 1, (pages * 16, pages * 16), 4, 1, 16, ("fixed", 48), (1, 1), SINK, WINDOW,
                                 budget_pages=5, pages_per_chunk=1, chunks_per_grid=1)


@pytest.mark.parametrize("pages", [63, 64, 65, 127, 255, 256, 257])
@pytest.mark.parametrize("rho_bp", [1, 700, 5000, 9990])
def test_levels_at_the_edges_of_the_cuts(pages, rho_bp):
    sp = spec_of(pages)
    wl = workload.generate(sp, 40 + pages)
    plan = plan_of(sp, plan=oracle.PLAN_RATIO, budget_pages=0, rho_g_bp=9000, rho_c_bp=9500, rho_p_bp=rho_bp)
    check_all(sp, wl, plan, max_sel=sp.max_pages, dense=False, label=f"{pages} pages, rho {rho_bp}")


@pytest.mark.parametrize("pages", [60, 200])
@pytest.mark.parametrize("shape", ["one_above", "one_below", "far_above", "two_values"])
@pytest.mark.parametrize("cut_rule", [oracle.CUT_COUNT, oracle.CUT_THRESHOLD])
def test_scores_with_little_to_search_by(pages, shape, cut_rule):
    sp = spec_of(pages)
    wl = workload.generate(sp, 7)
    base = wl.k_pool[wl.block_table[0, 3].item(), 0, 0].clone()
    for j in range(pages):
        row = base
        if shape == "one_above" and j == pages // 2:
            row = (base.float() + 0.01 * wl.q[0].float().sum(0).sign()).to(torch.bfloat16)
        elif shape == "one_below" and j == pages // 2:
            row = -base
        elif shape == "far_above" and j == pages // 3:
            row = (base.float() + 1e18 * wl.q[0].float().sum(0).sign()).to(torch.bfloat16)
        elif shape == "two_values" and j % 2:
            row = -base
        wl.k_pool[wl.block_table[0, j].item(), 0, :] = row
    plan = plan_of(sp, plan=oracle.PLAN_RATIO, budget_pages=0, rho_g_bp=8000, rho_c_bp=8000, rho_p_bp=3000, cut_rule=cut_rule)
    gpu, ref = check_all(sp, wl, plan, max_sel=sp.max_pages, dense=False, label=f"{shape}, {pages} pages")
    assert np.array_equal(gpu.ids, ref.ids)
