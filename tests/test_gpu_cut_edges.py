"""The cuts of a selection level at the sizes where one way of cutting hands over to the next (64 and 256 slots) and
where a search by value has the least to go by: all keys but one equal, one key far above the rest, k of 1 and of all
but one.  Page lists are compared with the oracle's exactly: both sides score in fp64 and rank by (score, index)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2602_20732_amd as pk
import workload
from gpu_common import config_of, gpu_plan, to_device
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


@pytest.mark.parametrize("pages,fans,rho", [(60, (1, 1), (9000, 9500, 2000)), (200, (1, 1), (9000, 9500, 300)),
                                            (768, (8, 8), (5500, 1700, 1000))])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_nan_scores_do_not_upset_a_cut(pages, fans, rho, sign):
    """Pages whose keys are NaN (their rank is not defined): every cut still keeps exactly what the general path keeps,
    which ranks the 64-bit keys, whatever the cluster and the schedule; nobody waits in vain.  The last shape merges the
    chunk level: 96 slots of which 56 (7 of 12 grids) compete."""
    sp = workload.WorkloadSpec("nan", 1, (pages * 16, pages * 16), 4, 1, 16, ("fixed", 48), (1, 1), SINK, WINDOW,
                               budget_pages=5, pages_per_chunk=fans[0], chunks_per_grid=fans[1])
    wl = workload.generate(sp, 50 + pages)
    for j in range(pages // 4, pages, 17):
        wl.k_pool[wl.block_table[0, j].item(), 0, 3] = sign * float("nan")
    d = to_device(wl)
    plan = gpu_plan(plan_of(sp, plan=oracle.PLAN_RATIO, budget_pages=0, rho_g_bp=rho[0], rho_c_bp=rho[1], rho_p_bp=rho[2]))
    lib = pk.Chess(config_of(sp, max_selected=sp.max_pages))
    summ = lib.new_summaries()
    lib.summarize(d.k_pool, d.block_table, d.seq_lens, summ)

    def lists(general, cluster, schedule):
        lib.debug_force_general_cut(general)
        lib.debug_force_cluster(cluster)
        lib.debug_force_schedule(schedule)
        ws, got = lib.new_workspace(), []
        ids = torch.full((1, 1, sp.max_pages), -7, dtype=torch.int32, device="cuda")
        nsel = torch.full((1, 1), -7, dtype=torch.int32, device="cuda")
        out = torch.empty((1, sp.n_q_heads, 128), device="cuda")
        lib.select(d.q, summ, d.seq_lens, plan, ids, nsel, ws)
        torch.cuda.synchronize()
        assert lib.workspace_error(ws) == 0, "a kernel gave up a bounded wait"
        got.append((ids.clone(), nsel.clone()))
        lib.decode_step(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, summ, plan, ids, nsel, out, ws)
        torch.cuda.synchronize()
        assert lib.workspace_error(ws) == 0, "a kernel gave up a bounded wait"
        got.append((ids, nsel))
        return got

    want = lists(True, 1, 1)[0]
    n = int(want[1])
    row = want[0][0, 0, :n].tolist()
    assert row == sorted(set(row)) and row[0] == 0 and row[-1] == pages - 1 and n < pages
    for cluster in (1, 2, 8):
        for schedule in (1, 2):
            for ids, nsel in lists(False, cluster, schedule):
                assert torch.equal(nsel, want[1]) and torch.equal(ids, want[0]), (cluster, schedule)
    lib.close()
