"""The fused step with more (sequence, KV head) rows than two workgroups a compute unit hold (its leaner kernel): empty and
one-token sequences, sequences that the safety pages cover, partial pages, the tail refresh, a ratio plan and a budget, against
the oracle, twice on one workspace."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_20732_amd as pk
import workload
from gpu_common import assert_summaries_equal, config_of, gpu_plan, host_views, run_oracle, to_device
from helpers import plan_of

pytestmark = pytest.mark.gpu
ATOL_TIGHT = 2e-3     # fp32 accumulation of bf16 inputs gives about 1e-6; the stated bar of the path is 1e-2


@pytest.mark.parametrize("page,group,fans", [(16, 1, (4, 2)), (16, 4, (16, 16)), (32, 7, (4, 2)), (32, 16, (2, 4))])
@pytest.mark.parametrize("refresh", [False, True])
def test_more_rows_than_two_workgroups_a_compute_unit(page, group, fans, refresh):
    heads = 8
    batch = 2 * torch.cuda.get_device_properties(0).multi_processor_count // heads + 3
    rng = np.random.default_rng(page + group)
    lens = [0, 1, page, 3 * page + 1, 900] + [int(x) for x in rng.integers(1, 900, batch - 5)]
    sp = workload.WorkloadSpec("rows", batch, (0, 900), heads * group, heads, page, ("fixed", 64), (1, 2), 1, 2, budget_pages=4,
                               pages_per_chunk=fans[0], chunks_per_grid=fans[1])
    wl = workload.generate(sp, 61, seq_lens=lens)
    d = to_device(wl)
    for kw in ({}, dict(sink_pages=0, window_pages=0, plan=oracle.PLAN_RATIO, rho_g_bp=5000, rho_c_bp=4000, rho_p_bp=3000)):
        plan = plan_of(sp, **kw)
        lib = pk.Chess(config_of(sp, max_selected=sp.max_pages))
        ref = run_oracle(wl, plan, sp.max_pages, dense=False)
        summ, ws = lib.new_summaries(), lib.new_workspace()
        lib.summarize(d.k_pool, d.block_table, d.seq_lens, summ)
        for turn in range(2):
            ids = torch.full((batch, heads, sp.max_pages), -7, dtype=torch.int32, device="cuda")
            nsel = torch.full((batch, heads), -7, dtype=torch.int32, device="cuda")
            out = torch.full((batch, sp.n_q_heads, 128), float("nan"), device="cuda")
            if refresh:                                           # stale tail vectors: the step has to renew them
                pv, cv, gv = lib.summary_views(summ)
                for b, L in enumerate(lens):
                    if L > 0:
                        p = -(-L // page) - 1
                        pv[b, :, p] = 5.0; cv[b, :, p // fans[0]] = -9.0; gv[b, :, p // fans[0] // fans[1]] = 3.0
            lib.decode_step(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, summ, gpu_plan(plan), ids, nsel, out, ws, refresh_tail=refresh)
            torch.cuda.synchronize()
            assert lib.workspace_error(ws) == 0
            assert np.array_equal(nsel.cpu().numpy(), ref.nsel) and np.array_equal(ids.cpu().numpy(), ref.ids), turn
            assert np.abs(out.cpu().numpy() - ref.out).max() <= ATOL_TIGHT

            class Got:
                pages, chunks, grids = host_views(lib, summ, batch)
            assert_summaries_equal(Got, ref, sp, lens)
        lib.close()


RATIO = dict(plan=oracle.PLAN_RATIO, rho_g_bp=4000, rho_c_bp=5000, rho_p_bp=3000)


@pytest.mark.parametrize("page,group,fans,pages,kw", [
    (16, 1, (1, 1), 1100, {}),                             # levels of 1100, some 300 and 60 slots
    (16, 4, (2, 2), 1100, RATIO),                          # 275, 220 and 220
    (16, 4, (4, 4), 1100, dict(plan=oracle.PLAN_FLAT)),    # every page in one level
    (32, 7, (1, 1), 600, RATIO),                           # 600, 240 and 120
    (32, 16, (8, 8), 1100, dict(budget_pages=40)),         # 18 of 18, 50 of 138, 400 slots
])
def test_long_rows_among_many(page, group, fans, pages, kw):
    """A few long sequences among rows enough for the leaner kernel: several trips of its scoring, and every cut but the smallest.
    The selection by itself as well, alone on its rows there."""
    batch = 2 * torch.cuda.get_device_properties(0).multi_processor_count + 5
    lens = [pages * page, pages * page - 7, (pages // 2) * page + 1] + [(7 * b) % (5 * page) for b in range(batch - 3)]
    sp = workload.WorkloadSpec("long_rows", batch, (0, pages * page), group, 1, page, ("geometric", 128), (1, 3), 1, 2, budget_pages=6,
                               pages_per_chunk=fans[0], chunks_per_grid=fans[1])
    wl = workload.generate(sp, 67, seq_lens=lens)
    d = to_device(wl)
    plan = plan_of(sp, **kw)
    max_sel = 400
    ref = run_oracle(wl, plan, max_sel, dense=False)
    lib = pk.Chess(config_of(sp, max_selected=max_sel))
    summ, ws = lib.new_summaries(), lib.new_workspace()
    lib.summarize(d.k_pool, d.block_table, d.seq_lens, summ)
    for turn in range(2):
        ids = torch.full((batch, 1, max_sel), -7, dtype=torch.int32, device="cuda")
        nsel = torch.full((batch, 1), -7, dtype=torch.int32, device="cuda")
        ids2, nsel2 = ids.clone(), nsel.clone()
        out = torch.full((batch, group, 128), float("nan"), device="cuda")
        lib.decode_step(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, summ, gpu_plan(plan), ids, nsel, out, ws, refresh_tail=True)
        lib.select(d.q, summ, d.seq_lens, gpu_plan(plan), ids2, nsel2, ws)
        torch.cuda.synchronize()
        for i, n in ((ids, nsel), (ids2, nsel2)):
            assert np.array_equal(n.cpu().numpy(), ref.nsel) and np.array_equal(i.cpu().numpy(), ref.ids), turn
        assert np.abs(out.cpu().numpy() - ref.out).max() <= ATOL_TIGHT
    lib.close()
