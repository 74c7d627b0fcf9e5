"""The fused step asks for the first phase's vectors before it knows a sequence's length, by the configuration's units: sequences far
shorter than the configuration allows (what their summaries do not have holds NaN), members without a share, the lazy, the merged and
the eager schedule, one workgroup to a row and several, levels that keep every grid; against the oracle, twice on one workspace."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_20732_amd as pk
import workload
from gpu_common import config_of, gpu_plan, run_oracle, to_device
from helpers import plan_of

pytestmark = pytest.mark.gpu
ATOL_TIGHT = 2e-3     # fp32 accumulation of bf16 inputs gives about 1e-6; the stated bar of the path is 1e-2
LENS = [9000, 0, 1, 16 * 16 + 1, 80, 1030, 5000]


@pytest.mark.parametrize("schedule,cluster", [(0, 0), (1, 1), (1, 3), (1, 12), (2, 2), (2, 12), (3, 5), (3, 32)])
@pytest.mark.parametrize("page,group,refresh", [(16, 4, True), (16, 1, False), (32, 7, True)])
def test_rows_shorter_than_the_configuration(schedule, cluster, page, group, refresh):
    sp = workload.WorkloadSpec("room", len(LENS), (0, 20000), 2 * group, 2, page, ("fixed", 96), (1, 2), 1, 2, budget_pages=9,
                               pages_per_chunk=4, chunks_per_grid=4)
    wl = workload.generate(sp, 977, seq_lens=LENS)
    d = to_device(wl)
    lib = pk.Chess(config_of(sp, max_selected=sp.max_pages))
    lib.debug_force_schedule(schedule)
    lib.debug_force_cluster(cluster)
    for kw in ({}, dict(budget_pages=200), dict(probe=oracle.PROBE_ANCHOR)):
        plan = plan_of(sp, **kw)
        renew = refresh and plan.probe != oracle.PROBE_ANCHOR
        ref = run_oracle(wl, plan, sp.max_pages, dense=False)
        summ, ws = lib.new_summaries(), lib.new_workspace()
        summ.fill_(0xFF)                                          # NaN, fp32 and bf16
        lib.summarize(d.k_pool, d.block_table, d.seq_lens, summ)
        for turn in range(2):
            ids = torch.full((len(LENS), 2, sp.max_pages), -7, dtype=torch.int32, device="cuda")
            nsel = torch.full((len(LENS), 2), -7, dtype=torch.int32, device="cuda")
            out = torch.full((len(LENS), sp.n_q_heads, 128), float("nan"), device="cuda")
            lib.decode_step(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, summ, gpu_plan(plan), ids, nsel, out, ws, refresh_tail=renew)
            torch.cuda.synchronize()
            assert lib.workspace_error(ws) == 0
            assert np.array_equal(nsel.cpu().numpy(), ref.nsel) and np.array_equal(ids.cpu().numpy(), ref.ids), (kw, turn)
            assert np.abs(out.cpu().numpy() - ref.out).max() <= ATOL_TIGHT, (kw, turn)
    lib.close()
