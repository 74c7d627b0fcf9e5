"""The merge of split partials where its shape changes: up to six, eight, twelve, sixteen splits and beyond, one pair of outputs
a thread and two (more than four query heads), splits without a tile; forced, against the same lists attended without a split."""
import pytest
import torch

import paper_2602_20732_amd as pk
import workload
from gpu_common import config_of, gpu_plan, to_device
from helpers import plan_of

pytestmark = pytest.mark.gpu
ATOL = 2e-5           # fp32 sums of weights that add up to 1 over |v| < 6, in another order


@pytest.mark.parametrize("group", [1, 4, 5, 7, 16])
def test_any_number_of_splits_gives_the_same_sums(group):
    sp = workload.WorkloadSpec("merge", 3, (0, 1600), 2 * group, 2, 16, ("fixed", 96), (1, 2), 1, 2, budget_pages=60,
                               pages_per_chunk=4, chunks_per_grid=4)
    d = to_device(workload.generate(sp, 17, seq_lens=[1590, 700, 40]))
    lib = pk.Chess(config_of(sp, max_selected=sp.max_pages))
    summ, ws = lib.new_summaries(), lib.new_workspace()
    lib.summarize(d.k_pool, d.block_table, d.seq_lens, summ)
    ids = torch.full((3, 2, sp.max_pages), -7, dtype=torch.int32, device="cuda")
    nsel = torch.full((3, 2), -7, dtype=torch.int32, device="cuda")
    lib.select(d.q, summ, d.seq_lens, gpu_plan(plan_of(sp)), ids, nsel, ws)
    want = torch.empty((3, sp.n_q_heads, 128), device="cuda")
    lib.debug_force_splits(1, 4)
    lib.sparse_decode(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, ids, nsel, want, ws)
    for waves in (4, 8):
        for splits in (2, 5, 6, 7, 8, 9, 12, 13, 16, 17, 40):
            lib.debug_force_splits(splits, waves)
            out = torch.full_like(want, float("nan"))
            lib.sparse_decode(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, ids, nsel, out, ws)
            torch.cuda.synchronize()
            assert lib.workspace_error(ws) == 0
            assert float((out - want).abs().max()) <= ATOL, (waves, splits)
    lib.close()
