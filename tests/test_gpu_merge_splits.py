"""The merge of split partials where its shape changes: up to six, eight, twelve, sixteen splits and beyond, one pair of outputs
a thread and two (more than four query heads), splits without a tile; forced, against the same lists attended without a split
and against softmax attention in fp64; and attention over every page, its splits dealt by length, against the latter."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_20732_amd as pk
import workload
from gpu_common import config_of, gpu_plan, host_arrays, to_device
from helpers import geom_of, plan_of

pytestmark = pytest.mark.gpu
ATOL = 2e-5           # fp32 sums of weights that add up to 1 over |v| < 6, in another order
ATOL_64 = 5e-5        # weights are carried to 2^-17 and values stay below about 5: 4e-5, and fp32 sums


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


@pytest.mark.parametrize("page", [16, 32])
@pytest.mark.parametrize("group", [1, 4, 5, 7, 9, 16])
def test_any_number_of_splits_against_64_bits(group, page):
    lens = [1590, 700, 40, 0]
    sp = workload.WorkloadSpec("merge64", 4, (0, 1600), 2 * group, 2, page, ("fixed", 96), (1, 2), 1, 2, budget_pages=960 // page,
                               pages_per_chunk=4, chunks_per_grid=4)
    wl = workload.generate(sp, 23 + group, seq_lens=lens)
    d = to_device(wl)
    lib = pk.Chess(config_of(sp, max_selected=sp.max_pages))
    summ, ws = lib.new_summaries(), lib.new_workspace()
    lib.summarize(d.k_pool, d.block_table, d.seq_lens, summ)
    ids = torch.full((4, 2, sp.max_pages), -7, dtype=torch.int32, device="cuda")
    nsel = torch.full((4, 2), -7, dtype=torch.int32, device="cuda")
    lib.select(d.q, summ, d.seq_lens, gpu_plan(plan_of(sp)), ids, nsel, ws)
    K, V, Q, bt, sl = host_arrays(wl)
    listed = oracle.attend(Q, K, V, bt, sl, geom_of(sp), ids.cpu().numpy(), nsel.cpu().numpy())
    every = oracle.attend(Q, K, V, bt, sl, geom_of(sp))
    for waves, splits in [(w, n) for w in (1, 4, 8) for n in (1, 2, 7, 8, 9, 10, 15, 16, 17, 24, 25, 33)] + [(4, 0)]:
        lib.debug_force_splits(splits, waves)                 # (0: every page is dealt by length)
        out, dense = (torch.full((4, sp.n_q_heads, 128), float("nan"), device="cuda") for _ in range(2))
        lib.sparse_decode(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, ids, nsel, out, ws)
        lib.dense_decode(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, dense, ws)
        torch.cuda.synchronize()
        assert np.abs(out.cpu().numpy() - listed).max() <= ATOL_64, (waves, splits)
        assert np.abs(dense.cpu().numpy() - every).max() <= ATOL_64, (waves, splits)
    lib.close()


@pytest.mark.parametrize("page,group", [(16, 1), (16, 4), (16, 16), (32, 4), (32, 7)])
def test_dealt_splits_of_long_sequences_against_64_bits(page, group):
    """Ragged lengths with one to some forty splits a sequence: every remainder of a merge that asks for eight at a time."""
    lens = [33000, 16000, 7000, 3000, 1200, 600, 130, 1]
    sp = workload.WorkloadSpec("dealt64", 8, (0, 33000), group, 1, page, ("fixed", 256), (1, 2), 1, 2, budget_pages=4)
    wl = workload.generate(sp, 7, seq_lens=lens)
    d = to_device(wl)
    K, V, Q, bt, sl = host_arrays(wl)
    want = oracle.attend(Q, K, V, bt, sl, geom_of(sp))
    lib = pk.Chess(config_of(sp))
    ws = lib.new_workspace()
    for n in (8, 5, 3, 2):                                    # fewer sequences: more splits for each
        out = torch.full((n, group, 128), float("nan"), device="cuda")
        lib.dense_decode(d.q[:n], d.k_pool, d.v_pool, d.block_table[:n], d.seq_lens[:n], out, ws)
        torch.cuda.synchronize()
        assert np.abs(out.cpu().numpy() - want[:n]).max() <= ATOL_64, n
    lib.close()
