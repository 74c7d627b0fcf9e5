"""Attention over a page list with eight waves to a workgroup, the shape forced: the reuse step against appending and
attending in two calls, bit for bit, while tokens open pages, a row of the list runs full, a sequence starts empty and one
is full; and both against the oracle.  List room of at most and of more than four tiles a wave (the reuse step's two
kernels), groups of 1, 7 and 16 query heads (sixteen need more than 64 KB of LDS)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2602_20732_amd as pk
import workload
from gpu_common import config_of, gpu_plan, to_device
from helpers import geom_of, plan_of

pytestmark = pytest.mark.gpu

SINK, WINDOW = 1, 2
ATOL = 5e-5      # weights are carried to 2^-17 and values stay below about 5: 4e-5, and fp32 sums


@pytest.mark.parametrize("page,tiles,splits", [(16, 8, 1), (16, 40, 1), (16, 40, 2), (32, 8, 1), (32, 40, 1)])
@pytest.mark.parametrize("group", [1, 7, 16])
def test_eight_waves(page, tiles, splits, group):
    room = tiles * 32 // page                                # list entries; the selection leaves one of them free
    k = room - SINK - WINDOW - 1
    cap = (room + 8) * page                                  # tokens a sequence can hold
    sp = workload.WorkloadSpec("waves8", 4, (0, cap), 2 * group, 2, page, ("fixed", 128), (2, 2), SINK, WINDOW,
                               budget_pages=k, pages_per_chunk=4, chunks_per_grid=4)
    steps = 2 * page + 2                                     # the second page the first sequence opens finds its row full
    start = [cap - 3 * page + 3, (room + 2) * page, 0, cap]
    lens_full = [min(n + steps, cap) for n in start]
    full = to_device(workload.generate(sp, 90 + group, seq_lens=lens_full))
    lib = pk.Chess(config_of(sp, max_selected=room))
    lib.debug_force_splits(splits, 8)
    lens = torch.tensor(start, dtype=torch.int32, device="cuda")
    summ, ws = lib.new_summaries(), lib.new_workspace()
    lib.summarize(full.k_pool, full.block_table, lens, summ)
    ids = torch.full((4, 2, room), -7, dtype=torch.int32, device="cuda")
    nsel = torch.full((4, 2), -7, dtype=torch.int32, device="cuda")
    lib.select(full.q, summ, lens, gpu_plan(plan_of(sp)), ids, nsel, ws)
    torch.cuda.synchronize()
    assert nsel[0].tolist() == [room - 1, room - 1]
    bt = full.block_table

    def state():
        st = dict(k=full.k_pool.clone(), v=full.v_pool.clone(), ids=ids.clone(), nsel=nsel.clone(), lens=lens.clone(),
                  out=torch.full((4, sp.n_q_heads, 128), float("nan"), device="cuda"))
        for b, n in enumerate(start):                        # nothing behind the current lengths is valid yet
            for j in range(n // page, -(-lens_full[b] // page)):
                phys, t0 = int(bt[b, j]), max(n - j * page, 0)
                st["k"][phys, :, t0:, :] = float("nan")
                st["v"][phys, :, :, t0:] = float("nan")
        return st

    A, B = state(), state()
    gen = torch.Generator(device="cuda").manual_seed(group)
    for step in range(steps):
        rk = torch.randn((4, 2, 128), device="cuda", generator=gen).to(torch.bfloat16)
        rv = torch.randn((4, 2, 128), device="cuda", generator=gen).to(torch.bfloat16)
        lib.append_kv(rk, rv, A["k"], A["v"], bt, A["lens"], A["ids"], A["nsel"])
        A["lens"] = torch.clamp(A["lens"] + 1, max=cap)
        lib.sparse_decode(full.q, A["k"], A["v"], bt, A["lens"], A["ids"], A["nsel"], A["out"], ws)
        lib.reuse_step(full.q, rk, rv, B["k"], B["v"], bt, B["lens"], B["ids"], B["nsel"], B["out"], ws)
        B["lens"] = torch.clamp(B["lens"] + 1, max=cap)
        torch.cuda.synchronize()
        assert torch.equal(A["nsel"], B["nsel"]), step
        live = torch.arange(room, device="cuda").view(1, 1, -1) < A["nsel"].unsqueeze(-1)
        assert torch.equal(torch.where(live, A["ids"], -1), torch.where(live, B["ids"], -1)), step
        assert torch.equal(A["out"], B["out"]), (step, (A["out"] - B["out"]).abs().max())
        if step in (0, steps - 1):
            K, V, Q = workload.bf16_bits(B["k"].cpu()), workload.bf16_bits(B["v"].cpu()), workload.bf16_bits(full.q.cpu())
            ref = oracle.attend(Q, K, V, bt.cpu().numpy(), B["lens"].cpu().numpy(), geom_of(sp), B["ids"].cpu().numpy(),
                                B["nsel"].cpu().numpy())
            assert np.abs(B["out"].cpu().numpy() - ref).max() <= ATOL, step
    assert int(B["nsel"][0, 0]) == room, "the row is full"
    # the split shape changes the order of additions, nothing else
    lib.debug_force_splits(splits, 4)
    four = torch.full_like(B["out"], float("nan"))
    lib.sparse_decode(full.q, B["k"], B["v"], bt, B["lens"], B["ids"], B["nsel"], four, ws)
    # every-page attention has no eight-wave kernel: a forced eight means four
    dense = [torch.full_like(four, float("nan")) for _ in range(2)]
    for waves, out in zip((8, 4), dense):
        lib.debug_force_splits(splits, waves)
        lib.dense_decode(full.q, B["k"], B["v"], bt, B["lens"], out, ws)
    torch.cuda.synchronize()
    assert (four - B["out"]).abs().max() <= ATOL
    assert torch.equal(dense[0], dense[1])
    lib.close()


def test_captured_launch_of_sixteen_heads():
    """Eight waves of sixteen query heads ask for more than 64 KB of LDS, by an attribute of the kernel that is set at each
    launch: also while a graph is being recorded.  Replays against the eager call, the lists changed in between."""
    group, page, room = 16, 16, 40
    sp = workload.WorkloadSpec("captured8", 2, (60 * page, 60 * page), 2 * group, 2, page, ("fixed", 128), (2, 2), SINK, WINDOW,
                               budget_pages=room - SINK - WINDOW, pages_per_chunk=4, chunks_per_grid=4)
    d = to_device(workload.generate(sp, 17))
    lib = pk.Chess(config_of(sp, max_selected=room))
    lib.debug_force_splits(2, 8)
    ws = lib.new_workspace()
    gen = torch.Generator().manual_seed(5)
    ids = torch.stack([torch.randperm(60, generator=gen)[:room].sort().values for _ in range(4)]).view(2, 2, room).to(torch.int32).cuda()
    nsel = torch.full((2, 2), room, dtype=torch.int32, device="cuda")
    out, want = (torch.empty((2, sp.n_q_heads, 128), device="cuda") for _ in range(2))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lib.sparse_decode(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, ids, nsel, out, ws)
    for n in (room, 33, 1, 0, room):
        nsel.fill_(n)
        out.fill_(float("nan"))
        graph.replay()
        lib.sparse_decode(d.q, d.k_pool, d.v_pool, d.block_table, d.seq_lens, ids, nsel, want, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, want), n
    lib.close()
