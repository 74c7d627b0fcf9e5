"""Attention over every page of ragged batches, where the workgroups of a head are dealt to the sequences by length:
lengths of 0 and 1, around a tile of 32 tokens, one long sequence among short ones, and batches around the 64 sequences
a wave deals at a time and around the size from which there are no workgroups to deal; lengths that change under a captured
launch; short sequences in a long context, which have nothing to split.  Reference: softmax attention in fp64."""
from __future__ import annotations

import math
import random

import pytest
import torch

import paper_2602_20732_amd as pk

pytestmark = pytest.mark.gpu

H, G, D = 2, 4, 128
ATOL = 5e-5      # weights are carried to 2^-17 and values stay below about 5: 4e-5, and fp32 sums


def lengths_of(shape, batch, most):
    r = random.Random(batch)
    if shape == "one_long":
        lens = [r.choice((0, 1, 31, 32, 33)) for _ in range(batch)]
        lens[r.randrange(batch)] = most
    elif shape == "equal":
        lens = [most] * batch
    elif shape == "empty":
        lens = [0] * batch
    else:
        lens = [r.randint(0, most) for _ in range(batch)]
    return lens


def pools(lens, page, max_pages, H, G, seed):
    """K and V pools, queries and the block table of sequences of these lengths, pages in random order."""
    gen = torch.Generator().manual_seed(seed)
    n_phys = max(1, sum(-(-n // page) for n in lens))
    order = torch.randperm(n_phys, generator=gen).to(torch.int32)
    table = torch.full((len(lens), max_pages), -1, dtype=torch.int32)
    at = 0
    for b, n in enumerate(lens):
        held = -(-n // page)
        table[b, :held] = order[at:at + held]
        at += held
    k = torch.randn((n_phys, H, page, D), generator=gen).to(torch.bfloat16)
    v = torch.randn((n_phys, H, D, page), generator=gen).to(torch.bfloat16)
    q = torch.randn((len(lens), H * G, D), generator=gen).to(torch.bfloat16)
    return q, k, v, table


def check(got, lens, q, k, v, table, H):
    page = k.shape[2]
    for b, n in enumerate(lens):
        if n == 0:
            assert (got[b] == 0).all()
            continue
        phys = table[b, :-(-n // page)].long()
        kb = k[phys].permute(1, 0, 2, 3).reshape(H, -1, D)[:, :n].double()
        vb = v[phys].permute(1, 0, 3, 2).reshape(H, -1, D)[:, :n].double()
        s = q[b].view(H, -1, D).double() @ kb.transpose(1, 2) / math.sqrt(D)
        ref = (torch.softmax(s, -1) @ vb).view(-1, D)
        assert (got[b].double() - ref).abs().max() <= ATOL, f"sequence {b} of {n} tokens"


@pytest.mark.parametrize("page", [16, 32])
@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65, 130])
@pytest.mark.parametrize("shape", ["one_long", "equal", "spread", "empty"])
def test_ragged_lengths(page, batch, shape):
    most = 4099 if batch <= 2 else 1100
    max_pages = -(-most // page)
    lens = lengths_of(shape, batch, most)
    q, k, v, table = pools(lens, page, max_pages, H, G, batch + page)
    lib = pk.Chess(pk.Config(H * G, H, page, batch, max_pages, 8))
    ws = lib.new_workspace()
    out = torch.full((batch, H * G, D), float("nan"), device="cuda")
    args = [x.cuda() for x in (q, k, v, table, torch.tensor(lens, dtype=torch.int32))]
    lib.dense_decode(*args, out, ws)
    first = out.cpu()
    lib.dense_decode(*args, out, ws)                       # the arrival counters are back at zero
    torch.cuda.synchronize()
    assert torch.equal(first, out.cpu())
    check(first, lens, q, k, v, table, H)
    lib.close()


@pytest.mark.parametrize("heads,group,batch", [(8, 4, 94), (8, 4, 95), (8, 4, 96), (8, 4, 97), (1, 1, 70), (1, 1, 300), (2, 16, 5), (2, 16, 100)])
def test_heads_groups_and_batches(heads, group, batch):
    """Eight heads leave 96 workgroups a head on 256 compute units: just enough to deal at 95, none at 97.  Sixteen query
    heads a group take more than 32 KB of LDS a workgroup."""
    lens = lengths_of("spread", batch, 700)
    q, k, v, table = pools(lens, 16, 64, heads, group, batch)
    lib = pk.Chess(pk.Config(heads * group, heads, 16, batch, 64, 8))
    ws, out = lib.new_workspace(), torch.full((batch, heads * group, D), float("nan"), device="cuda")
    lib.dense_decode(q.cuda(), k.cuda(), v.cuda(), table.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda"), out, ws)
    check(out.cpu(), lens, q, k, v, table, heads)
    lib.close()


@pytest.mark.parametrize("batch", [6, 80])
def test_captured_launch_follows_the_lengths(batch):
    most = 2000
    q, k, v, table = pools([most] * batch, 16, 125, H, G, 3)
    dev = [x.cuda() for x in (q, k, v, table)]
    lens = torch.full((batch,), most, dtype=torch.int32, device="cuda")
    lib = pk.Chess(pk.Config(H * G, H, 16, batch, 125, 8))
    ws, out, eager_out = lib.new_workspace(), torch.empty((batch, H * G, D), device="cuda"), torch.empty((batch, H * G, D), device="cuda")
    lib.dense_decode(*dev, lens, out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lib.dense_decode(*dev, lens, out, ws)
    r = random.Random(batch)
    swapped = [most if b % 3 == 0 else b % 2 for b in range(batch)]
    for now in ([most] * batch, swapped, swapped[::-1], [r.randint(0, most) for _ in range(batch)], [0] * batch, [31] * batch):
        lens.copy_(torch.tensor(now, dtype=torch.int32))
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        check(out.cpu(), now, q, k, v, table, H)
        lib.dense_decode(*dev, lens, eager_out, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, eager_out)
    lib.close()


@pytest.mark.parametrize("batch", [5, 150])
def test_short_sequences_in_a_long_context_are_not_split(batch):
    """Up to four tiles (128 tokens) are one workgroup's work however long a context the configuration allows: nothing is
    published to the workspace, whose partial rows stand at its start, and nothing is merged from it."""
    for lens in ([128] * batch, [1 + (37 * b) % 128 for b in range(batch)]):
        q, k, v, table = pools(lens, 16, 4096, 1, G, batch)
        lib = pk.Chess(pk.Config(G, 1, 16, batch, 4096, 8))
        ws, out = lib.new_workspace(), torch.empty((batch, G, D), device="cuda")
        rows = ws[:batch * G * D * 4]
        rows.fill_(0x5A)
        lib.dense_decode(q.cuda(), k.cuda(), v.cuda(), table.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda"), out, ws)
        check(out.cpu(), lens, q, k, v, table, 1)
        assert (rows == 0x5A).all()
        lib.close()
