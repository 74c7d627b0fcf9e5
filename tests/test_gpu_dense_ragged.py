"""Attention over every page of ragged batches, where the workgroups of a head are dealt to the sequences by length:
lengths of 0 and 1, around a tile of 32 tokens, one long sequence among short ones, and batches around the 64 sequences
a wave deals at a time.  Reference: softmax attention in fp64.  Tolerance: the weights are carried to 2^-17 and sums in
fp32, so outputs of unit-variance values differ by about 1e-5; 2e-4 is what the other attention tests allow."""
from __future__ import annotations

import math
import random

import pytest
import torch

import paper_2602_20732_amd as pk

pytestmark = pytest.mark.gpu

H, G, D = 2, 4, 128


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


@pytest.mark.parametrize("page", [16, 32])
@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65, 130])
@pytest.mark.parametrize("shape", ["one_long", "equal", "spread", "empty"])
def test_ragged_lengths(page, batch, shape):
    most = 4099 if batch <= 2 else 1100
    max_pages = -(-most // page)
    lens = lengths_of(shape, batch, most)
    gen = torch.Generator().manual_seed(batch + page)
    n_phys = max(1, sum(-(-n // page) for n in lens))
    order = torch.randperm(n_phys, generator=gen).to(torch.int32)
    table = torch.full((batch, max_pages), -1, dtype=torch.int32)
    at = 0
    for b, n in enumerate(lens):
        held = -(-n // page)
        table[b, :held] = order[at:at + held]
        at += held
    k = torch.randn((n_phys, H, page, D), generator=gen).to(torch.bfloat16)
    v = torch.randn((n_phys, H, D, page), generator=gen).to(torch.bfloat16)
    q = torch.randn((batch, H * G, D), generator=gen).to(torch.bfloat16)
    lib = pk.Chess(pk.Config(H * G, H, page, batch, max_pages, 8))
    ws = lib.new_workspace()
    out = torch.full((batch, H * G, D), float("nan"), device="cuda")
    args = [x.cuda() for x in (q, k, v, table, torch.tensor(lens, dtype=torch.int32))]
    lib.dense_decode(*args, out, ws)
    first = out.cpu()
    lib.dense_decode(*args, out, ws)                       # the arrival counters are back at zero
    torch.cuda.synchronize()
    assert torch.equal(first, out.cpu())
    for b, n in enumerate(lens):
        if n == 0:
            assert (first[b] == 0).all()
            continue
        phys = table[b, :-(-n // page)].long()
        kb = k[phys].permute(1, 0, 2, 3).reshape(H, -1, D)[:, :n].double()
        vb = v[phys].permute(1, 0, 3, 2).reshape(H, -1, D)[:, :n].double()
        s = q[b].view(H, G, D).double() @ kb.transpose(1, 2) / math.sqrt(D)
        ref = (torch.softmax(s, -1) @ vb).view(H * G, D)
        assert (first[b].double() - ref).abs().max() <= 2e-4, f"sequence {b} of {n} tokens"
