"""The entropy of rows that end inside, at and just past a 16-byte chunk and a split, with infinite logits among them, against fp64."""
from __future__ import annotations

import pytest
import torch

import paper_2602_20732_amd as pk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 3, 17])
@pytest.mark.parametrize("vocab", [1, 7, 8, 9, 4095, 8191, 8192, 8193, 8200, 32769, 151937])
def test_entropy_at_the_edges(vocab, batch):
    g = torch.Generator().manual_seed(vocab + batch)
    wide = (vocab + 7) // 8 * 8 + 8
    z = (3 * torch.randn((batch, wide), generator=g)).to(torch.bfloat16)
    z[:, vocab:] = float("inf")                                # beyond the vocabulary: never part of the sum
    if batch > 1 and vocab > 1:
        z[1, vocab // 2] = float("-inf")
        z[2, : vocab - 1] = float("-inf")                      # all the probability on the last entry
    lib = pk.Chess(pk.Config(1, 1, 16, batch, 8, 8))
    ws, got = lib.new_workspace(), torch.full((batch,), -1.0, device="cuda")
    d = z.cuda()
    for _ in range(2):                                         # the counters are armed again
        lib.entropy(d, got, ws, vocab=vocab)
    p = torch.softmax(z[:, :vocab].double(), -1)
    want = -torch.where(p > 0, p * torch.log(p), p).sum(-1)
    out = got.cpu().double()
    # fp32 sums of up to 151937 terms in trees of at most 32 + 64 + 4 + 32 steps, and a logarithm below 12
    assert float((out - want).abs().max()) < 2e-5
    lib.close()


@pytest.mark.parametrize("vocab", [1, 7, 8192, 8193, 32769])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_rows_without_an_entropy(vocab, bad):
    """A row whose first logit is infinite or a NaN has entropy 0, as does one of nothing but -inf; its neighbours are as they are."""
    z = torch.randn((4, (vocab + 7) // 8 * 8), generator=torch.Generator().manual_seed(vocab)).to(torch.bfloat16)
    lib = pk.Chess(pk.Config(1, 1, 16, 4, 8, 8))
    ws, want, got = lib.new_workspace(), torch.empty(4, device="cuda"), torch.full((4,), -1.0, device="cuda")
    lib.entropy(z.cuda(), want, ws, vocab=vocab)
    z[1, 0] = bad
    z[3] = float("-inf")
    lib.entropy(z.cuda(), got, ws, vocab=vocab)
    assert got[1].item() == 0.0 and got[3].item() == 0.0
    assert torch.equal(got[::2], want[::2])
    lib.close()
