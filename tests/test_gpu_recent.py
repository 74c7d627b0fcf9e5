"""The refresh of the last pages (summarize_recent, summarize_tail) against a pass over every page, bit for bit: hierarchies from 1 x 1 to
16 x 16 and beyond what one workgroup takes, one to sixteen recent pages and one more, lengths around the edges of pages, chunks and
grids, shorter than the recent pages, and empty; what does not change stays untouched."""
import pytest
import torch

import paper_2602_20732_amd as pk

pytestmark = pytest.mark.gpu
H, D = 3, 128


@pytest.mark.parametrize("fan_c,fan_g", [(1, 1), (2, 3), (8, 8), (8, 4), (16, 16), (5, 1), (17, 4), (4, 20)])
@pytest.mark.parametrize("page", [16, 32])
def test_recent_pages_equal_a_full_pass(fan_c, fan_g, page):
    ppg = fan_c * fan_g
    pages = sorted({1, 2, fan_c, fan_c + 1, ppg, ppg + 1, ppg + 7, 3 * ppg, 2 * ppg + fan_c - 1, 40})
    lens = [0] + [p * page - off for p in pages for off in (0, 1, page - 1)]
    most = max(pages) + 2
    g = torch.Generator().manual_seed(fan_c * 100 + fan_g * 10 + page)
    held = [-(-n // page) for n in lens]
    order = torch.randperm(sum(held), generator=g)
    table = torch.full((len(lens), most), -1, dtype=torch.int32)
    at = 0
    for b, n in enumerate(held):
        table[b, :n] = order[at:at + n]
        at += n
    k = torch.randn((sum(held), H, page, D), generator=g).to(torch.bfloat16).cuda()
    table, lens_d = table.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
    for dtype in (pk.SUMMARY_F32, pk.SUMMARY_BF16):
        lib = pk.Chess(pk.Config(H, H, page, len(lens), most, 8, fan_c, fan_g, summary_dtype=dtype))
        want = lib.new_summaries()
        lib.summarize(k, table, lens_d, want)
        for recent in (1, 2, 10, 15, 16, 17):
            got = want.clone()
            for b, n in enumerate(held):                          # what has to be renewed is made to differ
                fp = max(n - recent, 0)
                if n > 0:
                    for v, first, last in zip(lib.summary_views(got), (fp, fp // fan_c, fp // ppg), (n - 1, (n - 1) // fan_c, (n - 1) // ppg)):
                        v[b, :, first:last + 1] = 7.0
            lib.summarize_recent(k, table, lens_d, recent, got)
            torch.cuda.synchronize()
            assert torch.equal(got, want), (dtype, recent)
        lib.close()
