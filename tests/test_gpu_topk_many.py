"""Top-k of many segments at once: a launch with more shares than the device
runs together grows them, so segments of one launch use one, several or all of
their parts. Whole-number scores make ties everywhere."""
import pytest
import torch

import paper_2606_26439_amd as M

pytestmark = pytest.mark.gpu

CASES = {
    "even number, two parts": ([2100] * 1100, 100),
    "odd number, two parts": ([2100] * 1101, 1000),
    "six, several hundred parts": ([400_000] * 6, 10),
    "two of which one is empty": ([0, 2_700_000], 10),
    "four of uneven size": ([3_000_000, 5, 0, 1], 7),
    "a long one among short ones": ([700] * 299 + [900_000], 100),
    "the long one first, k above the short ones": ([900_000] + [700] * 300, 1000),
    "edges of a share": ([24575, 24576, 24577, 49152, 1, 0, 4097, 2048] * 40, 33),
    "one part each": ([50, 0, 1, 2048] * 400, 100),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("with_ids", [False, True])
def test_many_segments(name, with_ids):
    lens, k = CASES[name]
    n = sum(lens)
    g = torch.Generator(device="cuda").manual_seed(n)
    scores = torch.randint(-3000, 3000, (n,), generator=g, device="cuda").float()
    off = torch.zeros(len(lens) + 1, dtype=torch.int64)
    torch.cumsum(torch.tensor(lens), 0, out=off[1:])
    ids = torch.randperm(n, generator=g, device="cuda").to(torch.int32) if with_ids else None
    ts, ti = M.topk(scores, off.cuda(), k, ids=ids)
    # (score descending, id ascending): segment, then score, then id
    seg = torch.repeat_interleave(torch.arange(len(lens)), torch.tensor(lens)).cuda()
    pos = torch.arange(n, device="cuda") - off.cuda()[seg]
    key = ids.long() if with_ids else pos
    order = torch.argsort((seg << 46) + ((3000 - scores.long()) << 32) + key)
    want_s = torch.full((len(lens), k), float("-inf"), device="cuda")
    want_i = torch.full((len(lens), k), -1, dtype=torch.int32, device="cuda")
    keep = pos < k  # places within the segment, now read as ranks
    want_s[seg[keep], pos[keep]] = scores[order][keep]
    want_i[seg[keep], pos[keep]] = key[order][keep].to(torch.int32)
    assert torch.equal(ts.view_as(want_s), want_s)
    assert torch.equal(ti.view_as(want_i), want_i)
