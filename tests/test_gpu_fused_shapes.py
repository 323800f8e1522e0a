"""The shapes and query groups the fused scorer picks by itself: one query,
several in one unit, several units and candidate lists take different launch
shapes of the same arithmetic, so their scores are the same bits."""
import numpy as np
import pytest
import torch

import paper_2606_26439_amd as M
import workloads as W
from tests._gpu import dev, device_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16", "fp8"])
@pytest.mark.parametrize("dim,tokens,n_q", [
    (64, 64, 1), (64, 32, 2), (96, 43, 3), (128, 16, 2), (128, 20, 5), (144, 32, 2), (256, 10, 4),
    (256, 64, 2), (400, 32, 3), (512, 32, 4), (640, 32, 3), (768, 32, 2), (768, 17, 5),
    (768, 64, 1), (1024, 32, 2), (1024, 16, 7)])
def test_groups_units_and_candidates_agree(dtype, dim, tokens, n_q):
    if dtype == "f32" and dim > 512 and tokens > 32:
        pytest.skip("64 FP32 query tokens exceed the LDS")
    g = W.rng(dim + tokens)
    n_docs = 701
    d_off = W.offsets_from_lengths(g.integers(0, 40, size=n_docs))
    d = W.unit_tokens(int(d_off[-1]), dim, g)
    q_off = W.offsets_from_lengths([tokens] * n_q)
    q = W.unit_tokens(tokens * n_q, dim, g)
    Q, D = device_tokens(q, q_off, dtype), device_tokens(d, d_off, dtype)
    got = M.score(Q, D)
    ids = np.concatenate([g.permutation(n_docs) for _ in range(n_q)]).astype(np.int32)
    cand = M.Candidates(dev(W.offsets_from_lengths([n_docs] * n_q)), dev(ids))
    listed = M.score(Q, D, cand)
    for a in range(n_q):
        one = device_tokens(q[tokens * a:tokens * (a + 1)], [0, tokens], dtype)
        alone = M.score(one, D)
        sl = slice(a * n_docs, (a + 1) * n_docs)
        assert torch.equal(got[sl], alone), a
        assert torch.equal(listed[sl], alone[dev(ids[sl]).long()]), a
    ts, ti = M.score_topk(Q, D, 50)
    rs, ri = M.topk(got, dev(W.offsets_from_lengths([n_docs] * n_q)), 50)
    assert torch.equal(ts, rs) and torch.equal(ti, ri)
