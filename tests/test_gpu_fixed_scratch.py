"""What the fixed scratch of score_topk_noalloc takes: a problem that fits it
with one query per document read is not refused because larger groups of
queries would leave more top-k parts."""
import pytest
import torch

import paper_2606_26439_amd as M
import workloads as W
from tests._gpu import dev, device_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tokens,n_q,n_docs", [
    ("f16", 17, 4096, 1800), ("bf16", 17, 4100, 1800), ("f16", 9, 3700, 2000)])
def test_wide_queries_near_the_limit(dtype, tokens, n_q, n_docs):
    # parts for 1,024 results of every query and the spill array: 61 to 62 of
    # the 64 MiB with a query (of 9 tokens: two) for each document read, 64.1 to
    # 65.1 with twice as many
    g = W.rng(n_q)
    Q = device_tokens(W.unit_tokens(tokens * n_q, 768, g), W.offsets_from_lengths([tokens] * n_q), dtype)
    D = device_tokens(W.unit_tokens(2 * n_docs, 768, g), W.offsets_from_lengths([2] * n_docs), dtype)
    ts, ti = M.score_topk_noalloc(Q, D, 1024)
    rs, ri = M.topk(M.score(Q, D), dev(W.offsets_from_lengths([n_docs] * n_q)), 1024)
    assert torch.equal(ts, rs) and torch.equal(ti, ri)
