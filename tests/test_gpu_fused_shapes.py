"""The shapes and query groups the fused scorer picks by itself: one query,
several in one unit, several units and candidate lists take different launch
shapes of the same arithmetic, so their scores are the same bits."""
import json

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


@pytest.mark.parametrize("dtype,dim,tokens", [
    ("f16", 640, 16), ("bf16", 640, 9), ("fp8", 640, 32), ("f32", 320, 16), ("f16", 1008, 64),
    ("f16", 256, 64), ("fp8", 1024, 64)])
def test_top_k_fits_beside_the_query_blocks(dtype, dim, tokens):
    # wave-private query blocks that fill the LDS to the last byte leave the
    # top-k epilogue its part
    g = W.rng(dim + tokens)
    d_off = W.offsets_from_lengths(g.integers(1, 30, size=300))
    d = W.unit_tokens(int(d_off[-1]), dim, g)
    q = W.unit_tokens(tokens, dim, g)
    Q, D = device_tokens(q, [0, tokens], dtype), device_tokens(d, d_off, dtype)
    off = dev(np.array([0, 300], np.int64))
    ids = dev(np.arange(300, dtype=np.int32))
    want = M.topk(M.score(Q, D), off, 20)
    for cand in (None, M.Candidates(off, ids)):
        got = M.score_topk(Q, D, 20, cand)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("dtype,code,dim,tokens", [("f16", 2, 336, 64), ("bf16", 1, 720, 50)])
def test_a_saved_shape_of_narrower_chunks_still_runs(dtype, code, dim, tokens, tmp_path):
    g = W.rng(dim)
    d_off = W.offsets_from_lengths(g.integers(0, 40, size=200))
    d = W.unit_tokens(int(d_off[-1]), dim, g)
    q = W.unit_tokens(tokens, dim, g)
    Q, D = device_tokens(q, [0, tokens], dtype), device_tokens(d, d_off, dtype)
    want = M.score(Q, D)
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({"version": 1, "entries": [
        {"dtype": code, "dim": dim, "nqb": 4, "pf": 4, "nw": 8, "wg_per_cu": 0, "stage": 1}]}))
    M.load_tune_cache(str(path))
    assert torch.equal(M.score(Q, D), want)
    ts, ti = M.score_topk(Q, D, 10)
    rs, ri = M.topk(want, dev(np.array([0, 200], np.int64)), 10)
    assert torch.equal(ts, rs) and torch.equal(ti, ri)


def test_fixed_scratch_takes_what_one_workgroup_per_cu_fits():
    # 15.8M pairs and the largest k: the keys' spill array alone nearly fills
    # the 64 MiB, so the launch has to leave few top-k parts
    g = W.rng(3)
    n_docs, n_q, each = 2000, 8, 1_975_000
    d_off = W.offsets_from_lengths([2] * n_docs)
    Q = device_tokens(W.unit_tokens(32 * n_q, 128, g), W.offsets_from_lengths([32] * n_q), "f16")
    D = device_tokens(W.unit_tokens(2 * n_docs, 128, g), d_off, "f16")
    ids = torch.arange(n_q * each, dtype=torch.int32, device="cuda") % n_docs
    cand = M.Candidates(dev(W.offsets_from_lengths([each] * n_q)), ids)
    ts, ti = M.score_topk_noalloc(Q, D, 1024, cand)
    rs, ri = M.score_topk(Q, D, 1024, cand)
    assert torch.equal(ts, rs) and torch.equal(ti, ri)
