"""Top-k at the edges of its split into workgroups: segments of no, one and
many shares, shares that fit LDS and that do not, k from 1 to the largest,
ties, NaN and infinities, and merges whose answer sits in one part. Every
result must equal a sort of the same values on the CPU."""
import numpy as np
import pytest
import torch

import paper_2606_26439_amd as M
import workloads as W
from tests._gpu import dev, device_tokens

pytestmark = pytest.mark.gpu


def _order(scores, ids):
    """Positions by score descending (NaN last), then id ascending."""
    s = np.where(np.isnan(scores), -np.inf, scores).astype(np.float64)
    return np.lexsort((ids, -s, np.isnan(scores)))


def _check(top_s, top_i, scores, off, k, ids=None):
    top_s, top_i = top_s.cpu().numpy(), top_i.cpu().numpy()
    for a in range(len(off) - 1):
        sc = scores[off[a]:off[a + 1]]
        seg = np.arange(len(sc)) if ids is None else ids[off[a]:off[a + 1]]
        o = _order(sc, seg)[:k]
        n = len(o)
        assert np.array_equal(top_i[a, :n], seg[o]), a
        assert np.array_equal(top_s[a, :n], sc[o], equal_nan=True), a
        assert np.all(top_i[a, n:] == -1) and np.all(np.isneginf(top_s[a, n:])), a


@pytest.mark.parametrize("k", [1, 3, 10, 100, 1000, 1024])
@pytest.mark.parametrize("lens", [[1], [64, 0, 1, 65, 5], [6144], [6145, 12_287, 3], [150_000],
                                  [2047, 2048, 2049, 94_000, 7], [230_000], [2_300_000]])
def test_topk_segments(lens, k):
    off = W.offsets_from_lengths(lens)
    sc = W.random_scores(int(off[-1]), seed=k + len(lens))
    ts, ti = M.topk(dev(sc), dev(off), k)
    _check(ts, ti, sc, off, k)


@pytest.mark.parametrize("k", [10, 100, 1000])
@pytest.mark.parametrize("n_distinct", [1, 7, 3000])
def test_topk_ties_ids_and_special_values(n_distinct, k):
    off = W.offsets_from_lengths([30_000, 400, 9000])
    n = int(off[-1])
    g = W.rng(k)
    sc = W.random_scores(n, seed=n_distinct, n_distinct=n_distinct)
    sc[g.integers(0, n, 500)] = np.nan
    sc[g.integers(0, n, 500)] = -np.inf
    sc[g.integers(0, n, 5)] = np.inf
    sc[30_000:30_390] = np.nan  # a segment with more NaN than numbers
    ids = np.concatenate([g.permutation(2_000_000)[:m] for m in (30_000, 400, 9000)]).astype(np.int32)
    ts, ti = M.topk(dev(sc), dev(off), k, ids=dev(ids))
    _check(ts, ti, sc, off, k, ids)


@pytest.mark.parametrize("where", ["spread", "one part", "ascending"])
@pytest.mark.parametrize("k", [4, 100, 1000])
def test_topk_answer_in_one_part(where, k):
    n = 120_000
    sc = np.sort(W.random_scores(n, seed=3))
    if where == "spread":
        sc = W.rng(1).permutation(sc)
    elif where == "one part":
        sc[:n - 2000] = W.rng(2).permutation(sc[:n - 2000])
    ts, ti = M.topk(dev(sc), dev(np.array([0, n], np.int64)), k)
    _check(ts, ti, sc, [0, n], k)


@pytest.mark.parametrize("dtype,dim", [("f16", 128), ("f16", 64), ("fp8", 128), ("f32", 128)])
@pytest.mark.parametrize("k", [10, 100, 1000])
def test_score_topk_of_candidate_lists(dtype, dim, k):
    # lists shorter and longer than k, an empty one, repeated ids; queries of
    # one to four blocks
    g = W.rng(dim + k)
    lens = g.integers(0, 30, size=3000)
    d_off = W.offsets_from_lengths(lens)
    d = W.unit_tokens(int(d_off[-1]), dim, g)
    nq = [32, 64, 7, 17, 40]
    q_off = W.offsets_from_lengths(nq)
    q = W.unit_tokens(int(q_off[-1]), dim, g)
    sizes = [2500, 0, 3, 1, 900]
    c_off = W.offsets_from_lengths(sizes)
    ids = np.concatenate([g.permutation(3000)[:m] for m in sizes]).astype(np.int32)
    ids[2500:2503] = [5, 5, 5]
    Q, D = device_tokens(q, q_off, dtype), device_tokens(d, d_off, dtype)
    cand = M.Candidates(dev(c_off), dev(ids))
    sc = M.score(Q, D, cand).cpu().numpy()
    ts, ti = M.score_topk(Q, D, k, cand)
    _check(ts, ti, sc, c_off, k, ids)


@pytest.mark.parametrize("n_q", [8, 14, 16, 24])
@pytest.mark.parametrize("k", [0, 10, 1000])
def test_units_interleaved_over_workgroups(n_q, k):
    # several units of four 32-token queries over one document range: each
    # query's scores and ranking equal its own call's
    g = W.rng(n_q)
    lens = g.integers(0, 12, size=6001)
    d_off = W.offsets_from_lengths(lens)
    d = W.unit_tokens(int(d_off[-1]), 128, g)
    q_off = W.offsets_from_lengths([32] * n_q)
    q = W.unit_tokens(32 * n_q, 128, g)
    Q, D = device_tokens(q, q_off, "f16"), device_tokens(d, d_off, "f16")
    one = [device_tokens(q[32 * a:32 * a + 32], [0, 32], "f16") for a in range(n_q)]
    if k == 0:
        got = M.score(Q, D)
        for a in range(n_q):
            assert torch.equal(got[a * 6001:(a + 1) * 6001], M.score(one[a], D)), a
        return
    ts, ti = M.score_topk(Q, D, k)
    for a in range(n_q):
        sc = M.score(one[a], D).cpu().numpy()
        _check(ts[a:a + 1], ti[a:a + 1], sc, [0, 6001], k)
