"""The decode-into-MFMA PQ scorer's split of a launch over wavefronts: equal
shares of a batch's candidates whatever its lists' sizes, each query with its
own number of 16-token blocks, scores kept 64 documents at a time, codes
arriving four tiles ahead. Integer codebooks and queries make every sum exact,
so a misplaced code, document or score changes the result."""
import numpy as np
import pytest

import oracle
import paper_2606_26439_amd as M
import workloads as W
from tests._gpu import dev
from tests.test_gpu_parity import _pq_case, _pq_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 256, 16), (16, 256, 8), (4, 64, 32), (8, 100, 8),
                                   (16, 150, 32)])
@pytest.mark.parametrize("nq_lens", [[64, 1, 17, 33, 48, 16, 0], [32, 8, 31], [16, 3]])
def test_uneven_candidate_lists_and_query_lengths(shape, nq_lens):
    M_, K, dsub = shape
    if M_ * dsub == 512:  # two blocks of query operand at most (two waves share the codebooks)
        nq_lens = [min(n, 32) for n in nq_lens]
    q, q_off, cb, codes, d_off = _pq_case(400, M_, K, dsub, seed=K + sum(nq_lens), nq_lens=nq_lens,
                                          integer=True)
    g = W.rng(5)
    sizes = [700, 0, 3, 1, 65, 130, 64][:len(nq_lens)]
    off = W.offsets_from_lengths(sizes)
    ids = g.integers(0, 400, size=int(off[-1])).astype(np.int32)  # repeated ids
    ids[:3] = [0, 1, 0]  # document 0 has no tokens
    Q, D = _pq_device(q, q_off, cb, codes, d_off)
    got = M.pq_score(Q, D, M.Candidates(dev(off), dev(ids))).cpu().numpy().astype(np.float64)
    want = oracle.pq_decode_score(q.astype(np.float64), q_off, codes, cb.astype(np.float64), d_off,
                                  off, ids)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("n_q,lo,hi", [(1, 10, 10), (3, 1, 16), (45, 1, 16), (7, 20, 32)])
def test_many_short_documents_per_wave(n_q, lo, hi):
    # 0 to 3 tokens a document: a wave scores and writes several rows of 64
    g = W.rng(n_q)
    nq_lens = g.integers(lo, hi + 1, size=n_q)
    n_docs = 400_000 // n_q if n_q > 4 else 60_000
    d_off = W.offsets_from_lengths(g.integers(0, 4, size=n_docs))
    codes = g.integers(0, 256, size=(int(d_off[-1]), 8), dtype=np.uint8)
    cb = g.integers(-4, 5, size=(8, 256, 16)).astype(np.float16)
    q_off = W.offsets_from_lengths(nq_lens)
    q = g.integers(-3, 4, size=(int(q_off[-1]), 128)).astype(np.float16)
    Q, D = _pq_device(q, q_off, cb, codes, d_off)
    got = M.pq_score(Q, D).cpu().numpy().astype(np.float64)
    want = oracle.pq_decode_score(q.astype(np.float64), q_off, codes, cb.astype(np.float64), d_off)
    assert np.array_equal(got, want)
