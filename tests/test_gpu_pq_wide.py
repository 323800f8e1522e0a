"""PQ codebooks that nearly fill the LDS (M = 16, dsub = 32): up to K = 148 or
150 the decode scorer keeps its rings beside them, from there to K = 160 (all
160 KB) codes and scores stay in registers. Integer codebooks and queries make
every sum exact."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2606_26439_amd as M
import workloads as W
from paper_2606_26439_amd import _binding as B
from tests._gpu import dev
from tests.test_gpu_parity import _pq_case, _pq_device


@pytest.mark.parametrize("K", [148, 150, 151, 157, 158, 160])
@pytest.mark.parametrize("max_len,cand", [(10, False), (32, False), (32, True)])
def test_no_workspace_is_needed(K, max_len, cand):
    # (the table kernel, which larger codebooks take, has one of partial scores)
    q = B.CSR(2, 512, 3, 60, max_len, 0, 16, 16, None)
    d = B.PQ(16, K, 32, 2, 16, 16, 16, 1000, 50_000)
    c = ctypes.byref(B.Cand(16, 16, 500)) if cand else None
    need = M.lib().maxsim_pq_score_workspace_size
    assert need(ctypes.byref(q), ctypes.byref(d), c) == 0
    if max_len > 16:
        d.K = 161
        assert need(ctypes.byref(q), ctypes.byref(d), c) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("K", [148, 149, 151, 157, 158, 160])
@pytest.mark.parametrize("nq_lens", [[32, 8, 31, 1, 17, 16], [16, 3, 0, 9], [5], [30]])
def test_scores(K, nq_lens):
    q, q_off, cb, codes, d_off = _pq_case(700, 16, K, 32, seed=K + sum(nq_lens), nq_lens=nq_lens,
                                          integer=True)
    Q, D = _pq_device(q, q_off, cb, codes, d_off)
    q64, cb64 = q.astype(np.float64), cb.astype(np.float64)
    got = M.pq_score(Q, D).cpu().numpy().astype(np.float64)
    assert np.array_equal(got, oracle.pq_decode_score(q64, q_off, codes, cb64, d_off))
    g = W.rng(K)
    off = W.offsets_from_lengths([900, 0, 3, 1, 65, 130][:len(nq_lens)])
    ids = g.integers(0, 700, size=int(off[-1])).astype(np.int32)
    got = M.pq_score(Q, D, M.Candidates(dev(off), dev(ids))).cpu().numpy().astype(np.float64)
    assert np.array_equal(got, oracle.pq_decode_score(q64, q_off, codes, cb64, d_off, off, ids))
