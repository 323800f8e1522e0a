"""Host limits of the PQ decode and residual scorers' plans: a launch shares its
positions equally over the device, so what a wave counts in 32 bits is its own
share, whatever one query's list or the number of queries."""
import ctypes

import pytest

import paper_2606_26439_amd as M
from paper_2606_26439_amd import _binding as B


@pytest.mark.parametrize("n_q,n_total,fits", [
    (1, 1 << 31, True), (2048, 1 << 30, True), (2048, 1 << 31, True), (2048, 1 << 40, True),
    (2048, 1 << 43, False), (1, 1 << 43, False)])
def test_residual_candidates(n_q, n_total, fits):
    q = B.CSR(2, 64, n_q, 16 * n_q, 16, 0, 16, 16, None)
    d = B.Residual(64, 2, 100, 16, 16, 16, 16, 16, 1000, 50_000)
    c = B.Cand(16, 16, n_total)
    need = M.lib().maxsim_residual_score_workspace_size
    assert (need(ctypes.byref(q), ctypes.byref(d), ctypes.byref(c)) > 0) == fits


@pytest.mark.parametrize("n_q,n_docs,decode", [(64, 1 << 31, True), (1 << 20, 1 << 22, True),
                                               (1 << 20, 1 << 26, False)])
def test_pq_decode(n_q, n_docs, decode):
    # (the table kernel needs a workspace at this query length)
    q = B.CSR(2, 128, n_q, 32 * n_q, 32, 0, 16, 16, None)
    d = B.PQ(8, 256, 16, 2, 16, 16, 16, n_docs, 2 * n_docs)
    need = M.lib().maxsim_pq_score_workspace_size
    assert (need(ctypes.byref(q), ctypes.byref(d), None) == 0) == decode
