"""The residual scorer's table route, asserted to be the one that ran: a batch
of many short queries and a few long ones over few centroids takes the table
whatever the dimension, and the table is in the caller's workspace, which the
route that gathers centroids leaves alone. Every (bits, dimension, launch's
block count) is checked against the oracle, with queries of every own block
count up to it, and against the same queries on the other route, bit by bit."""
import numpy as np
import pytest
import torch

import paper_2606_26439_amd as M
from tests._gpu import assert_close_o1, dev
from tests.test_gpu_residual import _case, _device, _oracle

pytestmark = pytest.mark.gpu

LONG = {1: [16, 1, 15, 9], 2: [32, 17, 16, 31], 4: [64, 33, 48, 49, 17, 32, 16, 1]}
N_DOCS = 310


def _workspace(Q, D, cand=None):
    n = M.residual_workspace_bytes(Q, D) if cand is None else M.residual_workspace_bytes(Q, D, cand)
    return torch.full((n,), 255, dtype=torch.uint8, device="cuda")


def _written(ws):
    """Words of the workspace that the call wrote (none is a NaN of all ones)."""
    return int((ws.view(torch.int32) != -1).sum())


@pytest.mark.parametrize("blocks", sorted(LONG))
@pytest.mark.parametrize("nbits", [1, 2, 4])
@pytest.mark.parametrize("dim", [64, 128, 256])
def test_every_block_count_of_the_table(dim, nbits, blocks):
    first = LONG[blocks]
    lens = first + [(i * 5) % 13 + 1 for i in range(40 - len(first))]  # on average below 16
    n_c = 61
    c = _case(N_DOCS, dim, nbits, n_c, seed=dim + nbits + blocks, nq_lens=lens)
    Q, D = _device(c)
    ws = _workspace(Q, D)
    batch = M.residual_score(Q, D, workspace=ws)  # 40 x 21K tokens over 61 centroids
    # the table: every query's own blocks of 16 columns
    assert _written(ws) == n_c * 16 * sum((n + 15) // 16 for n in lens)
    assert_close_o1(batch.cpu().numpy(), _oracle(c), f"residual table {dim} {nbits} {blocks}")
    all_docs = M.Candidates(dev(np.array([0, N_DOCS], np.int64)),
                            dev(np.arange(N_DOCS, dtype=np.int32)))
    for a in range(len(first)):
        lo, hi = int(c["q_off"][a]), int(c["q_off"][a + 1])
        one = M.Tokens(Q.tokens[lo:hi].contiguous(), dev(np.array([0, hi - lo], np.int64)), "f16")
        ws = _workspace(one, D, all_docs)
        alone = M.residual_score(one, D, all_docs, workspace=ws)  # 21K tokens
        assert _written(ws) == 0
        assert torch.equal(alone, batch[a * N_DOCS:(a + 1) * N_DOCS]), lens[a]


@pytest.mark.parametrize("dim", [64, 128, 256])
def test_candidate_lists_on_the_table(dim):
    # the same with candidate lists of uneven length, repeated ids among them
    lens = LONG[4] + [(i * 5) % 13 + 1 for i in range(32)]
    c = _case(N_DOCS, dim, 2, 61, seed=dim, nq_lens=lens)
    Q, D = _device(c)
    g = np.random.default_rng(dim)
    sizes = np.array([700, 0, 3, 1, 65, 130, 64, 400] + [350] * 32)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    ids = g.integers(0, N_DOCS, size=int(off[-1])).astype(np.int32)
    cand = M.Candidates(dev(off), dev(ids))
    ws = _workspace(Q, D, cand)
    got = M.residual_score(Q, D, cand, workspace=ws)
    assert _written(ws) > 0
    assert_close_o1(got.cpu().numpy(), _oracle(c, off, ids), f"residual table lists {dim}")
