"""The residual scorer's two routes (a centroid-query table built first, or the
centroids gathered by the scorer) and its split of a batch over wavefronts.

A batch with many tokens per centroid takes the table, the same queries over
few candidates gather the centroids: the scores must have the same bits, and
must match the oracle. Query lengths cross each 16-token block count, lists
of very different sizes share a launch (empty ones, repeated ids), and
documents cross tile edges (0, 1, 16 and 17 tokens)."""
import numpy as np
import pytest
import torch

import paper_2606_26439_amd as M
import workloads as W
from tests._gpu import assert_close_o1, dev
from tests.test_gpu_residual import _case, _device, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbits", [1, 2, 4])
@pytest.mark.parametrize("dim", [64, 128, 256])
def test_table_and_direct_routes_give_the_same_bits(dim, nbits):
    nq = [16] * 36 + [1, 9, 16, 15]
    c = _case(310, dim, nbits, 257, seed=dim + nbits, nq_lens=nq)
    Q, D = _device(c)
    batch = M.residual_score(Q, D)  # 40 x 21K tokens over 257 centroids: table
    assert_close_o1(batch.cpu().numpy(), _oracle(c), f"residual table {dim} {nbits}")
    for a in (0, 36, 37, 39):
        lo, hi = int(c["q_off"][a]), int(c["q_off"][a + 1])
        one = M.Tokens(Q.tokens[lo:hi].contiguous(), dev(np.array([0, hi - lo], np.int64)), "f16")
        ids = dev(np.arange(309, -1, -1, dtype=np.int32))
        cand = M.Candidates(dev(np.array([0, 310], np.int64)), ids)
        alone = M.residual_score(one, D, cand)  # 21K tokens: centroids gathered
        assert torch.equal(alone.flip(0), batch[a * 310:(a + 1) * 310])


@pytest.mark.parametrize("nq_lens", [[64, 1, 17, 33, 48, 16], [32, 8, 31], [16, 3]])
def test_uneven_candidate_lists_share_a_launch(nq_lens):
    c = _case(500, 128, 2, 300, seed=sum(nq_lens), nq_lens=nq_lens)
    g = W.rng(7)
    sizes = [900, 0, 3, 1, 65, 130][:len(nq_lens)]
    off = W.offsets_from_lengths(sizes)
    ids = g.integers(0, 500, size=int(off[-1])).astype(np.int32)  # repeated ids
    ids[:4] = [0, 1, 2, 3]
    Q, D = _device(c)
    got = M.residual_score(Q, D, M.Candidates(dev(off), dev(ids))).cpu().numpy()
    assert_close_o1(got, _oracle(c, off, ids), f"residual uneven {nq_lens}")


@pytest.mark.parametrize("nbits,dim", [(1, 64), (2, 128), (4, 128), (2, 256)])
def test_each_query_uses_its_own_blocks(nbits, dim):
    # one to four blocks in one batch, over a table whose unwritten columns
    # hold NaN: every query's scores are the bits it has alone, on both routes
    nq = [64, 33, 48, 49, 17, 32, 16, 1] * 2
    c = _case(310, dim, nbits, 257, seed=dim + nbits, nq_lens=nq)
    Q, D = _device(c)
    ws = torch.full((M.residual_workspace_bytes(Q, D),), 255, dtype=torch.uint8, device="cuda")
    batch = M.residual_score(Q, D, workspace=ws)  # 16 x 21K tokens over 257 centroids: table
    assert_close_o1(batch.cpu().numpy(), _oracle(c), f"residual blocks {dim} {nbits}")
    for a in range(8):
        lo, hi = int(c["q_off"][a]), int(c["q_off"][a + 1])
        one = M.Tokens(Q.tokens[lo:hi].contiguous(), dev(np.array([0, hi - lo], np.int64)), "f16")
        cand = M.Candidates(dev(np.array([0, 310], np.int64)), dev(np.arange(310, dtype=np.int32)))
        alone = M.residual_score(one, D, cand)  # 21K tokens: centroids gathered
        assert torch.equal(alone, batch[a * 310:(a + 1) * 310]), nq[a]
