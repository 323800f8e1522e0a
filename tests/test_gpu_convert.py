"""FP8 conversion at the edges of its lane groups: a token is dim / 4 pieces
over 4, 8, 16, 32 or 64 lanes, one to four pieces per lane, several tokens per
wavefront. Codes and scales must equal the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_26439_amd as M
import workloads as W
from tests._gpu import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 257])
@pytest.mark.parametrize("dim", [16, 32, 48, 64, 80, 128, 144, 256, 272, 512, 528, 768, 784, 1024])
def test_fp8_conversion_bit_exact_at_group_edges(dim, n):
    g = W.rng(dim + n)
    x = W.unit_tokens(n, dim, g)
    x *= np.exp2(g.integers(-40, 40, size=(n, 1))).astype(np.float32)
    x[n // 2] = 0.0  # an all-zero token: scale 1
    x[-1, :] = 0.0
    x[-1, dim - 1] = -448.0  # the largest value in the last lane's last element
    tok, sc = M.quantize(dev(x), "fp8")
    torch.cuda.synchronize()
    _, payload = oracle.exact_values(x, "fp8")
    assert np.array_equal(tok.cpu().numpy(), payload[0])
    assert np.array_equal(sc.cpu().numpy(), payload[1])
