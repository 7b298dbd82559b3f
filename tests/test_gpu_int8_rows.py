"""mfma_i8_kernel, whose blocks make the bytes of their rows once: edges of its 128 x 128 tiles, and lengths of K either side of
its chunks of 128 positions, of the four chunks a load covers and of an odd and an even number of those."""
import numpy as np
import pytest
import torch

import oracle
from paper_2106_12169_amd import binding as B
from paper_2106_12169_amd import workloads as wl

pytestmark = pytest.mark.gpu
U, P = B.ENC_UNSIGNED, B.ENC_PM1


@pytest.mark.parametrize("M,N", [(1, 1), (127, 129), (128, 256), (130, 33)])
@pytest.mark.parametrize("K", [31, 128, 129, 512, 513, 1024, 1100, 1537])
@pytest.mark.parametrize("p,encW,q,encX", [(3, U, 5, U), (8, U, 8, U), (1, P, 6, U), (2, U, 3, U), (7, U, 1, P)])
def test_matches_oracle(M, N, K, p, encW, q, encX):
    W, X = wl.operand(81 + K, M, K, p, encW), wl.operand(82 + N, N, K, q, encX)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    B.apnn_debug_reset()
    B.apnn_debug_force("INT8", 2)
    try:
        Y = B.apnn_gemm(B.apnn_pack(dev(W), p, encW), B.apnn_pack(dev(X), q, encX), M, N, K, p, q, encW, encX)
        torch.cuda.synchronize()
    finally:
        B.apnn_debug_reset()
    assert np.array_equal(Y.cpu().numpy(), oracle.gemm(W, encW, p, X, encX, q))
