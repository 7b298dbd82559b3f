"""input_tile_kernel (image rows staged once per block) against the oracle: every number of byte-shifted copies (stride 1, 2, 3
and 4), one and two segments a kernel row, several blocks, ranges that cross images, rows shorter than a block's share of
threads, padding wider than the frame's edge groups, channel counts that are no multiple of the three in flight."""
import numpy as np
import pytest
import torch

import oracle
from paper_2106_12169_amd import binding as B
from paper_2106_12169_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu
U, P = B.ENC_UNSIGNED, B.ENC_PM1


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# BS, C, Cout, H, W, R, S, stride, pad, encW, p, q, q_out
@pytest.mark.parametrize("BS,C,Cout,H,W,R,S,stride,pad,encW,p,q,q_out", [
    (2, 3, 64, 37, 41, 7, 7, 2, 3, P, 1, 8, 2), (1, 3, 64, 30, 29, 3, 3, 1, 1, P, 1, 8, 2), (3, 3, 64, 43, 47, 11, 11, 4, 2, P, 1, 8, 2),
    (2, 4, 32, 19, 23, 5, 5, 3, 2, U, 2, 8, 1), (1, 1, 32, 8, 8, 1, 1, 1, 0, U, 1, 8, 2), (9, 2, 64, 5, 9, 3, 16, 1, 8, P, 1, 5, 2),
    (1, 7, 64, 12, 8, 3, 9, 2, 9, U, 3, 1, 2), (40, 3, 64, 9, 11, 7, 7, 2, 3, P, 1, 8, 2), (1, 3, 32, 3, 600, 3, 3, 1, 1, P, 1, 8, 1),
])
def test_matches_oracle(BS, C, Cout, H, W, R, S, stride, pad, encW, p, q, q_out):
    Wv = wl.operand(71, Cout, C * R * S, p, encW).reshape(Cout, C, R, S)
    img = wl.uniform_codes(72, (BS, C, H, W), 8)
    want = oracle.conv2d(Wv, encW, p, img & ((1 << q) - 1), U, q, stride, pad)
    scale = (wl.normals(73, (Cout,), 1.0, 0.2) / (np.std(want) + 1.0)).astype(np.float32)
    scale[1::7] *= -1
    bias = (1.5 - scale * np.mean(want) + wl.normals(74, (Cout,), 0.0, 0.3)).astype(np.float32)
    scale[3], bias[5], bias[6] = np.nan, np.inf, -1e-45
    d = B.Conv(BS, H, W, C, Cout, R, S, stride, pad, p, q, encW, U)
    Wp = B.apnn_pack_input_weights(dev(Wv), p, encW)
    got = {}
    for force in (0, 1):
        B.apnn_debug_reset()
        B.apnn_debug_force("INPUT_TILE", force)
        try:
            got[force] = B.apnn_input_layer(d, Wp, dev(img), q_out=q_out, scale=dev(scale), bias=dev(bias))
            torch.cuda.synchronize()
        finally:
            B.apnn_debug_reset()
    codes, pad_bits = hp.unpack_fmap(hp.words_u32(got[1]), BS, want.shape[2], want.shape[3], Cout, q_out)
    assert pad_bits == 0 and np.array_equal(codes, oracle.epilogue(want, scale, bias, q_out)[0])
    assert torch.equal(got[0], got[1])
