"""Max pooling by OR (one and two planes, windows up to 3 x 3) and the last layer with a class to a thread, against the oracle: every width
of load, buffers that are aligned to a word only, frames that are smaller than the window, channel counts at the form's edges."""
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


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("bits", [1, 2])
@pytest.mark.parametrize("k,stride,pad,C,H,W", [(3, 2, 1, 64, 14, 9), (3, 1, 2, 32, 5, 7), (2, 2, 0, 128, 6, 9), (2, 1, 1, 40, 3, 3),
                                                (1, 2, 0, 96, 7, 4), (3, 2, 1, 192, 1, 2), (3, 3, 0, 64, 9, 30)])
def test_maxpool(k, stride, pad, C, H, W, bits, shift):
    Xv = wl.uniform_codes(11, (3, C, H, W), bits)
    Xp = B.apnn_pack_fmap(dev(Xv), B.LAYOUT_NCHW, bits, U)
    X = torch.empty(Xp.numel() + 4, dtype=torch.int32, device="cuda")[shift:shift + Xp.numel()]
    X.copy_(Xp)
    want = oracle.maxpool(Xv, k, stride, pad)
    words = B.apnn_fmap_words(3 * want.shape[2] * want.shape[3], C, bits)
    out = torch.full((words + 4,), -1, dtype=torch.int32, device="cuda")[shift:shift + words]
    B.apnn_maxpool(X, 3, H, W, C, bits, k, stride, pad, out=out)
    torch.cuda.synchronize()
    codes, _ = hp.unpack_fmap(hp.words_u32(out), 3, want.shape[2], want.shape[3], C, bits)
    assert np.array_equal(codes, want)


@pytest.mark.parametrize("BS,C,bits,Cout,p,encW", [(70, 512, 2, 1000, 1, P), (300, 128, 1, 257, 1, U), (130, 256, 2, 513, 1, P),
                                                   (70, 544, 2, 1000, 1, P), (70, 512, 2, 1000, 2, U)])
def test_sumpool_fc(BS, C, bits, Cout, p, encW):
    """The last two are just outside the form: 17 channel words, two weight planes."""
    Xv = wl.uniform_codes(5 + C, (BS, C, 3, 3), bits)
    Wv = wl.operand(6 + Cout, Cout, C, p, encW)
    Y = B.apnn_sumpool_fc(B.apnn_pack_fmap(dev(Xv), B.LAYOUT_NCHW, bits, U), BS, 3, 3, C, bits, B.apnn_pack(dev(Wv), p, encW), Cout, p, encW,
                          out=torch.full((BS, Cout), -7, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy(), oracle.gemm(oracle.sumpool(Xv), U, 8, Wv, encW, p))
