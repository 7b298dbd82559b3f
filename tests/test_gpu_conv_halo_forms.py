"""The forms of conv_halo_kernel's blocks that test_gpu_conv_halo.py does not force: 128 channels to a block (eight waves), features staged as
bits and as codes, against the oracle: chunks of weights whose last one is short, digits on either side whose entries are odd in number,
a last channel tile that is half empty, blocks that walk with one buffer.  All results are whole numbers: compared exactly."""
import numpy as np
import pytest

import oracle
from paper_2106_12169_amd import binding as B
from paper_2106_12169_amd import workloads as wl
from tests import helpers as hp
from tests.test_gpu_conv_halo import LAYERS, P, U, _operands, _run, dev, test_layer as _layer

pytestmark = pytest.mark.gpu


# one-plane features, staged as one word of bits: weights that stay and that pass through, an odd number of channel words, pooling
ONE_PLANE = [
    (2, 128, 96, 9, 11, 3, 3, 1, 1, P, 1, U, 1, 2, 2, 0), (2, 96, 64, 7, 12, 3, 3, 1, 1, U, 1, U, 1, 2, 0, 0), (3, 256, 64, 9, 6, 3, 3, 1, 1, P, 1, U, 1, 1, 0, 0),
    (2, 256, 128, 8, 10, 3, 3, 1, 1, P, 1, U, 1, 2, 0, 1), (3, 64, 64, 12, 9, 3, 3, 2, 1, P, 1, U, 1, 2, 1, 2), (2, 64, 64, 9, 8, 3, 3, 1, 1, U, 3, U, 1, 2, 0, 0),
]


@pytest.mark.parametrize("force", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("layer", LAYERS + ONE_PLANE)
def test_forms(force, layer):
    _layer(force, *layer)


# BS, Cin, Cout, H, W, R, p, encW, q
INTS = [
    (2, 128, 192, 9, 13, 3, 1, P, 2),        # 18 steps that stay; a second pair of channel tiles that is half empty
    (2, 384, 128, 8, 9, 3, 1, P, 2),         # 54 steps in chunks, halves of six words
    (1, 192, 96, 11, 7, 3, 1, P, 2),         # 27 steps: the last granule of two is filled up
    (3, 32, 64, 9, 9, 3, 1, U, 5),           # nine steps of three digits
    (2, 256, 64, 6, 7, 1, 3, U, 3),          # four steps, two digits on either side
]


@pytest.mark.parametrize("force", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("BS,Cin,Cout,H,W,R,p,encW,q", INTS)
def test_integer_results(force, BS, Cin, Cout, H, W, R, p, encW, q):
    Wv, Xv, Wp, Xp = _operands(BS, Cin, Cout, H, W, R, R, encW, p, U, q)
    d = B.Conv(BS, H, W, Cin, Cout, R, R, 1, R // 2, p, q, encW, U)
    out = _run(force, lambda: B.apnn_conv2d(d, Wp, Xp))
    want = oracle.conv2d(Wv, encW, p, Xv, U, q, 1, R // 2)
    assert np.array_equal(out.cpu().numpy().reshape(want.transpose(0, 2, 3, 1).shape), want.transpose(0, 2, 3, 1))


# Cin, R, S, encW, p, q, pool: sums of one to three granules of one and of two steps
SHORT = [
    (32, 1, 1, P, 1, 1, 0), (32, 1, 1, P, 1, 2, 1), (64, 1, 1, U, 2, 2, 2), (32, 1, 2, P, 1, 2, 0), (128, 1, 1, U, 1, 2, 1), (96, 1, 1, P, 1, 2, 0),
    (32, 3, 1, P, 1, 2, 0), (192, 1, 1, P, 1, 1, 1), (256, 1, 1, P, 1, 2, 0), (160, 1, 1, P, 1, 2, 0), (64, 5, 1, U, 1, 2, 1), (192, 1, 2, P, 1, 2, 0),
    (32, 1, 1, P, 1, 3, 0), (32, 1, 1, U, 2, 6, 0), (64, 1, 1, U, 1, 4, 0), (128, 1, 1, P, 1, 4, 0), (96, 1, 1, U, 2, 5, 0), (32, 1, 3, P, 1, 4, 0),
]


@pytest.mark.parametrize("force", [1, 2, 5, 6, 7, 8])
@pytest.mark.parametrize("Cin,R,S,encW,p,q,pool", SHORT)
def test_short_sums(force, Cin, R, S, encW, p, q, pool):
    _layer(force, 3, Cin, 96, 10, 13, R, S, 1, 0, encW, p, U, q, 2, 0 if pool else 2, pool)


@pytest.mark.parametrize("force", [7, 8])
def test_blocks_walk_with_one_buffer(force):
    """Frames whose rows fill more than half of what two buffers would leave: every block walks over its tiles in one."""
    BS, Cin, Cout, H, W = 3, 64, 64, 200, 210
    Wv, Xv, Wp, Xp = _operands(BS, Cin, Cout, H, W, 3, 3, P, 1, U, 2)
    d = B.Conv(BS, H, W, Cin, Cout, 3, 3, 1, 1, 1, 2, P, U)
    want = oracle.conv2d(Wv, P, 1, Xv, U, 2, 1, 1)
    scale = np.full(Cout, 1.0 / (np.std(want) + 1.0), np.float32)
    bias = (1.5 - scale * np.mean(want)).astype(np.float32)
    out = _run(force, lambda: B.apnn_layer(d, Wp, Xp, q_out=2, scale=dev(scale), bias=dev(bias)))
    codes, pad_bits = hp.unpack_fmap(hp.words_u32(out), BS, H, W, Cout, 2)
    assert pad_bits == 0 and np.array_equal(codes, oracle.epilogue(want, scale, bias, 2)[0])
