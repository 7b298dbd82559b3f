"""The forms of conv_halo_kernel's blocks that test_gpu_conv_halo.py does not force: 128 channels to a block (eight waves), features staged as
bits and as codes, against the oracle: every kind of features, every width of the weight loads, pooling, residuals, weights that stay and
that pass through in chunks whose last one is short, digits on either side whose entries are odd in number, a last channel tile that is half
empty, blocks that walk over their tiles with one buffer and with two, sums of one granule and of a few.  That the layers listed here are staged,
in the form that the override names, is checked on the host: test_staged_forms.py.  All results are whole numbers: compared exactly."""
import numpy as np
import pytest

import oracle
from paper_2106_12169_amd import binding as B
from tests.test_gpu_conv_halo import LAYERS, P, U, _operands, _run, test_layer as _layer

pytestmark = pytest.mark.gpu


def applies(force, Cin, Cout, p, q):
    """Whether an override's form exists for a layer: eight waves want channel words in fours, more than 64 channels and one digit on
    either side, codes one digit."""
    one = p <= 2 and q <= 2
    return one if force >= 7 else force >= 5 or (one and Cin % 128 == 0 and Cout > 64)


# (BS, Cin, Cout, H, W, R, S, stride, pad, encW, p, encX, q, q_out, q_res, pool)
# one-plane features, staged as one word of bits: weights that stay and that pass through, an odd number of channel words, pooling
ONE_PLANE = [
    (2, 128, 96, 9, 11, 3, 3, 1, 1, P, 1, U, 1, 2, 2, 0), (2, 96, 64, 7, 12, 3, 3, 1, 1, U, 1, U, 1, 2, 0, 0), (3, 256, 64, 9, 6, 3, 3, 1, 1, P, 1, U, 1, 1, 0, 0),
    (2, 256, 128, 8, 10, 3, 3, 1, 1, P, 1, U, 1, 2, 0, 1), (3, 64, 64, 12, 9, 3, 3, 2, 1, P, 1, U, 1, 2, 1, 2), (2, 64, 64, 9, 8, 3, 3, 1, 1, U, 3, U, 1, 2, 0, 0),
]
# 128 channels a block, its last one short or half of it empty
EIGHT = [
    (2, 128, 128, 9, 11, 3, 3, 1, 1, P, 1, U, 2, 2, 2, 0),      # 8-byte weight loads, residual
    (2, 128, 160, 8, 9, 3, 3, 1, 1, U, 2, U, 2, 2, 0, 0),       # two planes of weights
    (2, 128, 192, 8, 9, 3, 3, 1, 1, P, 1, U, 1, 2, 1, 0),       # one-plane features
    (2, 128, 160, 7, 9, 3, 3, 2, 1, P, 1, P, 1, 2, 2, 0),       # -1/+1 features, stride
    (3, 256, 128, 9, 9, 1, 1, 1, 0, P, 1, U, 2, 1, 2, 0),       # 16-byte weight loads, four steps
    (2, 256, 224, 7, 9, 3, 1, 1, 1, U, 2, U, 1, 2, 0, 0),       # twelve, one-plane features
    (2, 256, 128, 8, 8, 3, 3, 1, 1, P, 1, U, 2, 2, 2, 0),       # 36 in chunks
    (1, 384, 96, 7, 8, 3, 3, 1, 1, U, 1, P, 1, 2, 0, 0),        # 54: the last chunk is short, 0/1 weights on -1/+1 features
    (1, 128, 128, 6, 7, 5, 5, 1, 2, P, 1, U, 1, 2, 0, 0),       # 50 in chunks of 8-byte loads
    (1, 384, 160, 8, 7, 3, 3, 1, 1, U, 2, U, 2, 2, 2, 0),       # two-plane features
    (2, 256, 128, 7, 9, 3, 3, 1, 1, P, 1, U, 1, 2, 1, 0),       # one-plane features, 16-byte loads
    (2, 256, 160, 8, 9, 2, 1, 1, 0, P, 1, P, 1, 2, 2, 0),       # -1/+1 features, eight steps that stay
    (2, 128, 128, 12, 10, 3, 3, 1, 1, P, 1, U, 2, 2, 0, 1),     # pooled: maximum, weights that stay
    (2, 128, 160, 9, 13, 3, 3, 1, 1, U, 2, U, 1, 2, 2, 2),      # sum, residual
    (2, 256, 128, 10, 8, 3, 3, 1, 1, P, 1, U, 2, 2, 2, 1),      # maximum, chunks, residual
    (2, 256, 192, 7, 12, 3, 3, 1, 1, U, 1, P, 1, 1, 0, 2),      # sum, chunks, -1/+1 features
]
FORMS = [(f, layer) for layer in LAYERS + ONE_PLANE + EIGHT for f in (3, 4, 5, 6, 7, 8) if applies(f, layer[1], layer[2], layer[10], layer[12])]


@pytest.mark.parametrize("force,layer", FORMS)
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
INT_FORMS = [(f, layer) for layer in INTS for f in (1, 2, 3, 4, 5, 6, 7, 8) if f < 3 or applies(f, layer[1], layer[2], layer[6], layer[8])]


@pytest.mark.parametrize("force,layer", INT_FORMS)
def test_integer_results(force, layer):
    BS, Cin, Cout, H, W, R, p, encW, q = layer
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


def short_layer(Cin, R, S, encW, p, q, pool):
    return (3, Cin, 96, 10, 13, R, S, 1, 0, encW, p, U, q, 2, 0 if pool else 2, pool)


SHORT_FORMS = [(f, s) for s in SHORT for f in (1, 2, 3, 4, 5, 6, 7, 8) if f < 3 or applies(f, s[0], 96, s[4], s[5])]


@pytest.mark.parametrize("force,short", SHORT_FORMS)
def test_short_sums(force, short):
    _layer(force, *short_layer(*short))


# Blocks that walk over their tiles, the last of which is ragged: override, buffers, layer.
WALKS = [
    (3, 2, (3, 128, 96, 149, 151, 1, 1, 1, 0, P, 1, U, 2, 2, 2, 0)),      # eight waves, residual
    (4, 2, (3, 256, 128, 690, 64, 1, 1, 1, 0, P, 1, U, 1, 2, 0, 0)),      # one-plane features, 16-byte weight loads
    (3, 1, (2, 256, 96, 890, 40, 3, 2, 1, 1, P, 1, P, 1, 2, 1, 0)),       # -1/+1 features, one buffer
    (4, 1, (2, 128, 96, 230, 160, 3, 3, 1, 1, P, 1, U, 2, 2, 0, 0)),
    (3, 2, (2, 128, 96, 282, 243, 1, 1, 1, 0, P, 1, U, 2, 2, 2, 1)),      # pooled: maximum, residual
    (4, 2, (3, 128, 96, 1401, 64, 1, 1, 1, 0, U, 2, U, 1, 2, 0, 2)),      # sum, one-plane features
    (3, 1, (2, 256, 96, 602, 60, 2, 2, 1, 1, P, 1, U, 2, 1, 0, 1)),       # one buffer
    (5, 2, (3, 64, 64, 761, 60, 3, 3, 1, 1, P, 1, U, 2, 2, 2, 0)),        # bits, four waves a SIMD
    (5, 2, (2, 32, 64, 1130, 60, 1, 1, 1, 0, P, 1, U, 5, 2, 0, 0)),       # of three digits
    (6, 1, (2, 96, 64, 214, 301, 3, 3, 1, 1, P, 1, U, 4, 2, 0, 0)),       # of two, one buffer
    (7, 1, (3, 64, 64, 200, 210, 3, 3, 1, 1, P, 1, U, 2, 2, 0, 0)),       # frames whose rows fill more than half of what two buffers would leave
    (8, 1, (4, 64, 64, 200, 210, 3, 3, 1, 1, P, 1, U, 2, 2, 0, 0)),
]


@pytest.mark.parametrize("force,buffers,layer", WALKS)
def test_blocks_walk(force, buffers, layer):
    _layer(force, *layer)
