"""conv_halo_kernel (convolutions with the input pixels staged once per block) against the oracle, forced onto small layers:
both sizes of tile, weights that stay in LDS and weights that pass through in chunks, every staging width, several
digits on either side, ragged last tiles of pixels and channels, ranges that cross images, pooling, residuals, int32
results, and the code thresholds at exact integers, infinities and NaN.  All results are whole numbers: compared exactly."""
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


def _operands(BS, Cin, Cout, H, W, R, S, encW, p, encX, q):
    Wv = wl.operand(61 + Cin, Cout, Cin * R * S, p, encW).reshape(Cout, Cin, R, S)
    Xv = wl.operand(62 + H, BS * Cin, H * W, q, encX).reshape(BS, Cin, H, W)
    return Wv, Xv, B.apnn_pack_conv_weights(dev(Wv), p, encW), B.apnn_pack_fmap(dev(Xv), B.LAYOUT_NCHW, q, encX)


def _run(force, call):
    B.apnn_debug_reset()
    B.apnn_debug_force("MFMA_HALO", force)
    try:
        out = call()
        torch.cuda.synchronize()
    finally:
        B.apnn_debug_reset()
    return out


# BS, Cin, Cout, H, W, R, S, stride, pad, encW, p, encX, q, q_out, q_res, pool
LAYERS = [
    (3, 64, 64, 13, 11, 3, 3, 1, 1, P, 1, U, 2, 2, 2, 0),       # ragged last tile, ranges across images
    (2, 128, 96, 9, 15, 3, 3, 1, 1, P, 1, U, 2, 2, 0, 0),       # a second channel tile that is half empty
    (1, 32, 32, 17, 9, 3, 3, 2, 1, U, 1, U, 2, 1, 1, 0),        # one channel word: a lane half without words
    (2, 96, 160, 8, 7, 3, 3, 1, 1, U, 2, U, 4, 2, 0, 0),        # odd channel words, two feature digits
    (2, 192, 64, 7, 9, 3, 3, 1, 1, P, 1, U, 3, 2, 2, 0),        # chunks of taps with three words a half, odd planes
    (2, 256, 64, 8, 8, 3, 3, 1, 1, P, 1, U, 2, 2, 2, 0),        # chunks of two taps
    (1, 512, 64, 7, 7, 3, 3, 1, 1, P, 1, U, 2, 2, 1, 0),        # chunks of one tap
    (1, 128, 64, 9, 9, 3, 3, 1, 1, U, 4, U, 4, 2, 0, 0),        # digits on both sides: several weight passes
    (5, 64, 64, 4, 3, 1, 1, 1, 0, U, 3, U, 1, 1, 0, 0),         # 1 x 1, one feature plane, odd weight planes
    (2, 64, 64, 9, 8, 5, 2, 3, 2, P, 1, P, 1, 2, 0, 0),         # -1/+1 features, padding beyond the kernel's reach
    (2, 256, 64, 6, 6, 3, 3, 1, 1, U, 1, P, 1, 1, 2, 0),        # the same through chunks
    (3, 64, 64, 11, 14, 3, 3, 1, 1, P, 1, U, 2, 2, 0, 1),       # pooling, odd frame
    (2, 256, 64, 10, 6, 3, 3, 1, 1, U, 2, U, 2, 2, 2, 2),       # pooled sum, chunks, residual
    (1, 96, 64, 9, 12, 2, 3, 2, 1, U, 1, P, 1, 1, 0, 1),        # pooling with stride, -1/+1 features
    (8, 64, 64, 20, 20, 3, 3, 1, 1, P, 1, U, 2, 2, 0, 0),       # a dozen tiles
    (1, 64, 64, 1, 1, 1, 1, 1, 0, P, 1, U, 2, 2, 0, 0),         # one pixel, one step
]


@pytest.mark.parametrize("force", [1, 2])
@pytest.mark.parametrize("BS,Cin,Cout,H,W,R,S,stride,pad,encW,p,encX,q,q_out,q_res,pool", LAYERS)
def test_layer(force, BS, Cin, Cout, H, W, R, S, stride, pad, encW, p, encX, q, q_out, q_res, pool):
    Wv, Xv, Wp, Xp = _operands(BS, Cin, Cout, H, W, R, S, encW, p, encX, q)
    d = B.Conv(BS, H, W, Cin, Cout, R, S, stride, pad, p, q, encW, encX)
    want = oracle.conv2d(Wv, encW, p, Xv, encX, q, stride, pad)
    if pool:
        want = oracle.gridpool(want, 2, oracle.POOL_MAX if pool == B.POOL_MAX2 else oracle.POOL_SUM)
    Hq, Wq = want.shape[2:]
    spread = np.std(want) + 1.0
    scale = (wl.normals(63, (Cout,), 1.0, 0.3) / spread).astype(np.float32)
    scale[::5] *= -1
    bias = (1.5 - scale * np.mean(want) + wl.normals(64, (Cout,), 0.0, 0.3)).astype(np.float32)
    res = wl.uniform_codes(65, (BS, Cout, Hq, Wq), q_res) if q_res else None
    kw = dict(q_out=q_out, scale=dev(scale), bias=dev(bias), pool=pool)
    if q_res:
        kw.update(residual=B.apnn_pack_fmap(dev(res), B.LAYOUT_NCHW, q_res, U), q_res=q_res, res_scale=0.37)
    out = _run(force, lambda: B.apnn_layer(d, Wp, Xp, **kw))
    codes, pad_bits = hp.unpack_fmap(hp.words_u32(out), BS, Hq, Wq, Cout, q_out)
    assert pad_bits == 0
    assert np.array_equal(codes, oracle.epilogue(want, scale, bias, q_out, res=res, res_scale=0.37)[0])


# Layers whose blocks walk over three tiles and more, the last one ragged, with the next tile's pixels in flight: kernel form, layer.
# (tests/sanitize/conv_halo_driver.cpp checks that the same layers get two buffers and as many tiles a block.)
WALKED = [
    (1, (2, 112, 111), (32, 512, 3, 3, 1, 1, P, 1, U, 2, 2, 2, 0)),     # eight channel tiles, ranges across images, residual
    (2, (2, 157, 158), (64, 480, 1, 1, 1, 0, P, 1, U, 2, 2, 1, 0)),     # 256 pixels a tile, the last channel tile half empty
    (1, (3, 105, 105), (32, 512, 1, 1, 1, 0, U, 1, U, 1, 1, 2, 0)),     # one feature plane
    (1, (3, 104, 105), (32, 512, 2, 1, 1, 1, P, 1, P, 1, 2, 0, 0)),     # -1/+1 features, padding
    (1, (3, 105, 105), (64, 512, 1, 1, 1, 0, P, 1, U, 3, 2, 2, 0)),     # two feature digits
    (1, (1, 550, 551), (32, 64, 1, 1, 1, 0, P, 1, U, 2, 2, 2, 0)),      # one channel tile
    (1, (2, 158, 159), (32, 512, 1, 1, 1, 0, P, 1, U, 2, 2, 2, 1)),     # pooled, 64 pooled pixels a tile
    (2, (2, 183, 183), (32, 512, 1, 1, 1, 0, P, 1, U, 2, 2, 0, 2)),     # pooled sum, 128
]


@pytest.mark.parametrize("force,frames,layer", WALKED)
def test_blocks_walk_over_tiles(force, frames, layer):
    BS, H, W = frames
    Cin, Cout, *rest = layer
    test_layer(force, BS, Cin, Cout, H, W, *rest)


@pytest.mark.parametrize("force", [1, 2])
@pytest.mark.parametrize("BS,Cin,Cout,H,W,R,S,stride,pad,encW,p,encX,q", [
    (2, 96, 36, 9, 7, 3, 3, 1, 1, U, 2, U, 4), (1, 64, 4, 12, 12, 3, 3, 2, 1, P, 1, U, 2), (1, 512, 132, 5, 5, 3, 3, 1, 1, P, 1, P, 1),
])
def test_int32(force, BS, Cin, Cout, H, W, R, S, stride, pad, encW, p, encX, q):
    Wv, Xv, Wp, Xp = _operands(BS, Cin, Cout, H, W, R, S, encW, p, encX, q)
    d = B.Conv(BS, H, W, Cin, Cout, R, S, stride, pad, p, q, encW, encX)
    Y = _run(force, lambda: B.apnn_conv2d(d, Wp, Xp))
    assert np.array_equal(Y.cpu().numpy().transpose(0, 3, 1, 2), oracle.conv2d(Wv, encW, p, Xv, encX, q, stride, pad))


@pytest.mark.parametrize("with_res", [False, True])
def test_code_thresholds(with_res):
    """t exactly on, just below and just above 1, 2, 3 and 4; constants that are infinite, NaN, denormal or huge."""
    BS, C, H = 2, 64, 9
    Wv, Xv, Wp, Xp = _operands(BS, 64, C, H, H, 3, 3, P, 1, U, 2)
    d = B.Conv(BS, H, H, 64, C, 3, 3, 1, 1, 1, 2, P, U)
    scale, bias = np.full(C, 0.25, np.float32), np.zeros(C, np.float32)
    scale[1::4], scale[2::4] = np.float32(1 / 3), np.nextafter(np.float32(0.25), np.float32(1))
    scale[3::4] = np.nextafter(np.float32(0.25), np.float32(0))
    odd = [np.inf, -np.inf, np.nan, 0.0, -0.0, 1e-40, -1e-40, 3e38, -3e38, 1e-45]
    scale[20:30], bias[30:40] = odd, odd
    scale[40:43], bias[40:43] = [np.inf, -np.inf, 0.0], [-np.inf, np.inf, np.nan]
    bias[43:48] = [1.0, np.nextafter(np.float32(1), np.float32(0)), 2.0, 3.0, 4.0]
    scale[43:48] = 0.0
    res = wl.uniform_codes(66, (BS, C, H, H), 2) if with_res else None
    kw = dict(q_out=2, scale=dev(scale), bias=dev(bias))
    if with_res:
        kw.update(residual=B.apnn_pack_fmap(dev(res), B.LAYOUT_NCHW, 2, U), q_res=2, res_scale=0.5)
    out = _run(2, lambda: B.apnn_layer(d, Wp, Xp, **kw))
    general = _run(0, lambda: B.apnn_layer(d, Wp, Xp, **kw))
    assert torch.equal(out, general)
    codes, _ = hp.unpack_fmap(hp.words_u32(out), BS, H, H, C, 2)
    want = oracle.epilogue(oracle.conv2d(Wv, P, 1, Xv, U, 2, 1, 1), scale, bias, 2, res=res, res_scale=0.5)[0]
    assert np.array_equal(codes, want)


def test_own_choice_has_the_same_planes():
    """The library's own choice against the other kernels, for layers either side of its rule (which one it takes:
    tests/sanitize/abi_host_driver.cpp)."""
    for BS in (8, 128):
        Wv, Xv, Wp, Xp = _operands(BS, 64, 64, 28, 28, 3, 3, P, 1, U, 2)
        d = B.Conv(BS, 28, 28, 64, 64, 3, 3, 1, 1, 1, 2, P, U)
        kw = dict(q_out=2, scale=torch.full((64,), 0.05, device="cuda"), bias=torch.full((64,), 1.5, device="cuda"))
        assert torch.equal(_run(-1, lambda: B.apnn_layer(d, Wp, Xp, **kw)), _run(0, lambda: B.apnn_layer(d, Wp, Xp, **kw)))
