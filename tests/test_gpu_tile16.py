"""mfma_tile16_kernel (products and convolutions with few outputs) against the oracle: edges of its 16 x 16 tiles, lengths of K either side of
its groups of 512 positions and of the groups that its four or eight waves share, every kind of operand, the whole epilogue,
and the sizes around the rule that takes it; for convolutions also the 32 x 32 tile whose K is split over eight waves.  All results are whole numbers, or floats of one rounding: compared exactly."""
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


def _run(force, call):
    B.apnn_debug_reset()
    if force == "32x8":                 # the 32 x 32 tile with K split over eight waves
        B.apnn_debug_force("MFMA_NSPLIT", 8)
    else:
        B.apnn_debug_force("MFMA_T16", force)
    B.apnn_debug_force("INT8", 0)
    try:
        out = call()
        torch.cuda.synchronize()
    finally:
        B.apnn_debug_reset()
    return out


@pytest.mark.parametrize("force", [4, 8])
@pytest.mark.parametrize("M,N", [(1, 1), (16, 33), (17, 16), (63, 95)])
@pytest.mark.parametrize("K", [1, 127, 512, 513, 2048, 2500, 4608, 16900])
@pytest.mark.parametrize("p,encW,q,encX", [(1, P, 2, U), (1, P, 1, P), (2, U, 1, U), (3, U, 1, P), (3, U, 4, U)])
def test_gemm(force, M, N, K, p, encW, q, encX):
    W, X = wl.operand(91 + K, M, K, p, encW), wl.operand(92 + N, N, K, q, encX)
    Y = _run(force, lambda: B.apnn_gemm(B.apnn_pack(dev(W), p, encW), B.apnn_pack(dev(X), q, encX), M, N, K, p, q, encW, encX))
    assert np.array_equal(Y.cpu().numpy(), oracle.gemm(W, encW, p, X, encX, q))


@pytest.mark.parametrize("force", [-1, 4, 8])
@pytest.mark.parametrize("BS,Cout,K,p,encW,q,encX,q_out,with_res",
                         [(1, 128, 9216, 1, P, 2, U, 2, False), (5, 96, 700, 1, P, 2, U, 2, True), (40, 32, 300, 2, U, 3, U, 8, True),
                          (17, 64, 1030, 1, P, 1, P, 1, True), (64, 1024, 1024, 1, U, 2, U, 3, False)])
def test_layer(force, BS, Cout, K, p, encW, q, encX, q_out, with_res):
    """The whole epilogue (residual, planes, int32 and float side outputs); a tile writes half a plane word."""
    Xv, Wv = wl.operand(93 + K, BS, K, q, encX), wl.operand(94, Cout, K, p, encW)
    want = oracle.gemm(Xv, encX, q, Wv, encW, p)
    scale = (wl.normals(95, (Cout,), 1.0, 0.2) * (1 << q_out) / 4 / (np.std(want) + 1)).astype(np.float32)
    bias = (0.5 * (1 << q_out) - scale * np.mean(want) + wl.normals(96, (Cout,), 0.0, 0.2)).astype(np.float32)
    res = wl.uniform_codes(97, (BS, Cout), 2) if with_res else None
    d = B.Conv(BS, 1, 1, K, Cout, 1, 1, 1, 0, p, q, encW, encX)
    acc = torch.empty((BS, Cout), dtype=torch.int32, device="cuda")
    tf = torch.empty((BS, Cout), dtype=torch.float32, device="cuda")
    kw = dict(is_gemm=True, q_out=q_out, scale=dev(scale), bias=dev(bias), acc_out=acc, float_out=tf)
    if with_res:
        kw.update(residual=B.apnn_pack_fmap(dev(res.reshape(BS, Cout, 1, 1)), B.LAYOUT_NCHW, 2, U), q_res=2, res_scale=0.5)
    out = _run(force, lambda: B.apnn_layer(d, B.apnn_pack(dev(Wv), p, encW), B.apnn_pack(dev(Xv), q, encX), **kw))
    want_codes, want_t = oracle.epilogue(want, scale, bias, q_out, res=res, res_scale=0.5, want_t=True)
    assert np.array_equal(acc.cpu().numpy(), want) and np.array_equal(tf.cpu().numpy(), want_t)
    codes, pad_bits = hp.unpack_fmap(hp.words_u32(out), BS, 1, 1, Cout, q_out)
    assert np.array_equal(codes.reshape(BS, Cout), want_codes) and pad_bits == 0


# BS, Cin, Cout, H, W, R, stride, pad, encW, p, encX, q, q_out, q_res, pool
CONVS = [
    (1, 256, 32, 6, 6, 6, 1, 0, P, 1, U, 2, 2, 0, 0),       # a fully connected layer: the kernel covers the frame
    (3, 512, 96, 1, 1, 1, 1, 0, P, 1, U, 2, 2, 3, 0),       # 1 x 1 frame, residual of three planes
    (2, 128, 64, 5, 7, 3, 1, 1, U, 2, U, 4, 3, 0, 0),       # 16-byte loads, two feature digits, three planes
    (1, 64, 32, 9, 5, 3, 2, 1, P, 1, U, 2, 1, 1, 0),        # 8-byte loads: two taps in one
    (2, 192, 32, 4, 4, 5, 1, 2, U, 3, U, 1, 2, 2, 0),
    (1, 32, 64, 7, 3, 3, 1, 1, U, 1, U, 3, 2, 0, 0),        # word by word: four taps in one
    (1, 96, 32, 6, 6, 5, 3, 2, P, 1, P, 1, 2, 0, 0),        # -1/+1 features, padding
    (2, 128, 32, 5, 5, 3, 1, 1, U, 1, P, 1, 1, 1, 0),
    (2, 64, 64, 7, 6, 3, 1, 1, P, 1, U, 2, 2, 0, 1),        # pooling, odd frame
    (1, 256, 32, 6, 4, 3, 1, 1, U, 2, U, 2, 3, 2, 2),       # pooled sum with residual
    (5, 32, 32, 4, 4, 3, 1, 1, U, 1, P, 1, 2, 3, 1),
]


@pytest.mark.parametrize("force", [-1, 4, 8, "32x8"])
@pytest.mark.parametrize("BS,Cin,Cout,H,W,R,stride,pad,encW,p,encX,q,q_out,q_res,pool", CONVS)
def test_conv(force, BS, Cin, Cout, H, W, R, stride, pad, encW, p, encX, q, q_out, q_res, pool):
    Wv = wl.operand(102 + Cin, Cout, Cin * R * R, p, encW).reshape(Cout, Cin, R, R)
    Xv = wl.operand(103 + H, BS * Cin, H * W, q, encX).reshape(BS, Cin, H, W)
    d = B.Conv(BS, H, W, Cin, Cout, R, R, stride, pad, p, q, encW, encX)
    want = oracle.conv2d(Wv, encW, p, Xv, encX, q, stride, pad)
    if pool:
        want = oracle.gridpool(want, 2, oracle.POOL_MAX if pool == B.POOL_MAX2 else oracle.POOL_SUM)
    Hq, Wq = want.shape[2:]
    scale = (wl.normals(104, (Cout,), 1.0, 0.3) * (1 << q_out) / 4 / (np.std(want) + 1.0)).astype(np.float32)
    scale[::5] *= -1
    bias = (0.5 * (1 << q_out) - scale * np.mean(want) + wl.normals(105, (Cout,), 0.0, 0.3)).astype(np.float32)
    res = wl.uniform_codes(106, (BS, Cout, Hq, Wq), q_res) if q_res else None
    acc = torch.empty((BS, Hq, Wq, Cout), dtype=torch.int32, device="cuda")
    kw = dict(q_out=q_out, scale=dev(scale), bias=dev(bias), pool=pool, acc_out=acc)
    if q_res:
        kw.update(residual=B.apnn_pack_fmap(dev(res), B.LAYOUT_NCHW, q_res, U), q_res=q_res, res_scale=0.37)
    Wp, Xp = B.apnn_pack_conv_weights(dev(Wv), p, encW), B.apnn_pack_fmap(dev(Xv), B.LAYOUT_NCHW, q, encX)
    out = _run(force, lambda: B.apnn_layer(d, Wp, Xp, **kw))
    codes, pad_bits = hp.unpack_fmap(hp.words_u32(out), BS, Hq, Wq, Cout, q_out)
    assert np.array_equal(acc.cpu().numpy().transpose(0, 3, 1, 2), want)
    assert pad_bits == 0 and np.array_equal(codes, oracle.epilogue(want, scale, bias, q_out, res=res, res_scale=0.37)[0])


def test_thresholds():
    """Infinities and NaN of the epilogue get the codes that the clamp gives them."""
    BS, Cout, K = 3, 32, 64
    Xv, Wv = wl.uniform_codes(98, (BS, K), 2), wl.fair_signs(99, (Cout, K))
    scale = np.resize(np.array([0, 1, -1, np.inf, np.nan, 0.25], np.float32), Cout)
    bias = np.resize(np.array([0, np.inf, -np.inf, np.nan, 1, 2, 3.4e38], np.float32), Cout)
    d = B.Conv(BS, 1, 1, K, Cout, 1, 1, 1, 0, 1, 2, P, U)
    call = lambda: B.apnn_layer(d, B.apnn_pack(dev(Wv), 1, P), B.apnn_pack(dev(Xv), 2, U), is_gemm=True, q_out=2, scale=dev(scale), bias=dev(bias))
    out, ref = _run(4, call), _run(0, call)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("M,N,K", [(256, 512, 640), (257, 512, 640), (16, 8224, 700), (17, 8224, 700), (512, 512, 256), (528, 512, 256)])
def test_rule(M, N, K):
    """Either side of the sizes up to which the rule takes the small tiles: the same results."""
    W, X = dev(wl.fair_signs(100, (M, K))), dev(wl.uniform_codes(101, (N, K), 2))
    call = lambda: B.apnn_gemm(B.apnn_pack(W, 1, P), B.apnn_pack(X, 2, U), M, N, K, 1, 2, P, U)
    want = (W.cpu().double() @ X.cpu().double().T).to(torch.int32)
    assert torch.equal(_run(-1, call).cpu(), want) and torch.equal(_run(0, call).cpu(), want)
