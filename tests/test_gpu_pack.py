"""GPU parity of the bit-plane packers: bit-exact against the source codes
(decoded from the packed words with numpy) and zero pad bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2106_12169_amd import binding as B
from paper_2106_12169_amd import workloads as wl
from tests import helpers as hp

pytestmark = pytest.mark.gpu
U, P = wl.ENC_UNSIGNED, wl.ENC_PM1


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("rows,K,bits,enc", [
    (128, 128, 1, P), (128, 128, 2, U), (37, 203, 3, U), (5, 31, 8, U), (300, 1000, 5, U),
    (64, 4096, 2, U), (1, 1, 1, U), (33, 96, 1, P), (7, 48, 4, U),
])
def test_pack_matrix(rows, K, bits, enc):
    src = wl.operand(100 + rows + K, rows, K, bits, enc)
    words = hp.words_u32(B.apnn_pack(dev(src), bits, enc))
    codes, pad = hp.unpack_matrix(words, rows, K, bits)
    want = hp.pm1_to_bits(src) if enc == P else src
    assert np.array_equal(codes, want)
    assert pad == 0 and words.size == B.apnn_packed_words(rows, K, bits)


def test_pack_ignores_bits_above_the_declared_width():
    src = wl.uniform_codes(5, (9, 70), 8)
    codes, _ = hp.unpack_matrix(hp.words_u32(B.apnn_pack(dev(src), 3, U)), 9, 70, 3)
    assert np.array_equal(codes, src & 7)


@pytest.mark.parametrize("layout", [B.LAYOUT_NHWC, B.LAYOUT_NCHW])
@pytest.mark.parametrize("N,C,H,W,bits", [(2, 64, 5, 7, 2), (1, 128, 9, 9, 2), (3, 32, 4, 4, 3), (1, 96, 6, 5, 1),
                                          (2, 64, 8, 8, 8), (1, 96, 6, 6, 2), (2, 40, 4, 6, 3), (3, 160, 28, 28, 2)])
def test_pack_fmap(layout, N, C, H, W, bits):
    nchw = wl.uniform_codes(7, (N, C, H, W), bits)
    src = nchw if layout == B.LAYOUT_NCHW else nchw.transpose(0, 2, 3, 1)
    words = hp.words_u32(B.apnn_pack_fmap(dev(src), layout, bits, U))
    codes, pad = hp.unpack_fmap(words, N, H, W, C, bits)
    assert np.array_equal(codes, nchw) and pad == 0


@pytest.mark.parametrize("layout", [B.LAYOUT_NHWC, B.LAYOUT_NCHW])
@pytest.mark.parametrize("N,C,H,W", [(2, 64, 4, 6), (1, 96, 5, 5), (2, 40, 8, 2)])
def test_pack_fmap_pm1(layout, N, C, H, W):
    nchw = wl.fair_signs(8, (N, C, H, W))
    src = nchw if layout == B.LAYOUT_NCHW else nchw.transpose(0, 2, 3, 1)
    words = hp.words_u32(B.apnn_pack_fmap(dev(src), layout, 1, P))
    codes, pad = hp.unpack_fmap(words, N, H, W, C, 1)
    assert np.array_equal(codes, hp.pm1_to_bits(nchw)) and pad == 0


def test_pack_conv_weights_layout():
    Cout, Cin, R, S = 5, 64, 3, 3
    w = wl.fair_signs(3, (Cout, Cin, R, S))
    words = hp.words_u32(B.apnn_pack_conv_weights(dev(w), 1, P))
    Cw = Cin // 32
    # [Cout][bits][R][S][Cw]: row (co, r, s) holds the channels of that tap
    codes, pad = hp.unpack_planes(words, Cout * R * S, Cin, 1, Cw)
    assert np.array_equal(codes.reshape(Cout, R, S, Cin), hp.pm1_to_bits(w).transpose(0, 2, 3, 1)) and pad == 0
    w2 = wl.uniform_codes(4, (Cout, Cin, R, S), 3)
    words = hp.words_u32(B.apnn_pack_conv_weights(dev(w2), 3, U)).reshape(Cout, 3, R * S, Cw)
    for t in range(3):
        plane, _ = hp.unpack_planes(words[:, t].reshape(-1), Cout * R * S, Cin, 1, Cw)
        assert np.array_equal(plane.reshape(Cout, R, S, Cin), ((w2 >> t) & 1).transpose(0, 2, 3, 1))


@pytest.mark.parametrize("rows,K", [(19, 333), (5, 256), (3, 1), (7, 31), (2, 1000), (64, 4096)])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_quantize_matches_oracle(bits, rows, K):
    x = wl.normals(9, (rows, K), 2.0, 3.0)
    special = [np.nan, np.inf, -np.inf, 0.0, -0.0, 1e30][:K]
    x[0, :len(special)] = special
    zero, step = -0.75, 0.37
    words = hp.words_u32(B.apnn_quantize(dev(x), zero, step, bits))
    codes, pad = hp.unpack_matrix(words, rows, K, bits)
    assert np.array_equal(codes, oracle.quantize(x, zero, step, bits)) and pad == 0


@pytest.mark.parametrize("bits,enc", [(1, P), (1, U), (2, U), (4, U), (5, U), (8, U)])
@pytest.mark.parametrize("K", [15, 31, 32, 33, 63, 65, 127, 1999])
def test_pack_rows_of_any_length_and_alignment(K, bits, enc):
    rows = 7
    src = wl.operand(200 + K, rows, K, bits, enc)
    buf = torch.zeros(rows * K + 3, dtype=dev(src).dtype, device="cuda")
    view = buf[3:].view(rows, K)                       # rows at odd addresses
    view.copy_(dev(src))
    codes, pad = hp.unpack_matrix(hp.words_u32(B.apnn_pack(view, bits, enc)), rows, K, bits)
    assert np.array_equal(codes, hp.pm1_to_bits(src) if enc == P else src) and pad == 0


@pytest.mark.parametrize("bits,enc", [(1, P), (2, U), (5, U)])
@pytest.mark.parametrize("N,C,H,W", [(2, 96, 27, 31), (1, 32, 1, 5), (1, 33, 1, 3), (3, 64, 5, 13), (1, 512, 17, 1), (40, 32, 65, 61)])
def test_pack_nchw_of_any_frame(N, C, H, W, bits, enc):
    nchw = wl.fair_signs(11, (N, C, H, W)) if enc == P else wl.uniform_codes(11, (N, C, H, W), bits)
    words = hp.words_u32(B.apnn_pack_fmap(dev(nchw), B.LAYOUT_NCHW, bits, enc))
    codes, pad = hp.unpack_fmap(words, N, H, W, C, bits)
    assert np.array_equal(codes, hp.pm1_to_bits(nchw) if enc == P else nchw) and pad == 0


@pytest.mark.parametrize("rows,K", [(3, 255), (2, 257), (2100, 513), (2050, 2049)])
@pytest.mark.parametrize("bits,step", [(2, 0.5), (8, 2.0 ** -7), (3, 0.7), (8, 1.0 / 3)])
def test_quantize_steps_and_segments(bits, step, rows, K):
    x = wl.normals(12, (rows, K), 1.0, 1.5)
    # values on and next to the boundaries of the codes
    edge = np.float32(-1.0) + np.float32(step) * np.arange(1, min(K, 1 << bits), dtype=np.float32)
    x[0, :edge.size] = edge
    x[1, :edge.size] = np.nextafter(edge, np.float32(-100.0))
    codes, pad = hp.unpack_matrix(hp.words_u32(B.apnn_quantize(dev(x), -1.0, step, bits)), rows, K, bits)
    assert np.array_equal(codes, oracle.quantize(x, -1.0, step, bits)) and pad == 0


@pytest.mark.parametrize("K", [260, 2048])
@pytest.mark.parametrize("zero,step", [(-1.0, 0.25), (0.5, 0.3), (0.0, 2.0 ** 100), (0.0, 3e-30)])
def test_quantize_of_infinities_nan_and_the_ends_of_the_range(zero, step, K):
    special = np.array([np.inf, -np.inf, np.nan, 3.4e38, -3.4e38, 1e-45, -1e-45, 0.0, -0.0], dtype=np.float32)
    x = np.resize(special, (2050, K))
    codes, pad = hp.unpack_matrix(hp.words_u32(B.apnn_quantize(dev(x), zero, step, 5)), 2050, K, 5)
    assert np.array_equal(codes, oracle.quantize(x, zero, step, 5)) and pad == 0


@pytest.mark.parametrize("bits,step", [(2, 0.5), (3, 0.7), (8, 1.0 / 3)])
@pytest.mark.parametrize("rows,K", [(1, 1), (3, 3), (7, 4), (5, 31), (9, 97), (33, 127), (6, 128), (8192, 5), (8195, 126), (32768, 2),
                                    (32783, 128), (2100, 700), (2050, 3001)])
def test_quantize_rows_that_share_a_wave_and_segments_partly_filled(bits, step, rows, K):
    """Rows of at most 128 values, two, four and sixteen to a wave, and the partial last wave; last segments of every width."""
    x = wl.normals(13, (rows, K), 1.0, 1.5)
    x[x < 0] = 0.0                                      # as a rectifier leaves them
    x[rows // 2] *= 1e6
    codes, pad = hp.unpack_matrix(hp.words_u32(B.apnn_quantize(dev(x), 0.0, step, bits)), rows, K, bits)
    assert np.array_equal(codes, oracle.quantize(x, 0.0, step, bits)) and pad == 0


@pytest.mark.parametrize("N,C,H,W,bits", [
    (40, 96, 65, 61, 2), (40, 96, 65, 61, 5),           # 256 pixels a block, several words a pixel
    (128, 1504, 2, 255, 1), (128, 1536, 2, 255, 1),     # 47 words a pixel: the last that 256 records leave room for; 48: 64 pixels
    (1, 768, 9, 8, 8), (2, 800, 9, 8, 8),               # 192, 200 words a pixel: the byte-by-byte kernel (191 at most fit)
    (1, 760, 9, 8, 7),                                  # 168
])
def test_pack_nchw_records_at_the_limits_of_a_block(N, C, H, W, bits):
    nchw = wl.uniform_codes(14, (N, C, H, W), bits)
    codes, pad = hp.unpack_fmap(hp.words_u32(B.apnn_pack_fmap(dev(nchw), B.LAYOUT_NCHW, bits, U)), N, H, W, C, bits)
    assert np.array_equal(codes, nchw) and pad == 0


def test_pack_nchw_of_more_frames_than_a_grid_has_blocks():
    """A launch has less than 2^32 threads: 2^24 blocks of 256."""
    src = torch.randint(0, 4, ((1 << 24) + 3, 1, 1, 5), dtype=torch.uint8, device="cuda")
    words = B.apnn_pack_fmap(src, B.LAYOUT_NCHW, 2, U).view(-1, 2)
    assert torch.equal(words[:, 0] + 2 * words[:, 1], src.view(-1).int())


@pytest.mark.parametrize("step", [2.0 ** 127, 2.0 ** 126, 2.0 ** -126, 1e-39, 1.3e38, 3e-38])
@pytest.mark.parametrize("rows,K", [(3, 40), (2, 300)])
def test_quantize_steps_whose_reciprocal_leaves_the_range(step, rows, K):
    """Reciprocals below 2^-126 or above 2^126 are not used: the kernel that divides takes those steps."""
    with np.errstate(over="ignore"):                    # (codes 0 .. 7 and beyond, or infinity)
        x = np.resize(np.float32(step) * np.arange(-1, 9, dtype=np.float32) / 2, (rows, K))
    x[:, ::7] = np.array([3.4e38, -3.4e38, 1e-45, 0.0, np.inf, -np.inf, np.nan], np.float32)[np.arange(x[:, ::7].shape[1]) % 7]
    codes, pad = hp.unpack_matrix(hp.words_u32(B.apnn_quantize(dev(x), 0.0, step, 3)), rows, K, 3)
    assert np.array_equal(codes, oracle.quantize(x, 0.0, step, 3)) and pad == 0


@pytest.mark.parametrize("call", ["pack", "quantize", "maxpool"])
def test_more_words_than_a_launch_has_threads(call):
    """2^32 words and a few: more than one launch."""
    n = (1 << 30) + 5
    if call == "maxpool":                               # one-pixel frames of one channel word
        x = torch.arange(n, dtype=torch.int32, device="cuda").repeat(4)
        out = B.apnn_maxpool(x, 4 * n, 1, 1, 32, 1, 1, 1, 0)
        assert torch.equal(out, x)
    else:                                               # rows of one value: four words each
        x = torch.randint(0, 2, (n, 1), dtype=torch.uint8, device="cuda")
        out = B.apnn_pack(x, 1, U) if call == "pack" else B.apnn_quantize(x.float(), 0.0, 1.0, 1)
        assert torch.equal(out.view(n, 4)[:, 0], x.view(-1).int()) and not out.view(n, 4)[:, 1:].any()
    del x, out
    torch.cuda.empty_cache()
