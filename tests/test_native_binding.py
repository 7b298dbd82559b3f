"""Host side of the native call path: what it refuses before the library is called, and the library's own errors."""
import numpy as np
import pytest
import torch

from paper_2106_12169_amd import binding as B


def test_refuses_host_tensors_and_wrong_argument_types():
    x = torch.zeros((4, 64), dtype=torch.uint8)
    w = torch.zeros(64, dtype=torch.int32)
    with pytest.raises(AssertionError):
        B.apnn_pack(x, 2, B.ENC_UNSIGNED, out=w)
    with pytest.raises(AssertionError):
        B.apnn_gemm(w, w, 4, 4, 64, 1, 2, B.ENC_PM1, B.ENC_UNSIGNED, out=torch.zeros((4, 4), dtype=torch.int32))
    with pytest.raises(AssertionError):
        B.apnn_layer(B.Conv(1, 4, 4, 32, 32, 3, 3, 1, 1), w, w, q_out=2, scale=w, bias=w, out=w)
    with pytest.raises(TypeError):
        B.native().gemm(1, 2)
    with pytest.raises(TypeError):
        B.native().gemm(w.numpy(), None, 4, 4, 64, 1, 2, 1, 0, None)


@pytest.mark.parametrize("call", [B.apnn_layer, B.apnn_input_layer])
@pytest.mark.parametrize("out", [torch.zeros(4), "no tensor"])
def test_an_output_that_is_not_written_is_not_looked_at(call, out):
    with pytest.raises(RuntimeError):                            # the library's refusal of null pointers (or: no device)
        call(B.Conv(1, 4, 4, 32, 32), None, None, q_out=0, out=out)


@pytest.mark.parametrize("flag", [np.bool_(True), 1.0])
def test_a_flag_is_whatever_converts_to_an_integer(flag):
    with pytest.raises(RuntimeError):
        B.apnn_layer(B.Conv(1, 1, 1, 32, 32), None, None, is_gemm=flag)


def test_an_empty_product_takes_any_empty_output():
    with pytest.raises(RuntimeError):                            # (no device; or the library: null operands)
        B.apnn_gemm(None, None, 4, 4, 64, 1, 2, B.ENC_PM1, B.ENC_UNSIGNED, out=torch.empty((0, 4), dtype=torch.int32))


@pytest.mark.filterwarnings("ignore:The PyTorch API of nested tensors")
def test_a_tensor_without_sizes_is_refused():
    x = torch.nested.nested_tensor([torch.zeros(3), torch.zeros(5)])
    with pytest.raises(RuntimeError):
        B.apnn_quantize(x, 0.0, 1.0, 2, out=torch.zeros(8, dtype=torch.int32))


@pytest.mark.gpu
def test_library_errors_arrive_with_status_and_text():
    with pytest.raises(B.ApnnError) as e:
        B.native().layer(B.Conv(1, 4, 4, 33, 32, 3, 3, 1, 1), None, None, False, 2, None, None, None, 0, 0.0, None, None, None, 0)
    assert e.value.status == 1 and "multiple of 32" in str(e.value)
    chain = B.native().Chain()
    chain.maxpool(None, 1, 8, 8, 64, 2, 3, 2, 3, None)          # recorded as it is, refused when it runs: pad >= window
    assert len(chain) == 1
    with pytest.raises(B.ApnnError) as e:
        chain.run(None)
    assert e.value.status == 1 and "pad" in str(e.value)


@pytest.mark.gpu
def test_a_recorded_step_checks_its_tensors_in_every_pass():
    X = torch.full((8 * 8 * 2 * 2,), -1, dtype=torch.int32, device="cuda")
    out = torch.empty(0, dtype=torch.int32, device="cuda")      # no storage yet when the step is recorded
    chain = B.native().Chain()
    chain.maxpool(X, 1, 8, 8, 64, 2, 2, 2, 0, out)
    out.data = torch.zeros(4 * 4 * 2 * 2, dtype=torch.int32, device="cuda")
    chain.run(None)
    assert (out.cpu() == -1).all()
    out.zero_()
    good = X.data
    for bad in (good.cpu(), good.repeat_interleave(2)[::2]):     # the host's memory, every second word
        X.data = bad
        with pytest.raises(AssertionError):
            chain.run(None)
    X.data = good
    assert (out.cpu() == 0).all()                                # a refused pass enqueues nothing
    chain.run(None)
    assert (out.cpu() == -1).all()
