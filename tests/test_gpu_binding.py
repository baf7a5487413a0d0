"""The native marshalling of the calls: what it refuses, and how."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_refusals(ds3):
    x = torch.randn(128, 256, device="cuda:0", dtype=torch.bfloat16)
    q, s = ds3.ds3_quant_act_1x128(x)
    w, sw = ds3.ds3_quant_w_128x128(x)
    with pytest.raises(ValueError, match="x must be 2-D with contiguous rows"):
        ds3.ds3_quant_act_1x128(x[:, ::2])
    with pytest.raises(TypeError, match="unsupported dtype torch.float16"):
        ds3.ds3_quant_act_128x1(x.half())
    with pytest.raises(TypeError):
        ds3.ds3_quant_w_128x128([1.0])
    with pytest.raises(ValueError, match="disagree on K"):
        ds3.ds3_gemm_fp8_bs(q, s, w[:, :128], sw)
    with pytest.raises(TypeError, match="unsupported dtype torch.float16"):
        ds3.ds3_gemm_fp8_bs(q, s, w, sw, out_dtype=torch.float16)
    with pytest.raises(ds3.Ds3Error) as e:
        ds3.ds3_gemm_fp8_bs(q[:, 1:129], s, w[:, 1:129], sw)
    assert e.value.status == 3 and "ds3_gemm_fp8_bs_v" in str(e.value)
    for bad in (s[:, 0], s[0, 0]):                        # scales without two strides
        with pytest.raises(IndexError):
            ds3.ds3_gemm_fp8_bs(q, bad, w, sw)
        with pytest.raises(IndexError):
            ds3.ds3_gemm_fp8_bs(q, s, w, bad)
    with pytest.raises(RuntimeError):                     # no memory of its own behind the tensor: its pointer throws
        torch.vmap(lambda t: ds3.ds3_quant_act_1x128(t)[0])(x[None])
    with pytest.raises(ds3.Ds3Error):                     # a workspace below the counters' size
        ds3.ds3_gemm_fp8_bs(q, s, w, sw, workspace=torch.zeros(16, dtype=torch.uint8, device="cuda:0"))


def test_layouts_of_the_outputs(ds3):
    x = torch.randn(130, 200, device="cuda:0")
    q, s = ds3.ds3_quant_act_1x128(x)
    assert q.shape == (130, 200) and q.stride() == (208, 1) and s.shape == (130, 2) and s.stride() == (1, 130)
    assert ds3.ds3_quant_act_1x128(x, k_major_scales=False)[1].stride() == (2, 1)
    q, s = ds3.ds3_quant_act_128x1(x)
    assert q.shape == (200, 130) and q.stride() == (144, 1) and s.shape == (200, 2)
    empty = ds3.ds3_quant_act_1x128(x[:0])
    assert empty[0].shape == (0, 200) and empty[1].shape == (0, 2)
    a, sa = ds3.ds3_quant_act_1x128(x[:, :128])
    b, sb = ds3.ds3_quant_w_128x128(x[:77, :128])
    y = ds3.ds3_gemm_fp8_bs(a, sa, b, sb)
    assert y.shape == (130, 77) and y.stride() == (80, 1) and y.dtype == torch.bfloat16
    c = torch.zeros(130, 80, device="cuda:0")
    assert ds3.ds3_gemm_fp8_bs(a, sa, b, sb, c=c[:, :77]).data_ptr() == c.data_ptr() and torch.all(c[:, 77:] == 0)
