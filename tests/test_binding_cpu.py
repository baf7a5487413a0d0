"""The native marshalling of the calls, as far as it goes without a GPU: a wrong argument is a Python exception, and
the interpreter goes on."""
import pytest
import torch


@pytest.mark.parametrize("which", ["sa", "sb"])
@pytest.mark.parametrize("pow2", [False, True])
def test_scales_without_two_strides(ds3, which, pow2):
    codes = torch.zeros((128, 128), dtype=torch.uint8)
    scales = {"sa": torch.ones((128, 1)), "sb": torch.ones((1, 1))}
    gemm = ds3.ds3_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_gemm_fp8_bs
    for bad in (scales[which][:, 0], scales[which][0, 0]):
        s = dict(scales, **{which: bad})
        with pytest.raises(IndexError):
            gemm(codes, s["sa"], codes, s["sb"])
