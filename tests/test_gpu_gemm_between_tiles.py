"""Tiles between the named configurations' sizes (192 rows or columns): one output element's operations are the main
kernel's, so a default call must equal a named variant without a workspace bit for bit -- NaN codes and any scales among
them, numbers of K-steps with every remainder of the stage ring, ragged last tiles, padded rows, both scale modes, kinds
and output types, with and without accumulation."""
import numpy as np
import pytest
import torch

from tests._gpu_util import announce, dev

pytestmark = pytest.mark.gpu

# (BF16 output with block scales, other calls): the tile each takes; 0: 256 weight rows x 192, 1: 192 x 128, 2: 192 x 256
CASES = [
    ((2561, 3841, 640), 2, 0), ((2817, 4095, 768), 0, 0),        # 176 and 192 tiles of 256x256
    ((2200, 2300, 2304), 1, 1), ((2050, 2001, 2432), 1, 1), ((130, 16500, 2560), 1, 1),   # more than one 128x128 tile a unit
    ((2305, 3585, 3072), 2, 0), ((2305, 3585, 3200), 2, 0),      # more than two
]


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("shape,bf16_tile,other_tile", CASES)
def test_between_tiles_equal_the_main_kernel(ds3, shape, bf16_tile, other_tile, per_row, pow2):
    m, n, k = shape
    mode = ds3.DS3_BSCALE_PER_ROW if per_row else ds3.DS3_BSCALE_128x128
    announce(f"between tiles {m}x{n}x{k} per_row={per_row} pow2={pow2}")
    for ct in (ds3.DS3_F32, ds3.DS3_BF16):
        want = bf16_tile if ct == ds3.DS3_BF16 and not per_row else other_tile
        assert ds3._L().ds3_gemm_between_tile(m, n, k, mode, ct, int(pow2), 256) == want
    rng = np.random.default_rng(m + n + k + per_row)
    lda, ldb = k + 16 * int(rng.integers(0, 3)), k + 16 * int(rng.integers(0, 3))
    a, b = rng.integers(0, 0x7F, (m, lda)).astype(np.uint8), rng.integers(0x80, 0xFF, (n, ldb)).astype(np.uint8)
    a[m // 3, k - 1], b[n // 2, 5] = 0x7F, 0xFF                  # NaN
    kb = k // 128
    exps = lambda r: np.ldexp(1.0, rng.integers(-3, 3, (r, kb))).astype(np.float32)
    sa, sb = exps(m), exps(n if per_row else (n + 127) // 128)
    if not pow2:
        sa, sb = (t * np.exp(rng.standard_normal(t.shape)).astype(np.float32) for t in (sa, sb))
    fn = ds3.ds3_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_gemm_fp8_bs
    args = (dev(a)[:, :k], dev(np.ascontiguousarray(sa.T)).t(), dev(b)[:, :k], dev(sb))
    ldc = (n + 7) // 8 * 8 + 8
    for dtype, accumulate in ((torch.bfloat16, False), (torch.float32, False), (torch.float32, True)):
        got, want = (torch.full((m + 1, ldc), 7.0, dtype=dtype, device="cuda:0") for _ in range(2))
        fn(*args, sb_mode=mode, c=got[:m, :n], accumulate=accumulate)
        fn(*args, sb_mode=mode, c=want[:m, :n], accumulate=accumulate, variant=2, workspace=None)
        assert torch.isnan(want[:m, :n]).any()
        assert torch.equal(got.nan_to_num(nan=1e30), want.nan_to_num(nan=1e30)), (shape, dtype, accumulate)
    assert torch.all(got[:, n:] == 7.0) and torch.all(got[m:] == 7.0), "wrote beyond the output"


def test_between_tiles_of_a_workspace_call(ds3):
    """These tiles need no workspace; one that is too small for the shape's tile walk is refused all the same."""
    m, n, k = 8192, 576, 1280                                    # (320 tiles of 128x128: nothing the walk would share)
    assert ds3.ds3_gemm_workspace_bytes(2304, 2048, 1280) > 0    # 288 tiles: a walk that could share them
    a, sa = ds3.ds3_quant_act_1x128(torch.randn(2304, k, device="cuda:0"))
    b, sb = ds3.ds3_quant_w_128x128(torch.randn(2048, k, device="cuda:0"))
    assert ds3._L().ds3_gemm_between_tile(2304, 2048, k, 0, ds3.DS3_BF16, 0, 256) == 1
    assert ds3.ds3_gemm_workspace_bytes(m, n, k) == 0
    with pytest.raises(ds3.Ds3Error):
        ds3.ds3_gemm_fp8_bs(a, sa, b, sb, workspace=torch.zeros(16, dtype=torch.uint8, device="cuda:0"))
    assert torch.equal(ds3.ds3_gemm_fp8_bs(a, sa, b, sb), ds3.ds3_gemm_fp8_bs(a, sa, b, sb, workspace=None))
