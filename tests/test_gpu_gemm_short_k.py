"""The GEMM for a short K and a large output: every number of K-steps, ranges of 32-row steps of unequal length and with
a ragged end, column tiles and 16-byte chunks of a row cut anywhere, both scale modes and kinds, both output types.  Codes
are small integers and scales powers of two, so the FP32 output must equal the oracle bit for bit (BF16: its rounding);
with any scales it must equal the main kernel's, whose operations these are."""
import numpy as np
import pytest
import torch

from oracle import ds3_oracle as orc
from tests._gpu_util import announce, dev, host

pytestmark = pytest.mark.gpu

TABLE = np.array([0x00, 0x38, 0x40, 0xB8, 0xC0, 0x80], dtype=np.uint8)   # 0, 1, 2, -1, -2, -0

SHAPES = [
    (1025, 4101, 128), (2049, 4162, 256), (1000, 8195, 384), (1056, 4100, 512), (4127, 1799, 512), (8191, 577, 384),
    (65, 66001, 512), (300, 40007, 256), (3001, 1415, 128),
]


def _case(shape, per_row, seed):
    m, n, k = shape
    rng = np.random.default_rng(seed)
    a, b = TABLE[rng.integers(0, 6, (m, k))], TABLE[rng.integers(0, 6, (n, k))]
    sa = np.ldexp(1.0, rng.integers(-2, 2, (m, k // 128))).astype(np.float32)
    sb = np.ldexp(1.0, rng.integers(-1, 3, (n if per_row else (n + 127) // 128, k // 128))).astype(np.float32)
    return rng, a, b, sa, sb


def _padded(x, ld):
    buf = torch.zeros((x.shape[0], ld), dtype=torch.uint8, device="cuda:0")
    buf[:, : x.shape[1]] = dev(x)
    return buf[:, : x.shape[1]]


def _reference(a, sa, b, sb, per_row):
    """The oracle's product, by FP32 arithmetic that is exact here (integers below 2^24 times a power of two)."""
    ad = orc.dequant_rows(a, sa).astype(np.float32)
    bd = (orc.dequant_rows(b, sb) if per_row else orc.dequant_blocks(b, sb)).astype(np.float32)
    return (torch.from_numpy(ad) @ torch.from_numpy(bd).t()).numpy()


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_short_k_exact(ds3, shape, per_row, pow2):
    m, n, k = shape
    mode = ds3.DS3_BSCALE_PER_ROW if per_row else ds3.DS3_BSCALE_128x128
    assert ds3._L().ds3_gemm_short_k(m, n, k, mode, 256) == 1
    rng, a, b, sa, sb = _case(shape, per_row, m * 7 + n * 3 + k + per_row + 2 * pow2)
    lda, ldb, ldc = k + 16 * int(rng.integers(0, 3)), k + 16 * int(rng.integers(0, 3)), (n + 3) // 4 * 4 + 4 * int(rng.integers(0, 3))
    announce(f"short K {m}x{n}x{k} per_row={per_row} pow2={pow2} ld=({lda},{ldb},{ldc})")
    ref = _reference(a, sa, b, sb, per_row)
    fn = ds3.ds3_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_gemm_fp8_bs
    args = (_padded(a, lda), dev(np.ascontiguousarray(sa.T)).t(), _padded(b, ldb), dev(sb))
    want = dev(ref)
    for accumulate in (False, True):
        cbuf = torch.full((m + 1, ldc), 7.0, dtype=torch.float32, device="cuda:0")
        cbuf[:m, :n] = -3.0
        fn(*args, sb_mode=mode, c=cbuf[:m, :n], accumulate=accumulate)
        assert torch.equal(cbuf[:m, :n], want - 3.0 if accumulate else want), (shape, accumulate)
        assert torch.all(cbuf[:, n:] == 7.0) and torch.all(cbuf[m:] == 7.0), "wrote beyond the output"
    cbuf = torch.full((m + 1, ldc), 7.0, dtype=torch.bfloat16, device="cuda:0")
    fn(*args, sb_mode=mode, c=cbuf[:m, :n])
    assert torch.equal(cbuf[:m, :n], want.bfloat16())
    assert torch.all(cbuf[:, n:] == 7.0) and torch.all(cbuf[m:] == 7.0), "wrote beyond the output"
    # row-major activation scales, K-block-major weight scales
    got = fn(args[0], dev(sa), args[2], dev(np.ascontiguousarray(sb.T)).t(), sb_mode=mode, out_dtype=torch.float32)
    assert torch.equal(got, want)


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("shape", [(1056, 4100, 512), (2049, 4162, 256), (3001, 1415, 128)])
def test_short_k_equals_the_main_kernel(ds3, shape, per_row, pow2):
    """Any codes and scales, NaN codes, and (FP32 scales) scales of zero, infinity and NaN among them."""
    m, n, k = shape
    announce(f"short K against the main kernel {m}x{n}x{k} per_row={per_row} pow2={pow2}")
    rng, a, b, sa, sb = _case(shape, per_row, m + n + k)
    a, b = rng.integers(0, 0x7F, (m, k)).astype(np.uint8), rng.integers(0x80, 0xFF, (n, k)).astype(np.uint8)
    a[m // 3, k - 1], b[n // 2, 5] = 0x7F, 0xFF
    if not pow2:
        sa, sb = (t * np.exp(rng.standard_normal(t.shape)).astype(np.float32) for t in (sa, sb))
        for t, vals in ((sa, (0.0, np.inf, np.nan)), (sb, (0.0, -np.inf))):
            for v in vals:
                t[rng.integers(0, t.shape[0]), rng.integers(0, t.shape[1])] = v
    fn = ds3.ds3_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_gemm_fp8_bs
    args = (dev(a), dev(np.ascontiguousarray(sa.T)).t(), dev(b), dev(sb))
    kw = dict(sb_mode=ds3.DS3_BSCALE_PER_ROW if per_row else ds3.DS3_BSCALE_128x128)
    for out in (torch.float32, torch.bfloat16):
        got, want = host(fn(*args, out_dtype=out, **kw)), host(fn(*args, out_dtype=out, variant=2, workspace=None, **kw))
        assert np.isnan(want).any() and np.array_equal(got, want, equal_nan=True)
