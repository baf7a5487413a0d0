"""The GEMM for few rows or few tiles: shapes at the edges of its tiles and of its split of K (K-steps that
do not divide among the wave groups, fewer K-steps than groups or stages), both scale modes and kinds, both
output types.  Codes are small integers and scales powers of two, so every order of summation is exact and
the FP32 output must equal the oracle bit for bit (BF16: its rounding)."""
import numpy as np
import pytest
import torch

from oracle import ds3_oracle as orc
from tests._gpu_util import announce, dev, host

pytestmark = pytest.mark.gpu

TABLE = np.array([0x00, 0x38, 0x40, 0xB8, 0xC0, 0x80], dtype=np.uint8)   # 0, 1, 2, -1, -2, -0

SHAPES = [
    (1, 1, 128), (1, 64, 256), (15, 31, 384), (16, 33, 640), (17, 96, 1152), (31, 32, 128), (32, 130, 2048),
    (33, 129, 896), (63, 4100, 512), (64, 8200, 384), (65, 257, 128), (129, 1000, 1408), (64, 18433, 256),
    (500, 2049, 384), (1000, 3001, 512), (2049, 65, 768), (1900, 1700, 256),
    # K split in four: K-step counts of every remainder (23, 24, 33, 26)
    (17, 130, 2944), (17, 130, 3072), (33, 96, 4224), (9, 130, 3328),
    # a decode batch's rows, wide layers
    (32, 18432, 1152), (31, 16500, 640), (1, 16461, 128), (20, 18435, 1024),
    # 128 weight rows, K split in two: more weight rows than one tile a compute unit takes, or a short K; K-steps of both
    # parities, fewer and more than the three stages hold
    (32, 24600, 1152), (17, 28675, 896), (31, 16500, 512), (9, 32700, 1664), (1, 24577, 384),
    # 64-row tiles whose ring of stages wraps, K split in two and not at all
    (200, 3000, 1280), (1000, 3001, 1152),
]


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_skinny_exact(ds3, shape, per_row, pow2):
    m, n, k = shape
    rng = np.random.default_rng(m * 7 + n * 3 + k + per_row + 2 * pow2)
    lda, ldb, ldc = k + 16 * int(rng.integers(0, 3)), k + 16 * int(rng.integers(0, 3)), (n + 3) // 4 * 4 + 8
    announce(f"skinny {m}x{n}x{k} per_row={per_row} pow2={pow2} ld=({lda},{ldb},{ldc})")
    a, b = TABLE[rng.integers(0, 6, (m, k))], TABLE[rng.integers(0, 6, (n, k))]
    sa = np.ldexp(1.0, rng.integers(-2, 2, (m, k // 128))).astype(np.float32)
    sb = np.ldexp(1.0, rng.integers(-1, 3, (n if per_row else (n + 127) // 128, k // 128))).astype(np.float32)
    c0 = rng.integers(-8, 9, (m, n)).astype(np.float32)
    ref = orc.gemm_fp8_bs(a, sa, b, sb, sb_per_row=per_row, c_in=None)

    def padded(x, ld):
        buf = torch.zeros((x.shape[0], ld), dtype=torch.uint8, device="cuda:0")
        buf[:, :k] = dev(x)
        return buf[:, :k]

    fn = ds3.ds3_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_gemm_fp8_bs
    sa_kmajor = dev(np.ascontiguousarray(sa.T)).t()
    args = (padded(a, lda), sa_kmajor, padded(b, ldb), dev(sb))
    mode = ds3.DS3_BSCALE_PER_ROW if per_row else ds3.DS3_BSCALE_128x128
    for accumulate in (False, True):
        cbuf = torch.full((m, ldc), 7.0, dtype=torch.float32, device="cuda:0")
        c = cbuf[:, :n]
        c.copy_(dev(c0))
        fn(*args, sb_mode=mode, c=c, accumulate=accumulate)
        want = ref + c0 if accumulate else ref
        assert np.array_equal(host(c).astype(np.float64), want), (shape, accumulate)
        assert torch.all(cbuf[:, n:] == 7.0), "wrote beyond the row"
    cbuf = torch.full((m + 1, ldc), 7.0, dtype=torch.bfloat16, device="cuda:0")
    fn(*args, sb_mode=mode, c=cbuf[:m, :n])
    assert torch.equal(cbuf[:m, :n].cpu(), torch.from_numpy(ref).float().bfloat16())
    assert torch.all(cbuf[:, n:] == 7.0) and torch.all(cbuf[m:] == 7.0), "wrote beyond the output"
    # row-major activation scales, K-block-major weight scales
    got = fn(args[0], dev(sa), args[2], dev(np.ascontiguousarray(sb.T)).t(), sb_mode=mode, out_dtype=torch.float32)
    assert np.array_equal(host(got).astype(np.float64), ref)


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("shape", [(33, 96, 4224), (33, 129, 896), (31, 16500, 640), (200, 3000, 1280), (1000, 3001, 512),
                                   (32, 24600, 1152), (31, 16500, 512)])
def test_skinny_special_values(ds3, shape, per_row, pow2):
    """NaN codes, and (FP32 scales) scales of zero, infinity and NaN: what the main kernel makes of them.  Everything
    else is exact in any order of summation."""
    m, n, k = shape
    announce(f"skinny special values {m}x{n}x{k} per_row={per_row} pow2={pow2}")
    rng = np.random.default_rng(m + n + k)
    a, b = TABLE[rng.integers(0, 6, (m, k))], TABLE[rng.integers(0, 6, (n, k))]
    sa = np.ldexp(1.0, rng.integers(-2, 2, (m, k // 128))).astype(np.float32)
    sb = np.ldexp(1.0, rng.integers(-1, 3, (n if per_row else (n + 127) // 128, k // 128))).astype(np.float32)
    a[m // 3, k - 1], b[n // 2, 5] = 0x7F, 0xFF
    if not pow2:
        for t, vals in ((sa, (0.0, np.inf, np.nan)), (sb, (0.0, -np.inf))):
            for v in vals:
                t[rng.integers(0, t.shape[0]), rng.integers(0, t.shape[1])] = v
    fn = ds3.ds3_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_gemm_fp8_bs
    args = (dev(a), dev(np.ascontiguousarray(sa.T)).t(), dev(b), dev(sb))
    kw = dict(sb_mode=ds3.DS3_BSCALE_PER_ROW if per_row else ds3.DS3_BSCALE_128x128)
    for out in (torch.float32, torch.bfloat16):
        got, want = host(fn(*args, out_dtype=out, **kw)), host(fn(*args, out_dtype=out, variant=2, workspace=None, **kw))
        assert np.isnan(want).any() and np.array_equal(got, want, equal_nan=True)


# one tile of 48 to 112 weight rows a compute unit, up to 32, 64 and 128 activation rows: odd numbers of waves side by side,
# activation rows that are no whole loads of all waves, K-steps of both parities and fewer or more than the stages hold
ONE_TILE = [
    (32, 8200, 1664), (1, 12288, 640), (17, 12300, 896), (20, 12417, 1664), (31, 16384, 1024), (32, 16401, 768), (9, 20480, 1408),
    (32, 20500, 640), (5, 24575, 1152), (33, 8200, 1664), (64, 12285, 640), (40, 13000, 896), (64, 17003, 768), (50, 20480, 1152),
    (63, 24570, 896),
    (65, 16400, 1280), (128, 20480, 1664), (97, 20481, 1408), (128, 24570, 1280), (80, 24577, 1792), (127, 28672, 1280),
    (1000, 1500, 1152), (130, 9000, 1024), (513, 3499, 1408),      # 128x64 tiles, two groups of waves
]


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("shape", ONE_TILE)
def test_one_tile_a_compute_unit(ds3, shape, per_row, pow2):
    mode = ds3.DS3_BSCALE_PER_ROW if per_row else ds3.DS3_BSCALE_128x128
    config = ds3._L().ds3_gemm_few_tiles_config(*shape, mode, 256)
    assert config >= 5 or (config == 3 and 32 < shape[0] <= 64)      # (64 weight rows by up to 64: one of the ranked tiles)
    test_skinny_exact(ds3, shape, per_row, pow2)


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("shape", [(32, 8200, 1664), (9, 20480, 1408), (40, 13000, 896), (64, 17003, 768), (97, 20481, 1408),
                                   (1000, 1500, 1152)])
def test_one_tile_special_values(ds3, shape, per_row, pow2):
    test_skinny_special_values(ds3, shape, per_row, pow2)
