"""Grouped GEMMs with few rows an expert (their own tiles up to a mean of 32 rows): group sizes at the edges of the
32- and 64-row tiles, empty groups, more experts than one wave counts at once, rows beyond the last group, widths
that are no multiple of a tile.  Every output element is the same sequence of operations as in the large tiles, so
the results must equal those bit for bit; the large tiles are what the oracle tests check."""
import numpy as np
import pytest
import torch

from tests._gpu_util import announce, dev

pytestmark = pytest.mark.gpu

GROUPS = {
    "one_row": [1],
    "edges32": [0, 1, 31, 32, 33, 0, 2, 15, 0, 0, 1],
    "edges64": [63, 64, 65, 0, 1, 20, 33, 31, 0],
    "129_experts": [i % 5 * 3 for i in range(129)],
    "last_only": [0] * 70 + [200],
    "empty": [0, 0, 0],
}
# group sizes, N (SwiGLU: output columns), K
PLAIN = [("one_row", 8, 128), ("edges32", 1000, 640), ("edges64", 132, 896), ("129_experts", 256, 256), ("129_experts", 896, 384),
         ("last_only", 390, 384), ("empty", 128, 128)]
SWIGLU = [("one_row", 128, 128), ("edges32", 384, 640), ("edges64", 256, 896), ("129_experts", 128, 256), ("last_only", 256, 384)]


def _inputs(sizes, n, k, pow2, extra, special=False):
    rng = np.random.default_rng(len(sizes) + n + k + pow2)
    g, m = len(sizes), sum(sizes) + extra
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)

    def codes(*shape):
        return (rng.integers(0, 0x7F, shape) | (rng.integers(0, 2, shape) << 7)).astype(np.uint8)

    def scales(lo, *shape):
        if pow2:
            return np.ldexp(1.0, rng.integers(lo, lo + 4, shape)).astype(np.float32)
        return (np.exp(0.5 * rng.standard_normal(shape)) * 2.0 ** lo).astype(np.float32)

    kb = k // 128
    a, sa, b, sb = codes(m, k), scales(-11, m, kb), codes(g, n, k), scales(-10, g, (n + 127) // 128, kb)
    if special:                                            # NaN codes; with FP32 scales also zero, infinity and NaN
        a[m // 2, k - 1], b[g // 2, n // 3, 7] = 0x7F, 0xFF
        if not pow2:
            sa[0, kb // 2], sa[m // 3, 0], sa[2 * m // 3, kb - 1], sb[g - 1, -1, 0] = 0.0, np.inf, np.nan, 0.0
    return (dev(a), dev(np.ascontiguousarray(sa.T)).t(), dev(off), dev(b), dev(sb)), m, int(off[-1])


def _bits(t):
    """The values as whole numbers, so that a NaN equals the same NaN."""
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("out", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("name,n,k", PLAIN)
def test_plain(ds3, name, n, k, out, pow2):
    announce(f"few rows an expert: {name} n={n} k={k} {out} pow2={pow2}")
    args, m, used = _inputs(GROUPS[name], n, k, pow2, 3)
    fn = ds3.ds3_grouped_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_grouped_gemm_fp8_bs
    got = torch.full((m + 1, (n + 11) // 4 * 4), 7.0, dtype=out, device="cuda:0")
    fn(*args, c=got[:m, :n])
    want = fn(*args, out_dtype=out, variant=0)
    assert torch.equal(got[:used, :n], want[:used])
    assert torch.all(got[used:] == 7.0) and torch.all(got[:, n:] == 7.0), "wrote beyond the groups"
    assert torch.equal(fn(args[0], args[1].contiguous(), *args[2:], out_dtype=out)[:used], want[:used])   # row-major scales


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("k_major", [False, True])
@pytest.mark.parametrize("name,inter,k", SWIGLU)
def test_swiglu_quant(ds3, name, inter, k, k_major, pow2):
    announce(f"few rows an expert, SwiGLU: {name} inter={inter} k={k} k_major={k_major} pow2={pow2}")
    (a, sa, off, b, sb), m, used = _inputs(GROUPS[name], 2 * inter, k, pow2, 2)
    g = b.shape[0]
    fused = ds3.ds3_grouped_gemm_swiglu_quant_fp8_bs_pow2 if pow2 else ds3.ds3_grouped_gemm_swiglu_quant_fp8_bs
    gemm = ds3.ds3_grouped_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_grouped_gemm_fp8_bs
    cast = ds3.ds3_swiglu_quant_1x128_pow2 if pow2 else ds3.ds3_swiglu_quant_1x128
    q, s = fused(a, sa, off, b, sb, k_major_scales=k_major)
    # the interleaved blocks in gate | up order, through the large tiles and the unfused cast
    order = lambda t, r: t.view(g, inter // 128, 2, r, -1).transpose(1, 2).reshape(t.shape).contiguous()
    h = gemm(a, sa, off, order(b, 128), order(sb, 1), variant=0)
    q2, s2 = cast(h[:used].contiguous())
    assert torch.equal(q[:used], q2) and torch.equal(s[:used], s2)
    q, s = fused(a, sa.contiguous(), off, b, sb, k_major_scales=k_major)                                  # row-major scales
    assert torch.equal(q[:used], q2) and torch.equal(s[:used], s2)


@pytest.mark.parametrize("pow2", [False, True])
@pytest.mark.parametrize("name", ["edges32", "edges64"])
def test_special_values(ds3, name, pow2):
    announce(f"few rows an expert, special values: {name} pow2={pow2}")
    n, k = 512, 640
    (a, sa, off, b, sb), m, used = _inputs(GROUPS[name], n, k, pow2, 2, special=True)
    g = b.shape[0]
    gemm = ds3.ds3_grouped_gemm_fp8_bs_pow2 if pow2 else ds3.ds3_grouped_gemm_fp8_bs
    for out in (torch.bfloat16, torch.float32):
        got, want = gemm(a, sa, off, b, sb, out_dtype=out)[:used], gemm(a, sa, off, b, sb, out_dtype=out, variant=0)[:used]
        assert torch.isnan(want).any() and torch.equal(_bits(got), _bits(want))
    fused = ds3.ds3_grouped_gemm_swiglu_quant_fp8_bs_pow2 if pow2 else ds3.ds3_grouped_gemm_swiglu_quant_fp8_bs
    q, s = fused(a, sa, off, b, sb)
    order = lambda t, r: t.view(g, n // 256, 2, r, -1).transpose(1, 2).reshape(t.shape).contiguous()
    h = gemm(a, sa, off, order(b, 128), order(sb, 1), variant=0)
    q2, s2 = (ds3.ds3_swiglu_quant_1x128_pow2 if pow2 else ds3.ds3_swiglu_quant_1x128)(h[:used].contiguous())
    assert torch.equal(q[:used], q2) and torch.equal(_bits(s[:used]), _bits(s2))
