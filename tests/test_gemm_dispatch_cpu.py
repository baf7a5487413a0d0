"""Which kernel a GEMM call takes, by size (host logic, 256 compute units): the lines that were measured, from both
sides, and that every configuration of the kernel for few rows or few tiles is reached."""
import pytest

from tests import test_gpu_gemm_grouped_few_rows as grouped_tests
from tests import test_gpu_gemm_skinny as dense_tests

BLOCK, ROW = 0, 1


@pytest.mark.parametrize("mode", [BLOCK, ROW])
@pytest.mark.parametrize("shape,few", [
    ((1, 1, 128), True), ((64, 32768, 18432), True), ((64, 128, 128), True),            # up to 64 rows: any K
    ((512, 2048, 18432), True), ((8192, 128, 65536), True),                             # 128 tiles of 64 rows: any K
    ((513, 2048, 12288), True), ((1024, 2048, 12288), True),                            # up to 256 tiles
    ((513, 2048, 12416), False), ((1024, 2048, 12416), False), ((4096, 512, 14336), False),
    ((1025, 2048, 3072), True), ((2048, 1920, 256), True),                              # more: a short K
    ((1025, 2048, 4224), False), ((384, 7168, 7168), False), ((2048, 1536, 18432), False),
    ((1025, 2048, 128), False), ((512, 7168, 128), False),                              # ... of two K-steps and more
    ((2048, 2048, 1024), False), ((65, 32768, 1024), False),                            # 256 tiles of 128 x 128
])
def test_dense(ds3, shape, few, mode):
    assert (ds3._L().ds3_gemm_few_tiles_config(*shape, mode, 256) >= 0) == few


def test_dense_by_row_gives_up_earlier(ds3):
    f = ds3._L().ds3_gemm_few_tiles_config
    for k, block, row in ((3072, True, True), (3200, True, False), (4096, True, False), (4224, False, False)):
        assert (f(2048, 1536, k, BLOCK, 256) >= 0, f(2048, 1536, k, ROW, 256) >= 0) == (block, row), k


@pytest.mark.parametrize("call,tile", [
    # experts, rows, N, K, SwiGLU epilogue
    ((32, 128, 4096, 7168, 1), 32), ((32, 128, 7168, 2048, 0), 32), ((8, 32, 7168, 2048, 0), 32),   # decode batches
    ((32, 512, 1024, 1024, 1), 32), ((32, 513, 1024, 1024, 1), 64), ((32, 1024, 512, 1024, 0), 64), ((32, 1025, 512, 1024, 0), 0),
    ((32, 512, 4096, 7168, 1), 0), ((64, 1024, 4096, 7168, 1), 0), ((32, 1024, 7168, 2048, 0), 0),  # uneven loads could cost
    ((256, 4096, 4096, 7168, 1), 0), ((256, 1024, 7168, 2048, 0), 0), ((1023, 1023, 2048, 1024, 0), 0),
    ((4, 64, 4096, 7168, 1), 32), ((4, 65, 4096, 7168, 1), 0), ((4, 65, 4096, 4096, 1), 64),        # a long K: 32 rows, gate|up
    ((12, 20, 4096, 14336, 0), 0), ((12, 20, 4096, 4096, 0), 32),
    ((1023, 16368, 1 << 20, 128, 0), 0), ((1, 1, 1 << 30, 128, 0), 0),                              # more workgroups than a launch holds
])
def test_grouped(ds3, call, tile):
    assert ds3._L().ds3_grouped_gemm_few_rows_tile(*call, 256) == tile


def test_the_gpu_tests_reach_every_configuration(ds3):
    """The shapes that the kernel's own tests run, which name no variant: every configuration, its ring of stages wrapped."""
    for mode in (BLOCK, ROW):
        config = lambda shapes: [ds3._L().ds3_gemm_few_tiles_config(*shape, mode, 256) for shape in shapes]
        assert min(config(dense_tests.SHAPES)) >= 0
        assert set(config(dense_tests.SHAPES + dense_tests.ONE_TILE)) == set(range(17)) - {10}, mode       # (10 would be 3)
        steps = {c: [s[2] // 128 for s in dense_tests.SHAPES + dense_tests.ONE_TILE if config([s])[0] == c] for c in range(17)}
        # (steps of a stage, stages): each configuration's ring of stages wraps, and K-steps are left over where they are split
        split = {0: (4, 4), 1: (2, 4), 2: (2, 3), 3: (2, 4), 4: (1, 3), 5: (2, 5), 6: (2, 5), 7: (2, 4), 8: (1, 6), 9: (2, 4), 11: (2, 3),
                 12: (1, 5), 13: (1, 5), 14: (1, 4), 15: (1, 4), 16: (2, 3)}
        for c, (wk, ns) in split.items():
            assert any(-(-k // wk) > ns for k in steps[c]) and (wk == 1 or any(k % wk for k in steps[c])), (mode, c, steps[c])
    tile = ds3._L().ds3_grouped_gemm_few_rows_tile
    groups = grouped_tests.GROUPS
    plain = {tile(len(groups[g]), sum(groups[g]) + 3, n, k, 0, 256) for g, n, k in grouped_tests.PLAIN}
    swiglu = {tile(len(groups[g]), sum(groups[g]) + 2, 2 * inter, k, 1, 256) for g, inter, k in grouped_tests.SWIGLU}
    assert plain == swiglu == {32, 64}


@pytest.mark.parametrize("mode", [BLOCK, ROW])
@pytest.mark.parametrize("shape,short", [
    ((8192, 32768, 512), 1), ((8192, 32768, 640), 0), ((18432, 7168, 128), 1),          # K in registers
    ((768, 16384, 512), 1), ((767, 16384, 512), 0), ((767, 65536, 256), 1),             # few rows: more than a round of large tiles
    ((1025, 2048, 512), 0), ((64, 32768, 512), 0), ((1025, 2048, 128), 1),              # the kernel for few rows or tiles comes first
])
def test_short_k(ds3, shape, short, mode):
    assert ds3._L().ds3_gemm_short_k(*shape, mode, 256) == short


@pytest.mark.parametrize("shape,c_type,mode,tile", [
    ((8192, 1536, 7168), 1, 0, 2), ((8192, 1536, 7168), 0, 0, -1), ((8192, 1536, 7168), 1, 1, -1),     # 192 tiles of 256x256: 256 of 192x256, 258 of 256x192
    ((1536, 7168, 8192), 0, 1, 0), ((1536, 7168, 640), 0, 1, 0), ((1536, 7168, 512), 0, 1, -1),        # 168: 224 of 256x192; the short-K kernel's
    ((4096, 4096, 7168), 1, 0, -1), ((4096, 18432, 7168), 1, 0, -1),                                   # a full round and more
    ((8192, 576, 7168), 1, 0, 1), ((8192, 576, 1280), 0, 1, 1), ((8192, 576, 1152), 1, 0, -1),         # 320 of 128x128: 192 of 192x128
    ((8192, 512, 7168), 1, 0, -1), ((8192, 800, 7168), 1, 0, -1),                                      # one each; no such tile fits
    ((4096, 2304, 1536), 1, 0, 2), ((4096, 2304, 1536), 0, 0, 0), ((4096, 2304, 1152), 1, 0, -1),      # 576 of 128x128
    ((64, 32768, 7168), 1, 0, -1), ((0, 576, 7168), 1, 0, -1), ((8192, 576, 7100), 1, 0, -1),
])
def test_between_tile(ds3, shape, c_type, mode, tile):
    assert ds3._L().ds3_gemm_between_tile(*shape, mode, c_type, 0, 256) == tile


@pytest.mark.parametrize("shape,c_type,mode,tile", [
    ((8192, 576, 2304), 1, 0, 1), ((8192, 576, 2176), 1, 0, -1), ((8192, 576, 1280), 0, 1, 1),
    ((4096, 2304, 3072), 0, 1, 0), ((4096, 2304, 2944), 0, 1, -1), ((4096, 2304, 1280), 1, 0, 2), ((1536, 7168, 640), 0, 1, 0),
])
def test_between_tile_with_power_of_two_scales(ds3, shape, c_type, mode, tile):
    assert ds3._L().ds3_gemm_between_tile(*shape, mode, c_type, 1, 256) == tile


@pytest.mark.parametrize("mode", [BLOCK, ROW])
@pytest.mark.parametrize("shape,few", [
    ((128, 16385, 7168), True), ((128, 28672, 7168), True), ((65, 18432, 1280), True),          # one tile a compute unit
    ((128, 16385, 18432), True), ((128, 16384, 18432), False), ((128, 28673, 7168), False), ((129, 18432, 7168), False),
])
def test_dense_one_tile_a_compute_unit(ds3, shape, few, mode):
    assert (ds3._L().ds3_gemm_few_tiles_config(*shape, mode, 256) >= 0) == few


@pytest.mark.parametrize("shape,c_type,mode,pow2,shared", [
    ((2048, 2048, 4096), 1, 0, 0, 1), ((2048, 2048, 3840), 1, 0, 0, 0),                # 256 tiles of 128x128: 16 of 32 K-steps saved, 15 of 30
    ((2048, 1152, 6144), 0, 1, 0, 1), ((2048, 1152, 4224), 1, 0, 0, 0),                # 144: 24 of 48, 11 of 33
    ((1024, 1152, 12800), 1, 0, 0, 1), ((1024, 1152, 15232), 1, 0, 0, 0),              # 72: 50 of 100, 17 of 119 (long runs)
    ((1228, 3404, 1152), 1, 0, 0, 0), ((2048, 2176, 2176), 1, 0, 1, 0),                # more than compute units
    ((2000, 9100, 2048), 0, 1, 0, 1), ((2000, 9100, 1920), 0, 1, 0, 0),                # 288 of 256x256: 8 and 7
    ((3072, 3072, 1536), 0, 1, 1, 1), ((3072, 3072, 1408), 0, 1, 1, 0),                # 576 of 128x128: 6 and 5
    ((4096, 4096, 7168), 1, 0, 0, 0), ((4096, 18432, 7168), 1, 0, 0, 0),               # no tail; half of the workgroups
    ((1333, 3000, 1536), 0, 0, 0, 0), ((8192, 32768, 512), 1, 0, 0, 0), ((32, 18432, 7168), 1, 0, 0, 0),   # other kernels
    ((0, 2048, 6144), 1, 0, 0, 0), ((2048, 2048, 6100), 1, 0, 0, 0),
])
def test_tail_shared(ds3, shape, c_type, mode, pow2, shared):
    assert ds3._L().ds3_gemm_tail_shared(*shape, mode, c_type, 0, pow2, 256) == shared


SHORT_K = 16


@pytest.mark.parametrize("mode", [BLOCK, ROW])
@pytest.mark.parametrize("shape,store,accumulate", [
    ((15489, 16763, 128), True, False), ((15489, 16764, 128), True, True),             # cut columns and a large output
    ((2391, 16379, 512), True, False), ((2390, 16379, 512), True, True),               # three columns of a piece, 7 * 2^24 in all
    ((2391, 16377, 512), True, True), ((7172, 16377, 512), True, False),               # one
    ((885, 15512, 512), False, True), ((885, 15360, 512), True, True), ((885, 15512, 256), True, True),    # 61 and 60 column tiles
    ((885, 8192, 512), True, True), ((770, 15512, 384), False, True), ((770, 10648, 384), True, True),     # 32; 5.7 and 3.9 MiB
    ((866, 8320, 512), False, True), ((866, 8321, 512), True, True), ((896, 8192, 512), True, True),       # 33 column tiles: 4.1 MiB
    ((1400, 4104, 384), False, True), ((1400, 4096, 384), True, True), ((2048, 3080, 512), False, True),   # 17: 1.503; 16; 13: 1.504
    ((2048, 3064, 512), True, True), ((1152, 6152, 256), False, True), ((2048, 4104, 384), True, True),    # 12; 25: 1.502; 528 of 128x128
])
def test_short_k_leaves_to_the_main_kernel(ds3, shape, store, accumulate, mode):
    f = lambda acc: ds3._L().ds3_gemm_default_kernel(*shape, mode, 0, acc, 0, 256)
    assert (f(0) == SHORT_K, f(1) == SHORT_K) == (store, accumulate)
    assert ds3._L().ds3_gemm_short_k(*shape, mode, 256) == store


@pytest.mark.parametrize("mode", [BLOCK, ROW])
@pytest.mark.parametrize("shape,tile,accumulating", [
    ((2305, 3585, 2944), 0, -1), ((2305, 3585, 3072), 0, 0), ((2305, 3588, 2944), 0, 0),      # more than two 128x128 tiles a unit
    ((2561, 3841, 640), 0, 0), ((2050, 2001, 2432), 1, 1),        # the other tiles lose nothing by it
])
def test_between_tile_of_an_accumulating_call(ds3, shape, tile, accumulating, mode):
    f = lambda acc: ds3._L().ds3_gemm_default_kernel(*shape, mode, 0, acc, 0, 256)
    assert (f(0), f(1)) == (8 + tile, 2 if accumulating < 0 else 8 + accumulating)
