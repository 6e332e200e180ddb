"""Which prefill launches take wide tiles (256 expert rows), by the library's host-only query."""
import pytest

moe = pytest.importorskip("paper_2606_10493_amd")

DEEPSEEK_V3 = (7168, 2048, 256, 8)


def _rows(dims, t):
    return moe.moe_prefill_tile_rows(moe.MoeDims(*dims), t)


@pytest.mark.parametrize("dims,t", [
    ((4096, 1536, 16, 2), 1023), ((4096, 1536, 16, 2), 1750), ((4096, 4096, 8, 2), 512), ((4096, 4096, 8, 2), 1750),
    ((4096, 2048, 32, 4), 1023), ((8192, 1024, 32, 4), 1023), ((4096, 512, 64, 4), 2500), ((7168, 2048, 32, 8), 512),
    ((3072, 1536, 64, 6), 1500), ((2048, 1024, 128, 8), 2048), ((7168, 2048, 64, 8), 1023),
])
def test_few_tiles_per_cu_stay_narrow(dims, t):
    """Up to two tiles per CU: wide ones took 1.05 to 1.33 times the time there under Zipf routing."""
    assert _rows(dims, t) == 128


@pytest.mark.parametrize("dims,t", [
    (DEEPSEEK_V3, 4096), (DEEPSEEK_V3, 8192), ((7168, 2048, 64, 8), 2048), ((4096, 1536, 16, 2), 8192),
    ((2048, 1024, 64, 8), 4096), ((4096, 4096, 8, 2), 3500), ((8192, 1024, 32, 4), 5000), ((4096, 512, 64, 4), 8192),
])
def test_many_rows_are_wide(dims, t):
    assert _rows(dims, t) == 256


def test_few_rows_per_expert_stay_narrow():
    assert [_rows(DEEPSEEK_V3, t) for t in (1, 1023, 3072)] == [128] * 3


def test_shapes_without_wide_tiles():
    """K in whole windows of four 128-blocks up to 8192, offsets of 32 bits."""
    assert _rows((2048, 768, 128, 8), 16384) == 128         # I is no multiple of 512
    assert _rows((7424, 2048, 256, 8), 16384) == 128        # nor H
    assert _rows((8192, 8192, 8, 2), 8192) == 256
    assert _rows((8704, 2048, 8, 2), 8192) == 128 and _rows((2048, 8704, 8, 2), 8192) == 128
    assert _rows((8192, 2048, 8, 2), (1 << 19) - 1) == 256  # T * H below 2^32
    assert _rows((8192, 2048, 8, 2), 1 << 19) == 128


def test_query_of_dims_that_the_regime_does_not_take():
    for dims in ((0, 512, 8, 2), (512, 0, 8, 2), (384, 512, 8, 2), (512, 500, 8, 2), (512, 512, 0, 2), (512, 512, 8, 0),
                 (65536, 512, 8, 2)):
        assert _rows(dims, 4096) == 0
    assert _rows(DEEPSEEK_V3, -1) == 0
    assert _rows(DEEPSEEK_V3, 1 << 28) == 0  # 2^31 slots
    assert _rows(DEEPSEEK_V3, 0) == 128
