"""The tile that a linear layer's launch takes (a rule on its sizes, host
code): measured times under each tile family on 256 compute units."""
import pytest

from paper_2605_01060_amd import surge as S


# (M, N, K), us with 128-wide, 192-row and 256-row tiles (for N not a multiple
# of 256 the last 128 features are 128-wide in each)
MEASURED = [
    ((262_144, 768, 64), 85.1, 87.4, 81.5), ((262_144, 2304, 64), 243.4, 242.8, 229.0),
    ((13_579, 2304, 64), 17.2, 20.6, 19.5), ((30_000, 1024, 64), 17.3, 20.4, 19.7),
    ((262_144, 768, 256), 153.2, 145.6, 132.5), ((100_000, 2304, 256), 168.5, 161.6, 150.1),
    ((262_144, 3072, 128), 410.2, 392.2, 369.2), ((100_000, 1024, 384), 101.3, 99.1, 97.5),
    ((8192, 768, 256), 8.0, 10.2, 11.7), ((13_579, 512, 384), 9.8, 12.2, 14.3),
    ((75_000, 256, 4096), 231.9, 183.4, 213.9), ((40_000, 512, 4096), 211.3, 172.5, 188.3),
    ((6144, 2304, 768), 28.0, 37.7, 24.2), ((8192, 2304, 768), 35.6, 38.5, 44.0),
    ((10_000, 2304, 768), 42.5, 40.7, 44.7), ((13_579, 2304, 768), 56.8, 56.7, 48.8),
    ((8192, 768, 3072), 43.4, 57.7, 65.4), ((13_579, 768, 3072), 79.5, 64.2, 67.1),
    ((17_000, 768, 3072), 87.6, 120.0, 72.2), ((262_144, 768, 3072), 1300.8, 1148.5, 1032.9),
    # an odd number of 128 features
    ((140_000, 1152, 64), 67.2, 75.7, 71.4), ((55_000, 1152, 384), 68.1, 69.3, 69.8),
    ((55_000, 1152, 3072), 406.1, 398.4, 381.7), ((75_000, 1152, 3072), 568.4, 577.3, 525.0),
    ((20_781, 640, 3072), 97.2, 112.2, 117.4), ((55_000, 640, 3072), 254.9, 272.3, 244.3),
    ((55_000, 896, 768), 84.3, 91.9, 87.9), ((75_000, 640, 3072), 333.6, 400.0, 372.8),
    ((262_144, 384, 768), 201.2, 230.1, 212.0), ((100_000, 384, 1536), 151.4, 194.1, 178.5),
]


@pytest.mark.parametrize("shape,us128,us192,us256", MEASURED)
def test_tile_is_the_fastest_measured(shape, us128, us192, us256):
    best = min((us128, (128, 128)), (us192, (192, 256)), (us256, (256, 256)))[1]
    assert S.surge_op_linear_tile(*shape) == best


def test_small_chunks_take_the_smallest_tile_of_one_per_cu():
    for n, k in ((768, 3072), (2304, 768), (128, 64)):
        last = 0
        for m in (1, 24, 300, 777, 1500, 2080, 5003):
            rows, cols = S.surge_op_linear_tile(m, n, k)
            tiles = -(-m // rows) * (n // cols)
            assert rows * cols >= last
            assert tiles <= 256 or (rows, cols) >= (128, 128)
            last = rows * cols
    # 64 x 64 tiles up to one per CU, then 64 x 128, then the large families
    assert S.surge_op_linear_tile(64 * 21, 768, 3072) == (64, 64)
    assert S.surge_op_linear_tile(64 * 21 + 1, 768, 3072) == (64, 128)
    assert S.surge_op_linear_tile(64 * 42 + 1, 768, 3072) == (128, 128)


def test_shapes_that_the_layer_refuses_have_no_tile():
    for m, n, k in ((0, 128, 64), (1 << 31, 128, 64), (1, 64, 64), (1, 192, 64), (1, 128, 32),
                    (1, 128, 96)):
        assert S.surge_op_linear_tile(m, n, k) == (0, 0)
    assert S.surge_op_linear_tile(100_000, 768, 768, 0) == (0, 0)
    # row strides beyond the wide tiles' 24-bit copy offsets
    assert S.surge_op_linear_tile(100_000, 768, (1 << 23) - 64) == (256, 256)
    assert S.surge_op_linear_tile(100_000, 768, 1 << 23) == (128, 128)
