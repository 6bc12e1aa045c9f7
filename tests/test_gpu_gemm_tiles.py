"""Layers whose projections take many of the tiles and k splits of the GEMM dispatch, with ragged token counts.

Tolerances are those of every bf16 layer test (storage rounding 2^-9 per tensor, fp32 sums).  Which launches the bf16 shapes
take is asked of the library in test_gemm_dispatch.py, which adds layers for those that none of them takes.
"""
import pytest

from paper_2405_16256_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2405_16256_amd import binding as hh
    c = hh.hh_ctx_create(0)
    yield c
    hh.hh_ctx_destroy(c)


@pytest.mark.parametrize("shape,packed", [
    # 64x64 tiles (whole and 4 shares of k) and 64x128 (whole, 4 and 8 shares)
    (I.LayerShape(1024, 4, 128, 2816, 150, 1), True),
    # the same with 70 tokens over grouped heads: single projections of 64 and 128 columns, k of 70 in the weight gradients
    (I.LayerShape(1024, 8, 64, 2816, 35, 2, n_kv_heads=1), False),
    # 192x128, 128x128 (one per CU: whole and 3 shares; two per CU: grouped, whole and 3 shares)
    (I.LayerShape(2048, 4, 128, 4096, 520, 1), True),
    # 128x128 in 2 and 3 shares, 128x256 in 3 shares and, in a group, whole and in 8
    (I.LayerShape(4096, 8, 128, 5632, 333, 1), True),
    # one token: a single row of C, a single k value in the weight gradients
    (I.LayerShape(2048, 2, 128, 1024, 1, 1), True),
])
def test_every_tile_of_the_gemm_dispatch(ctx, shape, packed):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, shape, True, 301, packed=packed, label="tiles")


@pytest.mark.parametrize("shape,packed", [
    # 64x64 tiles in the gate|up projection, k of 1000 and 700 (neither a multiple of the 32-wide stage)
    (I.LayerShape(1000, 4, 64, 2040, 700, 1), True),
    # 32x32 tiles with k of 8, 72 and 40: shorter than one stage, and a tail of a quarter stage
    (I.LayerShape(72, 1, 64, 40, 5, 2), False),
    (I.LayerShape(8, 1, 64, 8, 33, 1), True),
])
def test_both_tiles_of_the_fp32_gemm(ctx, shape, packed):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, shape, False, 302, packed=packed, label="f32 tiles")


@pytest.mark.parametrize("shape,packed", [
    # groups with and without k shares, B in two and three segments, some of them a single k tile wide
    (I.LayerShape(256, 4, 64, 704, 128, 1), True),
    (I.LayerShape(512, 8, 64, 64, 550, 2, n_kv_heads=2), False),
    (I.LayerShape(512, 3, 128, 1216, 77, 3, n_kv_heads=1), False),
    (I.LayerShape(4096, 8, 128, 256, 700, 1), True),
])
def test_problems_that_share_a_launch(ctx, shape, packed):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, shape, True, 303, packed=packed, label="groups")


@pytest.mark.parametrize("shape", [
    # 192x128 (q|k|v) and 192x192 (gate|up) on 333 rows; 192x256 (both) one row into a seventh tile.  The second layer, 385
    # rows, takes tiles of 64 and 128 rows.
    I.LayerShape(2048, 32, 128, 11008, 333, 1, n_kv_heads=32),
    I.LayerShape(1024, 24, 128, 5632, 385, 1, n_kv_heads=24),
    I.LayerShape(512, 24, 128, 4096, 1153, 1),
])
def test_tiles_of_192_rows(ctx, shape):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, shape, True, 304, label="192 rows")


@pytest.mark.parametrize("shape,packed", [
    # k loops of 4 to 87 stages of 32 side by side, ragged ones among them, separate weights
    (I.LayerShape(256, 4, 64, 688, 128, 1), True),
    (I.LayerShape(296, 3, 64, 1384, 37, 1), False),
    (I.LayerShape(64, 2, 64, 264, 500, 2, n_kv_heads=1), False),
    # 64x64 tiles for a whole group
    (I.LayerShape(1000, 4, 64, 2040, 1500, 1), True),
])
def test_fp32_problems_that_share_a_launch(ctx, shape, packed):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, shape, False, 305, packed=packed, label="f32 groups")


@pytest.mark.parametrize("shape,packed", [
    # all weight gradients in one launch of 256x256 tiles, from four and from seven problems, the last one's in two k shares
    (I.LayerShape(2048, 4, 128, 2048, 1100, 1, n_kv_heads=1), True),
    (I.LayerShape(2048, 4, 128, 2048, 750, 2, n_kv_heads=1), False),
    (I.LayerShape(2048, 16, 128, 2048, 1500, 1, n_kv_heads=4), False),
])
def test_weight_gradients_in_one_launch(ctx, shape, packed):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, shape, True, 306, packed=packed, label="dW together")


# the bf16 layers above
SHAPES = [(p if isinstance(p, tuple) else (p, True)) for f in (test_every_tile_of_the_gemm_dispatch, test_problems_that_share_a_launch,
                                                               test_tiles_of_192_rows, test_weight_gradients_in_one_launch)
          for m in f.pytestmark if m.name == "parametrize" for p in m.args[1]]
