"""Input gradients over separate weights, one segment after the other on 256x256 tiles, each but the first with what the ones before
it have left as its residual: one round of tiles and several, whole and in k shares, tiles that M and N do not fill."""
import pytest

from paper_2405_16256_amd import inputs as I
from tests import gemm_plans

# shape; the gradient and its k; tiles and k shares of the last round
CASES = [
    (I.LayerShape(5312, 1, 128, 512, 2397, 1), "d gate|up", (512, 512), 210, 1),
    (I.LayerShape(2368, 1, 128, 3648, 1801, 1), "d gate|up", (3648, 3648), 80, 3),
    (I.LayerShape(3648, 1, 128, 1024, 4489, 1), "d gate|up", (1024, 1024), 270, 4),      # a whole round before the shares
    (I.LayerShape(5696, 1, 128, 512, 4823, 1), "d gate|up", (512, 512), 437, 1),         # workgroups with a second tile
    (I.LayerShape(5568, 8, 128, 64, 2190, 1), "d qkv", (1024, 1024, 1024), 198, 1),
]
IDS = ["%s %d tiles" % (c[1], c[3]) for c in CASES]


@pytest.mark.parametrize("shape,name,ks,tiles,shares", CASES, ids=IDS)
def test_rule(shape, name, ks, tiles, shares):
    assert gemm_plans.layer_launches(shape, False)[name] == ("segments", "-", 1)
    for k in ks:
        assert gemm_plans.plan([(gemm_plans.NN, shape.tokens, shape.hidden, k)]) == [("alone", "256x256", shares)]
    assert -(-shape.tokens // 256) * -(-shape.hidden // 256) == tiles


@pytest.mark.gpu
@pytest.mark.parametrize("shape,name,ks,tiles,shares", CASES, ids=IDS)
def test_layer_against_the_oracle(shape, name, ks, tiles, shares):
    from paper_2405_16256_amd import binding as hh
    from tests.test_gpu_parity import check_layer
    ctx = hh.hh_ctx_create(0)
    check_layer(ctx, shape, True, 321, packed=False, label="segments")
    hh.hh_ctx_destroy(ctx)
