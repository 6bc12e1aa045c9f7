"""What the ring kernel does with a product on its way out (rotary embedding, SwiGLU forward and backward), at edges of tiles
and of the column order it needs, whole and in k shares, against the oracle.  Tolerances are those of every bf16 layer test."""
import pytest

from paper_2405_16256_amd import inputs as I
from tests import gemm_plans

pytestmark = pytest.mark.gpu

S = I.LayerShape
# shape, packed; (tile, k shares) of q|k|v (of q), gate|up (of gate) and d(m)
CASES = [
    (S(64, 1, 64, 64, 1, 1), True, ("64x64", 1), ("64x64", 1), ("64x64", 1)),                            # one token, one head
    (S(192, 3, 64, 64, 65, 2), True, ("64x64", 1), ("64x64", 1), ("64x64", 1)),                          # rows of two samples in a tile
    (S(128, 1, 128, 192, 33, 3, n_kv_heads=1), False, ("64x64", 1), ("64x64", 1), ("64x64", 1)),         # a head over two tiles
    (S(1024, 8, 128, 320, 40, 1, n_kv_heads=2), True, ("64x64", 1), ("64x64", 8), ("64x64", 8)),         # k shares: the reduction does it
    (S(2048, 4, 64, 192, 129, 1, n_kv_heads=1), True, ("64x64", 8), ("64x64", 8), ("64x64", 8)),
    (S(2048, 5, 64, 192, 70, 1), False, ("64x64", 8), ("64x64", 8), ("64x64", 8)),
]


def _got(shape, packed):
    p = gemm_plans.layer_launches(shape, packed)
    return tuple(p[n][1:] for n in (("qkv", "gate|up") if packed else ("q", "gate")) + ("d down",))


@pytest.mark.parametrize("shape,packed,qkv,gu,dm", CASES)
def test_against_the_oracle(shape, packed, qkv, gu, dm):
    from paper_2405_16256_amd import binding as hh
    from tests.test_gpu_parity import check_layer
    assert _got(shape, packed) == (qkv, gu, dm)
    ctx = hh.hh_ctx_create(0)
    check_layer(ctx, shape, True, 931, packed=packed, label="fused %s" % (shape,))
    hh.hh_ctx_destroy(ctx)
