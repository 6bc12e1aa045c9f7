"""What the ring kernel does with a product on its way out (rotary embedding, SwiGLU forward and backward), at edges of tiles
and of the column order it needs, whole and in k shares, and norms that add the shares of their input, against the oracle.
Tolerances are those of every bf16 layer test."""
import pytest

from paper_2405_16256_amd import inputs as I
from tests import gemm_plans

pytestmark = pytest.mark.gpu

S = I.LayerShape
# shape, packed; k shares of q|k|v (of q), gate|up (of gate), out, d(m), d(hn) and d(xn)
CASES = [
    (S(64, 1, 64, 64, 1, 1), True, (1, 1, 1, 1, 1, 1)),                               # one token, one head
    (S(192, 3, 64, 64, 65, 2), True, (1, 1, 1, 1, 1, 1)),                             # rows of two samples in a tile
    (S(128, 1, 128, 192, 33, 3, n_kv_heads=1), False, (1, 1, 1, 1, 1, 1)),            # a head over two tiles
    (S(1024, 8, 128, 320, 40, 1, n_kv_heads=2), True, (1, 8, 1, 8, 1, 8)),            # a wave a row, two vectors a lane
    (S(2048, 4, 64, 192, 129, 1, n_kv_heads=1), True, (8, 8, 1, 8, 1, 1)),
    (S(2048, 5, 64, 192, 70, 1), False, (8, 8, 1, 8, 1, 1)),
    (S(1536, 8, 64, 1024, 100, 1), True, (4, 4, 1, 6, 2, 8)),                         # a workgroup a row, a guarded length
    (S(512, 8, 64, 1408, 90, 2), True, (1, 1, 1, 1, 8, 8)),                           # a wave a row, one vector a lane
    (S(512, 32, 128, 64, 41, 1, n_kv_heads=1), True, (1, 1, 8, 1, 1, 8)),           # h from shares, of one tile row
    (S(2048, 16, 128, 1024, 300, 1, n_kv_heads=1), True, (1, 1, 1, 3, 3, 4)),         # two rows a workgroup
    (S(4096, 32, 128, 1024, 333, 1, n_kv_heads=1), True, (2, 4, 2, 4, 1, 2)),         # h from shares, larger tiles
    (S(6144, 16, 128, 512, 17, 1, n_kv_heads=8), True, (3, 8, 2, 8, 1, 1)),           # the longest rows whose gains' gradients the norm sums itself
    (S(6208, 16, 128, 512, 17, 1, n_kv_heads=8), True, (3, 8, 2, 8, 1, 1)),           # longer ones
    (S(8192, 32, 128, 4096, 17, 1, n_kv_heads=8), True, (2, 2, 2, 3, 2, 1)),          # the longest rows of shares, both norms
]


def _shares(shape, packed):
    p = gemm_plans.layer_launches(shape, packed)
    return tuple(p[n][2] for n in (("qkv", "gate|up") if packed else ("q", "gate")) + ("out", "d down", "d gate|up", "d qkv"))


@pytest.mark.parametrize("shape,packed,shares", CASES)
def test_against_the_oracle(shape, packed, shares):
    from paper_2405_16256_amd import binding as hh
    from tests.test_gpu_parity import check_layer
    assert _shares(shape, packed) == shares
    ctx = hh.hh_ctx_create(0)
    check_layer(ctx, shape, True, 931, packed=packed, label="fused %s" % (shape,))
    hh.hh_ctx_destroy(ctx)


# fp32: tiles of 32 with deep and shallow rings and of 64; an ffn in whole pieces of 16 columns and one that is not
@pytest.mark.parametrize("shape,packed", [
    (S(8, 1, 64, 8, 1, 1), True), (S(40, 3, 64, 48, 33, 2, n_kv_heads=1), True), (S(72, 1, 128, 40, 65, 1), False),
    (S(256, 4, 64, 688, 128, 1), True), (S(256, 2, 128, 336, 900, 1, n_kv_heads=1), True), (S(512, 8, 128, 1536, 1100, 1), False),
    (S(512, 8, 128, 1536, 1100, 1), True),
])
def test_fp32_against_the_oracle(shape, packed):
    from paper_2405_16256_amd import binding as hh
    from tests.test_gpu_parity import check_layer
    ctx = hh.hh_ctx_create(0)
    check_layer(ctx, shape, False, 932, packed=packed, label="fused fp32 %s" % (shape,))
    hh.hh_ctx_destroy(ctx)
