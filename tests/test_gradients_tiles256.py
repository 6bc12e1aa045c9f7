"""Weight gradients on 256x256 tiles, whose halves of rows change places in every other row of tiles: odd numbers of rows of tiles, the
last one not full, one k tile and several, whole and in k shares, written and added to."""
import numpy as np
import pytest

from paper_2405_16256_amd import inputs as I
from tests import gemm_plans

# shape; how the gradients of w_down and of w_gate|w_up are launched
CASES = [
    (I.LayerShape(1600, 1, 128, 6720, 50, 1), ("alone", "256x256", 1)),       # 7 and 53 rows of tiles, one k tile
    (I.LayerShape(1984, 1, 128, 8768, 128, 1), ("alone", "256x256", 1)),      # 8 and 69, two k tiles
    (I.LayerShape(1728, 1, 128, 1600, 516, 1), ("tiles256", "256x256", 1)),   # 7 and 13
    (I.LayerShape(2496, 1, 128, 4416, 685, 1), ("tiles256", "256x256", 2)),   # 10 and 35, the last round in k shares
]
IDS = ["%dx%d T%d" % (c[0].hidden, c[0].ffn, c[0].tokens) for c in CASES]


@pytest.mark.parametrize("shape,want", CASES, ids=IDS)
def test_rule(shape, want):
    got = gemm_plans.layer_launches(shape)
    assert got["dW down"] == got["dW gate|up"] == want


@pytest.mark.gpu
@pytest.mark.parametrize("shape,want", CASES, ids=IDS)
def test_against_the_oracle_and_added(shape, want):
    from paper_2405_16256_amd import binding as hh
    from paper_2405_16256_amd import glue as L
    from tests.test_gpu_parity import check_layer
    ctx = hh.hh_ctx_create(0)
    check_layer(ctx, shape, True, 331, label="dW 256")
    w = I.layer_weights(331, 0, shape, True)
    x, dy = I.activations(331, shape, 0, True)
    layer = L.DeviceLayer(w, shape, True)
    L.run_layer(ctx, shape, True, layer, x, dy)
    written = layer.grads_np()
    for t in layer.g.values():
        t.copy_((t * -3.0).flip(0))
    before = layer.grads_np()
    L.run_layer(ctx, shape, True, layer, x, dy, accumulate=True)
    added = layer.grads_np()
    for n in ("w_gate", "w_up", "w_down"):   # one fp32 addition at the end
        assert np.array_equal(added[n], (written[n].astype(np.float32) + before[n].astype(np.float32)).astype(np.float64)), n
    hh.hh_ctx_destroy(ctx)
