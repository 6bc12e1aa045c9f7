"""fp32 attention around the edges of its 16-row tiles and of the split of grouped heads over workgroups.

Sequence lengths sit one below, at and one above a tile and a round of four tiles.  The tolerance is the fp32 path's own
(1e-4 of each tensor's norm, against the fp64 oracle).
"""
import numpy as np
import pytest

from paper_2405_16256_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2405_16256_amd import binding as hh
    c = hh.hh_ctx_create(0)
    yield c
    hh.hh_ctx_destroy(c)


@pytest.mark.parametrize("heads,kv_heads,head_dim", [(2, 2, 64), (6, 2, 64), (4, 1, 128)])
@pytest.mark.parametrize("seq", [1, 15, 16, 17, 63, 65, 129])
def test_tile_edges(ctx, heads, kv_heads, head_dim, seq):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, I.LayerShape(128, heads, head_dim, 136, seq, 2, n_kv_heads=kv_heads), False, 501, label="attn f32")


def test_heads_that_share_keys_in_one_workgroup(ctx):
    # 2*4*64 tiles of keys fill the chip, so the two query heads of a key head stay together
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, I.LayerShape(64, 8, 64, 64, 1024, 2, n_kv_heads=4), False, 502, label="attn f32 wide")


@pytest.mark.parametrize("heads,kv_heads,head_dim,seq,batch", [(5, 1, 128, 1000, 1), (8, 8, 128, 650, 1), (16, 16, 64, 1001, 2), (16, 8, 64, 1030, 2)])
def test_backward_passes_together_and_apart(ctx, heads, kv_heads, head_dim, seq, batch):
    # 630 and 656 jobs of head_dim 128, 4032 and 4160 of head_dim 64: both sides of where the two passes share a launch
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, I.LayerShape(64, heads, head_dim, 64, seq, batch, n_kv_heads=kv_heads), False, 504, label="attn f32 passes")


@pytest.mark.parametrize("seq,at", [(50, 5), (50, 20), (33, 32)])
def test_values_that_are_not_finite_stay_behind_the_mask(ctx, seq, at):
    # the tile that holds the bad row is summed pair by pair, in another order: equal up to fp32 rounding of sums of at
    # most 136 terms of order 1 (136 * 2^-24 < 1e-5)
    from paper_2405_16256_amd import glue as L
    s = I.LayerShape(128, 2, 64, 136, seq, 1)
    w = I.layer_weights(503, 0, s, False)
    x, dy = I.activations(503, s, 0, False)
    layer = L.DeviceLayer(w, s, False)
    y0, dx0, _ = L.run_layer(ctx, s, False, layer, x, dy)
    bad = np.array(x)
    bad.reshape(seq, -1)[at, 3] = np.nan
    y, _, _ = L.run_layer(ctx, s, False, layer, bad, dy)
    y, y0 = y.reshape(seq, -1), y0.reshape(seq, -1)
    assert np.allclose(y[:at], y0[:at], rtol=1e-5, atol=1e-5) and np.all(np.isnan(y[at:]).any(axis=1))
    bad = np.array(dy)
    bad.reshape(seq, -1)[at, 3] = np.inf
    _, dx, _ = L.run_layer(ctx, s, False, layer, x, bad)
    dx, dx0 = dx.reshape(seq, -1), dx0.reshape(seq, -1)
    assert np.allclose(dx[at + 1:], dx0[at + 1:], rtol=1e-5, atol=1e-5) and not np.any(np.isfinite(dx[:at + 1]).all(axis=1))
