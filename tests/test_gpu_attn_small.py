"""bf16 attention on launches of few workgroups: keys split between two wave groups, both backward passes and delta in one
launch.  Sequence lengths around a 64-key tile, a pair of them and a 128-query block, with grouped heads (summed in one
workgroup or through partial sums), on both sides of the rules that choose these forms.

Tolerances are those of every bf16 layer test.
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


@pytest.mark.parametrize("heads,kv_heads,head_dim", [(2, 2, 64), (6, 2, 64), (3, 3, 128), (4, 1, 128)])
@pytest.mark.parametrize("seq,batch", [(1, 2), (63, 1), (65, 3), (128, 1), (129, 2), (257, 1), (1024, 1), (1025, 1)])
def test_edges(ctx, heads, kv_heads, head_dim, seq, batch):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, I.LayerShape(heads * head_dim, heads, head_dim, 128, seq, batch, n_kv_heads=kv_heads), True, 701, label="attn small")


def test_more_workgroups_than_cus(ctx):
    # 257 workgroups, each of the 100 queries of a sample: one group of waves per query block, two kernels backward
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, I.LayerShape(64, 1, 64, 64, 100, 257), True, 702, label="attn 257")


@pytest.mark.parametrize("heads,head_dim,seq", [(2, 64, 300), (1, 128, 300), (2, 64, 1100), (2, 64, 100)])
def test_scores_past_the_fp32_range(ctx, heads, head_dim, seq):
    # keys 64..127 score -1e40 with every query, i.e. -inf in fp32: weight zero, like any score far below the others, also
    # where these keys are the whole first tile of a group of waves (seq 300, 1100).  Channel pair (d/2 - 1, d - 1) turns
    # slowest under the rotation; only its second half is non-zero, in those keys, with x[0] set for them alone.
    import torch
    from oracle import decoder_oracle as O
    from paper_2405_16256_amd import binding as hh
    from paper_2405_16256_amd import glue as L
    s = I.LayerShape(128, heads, head_dim, 64, seq, 1)
    w = I.layer_weights(703, 0, s, True)
    x, _ = I.activations(703, s, 0, True)
    x[:, :, 0] = 0.0
    x[:, 64:128, 0] = 4.0
    x[:, :, 1] = 2.0
    for n, column, value in (("wq", 1, -2.0 ** 66), ("wk", 0, 2.0 ** 66)):
        w[n][head_dim // 2 - 1] = 0.0
        w[n][head_dim - 1] = 0.0
        w[n][head_dim - 1, column] = value
    cfg = L.cfg_of(s, True)
    layer = L.DeviceLayer(w, s, True)
    saved_b, ws_b = hh.hh_layer_sizes(cfg)
    xd = L.to_dev(x, True)
    yd = torch.empty_like(xd)
    ws = torch.empty(saved_b + ws_b, dtype=torch.uint8, device=L.DEV)
    hh.hh_layer_fwd(ctx, cfg, layer.wstruct, xd, yd, None, ws, L.stream_ptr())
    torch.cuda.synchronize()
    y = L.to_np(yd)
    want, _ = O.layer_forward(x, w, s.n_heads, s.head_dim, s.rms_eps, s.rope_base, s.kv_heads)
    assert np.all(np.isfinite(want)) and np.all(np.isfinite(y))
    # the last channel's scores swamp the others' among keys 64..127 only, whose weights are zero: the tolerance is
    # that of every bf16 output
    assert L.rel_err(y, want) <= 2e-2
