"""The launches that the bf16 GEMM dispatch can choose, each in a layer against the oracle.

Which kernel, tile and k split a projection takes follows from a cost model, so the shapes below would silently stop
reaching what they are listed for whenever its constants are fitted again.  The tests without a GPU ask the library for its
choice and fail then; the GPU tests run the same layers.  Tolerances are those of every bf16 layer test.
"""
import numpy as np
import pytest

from paper_2405_16256_amd import inputs as I
from tests import gemm_plans
from tests import test_gpu_gemm_tiles as tiles

# shape, packed weights, {GEMM: how, tile, k shares}
CASES = [
    # k shares of one wave's tile in a weight gradient, two workgroups of 128x128 per CU in a group
    (I.LayerShape(64, 1, 64, 2048, 277, 4), False, {"gate": "ring 128x128/2 1", "d down": "alone 64x128 1", "dW out": "ring 64x64 8"}),
    # one row past six tiles of 192: groups on 192x192, 192x128 and 192x256 tiles
    (I.LayerShape(64, 1, 64, 3392, 1153, 1), False, {"gate": "ring 192x192 1", "d down": "alone 128x128/2 1"}),
    (I.LayerShape(192, 1, 64, 2560, 769, 1), False, {"gate": "ring 192x128 1"}),
    (I.LayerShape(128, 1, 128, 4992, 769, 1), False, {"gate": "ring 192x256 1"}),
    # 256x256 tiles on two rows of them, alone and for a group of projections
    (I.LayerShape(64, 1, 128, 8256, 464, 1), True, {"gate|up": "alone 256x256 1"}),
    (I.LayerShape(64, 1, 64, 8896, 124, 4), False, {"gate": "tiles256 256x256 1", "up": "tiles256 256x256 1"}),
    (I.LayerShape(64, 1, 64, 12672, 59, 1), True, {"dW down": "alone 64x64 1", "dW gate|up": "alone 128x128/2 1"}),
    (I.LayerShape(448, 1, 128, 1728, 485, 4), False, {"gate": "ring 128x256 1"}),
    (I.LayerShape(1344, 1, 128, 256, 769, 4), False,
     {"out": "alone 128x128/2 1", "dW down": "ring 128x256 3", "dW q": "ring 128x128/2 6", "d qkv": "ring 128x128/2 1"}),
    (I.LayerShape(320, 1, 128, 5248, 1537, 1), True,
     {"gate|up": "alone 192x192 1", "d down": "alone 256x256 1", "dW down": "alone 64x128 1", "dW gate|up": "alone 128x128 1"}),
    (I.LayerShape(1728, 2, 128, 64, 961, 4), True, {"dW down": "ring 64x128 4", "dW qkv": "alone 128x128 3"}),
    # k shares of projections that share a launch, tiles of 192 rows among them
    (I.LayerShape(3776, 4, 128, 128, 324, 4, n_kv_heads=2), False, {"q": "ring 192x128 4", "k": "ring 192x128 4", "gate": "ring 64x64 3"}),
    (I.LayerShape(128, 1, 128, 9984, 1153, 4), True, {"down": "alone 128x128/2 6"}),
    (I.LayerShape(704, 1, 128, 3008, 1311, 4), True, {"dW down": "alone 128x256 3", "dW gate|up": "alone 256x256 3"}),
    (I.LayerShape(640, 1, 64, 4928, 914, 4), False, {"gate": "tiles256 256x256 2", "down": "alone 192x128 2", "d gate|up": "alone 128x128/2 3"}),
    # an input gradient over separate weights, one segment after the other
    (I.LayerShape(640, 1, 128, 3008, 1575, 4), False, {"q": "ring 128x128 1", "d gate|up": "segments - 1"}),
    (I.LayerShape(4096, 4, 128, 256, 1345, 1), False,
     {"q": "ring 128x256 3", "out": "alone 192x128 1", "gate": "ring 128x128 4", "d down": "alone 64x128 4"}),
    (I.LayerShape(960, 15, 128, 64, 486, 4), False, {"q": "tiles256 256x256 1", "k": "tiles256 256x256 1", "v": "tiles256 256x256 1"}),
    (I.LayerShape(576, 2, 128, 9920, 851, 4), True,
     {"gate|up": "alone 256x256 2", "down": "alone 192x192 4", "d down": "alone 256x256 2", "dW down": "alone 128x256 1", "dW qkv": "ring 128x128 4"}),
    (I.LayerShape(448, 1, 64, 10688, 1537, 4), True, {"down": "alone 192x256 3"}),
    (I.LayerShape(5760, 11, 64, 64, 917, 2), False, {"q": "tiles256 256x256 3"}),
    (I.LayerShape(5696, 11, 128, 256, 577, 1), False, {"q": "ring 128x128/2 3", "gate": "ring 64x128 6"}),
]

# What the dispatch chooses over 330000 random layers (hidden 64 to 6144, ffn up to 12800, 17 to 3000 tokens a sample, up to
# four samples) at least 40 times: kind, how, tiles without and with k shares.
OUTCOMES = {
    ("NT", "alone"): ("64x64 64x128 128x128 128x128/2 128x256 192x128 192x192 192x256 256x256",
                      "64x64 64x128 128x128 128x128/2 128x256 192x128 192x192 192x256 256x256"),
    ("NT", "ring"): ("64x64 64x128 128x128 128x128/2 128x256 192x128 192x192 192x256", "64x64 64x128 128x128 128x128/2 128x256 192x128"),
    ("NT", "tiles256"): ("256x256", "256x256"),
    ("NN", "alone"): ("64x64 64x128 128x128 128x128/2 128x256 256x256", "64x64 64x128 128x128 128x128/2 128x256 256x256"),
    ("NN", "ring"): ("64x64 64x128 128x128 128x128/2 128x256", "64x64 64x128 128x128 128x128/2 128x256"),
    ("NN", "segments"): ("-", ""),
    ("TN", "alone"): ("64x64 64x128 128x128 128x128/2 128x256 256x256", "128x128 128x256 256x256"),
    ("TN", "ring"): ("64x64 64x128 128x128 128x128/2 128x256", "64x64 64x128 128x128 128x128/2 128x256"),
    ("TN", "tiles256"): ("256x256", "256x256"),
}


def kind(gemm):
    return "TN" if gemm.startswith("dW") else "NN" if gemm.startswith("d ") else "NT"


def named(case):
    s, packed, _ = case
    return "%dx%d-%dx%d-%dx%d%s" % (s.hidden, s.ffn, s.n_heads, s.head_dim, s.micro_batch, s.seq, "" if packed else "-separate")


@pytest.mark.parametrize("case", CASES, ids=named)
def test_the_dispatch_chooses_what_a_case_is_listed_for(case):
    shape, packed, want = case
    got = {n: "%s %s %d" % r for n, r in gemm_plans.layer_launches(shape, packed).items()}
    assert {n: got[n] for n in want} == want


def test_the_layers_under_test_take_every_launch_of_the_dispatch():
    layers = [(s, packed) for s, packed, _ in CASES] + tiles.SHAPES
    got = {(kind(n), how, tile, shares > 1) for s, packed in layers
           for n, (how, tile, shares) in gemm_plans.layer_launches(s, packed).items()}
    for (k, how), both in OUTCOMES.items():
        for split, named_tiles in enumerate(both):
            for tile in named_tiles.split():
                assert (k, how, tile, bool(split)) in got, (k, how, tile, split)


@pytest.fixture(scope="module")
def ctx():
    from paper_2405_16256_amd import binding as hh
    c = hh.hh_ctx_create(0)
    yield c
    hh.hh_ctx_destroy(c)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=named)
def test_layer_against_the_oracle(ctx, case):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, case[0], True, 311, packed=case[1], label="dispatch")


@pytest.mark.gpu
@pytest.mark.parametrize("case", [c for c in CASES if any(n.startswith("dW") and int(r.split()[2]) > 1 for n, r in c[2].items())], ids=named)
def test_gradients_in_k_shares_add_to_what_the_buffers_hold(ctx, case):
    # `+=` adds the same sum that `=` writes, in one fp32 addition at the end: bit for bit
    from paper_2405_16256_amd import glue as L
    s, packed, _ = case
    w = I.layer_weights(312, 0, s, True)
    x, dy = I.activations(312, s, 0, True)
    layer = L.DeviceLayer(w, s, True, packed)
    L.run_layer(ctx, s, True, layer, x, dy)
    written = layer.grads_np()
    for t in layer.g.values():
        t.copy_((t * -3.0).flip(0))
    before = layer.grads_np()
    L.run_layer(ctx, s, True, layer, x, dy, accumulate=True)
    added = layer.grads_np()
    for n in I.WEIGHT_NAMES:
        want = (written[n].astype(np.float32) + before[n].astype(np.float32)).astype(np.float64)
        assert np.array_equal(added[n], want), n
