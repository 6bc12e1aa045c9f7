"""Small micro-batches of a stage step go through the launches side by side: every result must be what one micro-batch after
the other gives, bit for bit, and buffers that micro-batches share must keep their order."""
import numpy as np
import pytest
import torch

from paper_2405_16256_amd import inputs as I
from tests import gemm_plans, stage_plans

TINY = I.LayerShape(256, 4, 64, 704, 128, 1)
# shape, packed, layers, micro-batches, alive, added to the gradients, dx over dy; the number side by side
CASES = [
    (TINY, True, 2, 5, 2, False, False, 2),                                             # a last pass of one
    (TINY, True, 1, 9, 9, True, True, 8),                                               # more than one launch takes
    (I.LayerShape(128, 2, 64, 128, 1, 1), True, 1, 3, 3, False, False, 3),              # one token
    (I.LayerShape(128, 1, 128, 192, 37, 3, n_kv_heads=1), False, 2, 4, 3, True, False, 3),
    (I.LayerShape(512, 8, 64, 768, 1100, 2, n_kv_heads=2), False, 2, 3, 3, False, False, 3),   # split weight gradients
    (I.LayerShape(512, 4, 128, 64, 2049, 1, n_kv_heads=1), True, 1, 2, 2, True, True, 2),      # split ones, partial dK and dV
    (I.LayerShape(1024, 8, 128, 2048, 700, 1, n_kv_heads=2), True, 1, 4, 4, True, False, 3),   # larger tiles, passes of two
    (I.LayerShape(512, 8, 64, 768, 1100, 2, n_kv_heads=2), False, 2, 8, 8, True, True, 5),     # tensors in the pool's free slots
    (I.LayerShape(2048, 4, 128, 1408, 130, 1), True, 2, 7, 4, False, False, 4),
    (I.LayerShape(2048, 16, 128, 5632, 64, 1), True, 1, 4, 3, True, False, 3),                 # weight gradients that alone take 256x256
    (I.LayerShape(192, 3, 64, 64, 65, 40), True, 1, 2, 2, False, False, 2),                     # rows past a tile, many samples
]
# layers that leave their weight gradients to one launch at the end, of tensors that the attention branch must not overwrite before
DEFERRING = [
    (I.LayerShape(1536, 12, 128, 768, 400, 1), True, 1, 4, 4, False, False, 3),                        # passes of two, in the workspace
    (I.LayerShape(2176, 17, 128, 768, 426, 1, n_kv_heads=1), True, 2, 8, 8, True, True, 4),            # in the pool's free slots; partial dK and dV
    (I.LayerShape(2240, 35, 64, 2368, 397, 1, n_kv_heads=5), False, 1, 3, 2, True, False, 2),          # seven problems in two launches
    (I.LayerShape(1664, 26, 64, 704, 424, 1, n_kv_heads=1), False, 2, 3, 3, False, False, 3),
    (I.LayerShape(3392, 26, 128, 9536, 33, 1), False, 1, 2, 2, False, False, 2),                       # one k tile
]
CASES += DEFERRING
F32_CASES = [
    (I.LayerShape(256, 4, 64, 688, 128, 1), True, 2, 5, 5, False, False, 3),
    (I.LayerShape(72, 1, 128, 40, 33, 2), True, 1, 8, 8, True, True, 3),                  # no whole pieces of 16 columns
    (I.LayerShape(128, 4, 64, 256, 300, 1, n_kv_heads=1), True, 3, 8, 5, False, False, 3),     # partial dK and dV
    (I.LayerShape(512, 4, 128, 1536, 700, 1), True, 2, 4, 4, True, False, 2),             # tiles of 64
    (I.LayerShape(128, 4, 64, 192, 77, 1, n_kv_heads=2), False, 1, 6, 6, True, False, 2),   # B of the input gradients in segments
]
CASES = [c + (True,) for c in CASES] + [c + (False,) for c in F32_CASES]
IDS = ["%s%dx%d T%d M%d" % ("" if c[8] else "fp32 ", c[0].hidden, c[0].ffn, c[0].seq * c[0].micro_batch, c[3]) for c in CASES]


@pytest.mark.parametrize("shape,packed,k,M,n_live,acc,in_place,side,bf16", CASES, ids=IDS)
def test_rule(shape, packed, k, M, n_live, acc, in_place, side, bf16):
    buffers = stage_plans.boundary(shape, 2 if bf16 else 4, M, in_place)
    assert stage_plans.side_by_side(shape, k, M, n_live, packed, bf16, buffers=buffers) == side
    assert stage_plans.side_by_side(shape, k, M, 1, packed, bf16, buffers=buffers) == 1


def _random_shapes(n):
    rng = np.random.default_rng(17)
    for _ in range(n):
        d, hidden = int(rng.choice((64, 128))), 64 * int(np.exp(rng.uniform(np.log(2), np.log(192))))
        heads = max(1, int(hidden / d * rng.choice((0.125, 0.25, 0.5, 1.0))))
        kv = int(rng.choice([k for k in range(1, heads + 1) if heads % k == 0]))
        yield I.LayerShape(hidden, heads, d, 64 * int(rng.integers(max(1, hidden // 192), max(2, hidden // 20))), int(np.exp(rng.uniform(0, np.log(2500)))),
                           int(rng.choice((1, 1, 2))), n_kv_heads=kv), bool(rng.random() < 0.7)


def test_nothing_is_overwritten_before_its_last_reader():
    for case in DEFERRING:
        assert gemm_plans.defers(case[0], case[1])
    assert not any(gemm_plans.defers(c[0], c[1]) for c in CASES if c[8] and c[:8] not in DEFERRING)
    shapes = [(c[0], c[1]) for c in CASES if c[8]] + list(_random_shapes(300))
    for shape, packed in shapes:
        tensors, unit = stage_plans.side_tensors(shape, 2, packed)
        ends = sorted(e for _, e in tensors.values())
        assert ends[-1] <= unit, shape
        defer = gemm_plans.defers(shape, packed) and stage_plans.side_by_side(shape, 2, 16, 16, packed) > 1
        assert stage_plans.overwritten(tensors, stage_plans.backward_steps(defer)) == [], (shape, packed, defer)


def test_the_check_finds_a_tensor_overwritten():
    # a layer that does not defer, whose tensors are packed closer, run as if it did
    tensors, _ = stage_plans.side_tensors(TINY, 2)
    assert {t for _, t, _ in stage_plans.overwritten(tensors, stage_plans.backward_steps(True))} == {"m", "dgu"}


def test_rule_leaves_out():
    assert stage_plans.side_by_side(TINY, 2, 2, 2, bf16=False) == 1                    # fp32: no room for a second one's tensors
    assert stage_plans.side_by_side(I.CFG2, 1, 4, 4) == 1                              # no room in the workspace, tiles of 256
    x, y, dy, dx = stage_plans.boundary(TINY, 2, 3)
    bytes_ = 2 * 128 * 256

    def side(x=x, y=y, dy=dy, dx=dx):
        return stage_plans.side_by_side(TINY, 1, 3, 3, buffers=[x, y, dy, dx])
    assert side() == 3 and side(x=x[:1] * 3) == 3 and side(dy=dy[:1] * 3) == 3 and side(dx=dy) == 3
    for shared in (dict(y=y[:1] * 3), dict(dx=dx[:1] * 3), dict(dx=[dy[1], dy[2], dx[0]]), dict(dx=[dy[0], dx[1], dx[2]]),
                   dict(dy=y), dict(dy=dy[:1] * 3, dx=dy[:1] * 3), dict(y=[x[1], y[1], y[2]]), dict(dx=x),
                   dict(y=[y[0], y[0] + bytes_ - 16, y[2]]), dict(dy=x)):
        assert side(**shared) == 1, shared
    assert side(y=[y[0], y[0] + bytes_, y[2]]) == 3                                    # right behind one another
    pool_b, ws_b = [hh_sizes(TINY, 1, 3)[i] for i in (0, 1)]
    for inside in (stage_plans.POOL, stage_plans.POOL + pool_b - 256, stage_plans.WORKSPACE + ws_b - 256):
        assert side(y=[y[0], inside, y[2]]) == 1 and side(dx=[dx[0], dx[1], inside]) == 1 and side(dy=[inside] + dy[1:]) == 1
    assert side(y=[y[0], stage_plans.POOL + pool_b, stage_plans.WORKSPACE + ws_b]) == 3


def hh_sizes(shape, layers, live):
    from paper_2405_16256_amd import binding as hh
    from paper_2405_16256_amd import glue as L
    return hh.hh_stage_sizes(L.cfg_of(shape, True), layers, live)


def _tie(*names, layers=(0, 1)):
    def change(ws, gs):
        for n in names:
            setattr(gs[layers[1]], n, getattr(gs[layers[0]], n))
    return change


def test_rule_leaves_out_shared_gradients():
    def side(change):
        return stage_plans.side_by_side(TINY, 2, 3, 3, change=change)

    def tied_weights(ws, gs):
        for n in stage_plans.NAMES:
            setattr(ws[1], n, getattr(ws[0], n))

    def two_of_a_layer(ws, gs):
        gs[0].g_mlp = gs[0].g_attn

    def partly(ws, gs):
        gs[1].wo = gs[0].w_down + 4 * 256 * 704 - 256

    def behind(ws, gs):
        gs[1].wo = gs[0].w_down + 4 * 256 * 704

    def over_a_weight(ws, gs):
        gs[0].g_mlp = ws[0].g_mlp

    def input_is_a_weight(ws, gs):
        ws[0].wq = stage_plans.boundary(TINY, 2, 3)[0][0]

    def in_the_workspace(ws, gs):
        gs[1].g_attn = stage_plans.WORKSPACE
    assert side(None) == side(tied_weights) == side(behind) == 3
    for change in (_tie(*stage_plans.NAMES), _tie("wo"), _tie("g_mlp"), two_of_a_layer, partly, over_a_weight, input_is_a_weight, in_the_workspace):
        assert side(change) == 1, change


def _stage(hh, L, ctx, cfg, layers, n_live, xs, ys, dys, dxs, zero_first):
    pool_b, ws_b = hh.hh_stage_sizes(cfg, len(layers), n_live)
    pool = torch.full((pool_b + 4096,), 0xFF, dtype=torch.uint8, device=L.DEV)         # bf16 NaN wherever nothing is written
    ws = torch.full((ws_b + 4096,), 0xFF, dtype=torch.uint8, device=L.DEV)
    hh.hh_stage_step_1f1b(ctx, cfg, [l.wstruct for l in layers], n_live, xs, ys, dys, dxs, [l.gstruct for l in layers], zero_first,
                          pool[:pool_b], ws[:ws_b], L.stream_ptr())
    torch.cuda.synchronize()
    assert (pool[pool_b:] == 0xFF).all() and (ws[ws_b:] == 0xFF).all()


def _inputs(L, shape, packed, k, M, bf16=True):
    layers = [[L.DeviceLayer(I.layer_weights(811, l, shape, bf16), shape, bf16, packed) for l in range(k)] for _ in range(2)]
    for l in layers[0] + layers[1]:   # which GEMMs a layer has depends on whether these are one allocation
        for t in (l.w, l.g):
            for a, b in (("wq", "wk"), ("wk", "wv"), ("w_gate", "w_up")):
                assert (t[a].data_ptr() + t[a].numel() * t[a].element_size() == t[b].data_ptr()) == packed, (a, b)
    acts = [I.activations(811, shape, m, bf16) for m in range(M)]
    return layers, [L.to_dev(a[0], bf16) for a in acts], [L.to_dev(a[1], bf16) for a in acts]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,packed,k,M,n_live,acc,in_place,side,bf16", CASES, ids=IDS)
def test_same_bits_as_one_by_one(shape, packed, k, M, n_live, acc, in_place, side, bf16):
    from paper_2405_16256_amd import binding as hh
    from paper_2405_16256_amd import glue as L
    ctx = hh.hh_ctx_create(0)
    cfg = L.cfg_of(shape, bf16)
    (side_layers, one_layers), xs, dys = _inputs(L, shape, packed, k, M, bf16)
    out = []
    for layers, live in ((side_layers, n_live), (one_layers, 1)):
        for l in layers:
            for n in I.WEIGHT_NAMES:
                l.g[n].fill_(0.75 if acc else float("nan"))
        ys = [torch.full_like(t, float("nan")) for t in xs]
        g_in = [t.clone() for t in dys]
        dxs = g_in if in_place else [torch.full_like(t, float("nan")) for t in xs]
        _stage(hh, L, ctx, cfg, layers, live, xs, ys, g_in, dxs, not acc)
        out.append((ys, dxs))
    for m in range(M):
        assert torch.isfinite(out[0][0][m]).all() and torch.isfinite(out[0][1][m]).all()
        assert torch.equal(out[0][0][m], out[1][0][m]) and torch.equal(out[0][1][m], out[1][1][m]), m
    for a, b in zip(side_layers, one_layers):
        for n in I.WEIGHT_NAMES:
            assert torch.isfinite(a.g[n]).all() and torch.equal(a.g[n], b.g[n]), n
    hh.hh_ctx_destroy(ctx)


@pytest.mark.gpu
def test_micro_batches_that_share_an_output_keep_their_order():
    from paper_2405_16256_amd import binding as hh
    from paper_2405_16256_amd import glue as L
    ctx = hh.hh_ctx_create(0)
    cfg = L.cfg_of(TINY, True)
    (layers, ref), xs, dys = _inputs(L, TINY, True, 1, 3)
    y, dx = torch.empty_like(xs[0]), torch.empty_like(xs[0])
    _stage(hh, L, ctx, cfg, layers, 3, xs, [y] * 3, dys, [dx] * 3, True)
    ys, dxs = [torch.empty_like(t) for t in xs], [torch.empty_like(t) for t in xs]
    _stage(hh, L, ctx, cfg, ref, 1, xs, ys, dys, dxs, True)
    assert torch.equal(y, ys[2]) and torch.equal(dx, dxs[2])
    for n in I.WEIGHT_NAMES:
        assert np.array_equal(L.to_np(layers[0].g[n]), L.to_np(ref[0].g[n])), n
    hh.hh_ctx_destroy(ctx)


@pytest.mark.gpu
@pytest.mark.parametrize("names", [I.WEIGHT_NAMES, ("wo", "g_mlp")], ids=["all", "two"])
@pytest.mark.parametrize("zero_first", [False, True])
def test_layers_that_share_gradients_keep_their_order(names, zero_first):
    from paper_2405_16256_amd import binding as hh
    from paper_2405_16256_amd import glue as L
    ctx = hh.hh_ctx_create(0)
    cfg = L.cfg_of(TINY, True)
    (layers, ref), xs, dys = _inputs(L, TINY, True, 2, 3)
    out = []
    for both, live in ((layers, 3), (ref, 1)):
        for l in both:
            for n in I.WEIGHT_NAMES:
                l.g[n].fill_(0.75)
        both[1].gstruct = hh.make_grads({n: both[0 if n in names else 1].g[n] for n in I.WEIGHT_NAMES})
        ys, dxs = [torch.empty_like(t) for t in xs], [torch.empty_like(t) for t in xs]
        _stage(hh, L, ctx, cfg, both, live, xs, ys, dys, dxs, zero_first)
        out.append(dxs + [l.g[n] for l in both for n in I.WEIGHT_NAMES])
    assert all(torch.equal(a, b) for a, b in zip(*out))
    hh.hh_ctx_destroy(ctx)
