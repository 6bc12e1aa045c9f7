"""RMSNorm inside the launch of the projections that read it: which launches do it, and that xn and the factors it writes are the
bits of the norm's own launch."""
import ctypes as C

import pytest
import torch

from paper_2405_16256_amd import binding as hh
from paper_2405_16256_amd import inputs as I
from tests import gemm_plans

# heads of 64 columns; tokens at the edges of a tile of 64 rows, one and two 16-byte pieces a lane, whole and not
CASES = [(64, 1, True), (64, 130, False), (128, 63, True), (192, 64, True), (192, 65, False), (256, 200, True), (256, 17, False)]
MANY = 9000   # tokens of which no projection fits the rule


def norms(hidden, tokens, packed, ffn=192):
    s = I.LayerShape(hidden, hidden // 64, 64, ffn, tokens, 1)
    calls = {tuple(n for n, _ in call): [p for _, p in call] for call in gemm_plans._calls(s, packed)[0]}
    names = [("qkv",), ("gate|up",)] if packed else [("q", "k", "v"), ("gate", "up")]
    return [hh.lib.hh_internal_gemm_norms(gemm_plans._ints(calls[n]), len(calls[n])) for n in names]


def test_rule():
    for hidden, tokens, packed in CASES:
        assert norms(hidden, tokens, packed) == [1, 1], (hidden, tokens, packed)
        assert norms(hidden, MANY, packed) == [0, 0], (hidden, packed)
    assert norms(320, 64, True) == [0, 0]
    assert norms(256, 64, True, ffn=64 * 200) == [1, 0]      # more workgroups than CUs


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,tokens,packed", CASES)
def test_same_bits_as_a_launch_of_its_own(hidden, tokens, packed):
    from paper_2405_16256_amd import glue as L
    ctx = hh.hh_ctx_create(0)
    found = []
    for T in (tokens, MANY):
        s = I.LayerShape(hidden, hidden // 64, 64, 192, T, 1)
        cfg = L.cfg_of(s, True)
        layer = L.DeviceLayer(I.layer_weights(77, 0, s, True), s, True, packed)
        torch.manual_seed(3)
        x = (torch.randn(MANY, hidden) * torch.logspace(-3, 2, MANY)[torch.randperm(MANY)][:, None]).bfloat16()[:T].to(L.DEV).contiguous()
        y = torch.empty_like(x)
        lay = hh.hh_saved_layout_of(cfg)
        saved = torch.full((hh.hh_layer_sizes(cfg)[0],), 0xFF, dtype=torch.uint8, device=L.DEV)
        ws = torch.empty(hh.hh_layer_sizes(cfg)[1], dtype=torch.uint8, device=L.DEV)
        hh.hh_layer_fwd(ctx, cfg, layer.wstruct, x, y, saved, ws, L.stream_ptr())
        torch.cuda.synchronize()

        def part(name, dtype, n):
            at = getattr(lay, name)
            return saved[at:at + n * torch.empty(0, dtype=dtype).element_size()].view(dtype)
        xn, r1, r2 = part("xn", torch.bfloat16, T * hidden).view(T, hidden), part("r1", torch.float32, T), part("r2", torch.float32, T)
        h, hn = part("h", torch.bfloat16, T * hidden).view(T, hidden), part("hn", torch.bfloat16, T * hidden).view(T, hidden)
        for rows, r, out, g in ((x, r1, xn, "g_attn"), (h, r2, hn, "g_mlp")):
            exact = (rows.double().square().mean(1) + s.rms_eps).rsqrt()
            # a sum of at most 256 squares in 8 + 6 additions, a root and a division: under 20 roundings
            assert ((r.double() - exact).abs() <= 20 * 2.0 ** -24 * exact).all()
            assert torch.equal(out, (rows.float() * r[:, None] * layer.w[g].float()).bfloat16())
        found.append((xn[:tokens].clone(), r1[:tokens].clone()))
    assert all(torch.equal(a, b) for a, b in zip(*found))
    hh.hh_ctx_destroy(ctx)
