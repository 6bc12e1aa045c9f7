"""How many micro-batches a stage step takes through its launches side by side, asked of the library without a GPU."""
import ctypes as C

from paper_2405_16256_amd import binding as hh

NAMES = ("g_attn", "wq", "wk", "wv", "wo", "g_mlp", "w_gate", "w_up", "w_down")


def boundary(s, es, n_micro, in_place=False, base=1 << 40):
    """x, y, dy, dx as addresses of buffers of their own."""
    step = 2 * s.seq * s.micro_batch * s.hidden * es
    x, y, dy, dx = [[base + (4 * m + i) * step for m in range(n_micro)] for i in range(4)]
    return [x, y, dy, dy if in_place else dx]


def side_by_side(s, n_layers, n_micro, n_live, packed=True, bf16=True, buffers=None):
    es = 2 if bf16 else 4
    cfg = hh.make_cfg(s.hidden, s.n_heads, s.head_dim, s.ffn, s.seq, s.micro_batch, s.rms_eps, s.rope_base,
                      hh.HH_BF16 if bf16 else hh.HH_F32, n_kv_heads=s.kv_heads)
    rows = {"wq": s.attn, "wk": s.attn_kv, "wv": s.attn_kv, "w_gate": s.ffn, "w_up": s.ffn}

    def layer(struct, es):
        out, at = struct(), 1 << 36
        for n in NAMES:
            setattr(out, n, at)
            at += rows[n] * s.hidden * es + (0 if packed else 256) if n in rows else 1 << 30
        return out
    ws = (hh.hh_layer_weights * n_layers)(*[layer(hh.hh_layer_weights, es)] * n_layers)
    gs = (hh.hh_layer_grads * n_layers)(*[layer(hh.hh_layer_grads, 4)] * n_layers)
    ptrs = [(C.c_void_p * n_micro)(*b) for b in buffers or boundary(s, es, n_micro)]
    return hh.lib.hh_internal_side_by_side(C.byref(cfg), n_layers, ws, gs, n_micro, n_live, *ptrs)
