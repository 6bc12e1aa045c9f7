"""How many micro-batches a stage step takes through its launches side by side, asked of the library without a GPU."""
import ctypes as C

from paper_2405_16256_amd import binding as hh

NAMES = ("g_attn", "wq", "wk", "wv", "wo", "g_mlp", "w_gate", "w_up", "w_down")


def boundary(s, es, n_micro, in_place=False, base=1 << 40):
    """x, y, dy, dx as addresses of buffers of their own."""
    step = 2 * s.seq * s.micro_batch * s.hidden * es
    x, y, dy, dx = [[base + (4 * m + i) * step for m in range(n_micro)] for i in range(4)]
    return [x, y, dy, dy if in_place else dx]


def _stage(s, n_layers, packed, bf16):
    """cfg and the layers' weights and gradients, at addresses of their own."""
    cfg = hh.make_cfg(s.hidden, s.n_heads, s.head_dim, s.ffn, s.seq, s.micro_batch, s.rms_eps, s.rope_base,
                      hh.HH_BF16 if bf16 else hh.HH_F32, n_kv_heads=s.kv_heads)
    rows = {"wq": s.attn, "wk": s.attn_kv, "wv": s.attn_kv, "w_gate": s.ffn, "w_up": s.ffn}

    def layer(struct, es, at):
        out = struct()
        for n in NAMES:
            setattr(out, n, at)
            at += rows[n] * s.hidden * es + (0 if packed else 256) if n in rows else 1 << 32
        return out
    ws = (hh.hh_layer_weights * n_layers)(*[layer(hh.hh_layer_weights, 2 if bf16 else 4, (1 << 44) + (l << 36)) for l in range(n_layers)])
    gs = (hh.hh_layer_grads * n_layers)(*[layer(hh.hh_layer_grads, 4, (1 << 45) + (l << 36)) for l in range(n_layers)])
    return cfg, ws, gs


POOL, WORKSPACE = 1 << 46, 1 << 47


def side_by_side(s, n_layers, n_micro, n_live, packed=True, bf16=True, buffers=None, change=None):
    """change(weights, gradients): what to make of the layers' structs before."""
    cfg, ws, gs = _stage(s, n_layers, packed, bf16)
    if change:
        change(ws, gs)
    ptrs = [(C.c_void_p * n_micro)(*b) for b in buffers or boundary(s, 2 if bf16 else 4, n_micro)]
    return hh.lib.hh_internal_side_by_side(C.byref(cfg), n_layers, ws, gs, n_micro, n_live, *ptrs, C.c_void_p(POOL), C.c_void_p(WORKSPACE))


TENSORS = ("m", "dgu", "dhn", "dh", "da", "dqkv", "dvec", "dkv_part", "partial", "gbuf")


def side_tensors(s, n_layers, packed=True):
    """{tensor: (first byte, end)} in the memory of one of several bf16 micro-batches that go side by side, and its size."""
    cfg, ws, gs = _stage(s, n_layers, packed, True)
    at, dkv_part = (C.c_size_t * (len(TENSORS) + 1))(), C.c_size_t()
    hh.lib.hh_internal_side_layout(C.byref(cfg), n_layers, ws, gs, at, C.byref(dkv_part))
    T, H, Q3 = s.tokens, s.hidden, s.attn + 2 * s.attn_kv
    stats, gain = s.micro_batch * s.n_heads * s.seq * 4, (min(T, 256) * H * 4 + 255) // 256 * 256
    sizes = (T * s.ffn * 2, T * 2 * s.ffn * 2, T * H * 2, T * H * 2, T * s.attn * 2, T * Q3 * 2, stats, dkv_part.value, 2 * gain, T * H * 2)
    return {n: (at[i], at[i] + b) for i, (n, b) in enumerate(zip(TENSORS, sizes))}, at[len(TENSORS)]


def backward_steps(defer):
    """What the launches of a layer's backward pass read and write, in their order, of the tensors above."""
    to_wd, to_gu, to_o, to_qkv = ["gbuf", "m"], ["dgu"], ["dh"], ["dqkv"]
    late = to_wd + to_gu + to_o + to_qkv if defer else []
    return [("d(m), SwiGLU", ["gbuf"], ["m", "dgu"]), ("d(hn)", ["dgu"] + ([] if defer else to_wd + to_gu), ["dhn"]),
            ("MLP norm", ["dhn", "gbuf"], ["dh", "partial"]), ("d(a)", ["dh"], ["da"]),
            ("delta", ["da"], ["dvec"]), ("partial dK, dV", ["da", "dvec"], ["dkv_part"]), ("attention", ["da", "dvec", "dkv_part"], ["dqkv"]),
            ("d(xn)", ["dqkv"] + ([] if defer else to_qkv), ["dhn"]), ("weight gradients", late, []),
            ("attention norm", ["dhn", "dh", "partial"], ["gbuf"]), ("gain sums", ["partial"], [])]


def overwritten(tensors, steps):
    """[(launch, tensor, by)] where a launch reads a tensor after another one that overlaps it has been written, by which."""
    clobbered, found = {}, []
    for name, reads, writes in steps:
        found += [(name, r, clobbered[r]) for r in reads if r in clobbered]
        for w in writes:
            clobbered.pop(w, None)
            for t, (a, b) in tensors.items():
                if t != w and a < tensors[w][1] and tensors[w][0] < b:
                    clobbered[t] = w
    return found
