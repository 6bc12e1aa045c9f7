"""Which launches the bf16 GEMM dispatch chooses for a layer's projections, asked of the library without a GPU."""
import ctypes as C

from paper_2405_16256_amd import binding as hh

NT, NN, TN = 0, 1, 2


def _ints(problems):
    flat = [v for p in problems for v in (tuple(p) + (0, 0))[:6]]
    return (C.c_int * len(flat))(*flat)


def plan(problems):
    """[(how, tile, k shares)] of the problems (kind, M, N, K, first k of B's second and third segment) of one call."""
    out = C.create_string_buffer(1024)
    assert hh.lib.hh_internal_gemm_plan(_ints(problems), len(problems), out, C.c_size_t(len(out))) == 0
    rows = [line.split() for line in out.value.decode().splitlines()]
    return [(how, tile, int(shares)) for how, tile, shares in rows]


def _calls(s, packed):
    """The GEMMs of a layer, [(name, problem)] of each call: those up to d(m), and the three groups of the backward pass."""
    T, H, F, A, Akv = s.tokens, s.hidden, s.ffn, s.n_heads * s.head_dim, s.kv_heads * s.head_dim
    Q3 = A + 2 * Akv
    qkv, gu = ({"qkv": Q3}, {"gate|up": 2 * F}) if packed else ({"q": A, "k": Akv, "v": Akv}, {"gate": F, "up": F})
    calls = [[(n, (NT, T, w, H)) for n, w in qkv.items()], [("out", (NT, T, H, A))], [(n, (NT, T, w, H)) for n, w in gu.items()],
             [("down", (NT, T, H, F))], [("d down", (NN, T, F, H))]]
    groups = [[("dW down", (TN, H, F, T))] + [("dW " + n, (TN, w, H, T)) for n, w in gu.items()]
              + [("d gate|up", (NN, T, H, 2 * F, 0 if packed else F))],
              [("dW out", (TN, H, A, T)), ("d out", (NN, T, A, H))],
              [("dW " + n, (TN, w, H, T)) for n, w in qkv.items()] + [("d qkv", (NN, T, H, Q3) + (() if packed else (A, A + Akv)))]]
    return calls, groups


def defers(s, packed=True):
    """Whether the layer leaves its weight gradients to one launch at the end of its backward pass."""
    groups = _calls(s, packed)[1]
    defer = hh.lib.hh_internal_gemm_defer(_ints([p for g in groups for _, p in g]), (C.c_int * 3)(*[len(g) for g in groups]))
    assert defer in (0, 1)
    return bool(defer)


def layer_launches(s, packed=True):
    """{name of the GEMM: (how, tile, k shares)} of a forward and a backward pass of a layer."""
    calls, groups = _calls(s, packed)
    if defers(s, packed):
        calls += [g[-1:] for g in groups] + [[q for g in groups for q in g[:-1]]]
    else:
        calls += groups
    return {n: r for call in calls for (n, _), r in zip(call, plan([p for _, p in call]))}
