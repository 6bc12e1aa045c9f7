"""Several micro-batches in one launch: a weight gradient's products one after the other in a workgroup, or each in a workgroup of
its own, added by the reduction in the same order.  The bits are those of one micro-batch after the other."""
import ctypes as C
import random

import pytest

from paper_2405_16256_amd import binding as hh
from paper_2405_16256_amd import inputs as I
from tests import gemm_plans, stage_plans
from tests.test_stage_side_by_side import DEFERRING, hh_sizes
from tests.test_stage_side_by_side import test_same_bits_as_one_by_one as same_bits

MB = 1 << 20
# shape, micro-batches, add to the gradients; the groups (MLP, wo, wq|wk|wv) with gradients whose products are apart, and which
CASES = [
    (I.LayerShape(768, 12, 64, 2048, 1499, 1), 2, True, {1: 1}),                              # rows of a k tile left over
    (I.LayerShape(512, 8, 64, 768, 1100, 2, n_kv_heads=2), 3, False, {0: 3}),                 # beside gradients in k shares
    (I.LayerShape(448, 7, 64, 512, 1700, 1, n_kv_heads=1), 4, True, {0: 3, 1: 1, 2: 1}),   # columns of a tile left over
]
IDS = ["%dx%d T%d M%d" % (c[0].hidden, c[0].ffn, c[0].tokens, c[1]) for c in CASES]


def apart(problems, micro, room):
    return hh.lib.hh_internal_products_apart(gemm_plans._ints(problems), len(problems), micro, C.c_size_t(room))


def groups(shape):
    return [[p for _, p in call] for call in gemm_plans._calls(shape, True)[1]]


@pytest.mark.parametrize("shape,M,acc,want", CASES, ids=IDS)
def test_rule(shape, M, acc, want):
    side = stage_plans.side_by_side(shape, 1, M, M)
    room = hh_sizes(shape, 1, M)[1] - side * stage_plans.side_tensors(shape, 1)[1]
    assert side == M
    assert {i: b for i, g in enumerate(groups(shape)) for b in [apart(g, M, room)] if b > 0} == want
    assert all(apart(g, M, 0) in (0, -1) for g in groups(shape))        # no room for partial sums
    assert all(apart(g, 1, room) in (0, -1) for g in groups(shape))


def test_rule_leaves_short_sums():
    for tokens in (64, 128, 333):
        for g in groups(I.LayerShape(1024, 8, 128, 2752, tokens, 1)):
            assert apart(g, 8, 512 * MB) in (0, -1), tokens


def test_gradients_of_few_tokens_stay_in_one_workgroup():
    # those that 256x256 tiles would take alone: they are bound by the traffic of the gradients, which partial sums would add to
    rng, seen = random.Random(9), set()
    shapes = [(I.LayerShape(64 * rng.randint(24, 192), rng.choice((4, 8, 16, 32, 64)), 128, 64 * rng.randint(16, 448), rng.randint(1, 448), 1),
               rng.random() < 0.7) for _ in range(600)] + [c[:2] for c in DEFERRING]
    for shape, packed in shapes:
        M = rng.randint(2, 8)
        calls = gemm_plans._calls(shape, packed)[1]
        if gemm_plans.defers(shape, packed):
            calls = [[q for g in calls for q in g[:-1]]]
        for problems in ([p for _, p in c] for c in calls):
            plans = gemm_plans.plan(problems)
            of = sum(1 << i for i, (r, p) in enumerate(zip(plans, problems)) if r[1] == "256x256" and p[0] == gemm_plans.TN)
            bits = apart(problems, M, 1 << 40)
            if of and bits >= 0:
                assert bits & of == 0, (shape, packed, M)
                seen.add((plans[0][0], len(problems)))
    assert {("alone", 2), ("alone", 4), ("tiles256", 4), ("tiles256", 7)} <= seen


@pytest.mark.gpu
@pytest.mark.parametrize("shape,M,acc,want", CASES, ids=IDS)
def test_same_bits(shape, M, acc, want):
    same_bits(shape, True, 1, M, M, acc, False, M, True)
