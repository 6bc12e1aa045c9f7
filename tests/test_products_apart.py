"""Several micro-batches in one launch: a weight gradient's products one after the other in a workgroup, or each in a workgroup of
its own, added by the reduction in the same order.  The bits are those of one micro-batch after the other."""
import ctypes as C

import pytest

from paper_2405_16256_amd import binding as hh
from paper_2405_16256_amd import inputs as I
from tests import gemm_plans, stage_plans
from tests.test_stage_side_by_side import hh_sizes
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


@pytest.mark.gpu
@pytest.mark.parametrize("shape,M,acc,want", CASES, ids=IDS)
def test_same_bits(shape, M, acc, want):
    same_bits(shape, True, 1, M, M, acc, False, M, True)
