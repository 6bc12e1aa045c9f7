"""fp32 attention backward: whether both passes share a launch follows from the jobs of all samples and all micro-batches that go
side by side, and does not show in the results."""
import pytest

from paper_2405_16256_amd import binding as hh
from paper_2405_16256_amd import inputs as I
from tests import stage_plans
from tests.test_stage_side_by_side import test_same_bits_as_one_by_one as same_bits


def together(batch, seq, heads, kv_heads, head_dim, micro=1):
    return hh.lib.hh_internal_attn_f32_together(batch, seq, heads, kv_heads, head_dim, micro)


@pytest.mark.parametrize("head_dim,seq,heads,most", [(128, 500, 1, 10), (128, 44, 5, 21), (64, 640, 8, 6), (64, 128, 16, 16), (64, 1000, 10, 3)])
def test_samples_and_micro_batches_count(head_dim, seq, heads, most):
    # a sample's jobs: 64 and 30 of up to 640 at head_dim 128; 640, 256 and 1260 of 4096 at 64
    for n in range(1, 2 * most + 1):
        assert together(n, seq, heads, heads, head_dim) == (n <= most), n
        assert together(1, seq, heads, heads, head_dim, n) == (n <= most), n
        assert together(2, seq, heads, heads, head_dim, n) == (2 * n <= most), n


def test_workgroups_of_grouped_heads_count():
    # 22 tiles: 8 query heads and, for 2 key/value heads, 8 workgroups a tile; 352 jobs
    assert [together(1, 350, 8, 2, 128, n) for n in (1, 2)] == [1, 0]


# shape, micro-batches, side by side; the jobs of passes of 3 and 2 micro-batches, or of 2 and 1
CASES = [
    (I.LayerShape(64, 8, 128, 64, 220, 1), 7, 3),                   # 672 and 448
    (I.LayerShape(64, 8, 128, 64, 220, 1, n_kv_heads=2), 7, 3),
    (I.LayerShape(64, 3, 128, 64, 300, 1), 7, 3),                   # 342 and 228: 18 and 12 of a tile
    (I.LayerShape(64, 16, 64, 64, 700, 1), 7, 3),                   # 4224 and 2816
    (I.LayerShape(64, 16, 64, 64, 500, 2), 5, 2),                   # 4096 and 2048
]
IDS = ["%d heads on %d of %d, %d tokens" % (c[0].n_heads, c[0].kv_heads, c[0].head_dim, c[0].seq) for c in CASES]


@pytest.mark.parametrize("shape,M,side", CASES, ids=IDS)
def test_cases(shape, M, side):
    assert stage_plans.side_by_side(shape, 1, M, M, bf16=False) == side


@pytest.mark.gpu
@pytest.mark.parametrize("shape,M,side", CASES, ids=IDS)
def test_same_bits(shape, M, side):
    same_bits(shape, True, 1, M, M, True, False, side, False)
