"""bf16 attention on launches of few workgroups: keys split between two wave groups, both backward passes and delta in one
launch.  Sequence lengths around a 64-key tile, a pair of them and a 128-query block, with grouped heads (summed in one
workgroup or through partial sums), on both sides of the rules that choose these forms.

Tolerances are those of every bf16 layer test.
"""
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
    # 257 workgroups of at most 512 queries: one group of waves per query block, two kernels backward
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, I.LayerShape(64, 1, 64, 64, 100, 257), True, 702, label="attn 257")
