"""RMSNorm backward and the gain gradients at the edges of its kernels: a wave per row (up to 512 and 1024 bf16 elements,
256 and 512 fp32), a workgroup per row with a guarded and an exact length, rows that do not fit registers, one and several
rows per workgroup, and a workspace too small for a partial row per workgroup (narrow MLP).

The tolerance is that of every layer test: storage rounding for bf16, 1e-4 of each tensor's norm for fp32.
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


@pytest.mark.parametrize("bf16,hidden,ffn,seq,batch", [
    (True, 64, 64, 1, 1), (True, 512, 384, 300, 1), (True, 576, 384, 257, 1), (True, 1024, 64, 40, 1), (True, 1088, 704, 33, 2),
    (True, 2048, 64, 20, 1), (True, 2112, 704, 300, 1), (True, 12352, 128, 9, 1),
    (False, 8, 8, 3, 1), (False, 256, 688, 258, 1), (False, 264, 8, 65, 2), (False, 520, 72, 300, 1), (False, 1032, 344, 17, 1),
    (False, 6152, 64, 5, 1),
])
def test_row_lengths(ctx, bf16, hidden, ffn, seq, batch):
    from tests.test_gpu_parity import check_layer
    check_layer(ctx, I.LayerShape(hidden, 1, 64, ffn, seq, batch), bf16, 601, label="norm bwd")
