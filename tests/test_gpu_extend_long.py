"""Basis extension at the edges of the image rows' blocks, steps and turns, and on both sides of the rule for the sums of s."""
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_extend_wide import test_one_column as _one_column  # noqa: E402


# long rows: a block of u and a piece, with more rows than one turn of a launch takes; whole blocks and a piece; a step of
# 128 pieces and one less / more.  Sums of s by every workgroup: 32 slabs x 512 columns; by a launch of their own: 520
# columns, and fewer columns of very long rows
@pytest.mark.parametrize("d,K,k0,ms,dt", [(8200, 64, 3, (6200, 7), "bf16"), (16392, 64, 2, (9, 8), "bf16"), (4104, 64, 0, (3100,), "f32"),
                                          (1016, 64, 1, (1, 2), "bf16"), (1032, 64, 1, (15,), "bf16"), (512, 64, 5, (10,), "f32"),
                                          (2048, 512, 511, (8,), "bf16"), (2048, 520, 5, (17,), "bf16"),
                                          (131072, 160, 4, (5,), "bf16")])
def test_long_rows_and_sums(d, K, k0, ms, dt):
    _one_column(d, K, k0, ms, dt)
