"""Chain cycles of bf16 models at the sizes where the GEMMs on row fragments change form: row counts around 8, a K of 2048 and one block
more, K blocks that the wavefronts share unevenly, one to nine tiles per workgroup (q|k|v 1, 2, 3; gate|up 1, 2, 3, 4, 6, 7, 9; logits 1, 3, 5, 7
and 10, the last in two groups; O and down 1 and, 4128 wide, 2), a ragged last group, widths whose sums of squares are no multiple of
four, and a row width beyond what they serve.  Against the CPU oracle, as the passes of 9..16 rows are.  (Four tiles of q|k|v, nine of logits
and the longer rows of the other group sizes: the slices of the full widths in test_gpu_parity.py.)"""
import pytest

import test_gpu_rows16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,K,kw", [
    (1, 1, {}), (1, 6, dict(d=96, n_q_heads=3, n_kv_heads=1)), (1, 7, {}), (1, 8, dict(d=96, n_q_heads=3, n_kv_heads=1)),
    (1, 2, dict(d=2048, ffn=2080)), (2, 5, dict(d=2048, ffn=2080)), (1, 2, dict(d=2080, ffn=2048)), (2, 5, dict(d=2080, ffn=2048)),
    (1, 3, dict(ffn=5632, vocab=36880)), (2, 5, dict(ffn=5632, vocab=36880)),              # 3 tiles of gate|up, two groups of logits
    (1, 3, dict(ffn=8192, vocab=24592)), (3, 3, dict(ffn=14336, vocab=16400)),              # 4 and 7 tiles; 7 and 5 of logits
    (1, 3, dict(vocab=8208)), (2, 5, dict(vocab=8208)),                                     # 3 tiles of logits
    (1, 4, dict(n_q_heads=64, n_kv_heads=8)), (2, 5, dict(n_q_heads=64, n_kv_heads=8)),     # 2 tiles of q|k|v
    (1, 4, dict(ffn=18432, n_q_heads=48, n_kv_heads=8)), (2, 4, dict(ffn=10304, n_q_heads=96, n_kv_heads=48)),      # 9 and 6 tiles of gate|up; 1 and 3 of q|k|v
    (1, 3, dict(d=4128, ffn=64, n_layers=1)), (2, 4, dict(d=4128, ffn=64, n_layers=1)), (1, 2, dict(d=8224, ffn=64, n_layers=1)),
], ids=lambda x: "-".join(f"{k}{v}" for k, v in x.items()) if isinstance(x, dict) else str(x))
def test_sizes(batch, K, kw):
    test_gpu_rows16.test_rows_9_to_16(batch, K, kw)
