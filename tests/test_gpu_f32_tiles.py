"""Chain cycles of fp32 models whose rows fit one pass (up to 1024 values): every number of K blocks per wavefront, wavefronts with fewer or none,
1 to 16 rows, draft steps that add table rows (one to four sequences) and that run the fusion FC (five and more, also beyond the eight whose
cache lengths travel in the arguments)."""
import pytest

import synth                                            # noqa: F401  (puts the repository on the path)
import test_gpu_f32_widths as widths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,K,kw", [
    (1, 4, dict(d=16, ffn=16)), (1, 1, dict(d=64, ffn=32)), (1, 15, dict(d=144, ffn=272)), (2, 7, dict(d=256, ffn=688)), (3, 4, dict(d=272, ffn=528)),
    (4, 3, dict(d=528, ffn=768, qkv_bias=True)), (1, 4, dict(d=784, ffn=1008)), (3, 2, dict(d=1008, ffn=1024)), (1, 4, dict(d=1024, ffn=912)),
    (5, 2, dict(d=256, ffn=400)), (8, 1, dict(d=144, ffn=64, vocab=1040)), (9, 2, dict(d=272, ffn=144)), (10, 2, dict(d=64, ffn=272, qkv_bias=True)), (16, 1, dict(d=64, ffn=272)),
], ids=lambda x: "-".join(f"{k}{v}" for k, v in x.items()) if isinstance(x, dict) else str(x))
def test_one_pass(batch, K, kw):
    """(sums shorter than those the tolerance there is derived for)"""
    widths.test_cycles(batch, K, kw)
