"""Products of 17..64 rows (bf16): every column tile and both row tiles of their kernel, K of whole and ragged stages of four blocks, K slices,
products that end in SiLU(gate) * up.  The prompt's rows go through q|k|v, O, gate|up and down, and all of them reach what is compared."""
import numpy as np
import pytest

import synth
from oracle import HivisOracle
from test_gpu_prefill_shapes import cfg_of, check_prefill, rel, REL

pytestmark = pytest.mark.gpu


# heads of 64 with 4 key heads: q|k|v has 64 (hq + 8) columns, gate|up 2 ffn; 256 workgroups take 4, 6, 8, 10, 12, 16 and 20 column tiles from
# 0, 16385, 24577, 32769, 40961, 49153 and 65537 columns on
@pytest.mark.parametrize("rows", [(11, 9), (0, 32), (14, 19), (40, 21), (0, 64)], ids=str)
@pytest.mark.parametrize("hq,ffn", [(4, 704), (256, 10016), (384, 16000), (512, 20480), (640, 20512), (700, 25024), (800, 30016), (1024, 32800)], ids=str)
def test_column_tiles(rows, hq, ffn):
    check_prefill(cfg_of(n_vis=rows[0], n_text=rows[1], d=96, n_q_heads=hq, n_kv_heads=4, ffn=ffn, n_layers=1, vocab=128))


@pytest.mark.parametrize("d,ffn", [(416, 2720), (1024, 5632), (1056, 4128)], ids=str)
@pytest.mark.parametrize("rows", [(3, 17), (28, 33)], ids=str)
def test_slices(rows, d, ffn):
    """13, 32 and 33 K blocks, down 85, 176 and 129: slices of whole stages, the last one short"""
    check_prefill(cfg_of(n_vis=rows[0], n_text=rows[1], d=d, n_q_heads=d // 32, n_kv_heads=d // 32, head_dim=64, ffn=ffn))


def test_what_a_failed_pass_leaves():
    """A prompt with Inf in an embedding row fails and leaves Inf and NaN in the operand buffers and in LDS; the next prompt, whose K blocks do
    not fill their stages, has its own values"""
    from paper_2509_23928_amd import Hivis
    cfg = cfg_of(n_vis=0, n_text=20, d=416, n_q_heads=8, n_kv_heads=8, ffn=2720)
    w = synth.make_weights(cfg, seed=5)
    vis, ids = synth.make_prompt(cfg, seed=5)
    bad = ids.copy()
    bad[0, 3] = 7
    ids[ids == 7] = 8
    w["embed"] = w["embed"].copy()
    w["embed"][7, 5:9] = np.inf
    hv = Hivis(cfg, w)
    o = HivisOracle(cfg, w)
    x, ref = o.prefill(vis[0], ids[0])
    for _ in range(3):
        with pytest.raises(RuntimeError):
            hv.prefill(vis, bad)
        first = hv.prefill(vis, ids)
        assert rel(hv.get_logits(2)[0], ref) <= REL and int(first[0]) == x
        assert rel(hv.get_hidden(1)[0], o.f_next) <= REL
    hv.close()
