"""Products of 17..64 rows (bf16): every column tile and both row tiles of their kernel, K of one stage of four blocks and of more stages than are in flight, whole
and ragged, K slices, products that end in SiLU(gate) * up.  The prompt's rows go through q|k|v, O, gate|up and down, and all of them reach what is compared."""
import ctypes

import numpy as np
import pytest

import synth
from host_header import load
from oracle import HivisOracle
from test_gpu_prefill_shapes import cfg_of, check_prefill, rel, REL

pytestmark = pytest.mark.gpu


# heads of 64 with 4 key heads: q|k|v has 64 (hq + 8) columns, gate|up 2 ffn; 256 workgroups take 4, 6, 8, 10, 12, 16 and 20 column tiles from
# 0, 16385, 24577, 32769, 40961, 49153 and 65537 columns on.  Three K blocks: one stage
@pytest.mark.parametrize("rows", [(11, 9), (0, 32), (14, 19), (40, 21), (0, 64)], ids=str)
@pytest.mark.parametrize("hq,ffn", [(4, 704), (256, 10016), (384, 16000), (512, 20480), (640, 20512), (700, 25024), (800, 30016), (1024, 32800)], ids=str)
def test_column_tiles(rows, hq, ffn):
    check_prefill(cfg_of(n_vis=rows[0], n_text=rows[1], d=96, n_q_heads=hq, n_kv_heads=4, ffn=ffn, n_layers=1, vocab=128))


# The same with 33 K blocks in one slice: nine stages, one more than the most of the ring (4) and of the weights (4) ahead of it together, so that every place of
# both is used again; the last stage has one block.  form: what the plan takes for q|k|v and for gate|up, at 20 rows and at 61 (the widest tile is for 32)
@pytest.mark.parametrize("hq,ffn,form", [(240, 704, 0), (300, 10016, 1), (384, 16000, 2), (520, 20480, 3), (640, 20512, 4), (768, 25024, 5), (1024, 32800, 6)], ids=str)
def test_more_stages_than_are_in_flight(hq, ffn, form, tmp_path):
    lib = load("""#include "hivis_sizes.h"
using namespace hivis;
extern "C" void plans(int M, int kblks, int qkv, int gateup, int* out) {
    const WidePlan p = wide_plan(256, M, kblks, qkv / 16, true), w = wide_plan(256, M, kblks, gateup / 16, false), s = wide_plan(256, M, kblks, gateup / 16, true);
    const int v[] = {p.form, p.ksplit, p.kper / WIDE_STAGE, w.form, w.kper / WIDE_STAGE, tall_fused(w, s)};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}""", tmp_path)
    shapes = {20: (3, 17), 61: (40, 21)}
    for rows in shapes:
        got = (ctypes.c_int * 6)()
        lib.plans(rows, 33, 64 * (hq + 8), 2 * ffn, got)
        want = 3 if rows > 32 and form == 6 else form
        assert list(got) == [want, 1, 9, want, 9, 1], rows
    from paper_2509_23928_amd import Hivis
    cfg = {rows: cfg_of(n_vis=v, n_text=t, d=1056, n_q_heads=hq, n_kv_heads=4, ffn=ffn, n_layers=1, vocab=128) for rows, (v, t) in shapes.items()}
    w = synth.make_weights(cfg[61], seed=0)
    hv = Hivis(cfg[61], w)
    for rows in (20, 61, 20):
        vis, ids = synth.make_prompt(cfg[rows], seed=0)
        first = hv.prefill(vis, ids)
        o = HivisOracle(cfg[rows], w)
        x, ref = o.prefill(vis[0], ids[0])
        assert rel(hv.get_logits(2)[0], ref) <= REL and int(first[0]) == x
        assert rel(hv.get_hidden(1)[0], o.f_next) <= REL
    hv.close()


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
