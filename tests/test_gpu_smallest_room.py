"""Passes of 32 and 61 rows in the smallest contexts that hold them (64 rows of room), with an inner width that makes the MLP's
operand rows wider than the buffer of the others, with and without the phase programs."""
import numpy as np
import pytest

import synth
from parity_utils import SideBySide
from test_gpu_prefill_shapes import cfg_of
from test_gpu_tree import TreeSideBySide

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused", ["1", "0"])
@pytest.mark.parametrize("ffn", [1024, 2304])
def test_tree_of_61_rows(monkeypatch, fused, ffn):
    monkeypatch.setenv("HIVIS_FUSED", fused)
    cfg = cfg_of(n_vis=0, n_text=2, ffn=ffn)
    t = TreeSideBySide(cfg, 5, room=62)
    t.cycle(10, 6, 60)
    t.hv.close()


@pytest.mark.parametrize("fused", ["1", "0"])
def test_chain_of_32_rows(monkeypatch, fused):
    from paper_2509_23928_amd import Hivis
    monkeypatch.setenv("HIVIS_FUSED", fused)
    cfg = cfg_of(batch=4, K=7, n_vis=1, n_text=5, ffn=2304)
    w = synth.make_weights(cfg, seed=6)
    vis, ids = synth.make_prompt(cfg, seed=6)
    hv = Hivis(cfg, w, max_text=15)
    sbs = SideBySide(cfg, w, hv, vis, ids)
    sbs.cycle(cfg.K, planted=np.full((4, 7), 3, np.int32))
    hv.close()
