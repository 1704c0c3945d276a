"""The K sums of the LM head in passes of 9..64 rows, alone: the features that a pass returns are that product's operand, so the
logits are compared with the 64-bit product of the same high + low bf16 parts.  What is left is the rounding of the sums."""
import numpy as np
import pytest

import synth
from test_gpu_prefill_shapes import cfg_of

pytestmark = pytest.mark.gpu


def bf16(x):
    """nearest bf16 (ties to even) as float32"""
    u = np.ascontiguousarray(x, np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


# Relative 2-norm error with K = 4096.  A K block is four roundings of its sum, each 2^-24 / sqrt(3) * 0.7 of a value that grows with the root of the steps: a sum of n blocks errs
# by sqrt(2 n + 0.5) * 2.5e-8, and low parts added to the same sums make that n twice as large.  On 4096 columns n is 8 for all of these: 12 and 16 rows, eight
# wavefronts with two sums each of the high parts; 32 and 61 rows, 4 slices that four wavefronts share.  1.0e-7, measured 1.06e-7 to 1.09e-7; 1.4e-7 with the low parts in them.
# 61 rows on 32000 columns: one slice that two wavefronts share, n = 64: 2.8e-7, measured 2.75e-7; 4.0e-7 with the low parts.  The limits lie between the two.
@pytest.mark.parametrize("batch,K,nodes,vocab,limit", [(2, 5, 0, 4096, 1.25e-7), (2, 7, 0, 4096, 1.25e-7), (4, 7, 0, 4096, 1.25e-7), (1, 5, 60, 4096, 1.25e-7), (1, 5, 60, 32000, 3.4e-7)])
def test_lm_head_sums(batch, K, nodes, vocab, limit):
    from paper_2509_23928_amd import Hivis
    cfg = cfg_of(batch=batch, K=K, n_layers=1, d=4096, n_q_heads=2, n_kv_heads=2, head_dim=64, ffn=64, vocab=vocab, n_vis=9, n_text=7)
    w = synth.make_weights(cfg, seed=1)
    vis, ids = synth.make_prompt(cfg, seed=1)
    hv = Hivis(cfg, w, max_text=120)
    hv.prefill(vis, ids)
    if nodes:
        hv.tree_draft(10, 6, nodes)
        hv.tree_verify()
        rows = nodes + 1
    else:
        hv.draft(K)
        hv.verify()
        rows = batch * (K + 1)
    logits, g = hv.get_logits(0).reshape(rows, -1), hv.get_hidden(0).reshape(rows, -1)
    hv.close()
    hi = bf16(g)
    a = hi.astype(np.float64) + bf16(g - hi)
    head = np.asarray(w["lm_head"], np.float64)
    ref = a @ head.T
    err = np.linalg.norm(logits - ref) / np.linalg.norm(ref)
    print(f"{rows} rows: {err:.3e}")
    assert err <= limit
