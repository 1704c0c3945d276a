"""Prefill of bf16 models at the row counts and widths where its kernels change tiles, K slices or route, against the
CPU oracle.  Every row of the prompt reaches what is compared: the prompt's logits and the drafter's pending hidden state
attend to all rows' cached keys and values."""
import numpy as np
import pytest

import synth
from oracle import HivisOracle

pytestmark = pytest.mark.gpu

# Activations keep 16 mantissa bits between kernels (high + low bf16 part): every GEMM input carries a relative error of at
# most 2^-17, uncorrelated between elements, so a result's relative 2-norm error grows by at most that per contraction in
# the chain.  Two target layers and the drafter are 4 x 3 contractions plus fusion FC and LM head: 14 * 2^-17 = 1.1e-4.
REL = 14 * 2.0 ** -17


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b))


def check_prefill(cfg, seed=0, tol=REL):
    from paper_2509_23928_amd import Hivis
    w = synth.make_weights(cfg, seed=seed)
    vis, ids = synth.make_prompt(cfg, seed=seed)
    hv = Hivis(cfg, w)
    first = hv.prefill(vis, ids)
    logits, hidden = hv.get_logits(2), hv.get_hidden(1)
    for b in range(cfg.batch):
        o = HivisOracle(cfg, w)
        x, ref = o.prefill(vis[b], ids[b])
        assert rel(logits[b], ref) <= tol
        assert int(first[b]) == x
        assert rel(hidden[b], o.f_next) <= tol
    hv.close()


def cfg_of(**kw):
    base = dict(name="shapes", n_layers=2, d=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=704, vocab=512, dtype="bf16",
                n_vis=0, n_text=1, K=3, batch=1, gen_tokens=0, gen_cycles=1)
    base.update(kw)
    return synth.HivisConfig(**base)


@pytest.mark.parametrize("n_vis,n_text", [(0, 1), (0, 7), (0, 9), (3, 7), (0, 16), (0, 17), (30, 3), (0, 33), (0, 64), (64, 1), (0, 65), (17, 110),
                                          (0, 128), (100, 29), (0, 257), (383, 130)])
def test_row_counts(n_vis, n_text):
    check_prefill(cfg_of(n_vis=n_vis, n_text=n_text))


@pytest.mark.parametrize("kw", [
    dict(n_vis=1900, n_text=100, ffn=2048),                        # gate|up in one round of 256-column tiles
    dict(n_vis=1931, n_text=17, ffn=1792),                         # ... of 224-column tiles
    dict(n_vis=150, n_text=33, d=1024, n_q_heads=8, n_kv_heads=8, head_dim=128, ffn=2720),      # K slices in the O and down projections
    dict(n_vis=70, n_text=5, d=96, n_q_heads=3, n_kv_heads=1, head_dim=64, ffn=32),            # fewer columns and K blocks than one tile
    dict(n_vis=75, n_text=9, batch=3), dict(n_vis=0, n_text=5, batch=3), dict(n_vis=1, n_text=40, batch=2, qkv_bias=True),
    dict(n_vis=200, n_text=3, qkv_bias=True, n_q_heads=8, n_kv_heads=1),
], ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_widths(kw):
    check_prefill(cfg_of(**kw))


# the shared-tile attention: 64 rows per workgroup from 128 workgroups of 128 rows on, 128 rows from 512 on; last blocks of a few
# rows, key counts around the 32-key tile, and a prompt whose last block is one row
@pytest.mark.parametrize("kw", [dict(n_vis=513, n_text=32, n_q_heads=32, n_kv_heads=4), dict(n_vis=500, n_text=13, n_q_heads=32, n_kv_heads=32, head_dim=128),
                                dict(n_vis=380, n_text=33, n_q_heads=32, n_kv_heads=8, batch=4), dict(n_vis=350, n_text=35, n_q_heads=32, n_kv_heads=2, head_dim=128, batch=4),
                                dict(n_vis=480, n_text=32, n_q_heads=48, n_kv_heads=6, batch=3)],
                         ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_shared_attention(kw):
    check_prefill(cfg_of(**kw))


# query weights times 1, 16, 32, 128: over the key tiles a row's largest score grows by up to 0.7, 11, 22, 86 powers of two, below and above the growth (11) at
# which the shared-tile attention scales its sums.  A score s carries relative errors like any other result, and its weight that error times |s|:
# REL, and REL for each unit of the largest score (0.65 per factor of the weights).
@pytest.mark.parametrize("times", [1, 16, 32, 128])
@pytest.mark.parametrize("kw", [dict(n_vis=480, n_text=32, batch=1), dict(n_vis=400, n_text=33, batch=4)], ids=["64rows", "128rows"])
def test_shared_attention_of_growing_scores(kw, times):
    from paper_2509_23928_amd import Hivis
    cfg = cfg_of(n_q_heads=32, n_kv_heads=8, head_dim=128, **kw)
    w = synth.make_weights(cfg, seed=0)
    for layer in w["layers"] + [w["draft_layer"]]:
        layer["wq"] = layer["wq"] * np.float32(times)
    vis, ids = synth.make_prompt(cfg, seed=0)
    hv = Hivis(cfg, w)
    hv.prefill(vis, ids)
    logits, hidden = hv.get_logits(2), hv.get_hidden(1)
    hv.close()
    for b in range(cfg.batch):
        o = HivisOracle(cfg, w)
        _, ref = o.prefill(vis[b], ids[b])
        assert rel(logits[b], ref) <= REL * (1 + 0.65 * times)
        assert rel(hidden[b], o.f_next) <= REL * (1 + 0.65 * times)


# The same scores, with the low halves in sight: the first layer's attention (its output 64 times as large, no MLP) is what the results are made of, and they are compared
# with those of the kernel for few rows, which scales every block to its maximum and starts from the same queries and keys.  Weights without their low half, or
# values, put 1.4e-4 to 2.3e-4 between them (the oracle with such weights).  The two kernels' exponentials differ by 2^-24 of at most 125 powers of two, 7e-6, and
# what is left of that is rounded to 2^-17 in four contractions at most: 4e-5.
@pytest.mark.parametrize("times", [1, 32, 128])
@pytest.mark.parametrize("kw", [dict(n_vis=480, n_text=32, batch=1), dict(n_vis=400, n_text=33, batch=4)], ids=["64rows", "128rows"])
def test_shared_attention_keeps_low_halves(kw, times, monkeypatch):
    from paper_2509_23928_amd import Hivis
    cfg = cfg_of(n_q_heads=32, n_kv_heads=8, head_dim=128, **kw)
    w = synth.make_weights(cfg, seed=0)
    for layer in w["layers"] + [w["draft_layer"]]:
        layer["wd"] = layer["wd"] * np.float32(0)
    w["layers"][0]["wq"] = w["layers"][0]["wq"] * np.float32(times)
    w["layers"][0]["wo"] = w["layers"][0]["wo"] * np.float32(64)
    vis, ids = synth.make_prompt(cfg, seed=0)
    got = []
    for rows in ("128", "4096"):                                      # rows of a sequence from which the shared-tile kernel is taken
        monkeypatch.setenv("HIVIS_ATTN_SHARED_MIN", rows)
        hv = Hivis(cfg, w)
        hv.prefill(vis, ids)
        got.append((hv.get_logits(2), hv.get_hidden(1)))
        hv.close()
    for b in range(cfg.batch):
        for a, ref in zip(*got):
            err = rel(a[b], ref[b])
            print(f"times {times} sequence {b}: {err:.2e}")
            assert err <= 4e-5


@pytest.mark.parametrize("n_text", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17])
@pytest.mark.parametrize("heads", [(4, 4, 64), (6, 2, 64), (5, 1, 128)], ids=str)
def test_fp32_rows_of_an_attention_item(n_text, heads):
    """fp32 attention holds 1, 2, 4, 8 or 16 (head,row) pairs per work item.  32-bit sums of a few hundred terms in four layers'
    worth of contractions: 1e-5."""
    q, kv, hd = heads
    check_prefill(cfg_of(dtype="f32", n_vis=0, n_text=n_text, d=128, n_q_heads=q, n_kv_heads=kv, head_dim=hd, ffn=176), tol=1e-5)


# fp32 passes of many rows: 16, 8, 4, 2 and one (head,row) pairs per item, halved heads first, from even and odd counts, with one and with several key splits
@pytest.mark.parametrize("hq,hkv,hd,n_text", [(80, 80, 64, 32), (64, 64, 64, 31), (32, 32, 64, 32), (16, 16, 128, 32), (4, 4, 64, 32), (64, 8, 64, 4), (80, 40, 64, 5), (12, 4, 64, 11),
                                              (8, 8, 64, 333), (48, 16, 128, 290)], ids=str)
def test_fp32_rows_halved(hq, hkv, hd, n_text):
    check_prefill(cfg_of(dtype="f32", n_vis=0, n_text=n_text, d=128, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn=176), tol=1e-5)


def test_room_for_slices_grows_once(monkeypatch):
    """Without a reserve the first product that is cut into K slices allocates the room, for every row count of the context: the
    prompts after it, more and fewer rows, find it there."""
    import torch
    from paper_2509_23928_amd import Hivis
    monkeypatch.setenv("HIVIS_SPLITK_RESERVE", "0")
    cfg = cfg_of(n_vis=700, n_text=33, d=1024, n_q_heads=8, n_kv_heads=8, head_dim=128, ffn=2720, gen_cycles=4)
    w = synth.make_weights(cfg, seed=2)
    vis, ids = synth.make_prompt(cfg, seed=2)
    hv = Hivis(cfg, w)
    free = []
    for v, l in ((90, 33), (700, 33), (0, 20), (700, 11), (401, 9)):
        first = hv.prefill(vis[:, :v], ids[:, :l])
        free.append(torch.cuda.mem_get_info()[0])
        o = HivisOracle(cfg, w)
        x, ref = o.prefill(vis[0, :v], ids[0, :l])
        assert rel(hv.get_logits(2)[0], ref) <= REL and int(first[0]) == x
        assert rel(hv.get_hidden(1)[0], o.f_next) <= REL
    hv.close()
    assert len(set(free)) == 1, free
