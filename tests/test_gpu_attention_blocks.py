"""Attention over half-precision caches in blocks of 128 keys: cache lengths around one, two and three blocks, a tile of 16 and a key more or less,
key splits with a short or an empty last one; 64- and 128-wide heads; one to eight (head,row) pairs per item, and sixteen where a prompt's last
rows are more than eight."""
import itertools

import numpy as np
import pytest

import synth
from host_header import load
from oracle import HivisOracle
from test_gpu_prefill_shapes import REL, cfg_of, check_prefill, rel


def test_splits_take_as_few_blocks_as_they_can(tmp_path):
    lib = load("""#include "hivis_sizes.h"
extern "C" int splits(int keys, int most) { return hivis::attn_block_splits(keys, most); }""", tmp_path)
    for keys, most in itertools.product(range(1, 4000), [1, 2, 3, 8, 16]):
        n = lib.splits(keys, most)
        blocks = -(-keys // (128 * most))
        per = (-(-keys // n) + 15) // 16 * 16                   # a split's keys, as the kernel cuts them
        assert 1 <= n <= most and per <= 128 * blocks and (n == 1 or 128 * blocks * (n - 1) < keys), (keys, most, n)


LENGTHS = [1, 9, 112, 123, 124, 125, 140, 251, 252, 380, 381, 650]


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,hd,K,batch", [(4, 4, 128, 4, 1), (4, 4, 64, 4, 1), (6, 2, 128, 1, 1), (7, 1, 64, 1, 2), (32, 32, 128, 5, 1), (28, 4, 128, 6, 1), (16, 2, 64, 2, 3)],
                         ids=str)
def test_cache_lengths(hq, hkv, hd, K, batch, dtype="bf16", tol=REL):
    from paper_2509_23928_amd import Hivis
    cfg = cfg_of(name="blocks", dtype=dtype, n_layers=1, d=64, ffn=64, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, n_text=max(LENGTHS), K=K, batch=batch, gen_cycles=2)
    w = synth.make_weights(cfg, seed=4)
    vis, ids = synth.make_prompt(cfg, seed=4)
    hv = Hivis(cfg, w)
    for n in LENGTHS:
        first = hv.prefill(vis, np.ascontiguousarray(ids[:, :n]))
        hv.draft(K)
        hv.verify()
        drafts, dlog, vlog = hv.get_tokens()[0], hv.get_logits(1), hv.get_logits(0)
        hv.accept()
        hidden = hv.get_hidden(1)
        for b in range(batch):
            o = HivisOracle(cfg, w)
            assert o.prefill(vis[b], ids[b, :n])[0] == int(first[b])
            assert rel(dlog[:, b], o.draft(K, follow=drafts[b])[1]) <= tol, n
            g, ref, t = o.verify(drafts[b])
            assert rel(vlog[b], ref) <= tol, n
            o.accept(drafts[b], g, t)
            assert rel(hidden[b], o.f_next) <= tol, n
    hv.close()


# fp32 caches: one (head,row) pair per item and up to eight, one key split and several.  32-bit sums of a few hundred terms in two layers' worth of contractions: 1e-5.
@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,hd,K,batch", [(4, 4, 64, 4, 1), (6, 2, 128, 1, 1), (7, 1, 64, 1, 2), (32, 32, 128, 5, 1), (16, 2, 64, 2, 3), (28, 4, 128, 6, 1)], ids=str)
def test_fp32_cache_lengths(hq, hkv, hd, K, batch):
    test_cache_lengths(hq, hkv, hd, K, batch, dtype="f32", tol=1e-5)


@pytest.mark.gpu
@pytest.mark.parametrize("n_vis", [0, 79, 88, 216, 600])
@pytest.mark.parametrize("heads,n_text", [((32, 8, 64), 40), ((8, 8, 128), 33), ((6, 2, 64), 17), ((28, 4, 128), 61)], ids=str)
def test_last_rows_of_a_prompt(n_vis, heads, n_text):
    hq, hkv, hd = heads
    check_prefill(cfg_of(n_vis=n_vis, n_text=n_text, d=64, ffn=64, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd))
