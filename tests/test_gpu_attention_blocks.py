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


# the switches of the key splits: partials merged by a launch of their own; an item's splits over all XCDs (bit 1 clear), fences around its counter (bit 0 clear)
@pytest.mark.gpu
@pytest.mark.parametrize("name,value", [("HIVIS_ATTN_ELECT", "0"), ("HIVIS_ATTN_FLAGS", "0"), ("HIVIS_ATTN_FLAGS", "1"), ("HIVIS_ATTN_FLAGS", "2")])
def test_split_switches(name, value, monkeypatch):
    monkeypatch.setenv(name, value)
    monkeypatch.setitem(globals(), "LENGTHS", [9, 124, 381, 650])
    for hq, hkv, hd, K, batch in [(32, 32, 128, 5, 1), (7, 1, 64, 1, 2)]:
        test_cache_lengths(hq, hkv, hd, K, batch)
    test_fp32_cache_lengths(28, 4, 128, 6, 1)
    check_prefill(cfg_of(n_vis=600, n_text=61, d=64, ffn=64, n_q_heads=28, n_kv_heads=4, head_dim=128))        # items of 16 pairs


# ---- launches whose workgroups walk many blocks: the form without a barrier per block (attn_tiles_kernel)

def walks(tmp_path, hd, items, rm, keys, most):
    """Whether such a launch takes that form on 256 CUs."""
    lib = load("""#include "hivis_sizes.h"
using namespace hivis;
extern "C" int walks(int hd, int items, int rm, int keys, int most) { return attn_walks(256, hd, items, rm, attn_blocks(keys, attn_block_splits(keys, most))); }""", tmp_path)
    return bool(lib.walks(hd, items, rm, keys, most))


def test_walked_blocks_rule(tmp_path):
    for hd, items, rm, keys, most, want in [(128, 256, 16, 640, 1, False), (128, 256, 16, 641, 1, True), (64, 256, 16, 256, 1, False), (64, 256, 16, 257, 1, True), (128, 257, 8, 384, 1, False),
                                            (128, 257, 8, 385, 1, True), (64, 257, 8, 128, 1, False), (64, 257, 8, 129, 1, True), (128, 256, 8, 4000, 1, False), (128, 32, 16, 4000, 8, False)]:
        assert walks(tmp_path, hd, items, rm, keys, most) == want, (hd, items, rm, keys, most)


# a prompt's last rows, 16 pairs per item: more items than CUs, as many, and fewer (two key splits each); a short last block and row block
@pytest.mark.gpu
@pytest.mark.parametrize("heads,n_vis,n_text,items,most", [((40, 40, 128), 600, 127, 320, 1), ((32, 32, 128), 700, 113, 256, 1), ((36, 36, 64), 130, 127, 288, 1), ((32, 8, 64), 700, 61, 128, 2)], ids=str)
def test_walked_blocks_of_a_prompt(heads, n_vis, n_text, items, most, tmp_path):
    hq, hkv, hd = heads
    assert walks(tmp_path, hd, items, 16, n_vis + n_text, most)
    check_prefill(cfg_of(n_vis=n_vis, n_text=n_text, d=64, ffn=64, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd))


# decode passes of eight sequences, one and two rows each (K = 1); at 800 keys of 40 heads the caches outgrow the memory-side cache (256 MB) and are read with the hint
@pytest.mark.gpu
@pytest.mark.parametrize("heads,lengths", [((40, 40, 128), (385, 500, 800)), ((36, 36, 64), (129, 255, 300))], ids=str)
def test_walked_blocks_of_many_sequences(heads, lengths, tmp_path, monkeypatch):
    hq, hkv, hd = heads
    assert all(walks(tmp_path, hd, 8 * hkv, 8, n, 1) for n in lengths)
    monkeypatch.setitem(globals(), "LENGTHS", list(lengths))
    test_cache_lengths(hq, hkv, hd, 1, 8)


# rows of a draft tree: 61 rows of 36 heads over 3 and 4 blocks
@pytest.mark.gpu
def test_walked_blocks_of_a_tree(tmp_path):
    from test_gpu_tree import TreeSideBySide, small_bf16
    assert walks(tmp_path, 64, 36 * 4, 16, 300 + 9 + 61, 1)
    t = TreeSideBySide(small_bf16(n_q_heads=36, n_kv_heads=36, head_dim=64, n_vis=300, n_text=9), 3)
    t.cycle(10, 6, 60)
    t.cycle(10, 6, 60)
    t.hv.close()
