"""Chain cycles of fp32 models on rows of more than one K pass (1024 values), against the CPU oracle following the library's tokens: a
pass more by one block, two whole ones, three; draft steps of one to four sequences with the fusion FC on the LM head's launch
(hivis_draft and hivis_draft_noalloc in turn); matrices of at most one tile per workgroup, and of more."""
import numpy as np
import pytest

import synth
from oracle import HivisOracle, accept_length
from test_gpu_prefill_shapes import rel

pytestmark = pytest.mark.gpu

# A float32 sum of up to 2064 products runs in at least 32 chains (eight wavefronts, four K lanes of the matrix instruction), so its
# roundings of 2^-24 walk sqrt(2064 / 32) = 8 of them far.  Contractions in the chain: 21 up to the drafter's pending row, 9 per draft step.
REL = (21 + 9 * 3) * 8 * 2.0 ** -24


@pytest.mark.parametrize("batch,K,kw", [
    (1, 4, dict(d=1040)), (3, 3, dict(d=1040)), (1, 4, dict(d=2048, n_q_heads=16, n_kv_heads=4)), (4, 3, dict(d=2048, n_q_heads=16, n_kv_heads=4)),
    (1, 3, dict(d=2064)), (3, 3, dict(d=2064, qkv_bias=True)), (4, 3, dict(d=256)),
    (1, 3, dict(d=2064, n_q_heads=64, n_kv_heads=4, vocab=2048)), (3, 3, dict(d=1040, ffn=2064, vocab=4112)),      # more than 256 tiles: q|k|v; gate|up and LM head
], ids=lambda x: "-".join(f"{k}{v}" for k, v in x.items()) if isinstance(x, dict) else str(x))
def test_cycles(batch, K, kw):
    from paper_2509_23928_amd import Hivis
    base = dict(name="f32-widths", n_layers=2, d=1040, n_q_heads=8, n_kv_heads=4, head_dim=64, ffn=1056, vocab=528, dtype="f32",
                n_vis=20, n_text=11, K=K, batch=batch, gen_tokens=0, gen_cycles=3)
    base.update(kw)
    cfg = synth.HivisConfig(**base)
    w = synth.make_weights(cfg, seed=3)
    vis, ids = synth.make_prompt(cfg, seed=3)
    hv = Hivis(cfg, w)
    first = hv.prefill(vis, ids)
    oracles = [HivisOracle(cfg, w) for _ in range(batch)]
    for b, o in enumerate(oracles):
        assert o.prefill(vis[b], ids[b])[0] == int(first[b])
        assert rel(hv.get_hidden(1)[b], o.f_next) <= REL
    for cycle in range(2):
        (hv.draft_noalloc if cycle else hv.draft)(K)
        hv.verify()
        drafts, ttok = hv.get_tokens()
        dlog, vlog = hv.get_logits(1), hv.get_logits(0)
        n, toks = hv.accept()
        hidden = hv.get_hidden(1)
        for b, o in enumerate(oracles):
            _, ref = o.draft(K, follow=drafts[b])
            assert rel(dlog[:, b], ref) <= REL
            assert [int(x) for x in drafts[b]] == [int(x) for x in np.argmax(dlog[:, b], axis=-1)]
            g, ref, t = o.verify(drafts[b])
            assert rel(vlog[b], ref) <= REL
            assert list(ttok[b]) == [int(x) for x in np.argmax(vlog[b], axis=-1)]
            m = accept_length(drafts[b], ttok[b, :K])
            emitted = [int(x) for x in drafts[b, :m]] + [int(ttok[b, m])]
            assert int(n[b]) == m and [int(x) for x in toks[b, :m + 1]] == emitted
            o.accept(drafts[b], g, t, force=(m, emitted))
            assert rel(hidden[b], o.f_next) <= REL
    hv.close()


@pytest.mark.parametrize("kw,lengths", [
    (dict(n_q_heads=32, n_kv_heads=8, head_dim=128), [9, 2000]),             # verify and re-feed: items of one row each, then shared
    (dict(n_q_heads=32, n_kv_heads=8, head_dim=128, batch=2), [12, 1700, 30]),      # draft steps as well
], ids=["verify", "draft"])
def test_items_of_short_and_long_caches(kw, lengths):
    """One context (and its phase programs) on both sides of the rule that cuts the attention into items."""
    from paper_2509_23928_amd import Hivis
    K = 3
    cfg = synth.HivisConfig(**{**dict(name="f32-items", n_layers=1, d=64, ffn=64, vocab=528, dtype="f32", n_vis=0, n_text=max(lengths), K=K, batch=1,
                                      gen_tokens=0, gen_cycles=2), **kw})
    w = synth.make_weights(cfg, seed=4)
    vis, ids = synth.make_prompt(cfg, seed=4)
    hv = Hivis(cfg, w)
    for n in lengths * 2:
        first = hv.prefill(vis, np.ascontiguousarray(ids[:, :n]))
        hv.draft(K)
        hv.verify()
        drafts, dlog, vlog = hv.get_tokens()[0], hv.get_logits(1), hv.get_logits(0)
        hv.accept()
        hidden = hv.get_hidden(1)
        for b in range(cfg.batch):
            o = HivisOracle(cfg, w)
            assert o.prefill(vis[b], ids[b, :n])[0] == int(first[b])
            assert rel(dlog[:, b], o.draft(K, follow=drafts[b])[1]) <= REL
            g, ref, t = o.verify(drafts[b])
            assert rel(vlog[b], ref) <= REL
            o.accept(drafts[b], g, t)
            assert rel(hidden[b], o.f_next) <= REL
    hv.close()
