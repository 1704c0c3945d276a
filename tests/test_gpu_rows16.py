"""Chain cycles of bf16 models whose passes hold 9..16 rows, both ends of that range, ragged widths, against the CPU oracle following
the library's tokens: batch * (K + 1) rows of a verify and a re-feed, and batch rows of a draft step, whose fusion FC and layer run
where K >= 2 (batch 9 and 10: more sequences leave room for K = 1 only, which is the LM head alone)."""
import numpy as np
import pytest

import synth
from oracle import HivisOracle, accept_length
from test_gpu_prefill_shapes import REL, cfg_of, rel
from test_gpu_sampling import run_sampling

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,K,kw", [
    (3, 2, {}), (2, 4, {}), (2, 5, dict(ffn=2720, d=1024, n_q_heads=8, n_kv_heads=8, head_dim=128)), (4, 3, dict(n_q_heads=6, n_kv_heads=3, d=96, ffn=160)),
    (2, 7, dict(qkv_bias=True)), (1, 15, {}), (9, 1, {}), (12, 1, dict(vocab=1040)), (16, 1, {}),
    (9, 2, {}), (10, 2, dict(qkv_bias=True, vocab=1040)), (9, 2, dict(n_q_heads=6, n_kv_heads=3, d=96, ffn=160)),
], ids=lambda x: "-".join(f"{k}{v}" for k, v in x.items()) if isinstance(x, dict) else str(x))
def test_rows_9_to_16(batch, K, kw):
    from paper_2509_23928_amd import Hivis
    cfg = cfg_of(batch=batch, K=K, n_vis=20, n_text=11, gen_cycles=3, **kw)
    w = synth.make_weights(cfg, seed=3)
    vis, ids = synth.make_prompt(cfg, seed=3)
    hv = Hivis(cfg, w)
    first = hv.prefill(vis, ids)
    oracles = [HivisOracle(cfg, w) for _ in range(batch)]
    for b, o in enumerate(oracles):
        assert o.prefill(vis[b], ids[b])[0] == int(first[b])
    for _ in range(2):
        hv.draft(K)
        hv.verify()
        drafts, ttok = hv.get_tokens()
        dlog, vlog = hv.get_logits(1), hv.get_logits(0)
        n, toks = hv.accept()
        hidden = hv.get_hidden(1)
        for b, o in enumerate(oracles):
            _, ref = o.draft(K, follow=drafts[b])
            assert rel(dlog[:, b], ref) <= REL
            g, ref, t = o.verify(drafts[b])
            assert rel(vlog[b], ref) <= REL
            assert list(ttok[b]) == [int(x) for x in np.argmax(vlog[b], axis=-1)]
            m = accept_length(drafts[b], ttok[b, :K])
            emitted = [int(x) for x in drafts[b, :m]] + [int(ttok[b, m])]
            assert int(n[b]) == m and [int(x) for x in toks[b, :m + 1]] == emitted
            o.accept(drafts[b], g, t, force=(m, emitted))
            assert rel(hidden[b], o.f_next) <= REL
    hv.close()


def test_drawn_drafts_of_nine_sequences():
    run_sampling(cfg_of(batch=9, K=2, n_vis=5, n_text=7, gen_cycles=3, vocab=1040), 4, 2, 1.0)
