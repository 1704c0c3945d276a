"""Which draft rounds hivis_draft_noalloc takes, at the limit of its static array: grouped heads in float32, whose attention items of one
row each need more room than items that share their keys (the round then runs with the latter), and rounds beyond the limit, refused.
What is taken drafts the same tokens as hivis_draft."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# 16 MB; an attention phase of a step takes partials x 8 rows x (head_dim + 2) floats: 64 partials for 4 key heads, 256 for 32 items
BASE = dict(name="noalloc-room", n_layers=1, d=64, ffn=64, vocab=256, n_vis=0, n_text=20, batch=1, gen_tokens=0, gen_cycles=2)


@pytest.mark.parametrize("K,fits,kw", [
    (31, True, dict(dtype="f32", n_q_heads=32, n_kv_heads=4, head_dim=128)), (31, True, dict(dtype="f32", n_q_heads=32, n_kv_heads=8, head_dim=64)),
    (16, True, dict(dtype="f32", n_q_heads=32, n_kv_heads=4, head_dim=128)), (31, False, dict(dtype="f32", n_q_heads=32, n_kv_heads=32, head_dim=128)),
    (17, False, dict(dtype="bf16", n_q_heads=28, n_kv_heads=28, head_dim=128)),
], ids=lambda x: "-".join(str(v) for v in x.values()) if isinstance(x, dict) else str(x))
def test_room(K, fits, kw):
    from paper_2509_23928_amd import Hivis, HivisError, HIVIS_ECAP
    cfg = synth.HivisConfig(K=K, **BASE, **kw)
    w = synth.make_weights(cfg, seed=1)
    vis, ids = synth.make_prompt(cfg, seed=1)
    hv = Hivis(cfg, w)
    hv.prefill(vis, ids)
    if not fits:
        with pytest.raises(HivisError) as e:
            hv.draft_noalloc(K)
        assert e.value.code == HIVIS_ECAP
        hv.close()
        return
    hv.draft_noalloc(K)
    hv.verify()
    drafts, logits = hv.get_tokens()[0], hv.get_logits(1)
    hv.prefill(vis, ids)
    hv.draft(K)
    hv.verify()
    ref = hv.get_logits(1)
    # (float32 sums in another order, over 31 dependent steps of 9 contractions: the walk of 2^-24 per contraction)
    assert np.linalg.norm(logits - ref) <= 31 * 9 * 2.0 ** -24 * np.linalg.norm(ref)
    assert np.array_equal(drafts, hv.get_tokens()[0])
    hv.close()
