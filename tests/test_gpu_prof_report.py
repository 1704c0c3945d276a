"""HIVIS_PROF: the report of a verify pass names a time for every GEMM and attention launch of its middle, and where their workgroups ran."""
import re

import pytest

import synth

pytestmark = pytest.mark.gpu
PH_GEMM, PH_ATTN = 0, 1


# bf16 row fragments and key splits; fp32 one-tile kernels and others; more attention workgroups than are recorded (eight sequences of 192 heads: 1536 items)
@pytest.mark.parametrize("kw", [dict(dtype="bf16"), dict(dtype="f32"), dict(dtype="f32", d=1040, ffn=1056), dict(dtype="bf16", batch=8, K=1, n_q_heads=192, n_kv_heads=192, n_layers=4)], ids=str)
def test_report(kw, monkeypatch, capfd):
    from paper_2509_23928_amd import Hivis
    base = dict(name="prof", n_layers=6, d=256, n_q_heads=8, n_kv_heads=8, head_dim=64, ffn=704, vocab=1024, dtype="f32", n_vis=150, n_text=9, K=4, batch=1, gen_tokens=0, gen_cycles=2)
    base.update(kw)
    cfg = synth.HivisConfig(**base)
    monkeypatch.setenv("HIVIS_PROF", "1")
    hv = Hivis(cfg, synth.make_weights(cfg, seed=0))
    hv.prefill(*synth.make_prompt(cfg, seed=0))
    hv.draft(cfg.K)
    hv.verify()
    hv.get_hidden(0)
    hv.close()
    err = capfd.readouterr().err
    phases = re.findall(r"\[hivis prof\] phase (\d+) type (\d+) epi \d+: (.*)", err)
    assert len(phases) >= 8
    for p, kind, text in phases:
        if int(kind) in (PH_GEMM, PH_ATTN):
            entry = re.match(r"entry ([+-][\d.]+) us after the entry of phase (\d+);(.*)", text)
            assert entry and 0 < float(entry[1]) < 1000, (p, text)
            marks = [float(m) for m in re.findall(r"m\d ([+-][\d.]+)", entry[3])]
            assert marks and all(0 <= m < 1000 for m in marks), (p, text)
    groups = re.findall(r"\[hivis wg\] phase \d+ type (\d+) epi \d+: (\d+) workgroups, entries within ([\d.]+) us; exits min ([\d.-]+) .*? max ([\d.]+) us; latest:(.*?);.*mean exit per xcc:(.*)", err)
    assert len(groups) == 8 and any(int(g[0]) == PH_ATTN for g in groups)
    for kind, n, spread, first, last, latest, xcc in groups:
        assert 0 <= float(spread) <= float(last) < 1000 and float(first) >= 0
        assert 1 <= int(n) <= 1024
        counts = [int(c) for c in re.findall(r"\((\d+)\)", xcc)]
        assert sum(counts) == int(n) and (int(n) < 64 or min(counts) > 0), (kind, xcc)      # (all eight XCCs)
