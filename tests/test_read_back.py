"""Read-back calls where the rows that the library copies are not those of the binding's K: a draft round of another K, or a draft tree, since the pass that
the values belong to.  Rows that are not copied are zeros, and nothing is written behind an array."""
import ctypes as C
from types import SimpleNamespace

import numpy as np
import pytest

import synth


class Copies:
    """Stands for the library: counts rows as hivis_draft, hivis_verify and the tree calls do, and copies as many as they left."""

    def __init__(self, d, vocab):
        self.d, self.vocab, self.K, self.rows, self.nodes, self.sizes = d, vocab, 0, 0, 0, []

    def hivis_draft(self, ctx, K):
        self.K = K

    hivis_draft_noalloc = hivis_draft

    def hivis_draft_sample(self, ctx, K, t, u):
        self.K = K

    def hivis_set_drafts(self, ctx, tokens, K):
        self.K = K

    def hivis_verify(self, ctx):
        self.rows = self.K + 1

    def hivis_tree_draft(self, ctx, k, depth, n):
        self.nodes = n

    def hivis_tree_set(self, ctx, n, tokens, parents):
        self.nodes = n

    def hivis_tree_verify(self, ctx):
        self.rows = self.nodes + 1

    def copy(self, out, rows, width):
        np.ctypeslib.as_array(C.cast(out, C.POINTER(C.c_float)), (rows * width,))[:] = 1 + np.arange(rows).repeat(width)

    def hivis_get_logits(self, ctx, which, out):
        self.copy(out, {0: self.rows, 1: self.K, 2: 1}[which], self.vocab)

    def hivis_get_hidden(self, ctx, which, out):
        self.copy(out, {0: self.rows, 1: 1}[which], self.d)

    def hivis_get_tokens(self, ctx, drafts, target):
        np.ctypeslib.as_array(C.cast(drafts, C.POINTER(C.c_int32)), (self.K,))[:] = 1 + np.arange(self.K)
        np.ctypeslib.as_array(C.cast(target, C.POINTER(C.c_int32)), (self.K + 1,))[:] = 1 + np.arange(self.K + 1)


@pytest.fixture
def guarded(monkeypatch):
    """np.empty and np.zeros with guard words behind the array, checked at the end; np.empty filled with -1."""
    made = []

    def alloc(fill):
        def f(shape, dtype=np.float64):
            n = int(np.prod(shape))
            whole = np.full(n + 4096, 0x55 if np.issubdtype(dtype, np.integer) else np.float32(-7), dtype)
            made.append((whole, n))
            whole[:n] = fill
            return whole[:n].reshape(shape)
        return f

    from paper_2509_23928_amd import binding
    fake = SimpleNamespace(**{k: getattr(np, k) for k in ("prod", "float32", "int32", "uint16", "asarray", "ascontiguousarray", "ndarray")}, empty=alloc(-1), zeros=alloc(0))
    monkeypatch.setattr(binding, "np", fake)
    yield
    for whole, n in made:
        assert (whole[n:] == whole[-1]).all(), "written behind an array"


def rows_of(a):
    return [int(x) for x in a.reshape(-1, a.shape[-1])[:, 0]]


def context(d=16, vocab=48):
    from paper_2509_23928_amd import Hivis
    hv = Hivis.__new__(Hivis)
    hv.lib, hv.ctx, hv.B, hv.k_max, hv.cfg = Copies(d, vocab), None, 1, 8, SimpleNamespace(d=d, vocab=vocab)
    hv.K = hv._draft_K = hv._verify_rows = 0
    return hv


def test_other_k_since_the_pass(guarded):
    hv = context()
    hv.draft(2)
    hv.verify()
    assert rows_of(hv.get_logits(0)) == rows_of(hv.get_hidden(0)) == [1, 2, 3]
    hv.draft(5)                                              # more rows than the last verify had
    assert rows_of(hv.get_hidden(0)) == rows_of(hv.get_logits(0)) == [1, 2, 3, 0, 0, 0]
    assert rows_of(hv.get_logits(1)) == [1, 2, 3, 4, 5] and rows_of(hv.get_logits(2)) == [1]
    hv.verify()
    hv.draft_sample(1, 1.0)                                  # fewer
    assert rows_of(hv.get_hidden(0)) == [1, 2] and rows_of(hv.get_hidden(1)) == [1]
    hv.set_drafts([[0, 0, 0]])
    assert rows_of(hv.get_hidden(0)) == [1, 2, 3, 4]


def test_tree_and_chain_in_turn(guarded):
    hv = context()
    hv.tree_draft(3, 2, 6)
    assert rows_of(hv.get_logits(1)) == [0] * 6              # no chain round yet
    hv.tree_verify()
    assert rows_of(hv.get_logits(0)) == list(range(1, 8))
    hv.draft_noalloc(4)
    hv.tree_draft(3, 2, 6)
    assert rows_of(hv.get_logits(1)) == [1, 2, 3, 4, 0, 0]
    hv.tree_set([1, 2], [0, 1])
    assert rows_of(hv.get_logits(1)) == [1, 2]
    hv.tree_verify()
    dr, tt = hv.get_tokens()
    assert dr.tolist() == [[1, 2]] and tt.tolist() == [[1, 2, 3]]


@pytest.mark.gpu
def test_on_the_library():
    from paper_2509_23928_amd import Hivis
    cfg = synth.HivisConfig(name="rows", n_layers=1, d=64, n_q_heads=2, n_kv_heads=2, head_dim=64, ffn=64, vocab=2048, dtype="f32", n_vis=3, n_text=5, K=6, batch=1,
                            gen_tokens=0, gen_cycles=8)
    hv = Hivis(cfg, synth.make_weights(cfg, seed=1))
    hv.prefill(*synth.make_prompt(cfg, seed=1))
    assert hv.get_logits(1).shape == (0, 1, 2048)
    hv.draft(2)
    hv.verify()
    g = hv.get_hidden(0)
    hv.accept()
    hv.draft(6)
    later = hv.get_hidden(0)
    assert np.array_equal(later[:, :3], g) and not later[:, 3:].any()
    hv.verify()
    long = hv.get_hidden(0)
    hv.accept()
    hv.draft(1)
    assert np.array_equal(hv.get_hidden(0), long[:, :2])
    hv.verify()
    hv.accept()
    q = hv.get_logits(1)
    hv.tree_draft(2, 3, 5)
    d = hv.get_logits(1)
    assert d.shape == (5, 1, 2048) and np.array_equal(d[:1], q) and not d[1:].any()
    hv.tree_verify()
    assert hv.get_logits(0).shape == (1, 6, 2048) and hv.get_logits(0)[0, 5].any()
    hv.close()
