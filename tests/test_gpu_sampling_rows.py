"""Sampling at the vocabulary sizes where its passes over a row change shape: fewer logits than one step of the walk (512) or
than one load per thread, ragged last steps and segments, more than one trip.  Every decision is re-taken in float64 from the
library's own logits; a difference is accepted only within 1e-5 of a boundary of the running sum."""
import pytest

from test_gpu_prefill_shapes import cfg_of
from test_gpu_sampling import run_sampling

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,dtype,T", [(48, "bf16", 1.0), (528, "bf16", 2.0), (4112, "bf16", 1.0), (8208, "bf16", 0.7), (33040, "bf16", 1.0),
                                           (64, "f32", 1.5), (1040, "f32", 1.0)])
def test_vocabulary_sizes(vocab, dtype, T):
    run_sampling(cfg_of(vocab=vocab, dtype=dtype, n_vis=5, n_text=7, gen_cycles=4), 3, 3, T, sample_first=True)
