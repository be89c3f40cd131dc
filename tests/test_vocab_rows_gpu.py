"""Gradient of the word matrix's last rows when the vocabulary is no multiple of four: in fp32 mode they are the last columns
of the k-strided logit gradient, whose rows are wider, and the last row of it ends inside a 16-byte chunk."""
import numpy as np
import pytest

from paper_2011_13635_amd import synth
from parity_util import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [1021, 1022, 1023, 1025, 1026])
@pytest.mark.parametrize("B,S", [(1, 8), (2, 16), (5, 50)])
def test_last_rows_of_the_word_gradient(vocab, B, S):
    # one, four and 35 predicted positions: with one, its row of logit gradients is the whole contraction
    sh = synth.ModelShape(n_layers=1, hidden=128, n_heads=2, ffn=512, vocab=vocab, max_pos=512)
    r = run_case(sh, B, S, 0, 1, True, 0, seed=6, std=0.08, perturb=0.1)
    got, ref = (np.asarray(r[k]["emb.word"][-8:], dtype=np.float64) for k in ("grads", "ref_grads"))
    scale = np.abs(ref).max(axis=1)                      # every row by its own scale
    assert (scale > 0).all()
    assert (np.abs(got - ref).max(axis=1) <= 1e-4 * scale).all()
    r["model"].close()
