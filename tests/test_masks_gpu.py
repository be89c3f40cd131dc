"""Key masks a training run can meet besides the padding of a few last tokens: biases as low as the type goes or
infinite, sequences whose first keys are masked, and sequences without any open key that fill up a batch.  A masked key
next to an open one has probability zero for any such bias; without an open key the bias is the same for all keys and
cancels.  The oracle adds -1e9 in float64, which leaves nine digits of a score and is exactly that."""
import dataclasses

import numpy as np
import pytest

from oracle import mslt_oracle as O
from paper_2011_13635_amd import synth
from parity_util import TOL, grads_dict, make_model, rel_errors

pytestmark = pytest.mark.gpu

LOWEST = float(np.finfo(np.float32).min)


@pytest.mark.parametrize("bias", [LOWEST, -np.inf, -1e9, -10000.0])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("S,heads", [(70, 2), (128, 2), (131, 2), (70, 4)])   # heads 4: wave-per-row attention
def test_low_masks_first_keys_masked_and_empty_sequences(bias, precision, S, heads):
    B = 14
    sh = synth.ModelShape(n_layers=3, hidden=128, n_heads=heads, ffn=512, vocab=1024, max_pos=512, nsp=True, mask_bias=bias)
    W = synth.make_weights(sh, seed=3, perturb=0.05)
    batch = synth.make_batch(sh, B, S, seed=4, ragged=True)
    batch["attn_mask"][0] = 0                      # empty sequences, first and last of the batch
    batch["attn_mask"][B - 1] = 0
    batch["attn_mask"][1] = 1
    batch["attn_mask"][1, :S - 4] = 0              # only the last keys open (more than 64 masked before them)
    for b in (0, B - 1):
        batch["labels"][b] = -100
    m = make_model(sh, B, S, precision)
    m.mslt_load_params(synth.pack_weights(sh, W))
    loss = m.mslt_stage_step(1, 2, False, m.device_batch(batch))
    prefix = m.mslt_debug_prefix_output(B, S)
    g = grads_dict(m, sh, 1, 2, False)
    m.close()
    ref_loss, ref_g, info = O.stage_step(dataclasses.replace(sh, mask_bias=-1e9), W, batch, 1, 2, False)
    assert all(np.isfinite(v).all() for v in g.values())
    assert abs(loss - ref_loss) < TOL[precision] * abs(ref_loss)
    assert np.abs(prefix - info["prefix_out"]).max() < TOL[precision] * np.abs(info["prefix_out"]).max()
    errs = rel_errors(g, ref_g)
    worst = max(errs, key=errs.get)
    print(bias, precision, S, heads, worst, errs[worst], flush=True)
    assert errs[worst] < TOL[precision], (worst, errs[worst])
