"""The stream a model is created on has no part in the result: a step gives the same bits on the default stream and on
a named one (products are planned the same way on both)."""
import numpy as np
import pytest

from paper_2011_13635_amd import binding, synth
from test_parity_gpu import small_shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,B,S,precision", [
    (synth.tiny_shape(3), 11, 50, 0),              # fp32 mode: the feed-forward products split their contraction
    (small_shape(2), 11, 13, 1),                   # bf16, hidden size no multiple of 128: the same kernel
    (synth.tiny_shape(3), 4, 64, 1),               # bf16 on the few-tile kernel
])
def test_step_on_a_named_stream_gives_the_bits_of_the_default_stream(shape, B, S, precision):
    import torch
    W = synth.pack_weights(shape, synth.make_weights(shape, seed=5))
    batch = synth.make_batch(shape, B, S, seed=6, ragged=True)
    out = []
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        m = binding.Model(binding.make_config(shape, B, S, precision), stream=stream)
        m.mslt_load_params(W)
        loss = m.mslt_stage_step(1, 1, False, m.device_batch(batch))
        out.append((loss, m.mslt_debug_prefix_output(B, S), m.mslt_get_grads()))
        m.close()
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1])
    assert np.array_equal(out[0][2], out[1][2])
