"""Tiles of a matrix product whose rows are no multiple of the tile: the right result in every row and none past the end
written; and a step whose two forward chains meet inside a tile.  (Whether rows past the end of A are read shows in no
result: they would feed rows that are not written.)"""
import numpy as np
import pytest

from paper_2011_13635_amd import binding, synth
from test_gemm_gpu import _operands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tm,tn", [(256, 256), (256, 384), (256, 128), (128, 256), (128, 192), (64, 64), (32, 32)])
@pytest.mark.parametrize("bkc", [1, 0])
@pytest.mark.parametrize("M,K", [(1, 64), (31, 128), (129, 704), (384, 192), (515, 832)])
def test_any_row_count(tm, tn, bkc, M, K):
    # one to thirteen k tiles; products and partial sums of these operands are exact in fp32
    import torch
    N = 768
    ta, tb, ref = _operands(torch, M, N, K, 1, bkc, seed=70 + M)
    for dtype in (torch.float32, torch.bfloat16):
        c = torch.full((M + 256, N), float("nan"), dtype=dtype, device="cuda:0")
        binding.mslt_debug_gemm(ta, tb, c, M, N, K, 1, bkc, 5, tm, tn, 64, 1, None)
        torch.cuda.synchronize()
        want = torch.tensor(ref, dtype=torch.float64).to(torch.float32).to(dtype)
        assert torch.equal(c[:M].cpu(), want)
        assert bool(torch.isnan(c[M:]).all())


# (10 x 65 and 15 x 40: few-tile products, and with the padded rows the second half is the larger one or as large)
@pytest.mark.parametrize("B,S,dropout", [(27, 203, 0.1), (9, 128, 0.0), (3, 510, 0.1), (10, 65, 0.1), (15, 40, 0.0)])
def test_chains_of_unequal_halves_give_the_bits_of_one_chain(B, S, dropout):
    import torch
    shape = synth.bert_base_shape(2)
    W = synth.pack_weights(shape, synth.make_weights(shape, seed=11))
    batch = synth.make_batch(shape, B, S, seed=12, ragged=True)
    m = binding.Model(binding.make_config(shape, B, S, 1))
    m.mslt_load_params(W)
    bt = m.device_batch(batch)
    out = []
    for one_chain in (False, True, False):
        m.mslt_profile_enable(one_chain)
        if dropout:
            m.mslt_set_dropout(dropout, 3, 0)
        loss = m.mslt_stage_step(1, 1, False, bt)
        out.append((loss, m.mslt_debug_prefix_output(B, S), m.mslt_get_grads()))
    m.close()
    for o in out[1:]:
        assert o[0] == out[0][0]
        assert np.array_equal(o[1], out[0][1])
        assert np.array_equal(o[2], out[0][2])
