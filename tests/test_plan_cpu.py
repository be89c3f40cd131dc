"""Which kernel a step takes for a product, and how many chains its forward runs as: the lines between them, from the plans
alone (no GPU)."""
import pytest

from paper_2011_13635_amd import binding, synth

GUARDED_F32, F32 = 4, 6


@pytest.mark.parametrize("M,N,K,akc,bkc,kernel,splitk", [
    # many tiles of a short contraction stay with the guarded kernel: the vocabulary's weight gradient over a few predicted
    # positions, the feed-forward one over a short batch
    (30592, 768, 20, 0, 0, GUARDED_F32, 1), (30592, 768, 304, 0, 0, GUARDED_F32, 1), (3072, 768, 128, 0, 0, GUARDED_F32, 1),
    (304, 30592, 256, 1, 1, GUARDED_F32, 1), (2304, 768, 32, 0, 0, GUARDED_F32, 1),
    # on the other side of each line: 11 slabs of 32, 512 tiles, two slabs on 432 tiles
    (3072, 768, 352, 0, 0, F32, 1), (2048, 1024, 128, 0, 0, F32, 1), (2304, 768, 64, 0, 0, F32, 1), (768, 768, 32, 0, 0, F32, 1),
    # parts of a split: short ones and those that start a second round stay, longer ones and other splits do not
    (256, 768, 768, 1, 0, GUARDED_F32, 5), (4, 768, 30592, 1, 0, GUARDED_F32, 64), (1024, 768, 3072, 1, 0, GUARDED_F32, 4),
    (304, 1024, 30592, 1, 0, F32, 6), (100, 768, 3072, 1, 1, F32, 10),
    # rows that are not 16-byte aligned
    (64, 64, 66, 1, 1, GUARDED_F32, 1)])
def test_fp32_products(M, N, K, akc, bkc, kernel, splitk):
    assert binding.mslt_debug_plan_gemm(0, M, N, K, akc, bkc, 1) == (kernel, 64, 64, splitk)


@pytest.mark.parametrize("hidden,B,S,rows", [
    # halves of unequal rows whose larger one is past the 32-wide few-tile kernel, while one chain stays with the 64-wide: one
    (768, 5, 112, (640, 0)), (768, 5, 128, (640, 0)), (768, 3, 200, (640, 0)), (768, 13, 40, (640, 0)), (768, 3, 180, (640, 0)),
    (768, 6, 106, (640, 0)), (1024, 3, 140, (512, 0)), (1024, 10, 40, (512, 0)), (1024, 5, 100, (512, 0)),
    # on either side of the lines two: 320 (256) rows each, 320 against 192, past the few-tile kernel, equal halves
    (768, 15, 40, (320, 320)), (768, 4, 160, (320, 320)), (768, 5, 100, (300, 212)), (768, 3, 160, (320, 192)),
    (768, 7, 100, (400, 368)), (768, 9, 128, (640, 512)), (768, 27, 203, (2842, 2662)), (768, 64, 128, (4096, 4096)),
    (1024, 3, 128, (256, 128)), (1024, 7, 64, (256, 256)), (1024, 13, 40, (280, 360)), (1024, 5, 128, (384, 256)),
    # one sequence, and products of at most 2^30 operations
    (768, 1, 512, (512, 0)), (768, 1, 100, (128, 0)), (128, 64, 64, (4096, 0)), (512, 4, 128, (512, 0)),
    # narrower than BERT-Base: unequal halves only from twice that on, equal ones as everywhere
    (512, 5, 128, (640, 0)), (512, 25, 40, (1024, 0)), (640, 9, 40, (384, 0)), (512, 3, 512, (1024, 512)), (512, 6, 128, (384, 384))])
def test_forward_chains(hidden, B, S, rows):
    base = synth.bert_base_shape(2).as_dict()
    base.update(hidden=hidden, ffn=4 * hidden, n_heads=hidden // 64)
    cfg = binding.make_config(synth.ModelShape(**base), 64, 512, 1)
    assert binding.mslt_debug_plan_chains(cfg, B, S) == rows
    assert binding.mslt_debug_plan_chains(binding.make_config(synth.ModelShape(**base), 64, 512, 0), B, S) == (B * S, 0)


def test_forward_chains_with_dropout_meet_where_its_quads_do():
    sh = synth.bert_base_shape(2)
    cfg = binding.make_config(sh, 64, 512, 1)
    assert binding.mslt_debug_plan_chains(cfg, 27, 203, True) == (2842, 2662)        # 12 heads: any offset is a multiple of 4
    sh = sh.as_dict()
    sh.update(n_heads=6)
    cfg = binding.make_config(synth.ModelShape(**sh), 64, 512, 1)
    assert binding.mslt_debug_plan_chains(cfg, 25, 203, True) == (5120, 0) != binding.mslt_debug_plan_chains(cfg, 25, 203)


@pytest.mark.parametrize("N,tile", [(16384, (256, 256)), (16256, (256, 128))])
def test_offsets_of_loads_past_the_last_k_tile_count(N, tile):
    # the turn-taking tiles queue up to three k tiles past the end: the byte offset of a k-strided operand's row K + 190 has to
    # fit 31 bits, where those of the operand itself do
    limit = 2**31
    fits = (limit // (2 * N) - 256 - 1) // 64 * 64
    beyond = (limit // (2 * N) - 1) // 64 * 64
    assert 2 * N * (fits + 256) < limit and 2 * N * beyond < limit < 2 * N * (beyond + 190)
    assert binding.mslt_debug_plan_gemm(1, 4096, N, fits, 1, 0)[:3] == (5,) + tile
    assert binding.mslt_debug_plan_gemm(1, 4096, N, beyond, 1, 0)[:3] != (5,) + tile
