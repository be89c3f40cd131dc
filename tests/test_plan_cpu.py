"""Which kernel a step takes for a product: the lines between the kernels, from the plan alone (no GPU)."""
import pytest

from paper_2011_13635_amd import binding

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
