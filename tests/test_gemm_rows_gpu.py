"""Tiles of a matrix product whose rows are no multiple of the tile: the right result in every row, none past the end
written, none past the end of A read (its buffer ends there)."""
import pytest

from paper_2011_13635_amd import binding
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

