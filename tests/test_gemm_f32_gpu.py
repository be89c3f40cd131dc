"""The fp32 matrix product of a step, at the edges of its 64x64 tiles and 32-wide slabs, in every layout and split: equal
to the float64 product of operands whose products and partial sums are exact in fp32."""
import numpy as np
import pytest

from paper_2011_13635_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,splitk", [(64, 64, 32, 1), (4, 4, 4, 1), (68, 128, 36, 1), (60, 188, 100, 3), (132, 64, 352, 2),
                                          (128, 132, 388, 5), (8, 260, 1028, 7)])
@pytest.mark.parametrize("akc,bkc", [(1, 1), (1, 0), (0, 0), (0, 1)])
def test_equals_the_float64_product(M, N, K, splitk, akc, bkc):
    import torch
    A = ((synth.rand_u64(7, 11, np.arange(M * K)) % 2049).astype(np.float64) - 1024.0).reshape(M, K) / 1024.0
    B = ((synth.rand_u64(7, 12, np.arange(N * K)) % 3).astype(np.float64) - 1.0).reshape(N, K)
    ta = torch.tensor(A if akc else A.T.copy(), dtype=torch.float32, device="cuda:0")
    tb = torch.tensor(B if bkc else B.T.copy(), dtype=torch.float32, device="cuda:0")
    partials = torch.full((splitk * M * N,), float("nan"), device="cuda:0") if splitk > 1 else None
    c = torch.full((M + 1, N), float("nan"), dtype=torch.float32, device="cuda:0")
    binding.mslt_debug_gemm(ta, tb, c, M, N, K, akc, bkc, 6, splitk=splitk, partials=partials)
    torch.cuda.synchronize()
    assert np.array_equal(c[:M].cpu().numpy().astype(np.float64), A @ B.T)
    assert bool(torch.isnan(c[M:]).all())


def test_odd_contraction_of_two_strided_operands():
    # k past the end lies past the end of both operands; M and N stay multiples of four
    import torch
    for K in (1, 33, 550, 31):
        A = ((synth.rand_u64(7, 11, np.arange(68 * K)) % 2049).astype(np.float64) - 1024.0).reshape(K, 68) / 1024.0
        B = ((synth.rand_u64(7, 12, np.arange(128 * K)) % 3).astype(np.float64) - 1.0).reshape(K, 128)
        ta, tb = (torch.tensor(x, dtype=torch.float32, device="cuda:0") for x in (A, B))
        c = torch.full((68, 128), float("nan"), device="cuda:0")
        binding.mslt_debug_gemm(ta, tb, c, 68, 128, K, 0, 0, 6)
        torch.cuda.synchronize()
        assert np.array_equal(c.cpu().numpy().astype(np.float64), A.T @ B), K


def test_rows_that_are_not_aligned_are_refused():
    import torch
    t = torch.zeros(66 * 66, device="cuda:0")
    for M, N, K, akc, bkc in ((64, 64, 66, 1, 1), (66, 64, 64, 0, 0)):
        with pytest.raises(binding.MsltError) as ei:
            binding.mslt_debug_gemm(t, t, t, M, N, K, akc, bkc, 6)
        assert ei.value.code == binding.MSLT_ERR_ARG
