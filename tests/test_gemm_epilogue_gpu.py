"""How a product ends (bias, dropout, GELU, multiplication by the stored derivative, addition, accumulation), alone, through
the C ABI, on every tile of a step that ends a product in its own way: against float64.

The operands' products and partial sums, the bias among them, are exact in fp32, so all ends but GELU have one right result:
fp32 operations on exact values, rounded once to the output's type.  GELU: the three-term erf of the bf16 path is off by at
most 2.5e-5, Phi by half of that, and 2^-9 of the value is half a unit of bf16; its derivative is stored in steps of 2^-15."""
import math

import numpy as np
import pytest

from oracle import mslt_oracle as O
from paper_2011_13635_amd import binding, synth
from test_gemm_gpu import _operands

pytestmark = pytest.mark.gpu

P, SEED, N, K = 0.1, 41, 768, 192
TILES = [(5, 256, 256), (5, 256, 384), (5, 256, 128), (5, 128, 256), (5, 128, 192), (5, 64, 64), (5, 32, 32), (1, 128, 0)]


def _erf(x):
    return np.vectorize(math.erf)(x)


def _small(seed, n, steps=33, unit=16.0):
    return ((synth.rand_u64(seed, 13, np.arange(n)) % steps).astype(np.float64) - steps // 2) / unit


def _product(torch, kernel, tm, tn, M, akc, bkc, end, out_dtype, fill=float("nan"), rows_past=256, n=N, k=K):
    """Runs a product into the first M rows of a larger buffer; returns those rows and the operands' float64 product."""
    ta, tb, ref = _operands(torch, M, n, k, akc, bkc, seed=90 + M)
    c = torch.full((M + rows_past, n), fill, dtype=out_dtype, device="cuda:0")
    binding.mslt_debug_gemm(ta, tb, c, M, n, k, akc, bkc, kernel, tm, tn, 64, 1, None, epilogue=end)
    torch.cuda.synchronize()
    past = c[M:].float().cpu()
    assert bool(torch.isnan(past).all()) if math.isnan(fill) else bool((past == fill).all())
    return c[:M].cpu(), ref


def _rounded(torch, x, dtype):
    return torch.tensor(np.asarray(x, dtype=np.float32)).to(dtype)


@pytest.mark.parametrize("kernel,tm,tn", TILES)
@pytest.mark.parametrize("bkc", [1, 0])
@pytest.mark.parametrize("M", [515, 31])
def test_exact_ends(kernel, tm, tn, bkc, M):
    import torch
    if kernel == 1:
        M = 512 if M > 128 else 128
    f32, bf16 = torch.float32, torch.bfloat16
    bias = _small(1, N)
    tbias = torch.tensor(bias, dtype=f32, device="cuda:0")
    keep = O.Dropout(P, SEED, 0).mask(0, O.SITE_ATTN_OUT, (M, N)) != 0
    scale = np.float32(1.0) / (np.float32(1.0) - np.float32(P))
    code = (synth.rand_u64(3, 14, np.arange(M * N)) % 49152).astype(np.int64).reshape(M, N)        # derivatives -1/4 .. 5/4
    tcode = torch.from_numpy(code.astype(np.uint16).view(np.int16)).to("cuda:0")
    add = _small(2, M * N, 257, 64.0).reshape(M, N)
    for out in (bf16, f32):
        # rounding happens after the last operation: exact sums, one fp32 operation, the output's type
        end = {"bias": tbias}
        got, ref = _product(torch, kernel, tm, tn, M, 1, bkc, end, out)
        assert torch.equal(got, _rounded(torch, ref + bias, out)), "bias"
        got, ref = _product(torch, kernel, tm, tn, M, 1, bkc, {**end, "act": 2, "aux": tcode}, out)
        want = (ref + bias).astype(np.float32) * (code / 32768.0 - 0.25).astype(np.float32)
        assert torch.equal(got, _rounded(torch, want, out)), "multiply"
        for dt in (bf16, f32):
            aux = torch.tensor(add, dtype=dt, device="cuda:0")
            got, ref = _product(torch, kernel, tm, tn, M, 1, bkc, {"act": 3, "aux": aux, "aux_f32": int(dt == f32)}, out)
            want = ref.astype(np.float32) + aux.float().cpu().numpy()
            assert torch.equal(got, _rounded(torch, want, out)), "add"
    got, ref = _product(torch, kernel, tm, tn, M, 1, bkc, {"bias": tbias, "dropout": P, "seed": SEED}, bf16)
    want = np.where(keep, (ref + bias).astype(np.float32) * scale, np.float32(0.0))
    assert torch.equal(got.float(), _rounded(torch, want, bf16).float()), "dropout"
    assert 0.08 < 1.0 - keep.mean() < 0.12


@pytest.mark.parametrize("kernel,tm,tn", TILES)
@pytest.mark.parametrize("M", [515, 31])
def test_gelu_and_its_derivative(kernel, tm, tn, M):
    import torch
    if kernel == 1:
        M = 512 if M > 128 else 128
    bias = _small(1, N)
    tbias = torch.tensor(bias, dtype=torch.float32, device="cuda:0")
    grad = torch.zeros((M + 256, N), dtype=torch.int16, device="cuda:0")
    for with_grad in (True, False):
        end = {"bias": tbias, "act": 1, **({"gelu_grad": grad} if with_grad else {})}
        got, ref = _product(torch, kernel, tm, tn, M, 1, 1, end, torch.bfloat16)
        u = ref + bias
        cdf = 0.5 * (1.0 + _erf(u / math.sqrt(2.0)))
        e = 1.3e-5 * np.abs(u) + 1e-7
        err = np.abs(got.double().numpy() - u * cdf)
        assert (err <= e + 2.0 ** -8 * (np.abs(u * cdf) + e)).all(), err.max()
    g = (grad[:M].cpu().numpy().astype(np.int64) & 0xffff) / 32768.0 - 0.25
    assert np.abs(g - (cdf + u * np.exp(-0.5 * u * u) / math.sqrt(2.0 * math.pi))).max() <= 2.0 ** -16 + 1.4e-5
    assert not grad[M:].any()


@pytest.mark.parametrize("tm,tn", [(256, 256), (256, 128), (128, 128)])
@pytest.mark.parametrize("M,n,k", [(256, 512, 64), (768, 256, 192), (512, 768, 448)])
def test_grouped_weight_gradients_accumulate(tm, tn, M, n, k):
    # the first layer of a parameter set writes, the others add to what is there
    import torch
    got, ref = _product(torch, 7, tm, tn, M, 0, 0, {}, torch.float32, n=n, k=k)
    assert np.array_equal(got.numpy(), ref.astype(np.float32))
    got, ref = _product(torch, 7, tm, tn, M, 0, 0, {"accumulate": 1}, torch.float32, fill=0.3125, n=n, k=k)
    assert np.array_equal(got.numpy(), (ref + 0.3125).astype(np.float32))


def test_parts_that_do_not_belong_together_are_refused():
    import torch
    t = torch.zeros(256 * 256, dtype=torch.bfloat16, device="cuda:0")
    c = torch.zeros((256, 256), dtype=torch.bfloat16, device="cuda:0")
    for end in ({"act": 4}, {"act": 2}, {"act": 1, "aux": t}, {"gelu_grad": t}, {"accumulate": 1}, {"dropout": 1.0},
                {"act": 2, "aux": t, "aux_f32": 1}):
        with pytest.raises(binding.MsltError) as ei:
            binding.mslt_debug_gemm(t, t, c, 256, 256, 256, 1, 1, 5, 256, 256, epilogue=end)
        assert ei.value.code == binding.MSLT_ERR_ARG


@pytest.mark.parametrize("kernel,tm,tn", [(1, 128, 0), (2, 256, 256), (2, 128, 256), (2, 128, 128)])
@pytest.mark.parametrize("bkc", [1, 0])
def test_split_contraction_gets_its_bias_once(kernel, tm, tn, bkc):
    import torch
    M, n, k, parts = 256, 768, 448, 3
    bias = _small(1, n)
    end = {"bias": torch.tensor(bias, dtype=torch.float32, device="cuda:0")}
    ta, tb, ref = _operands(torch, M, n, k, 1, bkc, seed=17)
    partials = torch.empty(parts * M * n, device="cuda:0")
    for out in (torch.bfloat16, torch.float32):
        c = torch.full((M, n), float("nan"), dtype=out, device="cuda:0")
        binding.mslt_debug_gemm(ta, tb, c, M, n, k, 1, bkc, kernel, tm, tn, 64, parts, partials, epilogue=end)
        assert torch.equal(c.cpu(), _rounded(torch, ref + bias, out))
