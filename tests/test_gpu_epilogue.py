"""GPU: activations of bf16 products are as exact as those of fp32 ones.  The residual subtracts the bf16 rounding of the result,
so that what is stored is the part below it; most of that part's bits are seen where it is small."""
import pytest

from util import draw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2401_10652_amd import binding
    binding.lib()
    return binding


def below_bf16(B, activation, std, k=128, n=64, m=8192):
    """(what a bf16 product of these pre-activations stores, what an fp32 product's activation gives for it)."""
    import torch
    hi, lo = draw((m, n), 440, "bf16", std), draw((m, n), 441, "bf16", std * 2 ** -8)   # hi + lo is exact in fp32
    a, w = torch.zeros((m, k), device="cuda"), torch.zeros((n, k), device="cuda")
    a[:, :n], a[:, n:2 * n] = B.to_device(hi, "f32"), B.to_device(lo, "f32")
    w[:, :n] = w[:, n:2 * n] = torch.eye(n, device="cuda")
    y = torch.empty((m, n), device="cuda")
    B.ac_op_linear(a, w, y, activation=activation)
    rounded = y.bfloat16()
    out = torch.empty_like(rounded)
    B.ac_op_linear(a.bfloat16(), w.bfloat16(), out, residual=-rounded, activation=activation)
    torch.cuda.synchronize()
    return out, (y - rounded.float()).bfloat16()


@pytest.mark.parametrize("std", [0.5, 2.0, 8.0])
def test_sigmoid_of_a_bf16_product(B, std):
    import torch
    out, ref = below_bf16(B, B.AC_ACT_SIGMOID, std)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("std", [0.02, 0.5, 2.0])
def test_tanh_gelu_of_a_bf16_product(B, std):
    import torch
    out, ref = below_bf16(B, B.AC_ACT_GELU_TANH, std)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("k,m", [(136, 8192), (136, 100), (200, 8192)])
def test_erf_gelu_of_a_bf16_product_of_ragged_depth(B, k, m):
    """(A depth of whole tiles takes the table, whose error a bf16 result hides.)"""
    import torch
    out, ref = below_bf16(B, B.AC_ACT_GELU_ERF, 1.0, k=k, m=m)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("m,n,k", [(128, 64, 128), (512, 256, 64), (3072, 1024, 512), (16384, 1024, 256)])
def test_operands_and_results_in_descending_order(B, m, n, k):
    """The factor, the residual and the strided result with negative row strides: the bits of the same rows in ascending order, and nothing
    outside them read or written."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    a, w, mul, res = (torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((m, k), (n, k), (m, n), (m, n)))
    ref, ref_t = torch.empty((m, n), device="cuda", dtype=torch.bfloat16), torch.empty((n, m), device="cuda", dtype=torch.bfloat16)
    B.ac_op_linear(a, w, ref, mul=mul, residual=res)
    B.ac_op_linear(a, w, None, mul=mul, residual=res, out_t=ref_t, n_split=0, t_s2=1, t_s3=m)

    def among_nan(t):
        buf = torch.full((3, *t.shape), float("nan"), device="cuda", dtype=torch.bfloat16)
        buf[1] = t
        return buf
    up, down = (among_nan(mul), among_nan(res)), (among_nan(mul.flip(0)), among_nan(res.flip(0)))
    stream = torch.cuda.current_stream().cuda_stream
    for mul_down in (False, True):
        for res_down in (False, True):
            bm, br = (down if mul_down else up)[0], (down if res_down else up)[1]
            mul_at, ldmul = (bm[1, m - 1].data_ptr(), -n) if mul_down else (bm[1].data_ptr(), n)
            res_at, ldr = (br[1, m - 1].data_ptr(), -n) if res_down else (br[1].data_ptr(), n)
            out, out_t = torch.full_like(ref, float("nan")), torch.full((3, n, m), float("nan"), device="cuda", dtype=torch.bfloat16)
            args = (a.data_ptr(), k, w.data_ptr(), k, None, mul_at, ldmul, res_at, ldr)
            assert B.lib().ac_op_linear(*args, out.data_ptr(), n, None, n, 0, 0, 0, 0, m, n, k, B.AC_ACT_NONE, B.AC_BF16, stream) == 0
            assert B.lib().ac_op_linear(*args, None, 0, out_t[1, n - 1].data_ptr(), 0, 0, 0, 1, -m, m, n, k, B.AC_ACT_NONE, B.AC_BF16, stream) == 0
            torch.cuda.synchronize()
            assert torch.equal(out, ref) and torch.equal(out_t[1].flip(0), ref_t)
            assert bool(out_t[0].isnan().all()) and bool(out_t[2].isnan().all())


@pytest.mark.parametrize("k", [64, 128])
def test_strided_results_of_fused_projections_in_descending_order(B, k):
    import torch
    m, n = 4096, 192
    g = torch.Generator(device="cuda").manual_seed(8)
    x, w, gain, shift = (torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((m, k), (n, k), (k,), (k,)))
    ref = torch.empty((n, m), device="cuda", dtype=torch.bfloat16)
    out = torch.full((3, n, m), float("nan"), device="cuda", dtype=torch.bfloat16)
    B.ac_op_ln_linear(x, gain, shift, [dict(w=w, out_t=ref, t_s2=1, t_s3=m)])
    B.ac_op_ln_linear(x, gain, shift, [dict(w=w, out_t=out[1, n - 1], t_s2=1, t_s3=-m)])
    torch.cuda.synchronize()
    assert torch.equal(out[1].flip(0), ref) and bool(out[0].isnan().all()) and bool(out[2].isnan().all())
