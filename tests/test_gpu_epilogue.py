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
