"""fp32 layers of 32, 64 and 128 channels, whose LayerNorm 1 and projection (64 and 128) and whose tail (32, 64, and 128 where rows are neither few nor
many) are one kernel each: the bits of the separate kernels (each op called by itself), row counts around the blocks' 16 rows, every activation, chunked plans, several layers."""
import pytest

from paper_2401_10652_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2401_10652_amd import binding
    binding.lib()
    return binding


def layer_by_ops(B, x, w, heads, causal, act):
    import torch
    rows, d = x.shape
    u, qkv, ctx, h, y = torch.empty_like(x), torch.empty(rows, 3 * d, device="cuda"), torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
    hid = torch.empty(rows, w["w_1"].shape[0], device="cuda")
    B.ac_op_layernorm(x, w["ln1_g"], w["ln1_b"], u, 1e-5)
    B.ac_op_linear(u, w["w_qkv"], qkv, bias=w["b_qkv"])
    B.ac_op_attention(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:], ctx, heads, d // heads, causal=causal)
    B.ac_op_linear(ctx, w["w_o"], h, bias=w["b_o"], residual=x)
    B.ac_op_layernorm(h, w["ln2_g"], w["ln2_b"], u, 1e-5)
    B.ac_op_linear(u, w["w_1"], hid, bias=w["b_1"], activation=act)
    B.ac_op_linear(hid, w["w_2"], y, bias=w["b_2"], residual=h)
    return y


@pytest.mark.parametrize("seq,d,heads,layers,causal,activation", [
    (1, 64, 4, 1, False, "gelu_erf"), (15, 32, 2, 2, True, "relu"), (16, 128, 4, 1, False, "gelu_tanh"), (17, 64, 2, 3, True, "gelu_erf"), (33, 128, 8, 2, False, "relu"),
    (256, 64, 4, 1, False, "gelu_erf"), (1000, 32, 2, 1, True, "gelu_tanh"), (5003, 128, 2, 1, True, "gelu_erf")])
def test_layers_equal_the_separate_kernels(B, seq, d, heads, layers, causal, activation):
    import torch
    cfg = I.TransformerConfig("tfc", 48, layers, seq, d, heads, 4 * d, causal, "f32", None, activation=activation)
    shapes = I.transformer_layer_shapes(cfg)
    g = torch.Generator(device="cuda").manual_seed(48)
    x = torch.randn((seq, d), generator=g, device="cuda")
    ws = [{n: torch.randn(shapes[n], generator=g, device="cuda") * shapes[n][-1] ** -0.5 for n in I.TRANSFORMER_LAYER_TENSORS} for _ in range(layers)]
    act = {"gelu_erf": B.AC_ACT_GELU_ERF, "gelu_tanh": B.AC_ACT_GELU_TANH, "relu": B.AC_ACT_RELU}[activation]
    ref = x
    for w in ws:
        ref = layer_by_ops(B, ref, w, heads, causal, act)
    kinds = (B.AC_REGION_QKV, B.AC_REGION_ATTENTION, B.AC_REGION_OUT_PROJ, B.AC_REGION_FFN)
    for chunk, flags in ((seq, 0), ((seq + 2) // 3, 0), ((seq + 4) // 5, B.AC_FLAG_TWO_SEGMENTS_IN_FLIGHT)):
        plan = B.Plan(B.transformer_desc(cfg, flags=flags), [(k, B.AC_DIM_SEQ, chunk) for k in kinds])
        info = plan.ac_plan_query()
        plan.ac_plan_bind_weights([w[n] for w in ws for n in I.TRANSFORMER_LAYER_TENSORS])
        space = torch.full((int(info.workspace_bytes),), 0xff, dtype=torch.uint8, device="cuda")
        y = torch.full_like(x, float("nan"))
        assert plan.ac_execute(x, y, space) == info.peak_bytes_planned
        torch.cuda.synchronize()
        plan.close()
        assert torch.equal(y, ref), (chunk, flags)
