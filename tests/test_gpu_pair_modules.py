"""The one-kernel ends of the triangle updates and the one-kernel transition, module by module against the oracle: row counts around their tiles of
64 and 128 rows, each channel count, activation and hidden width, row and column chunks; the bits do not depend on the chunks."""
import pytest

from oracle import pairstack as P
from paper_2401_10652_amd import inputs as I
from util import check, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2401_10652_amd import binding
    binding.lib()
    return binding


def module(B, cfg, kind, settings):
    """One module under each (dim, chunk) of `settings`: every result the same, from a workspace full of NaN; returns it and the oracle's."""
    import torch
    z, w = I.pair_inputs(cfg, bias_std=0.1, ln_jitter=0.1)
    dz = B.to_device(z, "bf16")
    dw = [B.to_device(w[n], "bf16") for n, _ in I.pair_tensor_shapes(cfg)]
    first = None
    for dim, chunk, flags in settings:
        plan = B.Plan(B.pair_desc(cfg, flags=flags | B.AC_FLAG_LISTED_REGIONS_ONLY), [(kind, dim, chunk)])
        plan.ac_plan_bind_weights(dw)
        ws = torch.full((int(plan.ac_plan_query().workspace_bytes),), 0xff, dtype=torch.uint8, device="cuda")
        y = torch.full_like(dz, float("nan"))
        plan.ac_execute(dz, y, ws)
        torch.cuda.synchronize()
        plan.close()
        first = y if first is None else first
        assert torch.equal(y, first), (dim, chunk, flags)
    return host(first), P.pair_module(P.PAIR_MODULES[kind - B.AC_REGION_TRIMUL_OUT], z, w, cfg.heads, cfg.activation, cfg.ln_eps)


def settings(B, n):
    chunks = sorted({1, (n + 2) // 3, n})
    return [(d, c, 0) for d in (B.AC_DIM_ROW, B.AC_DIM_COL) for c in chunks] + [(B.AC_DIM_ROW, chunks[0], B.AC_FLAG_TWO_SEGMENTS_IN_FLIGHT)]


@pytest.mark.parametrize("c_z,c_hidden", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("n", [8, 16, 24, 72, 200])
def test_triangle_update(B, n, c_z, c_hidden):
    cfg = I.PairConfig("tpm", 46, n, c_z, c_hidden, 2, 32, 2, "bf16")
    for kind in (B.AC_REGION_TRIMUL_OUT, B.AC_REGION_TRIMUL_IN):
        y, ref = module(B, cfg, kind, settings(B, n))
        check(y, ref, "bf16", what=f"kind {kind}")


@pytest.mark.parametrize("n,c_z,factor,activation", [
    (8, 64, 1, "relu"), (8, 128, 1, "gelu_erf"), (16, 64, 4, "gelu_tanh"), (24, 128, 4, "relu"), (40, 128, 8, "gelu_tanh"), (48, 64, 3, "gelu_erf"),
    (72, 128, 2, "gelu_tanh"), (104, 128, 4, "gelu_erf"), (16, 128, 9, "relu"),     # (nine times as wide: two launches)
    (24, 128, 2, "relu"), (72, 128, 4, "relu"), (96, 64, 8, "gelu_erf"), (112, 128, 8, "gelu_tanh")])   # (the last three: one kernel whole, two launches in parts)
def test_transition(B, n, c_z, factor, activation):
    cfg = I.PairConfig("tpt", 47, n, c_z, 64, 2, 32, factor, "bf16", activation=activation)
    y, ref = module(B, cfg, B.AC_REGION_PAIR_TRANSITION, settings(B, n))
    check(y, ref, "bf16")


@pytest.mark.parametrize("k", [64, 128])
@pytest.mark.parametrize("rows", [8, 64, 1000, 8200, 33008, 131072 + 72])      # (two gated pairs: from 16384 or 32768 rows on; 131072: tiles of 64 rows)
@pytest.mark.parametrize("parts", ["four", "two", "pairs", "narrow"])
def test_projections_of_whole_slices(B, rows, k, parts):
    """256 or 512 weight columns (and a few more of a part stored strided): the bits of the same projections with four columns more, which the kernel of 64-column tiles takes."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(49)
    def t(*shape, std=1.0):
        return torch.randn(shape, generator=g, device="cuda").mul_(std).bfloat16()
    x, gain, shift, period = t(rows, k), t(k, std=0.1) + 1, t(k, std=0.1), 8 if rows % 1000 else 1000
    w = [t(132, k, std=k ** -0.5) for _ in range(4)]
    b = [t(132, std=0.2) for _ in range(4)]
    def run(n):
        def nan(*shape):
            return torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        if parts == "pairs":
            out = [nan(n, rows), nan(n, rows)]
            specs = [dict(w=w[2 * i][:n], bias=b[2 * i], w_gate=w[2 * i + 1][:n], bias_gate=b[2 * i + 1], out_t=out[i], t_s2=1, t_s3=rows) for i in range(2)]
        else:
            out = [nan(rows, n), nan(rows, n), nan(rows, n), nan(rows // period, n, period)]
            specs = [dict(w=w[0][:n], out=out[0]), dict(w=w[1][:n], bias=b[1], activation=B.AC_ACT_SIGMOID, out=out[1]), dict(w=w[2][:n], bias=b[2], out=out[2]),
                     dict(w=w[3][:n], bias=b[3], out_t=out[3], t_period=period, t_s1=n * period, t_s2=1, t_s3=period)]
            if parts in ("two", "narrow"):
                specs, out = specs[1::2], out[1::2]
            if parts == "narrow":             # beside them a part of 12 columns, as the pair bias is
                out.append(nan(12, rows))
                specs.insert(0, dict(w=w[0][:12], bias=b[0], out_t=out[2], t_s2=1, t_s3=rows))
        B.ac_op_ln_linear(x, gain, shift, specs)
        torch.cuda.synchronize()
        return out
    for i, (ours, other) in enumerate(zip(run(128), run(132))):
        other = other[:128] if parts == "pairs" or i == 2 and parts == "narrow" else other[:, :128]
        assert torch.equal(ours, other), i
