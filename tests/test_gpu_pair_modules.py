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
    (72, 128, 2, "gelu_tanh"), (104, 128, 4, "gelu_erf"), (16, 128, 9, "relu")])     # (nine times as wide: two launches)
def test_transition(B, n, c_z, factor, activation):
    cfg = I.PairConfig("tpt", 47, n, c_z, 64, 2, 32, factor, "bf16", activation=activation)
    y, ref = module(B, cfg, B.AC_REGION_PAIR_TRANSITION, settings(B, n))
    check(y, ref, "bf16")
