"""GPU parity of the fp32 matrix-core kernels at the edges of their tiles, against the fp64 oracle, through the C-ABI."""
import math

import numpy as np
import pytest

from oracle import transformer as O
from util import check, draw, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2401_10652_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("m,n,k", [
    (1, 4, 4),                       # one row, less than one step of k: three of the four runs of k empty
    (15, 20, 12), (17, 16, 68),      # 16x16 tiles; a run that ends inside a step
    (64, 33, 64),                    # columns that end inside a 16-byte store
    (250, 520, 2052),                # 32x32 tiles, ragged last run
    (700, 1020, 260),                # 32x32 tiles, ragged both ways
    (1100, 2100, 100),               # 32x64 tiles, ragged both ways
    (204, 449, 200),                 # 32x16 tiles, ragged all ways
    (859, 65, 72),
    (745, 602, 232),                 # 32x64 tiles, ragged all ways
    (274, 929, 68),
])
def test_linear_f32(B, m, n, k):
    import torch
    a, w = draw((m, k), 110, "f32"), draw((n, k), 111, "f32", 1 / math.sqrt(k))
    bias, res = draw((n,), 112, "f32", 0.5), draw((m, n), 113, "f32")
    da, dw, db, dr = (B.to_device(t, "f32") for t in (a, w, bias, res))
    out = torch.full((m, n), float("nan"), device="cuda")
    B.ac_op_linear(da, dw, out, bias=db, residual=dr)
    torch.cuda.synchronize()
    check(host(out), O.linear(a, w, bias) + res, "f32")
    # a row's bits do not depend on the launch it falls in (nor on the tile shape: launches of 33 rows take 16x16)
    tile = {(250, 520): "32x32", (700, 1020): "32x32", (1100, 2100): "32x64", (204, 449): "32x16", (859, 65): "32x16",
            (745, 602): "32x64", (274, 929): "32x64"}.get((m, n), "16x16")
    assert B.ac_linear_kernel(m, n, k, "f32") == "f32 " + tile and B.ac_linear_kernel(min(m, 33), n, k, "f32") == "f32 16x16"
    part = torch.full((m, n), float("nan"), device="cuda")
    for r0 in range(0, m, 33):
        r1 = min(m, r0 + 33)
        B.ac_op_linear(da[r0:r1], dw, part[r0:r1], bias=db, residual=dr[r0:r1])
    torch.cuda.synchronize()
    assert torch.equal(part, out)


@pytest.mark.parametrize("m,n,k,kernel", [
    (1024, 512, 512, "f32-ring-deep 32x32"), (1100, 1540, 128, "f32-ring 32x32"), (1531, 601, 256, "f32-ring 32x64"), (5900, 65, 1152, "f32-ring 32x32"),
    (5000, 96, 384, "f32-ring 32x32"), (250, 2100, 640, "f32-ring 32x64"), (260, 516, 1024, "f32 32x32"), (520, 516, 1024, "f32-ring-deep 32x32"),
    (2066, 200, 1024, "f32-ring-deep 32x32"), (700, 516, 256, "f32-ring-deep 32x32")])
def test_linear_f32_depths_of_whole_tiles(B, m, n, k, kernel):
    """Launches of a ring of tiles, odd rows and columns among them: the oracle's values, and the bits of launches of 33 rows (waves that share out k)."""
    import torch
    a, w = draw((m, k), 114, "f32"), draw((n, k), 115, "f32", 1 / math.sqrt(k))
    bias, res = draw((n,), 116, "f32", 0.5), draw((m, n), 117, "f32")
    da, dw, db, dr = (B.to_device(t, "f32") for t in (a, w, bias, res))
    guard = torch.full((m + 2, n), float("nan"), device="cuda")
    out = guard[1:-1]
    B.ac_op_linear(da, dw, out, bias=db, residual=dr)
    torch.cuda.synchronize()
    check(host(out), O.linear(a, w, bias) + res, "f32")
    assert bool(torch.isnan(guard[0]).all()) and bool(torch.isnan(guard[-1]).all())
    assert B.ac_linear_kernel(m, n, k, "f32") == kernel and B.ac_linear_kernel(33, n, k, "f32").startswith("f32 ")
    part = torch.full((m, n), float("nan"), device="cuda")
    for r0 in range(0, m, 33):
        r1 = min(m, r0 + 33)
        B.ac_op_linear(da[r0:r1], dw, part[r0:r1], bias=db, residual=dr[r0:r1])
    torch.cuda.synchronize()
    assert torch.equal(part, out)


@pytest.mark.parametrize("dh", [16, 32, 64, 128])
@pytest.mark.parametrize("sq,sk,causal,off", [
    (1, 1, False, 0), (16, 32, False, 0), (17, 33, True, 16), (70, 129, False, 0), (200, 200, True, 0), (40, 300, True, 260)])
def test_attention_f32(B, dh, sq, sk, causal, off):
    """Row counts around 16 and key counts around 32 (a wave without a tile, a ragged last tile), segments inside a
    causal sequence; q, k and v are column blocks of one packed tensor."""
    import torch
    heads = 2
    d = heads * dh
    q, k, v = draw((sq, d), 120, "f32"), draw((sk, d), 121, "f32"), draw((sk, d), 122, "f32")
    packed = torch.zeros((max(sq, sk), 3 * d), device="cuda")
    packed[:sq, :d], packed[:sk, d:2 * d], packed[:sk, 2 * d:] = (B.to_device(t, "f32") for t in (q, k, v))
    ctx = torch.full((sq, d), float("nan"), device="cuda")
    views = packed[:sq, :d], packed[:sk, d:2 * d], packed[:sk, 2 * d:]
    B.ac_op_attention(*views, ctx, heads, dh, causal=causal, q_offset=off)
    torch.cuda.synchronize()
    check(host(ctx), O.attention(q, k, v, heads, causal, q_offset=off), "f32")
    part = torch.full((sq, d), float("nan"), device="cuda")
    for r0 in range(0, sq, 7):
        r1 = min(sq, r0 + 7)
        B.ac_op_attention(views[0][r0:r1], views[1], views[2], part[r0:r1], heads, dh, causal=causal, q_offset=off + r0)
    torch.cuda.synchronize()
    assert torch.equal(part, ctx)


@pytest.mark.parametrize("dh", [16, 64, 128])
def test_attention_f32_mask_values(B, dh):
    """An additive mask written with the type's lowest value: masked keys have no weight beside others (also where they are all the
    keys of a wave), and a row of nothing but masked keys averages its values.  A mask of -inf drops its keys likewise."""
    import torch
    heads, sq, sk = 2, 40, 200
    d, low = heads * dh, np.finfo(np.float32).min
    q, k, v = draw((sq, d), 130, "f32"), draw((sk, d), 131, "f32"), draw((sk, d), 132, "f32")
    bias = draw((heads, sq, sk), 133, "f32").astype(np.float32)
    bias[:, 0] = low                                            # nothing but masked keys
    bias[:, 1, 5:] = low                                        # five visible ones, all in one wave's tile
    bias[:, 2, 32:64] = low                                     # one wave's tile masked
    bias[:, 3, 32:64] = -np.inf
    ctx = torch.full((sq, d), float("nan"), device="cuda")
    B.ac_op_attention(*(B.to_device(t, "f32") for t in (q, k, v)), ctx, heads, dh, bias=B.to_device(bias, "f32"))
    torch.cuda.synchronize()
    ref = np.empty((sq, d))
    for h in range(heads):
        c = slice(h * dh, (h + 1) * dh)
        # (scores and the mask meet in fp32, where lowest + score is lowest; everything else in fp64)
        s = ((q[:, c].astype(np.float64) @ k[:, c].astype(np.float64).T / math.sqrt(dh)).astype(np.float32) + bias[h]).astype(np.float64)
        p = np.exp(s - s.max(-1, keepdims=True))
        ref[:, c] = p / p.sum(-1, keepdims=True) @ v[:, c].astype(np.float64)
    check(host(ctx), ref, "f32")


@pytest.mark.parametrize("dh", [16, 64])
@pytest.mark.parametrize("tile", [1, 3, 6])
def test_attention_f32_nan_keys(B, dh, tile):
    """NaN in every key of one 32-key tile (all that one wave sees, or the last, ragged one) reaches every row that sees the tile, and no other."""
    import torch
    heads, s = 2, 200
    q, k, v = (draw((s, heads * dh), 140 + i, "f32") for i in range(3))
    k[32 * tile:32 * tile + 32] = np.nan
    ctx = torch.zeros((s, heads * dh), device="cuda")
    B.ac_op_attention(*(B.to_device(t, "f32") for t in (q, k, v)), ctx, heads, dh)
    torch.cuda.synchronize()
    assert torch.isnan(ctx).all()
    B.ac_op_attention(*(B.to_device(t, "f32") for t in (q, k, v)), ctx, heads, dh, causal=True)
    torch.cuda.synchronize()
    assert torch.isnan(ctx[32 * tile:]).all()
    check(host(ctx[:32 * tile]), O.attention(q, k, v, heads, True)[:32 * tile], "f32")


def test_attention_f32_many_blocks(B):
    """257 heads x 65535 problems of 16 queries: as blocks of 256 threads per 16 rows more threads than a grid of one dimension can have."""
    import torch
    heads, dh, batch, sq, sk = 257, 16, 65535, 16, 4
    d = heads * dh
    q, k, v = draw((sq, d), 150, "f32"), draw((sk, d), 151, "f32"), draw((sk, d), 152, "f32")
    ctx = torch.zeros((batch, sq, d), device="cuda")
    B.ac_op_attention(*(B.to_device(t, "f32") for t in (q, k, v)), ctx[0], heads, dh, batch=batch, strides=(0, 0, 0, 0, sq * d))
    torch.cuda.synchronize()
    check(host(ctx[0]), O.attention(q, k, v, heads, False), "f32")
    assert all(torch.equal(ctx[i:i + 1], ctx[:1]) for i in range(1, batch, 1093)) and torch.equal(ctx[-1], ctx[0])


@pytest.mark.parametrize("batch,m,n,k,kernel", [(64, 128, 128, 128, "f32-ring 32x32"), (48, 100, 130, 128, "f32-ring 32x32"), (16, 256, 250, 256, "f32-ring 32x64"),
                                                (16, 150, 140, 512, "f32-ring-deep 32x32")])
def test_many_products_f32_of_whole_tile_depths(B, batch, m, n, k, kernel):
    """Batched launches of the rings, odd rows and columns among them, operands and results apart from their neighbours: the oracle's values, and the bits of
    each product by itself in launches of 33 rows."""
    import torch
    assert B.ac_linear_kernel(m, n, k, "f32", batch=batch) == kernel
    a, w = draw((batch, m, k), 118, "f32"), draw((batch, n, k), 119, "f32", 1 / math.sqrt(k))
    da, dw = (torch.full((batch, r + 3, k + 4), float("nan"), device="cuda") for r in (m, n))
    da[:, :m, :k], dw[:, :n, :k] = B.to_device(a, "f32"), B.to_device(w, "f32")
    out = torch.full((batch, m + 1, n + 6), float("nan"), device="cuda")
    B.ac_op_triangle_contract(da[:, :m, :k], dw[:, :n, :k], out[:, :m, :n])
    torch.cuda.synchronize()
    check(host(out[:, :m, :n]), np.matmul(a.astype(np.float64), w.astype(np.float64).transpose(0, 2, 1)), "f32")
    assert bool(torch.isnan(out[:, m]).all()) and bool(torch.isnan(out[:, :, n:]).all())
    part = torch.full((batch, m, n), float("nan"), device="cuda")
    for b in range(0, batch, 5):
        for r0 in range(0, m, 33):
            B.ac_op_linear(da[b, r0:min(m, r0 + 33), :k], dw[b, :n, :k], part[b, r0:r0 + 33])
    torch.cuda.synchronize()
    assert torch.equal(part[::5], out[::5, :m, :n])


def test_pair_stack_f32_of_whole_tile_depths(B):
    """The contraction over 128 residues on a ring, batches in either order, rows and columns in chunks: the oracle's values, the same bits."""
    import torch
    from oracle import pairstack as P
    from paper_2401_10652_amd import inputs as I
    n, kinds = 128, (B.AC_REGION_TRIMUL_OUT, B.AC_REGION_TRIMUL_IN)
    assert B.ac_linear_kernel(n, n, n, "f32", batch=64) == "f32-ring 32x32"
    cfg = I.PairConfig("tpr", 45, n, 16, 64, 2, 16, 2, "f32")
    z, w = I.pair_inputs(cfg, bias_std=0.1, ln_jitter=0.1)
    dz = B.to_device(z, "f32")
    dw = [B.to_device(w[name], "f32") for name, _ in I.pair_tensor_shapes(cfg)]
    for kind, name in zip(kinds, P.PAIR_MODULES):
        first = None
        for dim, chunk in ((B.AC_DIM_ROW, n), (B.AC_DIM_ROW, 40), (B.AC_DIM_COL, 64)):
            plan = B.Plan(B.pair_desc(cfg, flags=B.AC_FLAG_LISTED_REGIONS_ONLY), [(kind, dim, chunk)])
            plan.ac_plan_bind_weights(dw)
            y = torch.full_like(dz, float("nan"))
            plan.ac_execute(dz, y, B.empty_workspace(plan.ac_plan_query().workspace_bytes))
            torch.cuda.synchronize()
            plan.close()
            first = y if first is None else first
            assert torch.equal(y, first), (name, dim, chunk)
        check(host(first), P.pair_module(name, z, w, cfg.heads, cfg.activation, cfg.ln_eps), "f32", what=name)
