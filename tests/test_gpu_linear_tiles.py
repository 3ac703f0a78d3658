"""GPU parity of the bf16 GEMM's tile shapes at their edges: k of one to seven tiles (shorter than, equal to and longer than the ring of
LDS buffers), rows and columns that end inside a tile, batched products, and equal bits whatever shape a launch takes."""
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


@pytest.mark.parametrize("m,n", [
    (5000, 5000),      # 256x256 (one tile of k: 128x128 through registers)
    (8100, 1020),      # 256x128
    (4000, 760),       # 128x128 with a ring
    (1000, 640),       # 64x64, at most one per CU
    (1990, 2040),      # 128x128 with a ring, its 1017-row launches also 128x64
    (100, 100),        # 32x64 (one tile of k: 64x64)
])
@pytest.mark.parametrize("k", [64, 128, 192, 320, 448])
def test_linear_tiles(B, m, n, k):
    """One launch against fp64 on sampled rows, and against the same rows in launches of other tile shapes, bit for bit."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    a = torch.randn((m, k), generator=g, device="cuda").bfloat16()
    w = (torch.randn((n, k), generator=g, device="cuda") / math.sqrt(k)).bfloat16()
    res = torch.randn((m, n), generator=g, device="cuda").bfloat16()
    out = torch.full((m, n), float("nan"), device="cuda", dtype=torch.bfloat16)
    B.ac_op_linear(a, w, out, residual=res)
    rows = np.unique(np.concatenate([np.arange(min(m, 40)), np.arange(max(0, m - 40), m), np.arange(0, m, 61)]))
    t = torch.from_numpy(rows).cuda()
    check(host(out[t]), O.linear(host(a[t]), host(w)) + host(res[t]), "bf16")
    part = torch.full((m, n), float("nan"), device="cuda", dtype=torch.bfloat16)
    for r0 in range(0, m, 1017):
        r1 = min(m, r0 + 1017)
        B.ac_op_linear(a[r0:r1], w, part[r0:r1], residual=res[r0:r1])
    assert torch.equal(part, out)


@pytest.mark.parametrize("tile,m,n,k", [
    ("quad 256x256", 1684, 5708, 64), ("quad 256x256", 1445, 5780, 128), ("quad 256x256", 7215, 1096, 256),
    ("ring 256x128", 773, 5000, 64), ("ring 256x128", 5473, 708, 192),
    ("ring 128x128", 8267, 68, 64), ("ring 128x128", 291, 5448, 256),
    ("staged 128x128", 1314, 5464, 64), ("staged 128x128", 2371, 3408, 192),
    ("ring 128x64", 8270, 408, 64), ("ring 128x64", 4785, 196, 256),
    ("ring 64x64", 150, 8, 64), ("ring 64x64", 1000, 644, 448),
    ("staged 64x64", 1000, 644, 512), ("staged 64x64", 950, 1020, 1024),
    ("staged 32x64", 500, 1020, 4096), ("staged 32x64", 201, 500, 2048),
])
def test_every_tile(B, tile, m, n, k):
    """Each kernel and tile, one and more tiles of k, rows and columns that end inside a tile: against fp64 on sampled rows and bit for
    bit against launches of 97 rows, which take other tiles (GELU and the residual in the epilogue)."""
    import torch
    assert B.ac_linear_kernel(m, n, k, "bf16") == tile
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    a = torch.randn((m, k), generator=g, device="cuda").bfloat16()
    w = (torch.randn((n, k), generator=g, device="cuda") / math.sqrt(k)).bfloat16()
    res = torch.randn((m, n), generator=g, device="cuda").bfloat16()
    out, part = (torch.full((m, n), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    B.ac_op_linear(a, w, out, residual=res, activation=B.AC_ACT_GELU_ERF)
    rows = np.unique(np.concatenate([np.arange(min(m, 40)), np.arange(max(0, m - 40), m), np.arange(0, m, 61)]))
    t = torch.from_numpy(rows).cuda()
    check(host(out[t]), O.gelu_erf(O.linear(host(a[t]), host(w))) + host(res[t]), "bf16")
    for r0 in range(0, m, 97):
        B.ac_op_linear(a[r0:r0 + 97], w, part[r0:r0 + 97], residual=res[r0:r0 + 97], activation=B.AC_ACT_GELU_ERF)
    assert torch.equal(part, out)


@pytest.mark.parametrize("c,ni,nj,nk", [(16, 64, 1024, 1024), (3, 700, 900, 192), (5, 40, 72, 64)])
def test_batched_products(B, c, ni, nj, nk):
    import torch
    a, b = draw((c, ni, nk), 140, "bf16"), draw((c, nj, nk), 141, "bf16", 1 / math.sqrt(nk))
    out = torch.full((c, ni, nj), float("nan"), device="cuda", dtype=torch.bfloat16)
    B.ac_op_triangle_contract(B.to_device(a, "bf16"), B.to_device(b, "bf16"), out)
    torch.cuda.synchronize()
    check(host(out), np.matmul(a.astype(np.float64), b.astype(np.float64).transpose(0, 2, 1)), "bf16")


@pytest.mark.parametrize("c,ni,nj,nk", [(6, 40, 200, 200), (3, 70, 72, 8), (2, 100, 136, 72), (128, 33, 328, 328), (4, 2000, 2100, 1000), (128, 197, 200, 200), (128, 200, 200, 72)])
def test_depth_that_is_no_multiple_of_a_tile(B, c, ni, nj, nk):
    """k of whole 16-byte chunks that ends inside a tile of 64 (64x64 tiles, the last three 256x128): what lies past the end of a row must not
    count, so the operands are column blocks of tensors whose other columns hold NaN."""
    import torch
    assert B.ac_linear_kernel(ni, nj, nk, "bf16", lda=nk + 64, ldw=nk + 64, batch=c) == ("ragged 256x128" if c * ni >= 8000 else "ragged 64x64")
    a, b = draw((c, ni, nk), 150, "bf16"), draw((c, nj, nk), 151, "bf16", 1 / math.sqrt(nk))
    wide_a = torch.full((c, ni, nk + 64), float("nan"), device="cuda", dtype=torch.bfloat16)
    wide_b = torch.full((c, nj, nk + 64), float("nan"), device="cuda", dtype=torch.bfloat16)
    wide_a[..., :nk], wide_b[..., :nk] = B.to_device(a, "bf16"), B.to_device(b, "bf16")
    out = torch.full((c, ni, nj), float("nan"), device="cuda", dtype=torch.bfloat16)
    B.ac_op_triangle_contract(wide_a[..., :nk], wide_b[..., :nk], out)
    torch.cuda.synchronize()
    check(host(out), np.matmul(a.astype(np.float64), b.astype(np.float64).transpose(0, 2, 1)), "bf16")
    part = torch.full_like(out, float("nan"))
    B.ac_op_triangle_contract(wide_a[:, :17, :nk], wide_b[..., :nk], part[:, :17])
    torch.cuda.synchronize()
    assert torch.equal(part[:, :17], out[:, :17])


@pytest.mark.parametrize("m,n", [(70, 60), (200, 520)])
@pytest.mark.parametrize("side", ["a", "w"])
def test_long_row_strides(B, m, n, side):
    """Operand rows 2^22 elements apart: equal bits to the same rows side by side."""
    import torch
    k = 192
    a, w = B.to_device(draw((m, k), 160, "bf16"), "bf16"), B.to_device(draw((n, k), 161, "bf16", 1 / math.sqrt(k)), "bf16")
    ref, out = (torch.full((m, n), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    B.ac_op_linear(a, w, ref)
    near = a if side == "a" else w
    far = torch.empty(((near.shape[0] - 1) << 22) + k, device="cuda", dtype=torch.bfloat16).as_strided(near.shape, (1 << 22, 1))
    far.copy_(near)
    B.ac_op_linear(*((far, w) if side == "a" else (a, far)), out)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


@pytest.mark.parametrize("m,n,k", [(6399, 764, 1600), (3001, 1500, 1664), (6273, 708, 3072)])
def test_192_column_tiles(B, m, n, k):
    """Rows and columns that end inside a 128x192 tile: as test_every_tile."""
    test_every_tile(B, "ring 128x192", m, n, k)


@pytest.mark.parametrize("images,h,w,ci,co", [(5, 57, 56, 128, 320), (2, 91, 90, 128, 320), (1, 1, 16003, 192, 320)])
def test_192_column_tiles_of_the_convolution(B, images, h, w, ci, co):
    """Against fp64 on sampled pixels, and bit for bit against launches of one image or of fewer columns (64x64 tiles)."""
    import torch
    assert B.ac_linear_kernel(images * h * w, co, 9 * ci, "bf16", lda=ci, conv=True) == "conv 128x192"
    g = torch.Generator(device="cuda").manual_seed(co)
    x = torch.randn((images, h, w, ci), generator=g, device="cuda").bfloat16()
    wt = (torch.randn((co, 3, 3, ci), generator=g, device="cuda") / math.sqrt(9 * ci)).bfloat16()
    res = torch.randn((images, h, w, co), generator=g, device="cuda").bfloat16()
    out = torch.full((images, h, w, co), float("nan"), device="cuda", dtype=torch.bfloat16)
    B.ac_op_conv3x3(x, wt, out, residual=res)
    pad = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    ref = sum(pad[:, i:i + h, j:j + w] @ wt[:, i, j].double().T.contiguous() for i in range(3) for j in range(3)) + res.double()
    check(host(out), ref.cpu().numpy(), "bf16")
    for i in range(images):
        for n0 in range(0, co, 40):
            part = torch.full((1, h, w, 40), float("nan"), device="cuda", dtype=torch.bfloat16)
            B.ac_op_conv3x3(x[i:i + 1], wt[n0:n0 + 40].contiguous(), part, residual=res[i:i + 1, ..., n0:n0 + 40].contiguous())
            assert torch.equal(part[0], out[i, ..., n0:n0 + 40])
