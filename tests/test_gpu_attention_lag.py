"""The attention kernel's exponent reference, which moves only when a score passes it, and the pipelined loop with a ragged last tile:
against the fp64 oracle, with NaN in whatever lies behind the keys."""
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


def run(B, q, k, v, heads, causal, q_offset=0, bias=None, n_splits=1):
    """One problem; k [sk, d] and v [sk, d] handed over in buffers whose rest is NaN."""
    import torch
    sq, sk, d = q.shape[0], k.shape[0], q.shape[1]
    kb = torch.full((sk + 80, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    vb = torch.full((d + 1, sk + (-sk) % 8 + 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    kb[:sk], vb[:d, :sk] = B.to_device(k, "bf16"), B.to_device(v, "bf16").T
    ctx = torch.full((sq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = B.empty_workspace(max(256, B.ac_attention_split_workspace_bytes(sq, heads, 1, d // heads, n_splits)))
    db = None
    if bias is not None:
        db = torch.full((heads, sq, sk + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        db[:, :, :sk] = B.to_device(bias, "bf16")
    B.ac_op_attention(B.to_device(q, "bf16"), kb[:sk], vb[:d], ctx, heads, d // heads, causal=causal, q_offset=q_offset, bias=db,
                      v_transposed=True, n_splits=n_splits, split_workspace=ws)
    torch.cuda.synchronize()
    return host(ctx)


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("sq,sk,causal,q_offset,n_splits", [
    (100, 328, False, 0, 1), (33, 520, True, 487, 1), (300, 1032, False, 0, 2), (64, 72, True, 8, 1), (200, 392, True, 150, 1),
    (130, 1096, True, 966, 3), (129, 320, True, 0, 1), (40, 312, False, 0, 1)])
@pytest.mark.parametrize("growth", [1.0, 40.0])
def test_ragged_key_tiles(B, dh, sq, sk, causal, q_offset, n_splits, growth):
    heads = 2
    q, k, v = (draw((n, heads * dh), 300 + i, "bf16") for i, n in enumerate((sq, sk, sk)))
    # the scores' spread grows along the keys to `growth` units: hundreds of binary orders, raised several times over
    k = (k * (growth / 2 * np.linspace(0.05, 1.0, sk)[:, None] if growth > 1 else k * 0 + 1)).astype(np.float32)
    from paper_2401_10652_amd.inputs import round_to_storage
    k = round_to_storage(k, "bf16")
    check(run(B, q, k, v, heads, causal, q_offset, None, n_splits), O.attention(q, k, v, heads, causal, q_offset=q_offset), "bf16")


@pytest.mark.parametrize("dh,biased", [(32, False), (64, False), (64, True), (128, False)])
@pytest.mark.parametrize("sk,n_splits", [(384, 1), (392, 1), (328, 1), (1096, 2)])
@pytest.mark.parametrize("order", [100, 114, -100])
def test_values_near_the_ends_of_the_range(B, dh, biased, sk, n_splits, order):
    """Scores that grow along the keys, some of them by up to tens of binary orders between two moves of the reference: no product
    or sum of probabilities and values may leave the range that the result stays in."""
    from paper_2401_10652_amd.inputs import round_to_storage
    heads, sq = 2, 100
    q, k, v = (draw((n, heads * dh), 340 + i, "bf16") for i, n in enumerate((sq, sk, sk)))
    k = round_to_storage((k * (6.0 * np.linspace(0.05, 1.0, sk)[:, None])).astype(np.float32), "bf16")
    v = np.clip(v, -2, 2) * 2.0 ** order
    bias = draw((heads, sq, sk), 343, "bf16") if biased else None
    got = run(B, q, k, v.astype(np.float32), heads, False, bias=bias, n_splits=n_splits)
    check(got * 2.0 ** -order, O.attention(q, k, v * 2.0 ** -order, heads, False, bias=bias), "bf16")


@pytest.mark.parametrize("dh,sq,sk,batch", [(64, 264, 328, 256), (128, 260, 136, 256)])
def test_ragged_key_tiles_in_256_row_blocks(B, dh, sq, sk, batch):
    import torch
    heads, d = 2, 2 * dh
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((batch, n, d), generator=gen, device="cuda").bfloat16() for n in (sq, sk, sk))
    vt = v.transpose(1, 2).contiguous()
    ctx = torch.full_like(q, float("nan"))
    B.ac_op_attention(q[0], k[0], vt[0], ctx[0], heads, dh, v_transposed=True, batch=batch, strides=(sq * d, sk * d, d * sk, 0, sq * d))
    torch.cuda.synchronize()
    for b in (0, 100, batch - 1):
        check(host(ctx[b]), O.attention(host(q[b]), host(k[b]), host(v[b]), heads, False), "bf16")


@pytest.mark.parametrize("dh", [32, 64])
@pytest.mark.parametrize("sk", [192, 200])
@pytest.mark.parametrize("mask", [-1e30, float("-inf"), float(np.finfo(np.float32).min)])
def test_masks_over_the_first_tiles(B, dh, sk, mask):
    """Rows whose first tiles are masked altogether, and later tiles far above the first ones."""
    heads, sq = 2, 70
    q, k, v = (draw((n, heads * dh), 310 + i, "bf16") for i, n in enumerate((sq, sk, sk)))
    bias = draw((heads, sq, sk), 313, "bf16", 3.0)
    bias[:, :, 128:] += 90.0
    from paper_2401_10652_amd.inputs import round_to_storage
    bias = round_to_storage(bias, "bf16").astype(np.float64)
    if np.isfinite(mask):   # the largest bf16 below: what such a mask is in storage
        mask = max(mask, -3.3895313892515355e38)
    bias[:, 10:40, :130] = mask
    bias[:, 50:, 64:] = mask
    if mask == -1e30:
        bias[:, 45:48] = mask          # a row of nothing else averages its values
    b32 = round_to_storage(bias.astype(np.float32), "bf16")
    check(run(B, q, k, v, heads, False, bias=b32), O.attention(q, k, v, heads, False, bias=b32), "bf16")


@pytest.mark.parametrize("ldv", [8454656, 8454664, 9437184])
def test_values_in_far_rows(B, ldv):
    """Rows of V^T up to the 2^31 bytes of the pipelined loop's buffer, and beyond."""
    import torch
    sq, sk, dh = 100, 328, 128
    q, k, v = (draw((n, dh), 320 + i, "bf16") for i, n in enumerate((sq, sk, sk)))
    vb = torch.empty((dh, ldv), dtype=torch.bfloat16, device="cuda")
    vb[:, :sk], vb[:, sk:sk + 64] = B.to_device(v, "bf16").T, float("nan")
    ctx = torch.full((sq, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.ac_op_attention(B.to_device(q, "bf16"), B.to_device(k, "bf16"), vb, ctx, 1, dh, v_transposed=True)
    torch.cuda.synchronize()
    check(host(ctx), O.attention(q, k, v, 1, False), "bf16")


@pytest.mark.parametrize("dh,sk,causal", [(64, 384, True), (64, 392, False), (128, 384, False), (128, 392, True)])
@pytest.mark.parametrize("which", ["k", "v"])
def test_rows_in_descending_order(B, dh, sk, causal, which):
    """A key or a value operand whose rows lie behind each other (a negative stride), in the middle of memory it must not reach beyond."""
    import torch
    sq = 150
    q, k, v = (draw((n, dh), 330 + i, "bf16") for i, n in enumerate((sq, sk, sk)))
    dq, dk, dv = B.to_device(q, "bf16"), B.to_device(k, "bf16"), B.to_device(v, "bf16").T.contiguous()

    def placed(t, descending):
        """(address of row 0, row stride, the buffer)"""
        buf = torch.full((3, *t.shape), float("nan"), dtype=t.dtype, device="cuda")
        buf[1] = t.flip(0) if descending else t
        row = t.shape[1]
        return buf[1, t.shape[0] - 1 if descending else 0].data_ptr(), -row if descending else row, buf
    kp, ldk, kb = placed(dk, which == "k")
    vp, ldv, vb = placed(dv, which == "v")
    ctx = torch.full((sq, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    status = B.lib().ac_op_attention(dq.data_ptr(), dh, 0, kp, ldk, 0, vp, ldv, 0, 1, None, 0, 0, None, 0, 0, ctx.data_ptr(), dh, 0, 1, sq, sk, 1, dh,
                                     int(causal), sk - sq if causal else 0, 1, None, 0, B.AC_BF16, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert status == 0
    check(host(ctx), O.attention(q, k, v, 1, causal, q_offset=sk - sq if causal else 0), "bf16")


@pytest.mark.parametrize("dh", [32, 64])
def test_masked_rows_leave_their_neighbours_alone(B, dh):
    """Rows whose biases lie far from zero among others: the others' bits are those of a launch without them."""
    import torch
    heads, sq, sk = 2, 160, 192
    g = torch.Generator(device="cuda").manual_seed(77)
    q, k = (torch.randn((s, heads * dh), generator=g, device="cuda").bfloat16() for s in (sq, sk))
    vt = torch.randn((heads * dh, sk), generator=g, device="cuda").bfloat16()
    bias = torch.randn((heads, sq, sk), generator=g, device="cuda").mul_(3).bfloat16()
    plain, mixed = torch.empty_like(q), torch.empty_like(q)
    B.ac_op_attention(q, k, vt, plain, heads, dh, bias=bias, v_transposed=True)
    far = bias.clone()
    far[:, ::3] -= 1e9
    B.ac_op_attention(q, k, vt, mixed, heads, dh, bias=far, v_transposed=True)
    torch.cuda.synchronize()
    others = [r for r in range(sq) if r % 3]
    assert torch.equal(plain[others], mixed[others]) and bool(torch.isfinite(mixed.float()).all())


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("sk", [192, 200])
@pytest.mark.parametrize("common", [-1e3, -1e4, -1e5, -6e5, -1e6, 1e5])
def test_rows_whose_keys_share_a_large_bias(B, dh, sk, common):
    """A score is rounded once at the bias's magnitude, in log2 units, whatever the head's width (the bias's own rounding there is the same for all keys):
    the relative error of a probability, uniform within that half unit, is that of the context in 2-norm, beside the bf16 roundings of probabilities and
    result.  Every third row is such a row; the others are as exact as ever."""
    from paper_2401_10652_amd.inputs import round_to_storage
    heads, sq = 4, 160
    q, k, v = (draw((n, heads * dh), 350 + i, "bf16") for i, n in enumerate((sq, sk, sk)))
    bias = draw((heads, sq, sk), 353, "bf16")
    bias[:, ::3] = common
    bias = round_to_storage(bias.astype(np.float32), "bf16")
    got, ref = run(B, q, k, v, heads, False, bias=bias), O.attention(q, k, v, heads, False, bias=bias)
    shared = np.arange(sq) % 3 == 0
    half_unit = float(np.spacing(np.float32(abs(bias[0, 0, 0]) * 1.4426950408889634))) / 2 * np.log(2)
    for rows, h in ((shared, half_unit), (~shared, 0.0)):
        err = np.linalg.norm(got[rows] - ref[rows]) / np.linalg.norm(ref[rows])
        # (uniform errors: a third of the half units' squares; bf16's are 2^-8 of a value at the foot of a binade, 0.54 of its square in the mean over it)
        bound = 1.25 * np.sqrt((2 * 0.54 * 2.0 ** -16 + h * h) / 3)
        assert err <= bound, (err, bound)


@pytest.mark.parametrize("dtype,batch,sq,heads,dh", [
    ("bf16", 256, 200, 1, 64), ("bf16", 3, 256, 2, 128), ("bf16", 12, 500, 4, 64), ("bf16", 7, 1000, 6, 64), ("bf16", 5, 700, 3, 128), ("bf16", 2, 4200, 2, 64),
    ("f32", 1, 520, 8, 32), ("f32", 2, 1100, 4, 64), ("f32", 3, 520, 2, 32), ("f32", 5, 300, 8, 16), ("f32", 1, 2431, 4, 64)])
def test_causal_blocks_in_whatever_order(B, dtype, batch, sq, heads, dh):
    """Heads of one, two, four, eight and other numbers of blocks, whole numbers of heads per XCD and others: each problem's rows are those of a launch
    with this problem alone, one head after another."""
    import torch
    d = heads * dh
    gen = torch.Generator(device="cuda").manual_seed(6)
    q, k, v = (torch.randn((batch, sq, d), generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(3))
    vt = v.transpose(1, 2).contiguous() if dtype == "bf16" else v
    ctx, alone = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    B.ac_op_attention(q[0], k[0], vt[0], ctx[0], heads, dh, causal=True, v_transposed=dtype == "bf16", batch=batch, strides=(sq * d, sq * d, sq * d, 0, sq * d))
    for b in range(batch) if batch <= 12 else (0, 1, batch // 2, batch - 1):
        for h in range(heads):
            c = slice(h * dh, (h + 1) * dh)
            B.ac_op_attention(q[b, :, c], k[b, :, c], vt[b, c] if dtype == "bf16" else vt[b, :, c], alone[b, :, c], 1, dh, causal=True, v_transposed=dtype == "bf16")
        torch.cuda.synchronize()
        assert torch.equal(ctx[b], alone[b]), b
    assert bool(torch.isfinite(ctx.float()).all())
