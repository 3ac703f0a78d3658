"""Segments that share launches in idle memory: the same bits as the plan in one segment and as the plan whose two lanes keep the
caller's segments apart (to rounding where attention cuts the keys of their launches differently), from a workspace and an output full of
NaN, and not a byte outside either.  (The peak that such a plan reports counts all that its loops are handed, so its equality with the planned
one says that the plan is kept to; that it suffices is what the bytes outside show.)"""
import pytest

from paper_2401_10652_amd import inputs as I
from util import check, host

pytestmark = pytest.mark.gpu
GUARD = 4096


@pytest.fixture(scope="module")
def B():
    from paper_2401_10652_amd import binding
    binding.lib()
    return binding


def execute(B, desc, weights, x, regs, share=()):
    """The result; the regions of the kinds `share` must take fewer launches than they have segments."""
    import torch
    plan = B.Plan(desc, regs)
    info = plan.ac_plan_query()
    plan.ac_plan_bind_weights(weights)
    need, size = int(info.workspace_bytes), x.numel() * x.element_size()
    ws = torch.full((need + GUARD,), 0xff, dtype=torch.uint8, device="cuda")         # (0xff..ff is a NaN in either type)
    out = torch.full((GUARD + size + GUARD,), 0xff, dtype=torch.uint8, device="cuda")
    y = out[GUARD:GUARD + size].view(x.dtype).view(x.shape)
    x0 = x.clone()
    for _ in range(2):                                                               # the second on what the first left behind
        assert plan.ac_execute(x, y, ws[:need]) == info.peak_bytes_planned
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xff).all()) and bool((out[:GUARD] == 0xff).all()) and bool((out[GUARD + size:] == 0xff).all())
    assert torch.equal(x, x0)
    launches = {r.kind: (r.n_segments, r.launches) for r in info.regions[:info.n_regions]}
    assert all(launches[k][1] < launches[k][0] for k in share), launches
    plan.close()
    return y.clone()


def compare(B, make_desc, shapes, x_shape, dtype, regions, share, seed, exact=True):
    import torch
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(x_shape, generator=gen, device="cuda").to(dt)
    weights = [torch.randn(s, generator=gen, device="cuda").mul_(s[-1] ** -0.5).to(dt) for s in shapes]
    ys = execute(B, make_desc(0), weights, x, regions, share)
    assert bool(torch.isfinite(ys.float()).all())
    for flags, regs in ((0, [(k, dim, 0) for k, dim, _ in regions]), (B.AC_FLAG_TWO_SEGMENTS_IN_FLIGHT, regions)):
        other = execute(B, make_desc(flags), weights, x, regs)
        if exact:
            assert torch.equal(ys, other)
        else:
            check(host(ys), host(other), dtype)


@pytest.mark.parametrize("dtype,batch,seq,chunk,dim,layers,ffn", [
    ("bf16", 1, 520, 72, 1, 3, 512), ("bf16", 3, 136, 40, 1, 1, 1024), ("bf16", 5, 64, 1, 0, 2, 2048), ("f32", 1, 201, 13, 1, 2, 512)])
def test_transformer(B, dtype, batch, seq, chunk, dim, layers, ffn):
    cfg = I.TransformerConfig("tsh", 71, layers, seq, 128, 2, ffn, True, dtype, None, batch=batch)
    shapes = I.transformer_layer_shapes(cfg)
    kinds = (B.AC_REGION_QKV, B.AC_REGION_ATTENTION, B.AC_REGION_OUT_PROJ, B.AC_REGION_FFN)
    compare(B, lambda f: B.transformer_desc(cfg, flags=f), [shapes[n] for _ in range(layers) for n in I.TRANSFORMER_LAYER_TENSORS],
            (cfg.tokens, 128), dtype, [(k, dim, chunk) for k in kinds], kinds, 71)


@pytest.mark.parametrize("dtype,n,c_z,c_hidden,heads,head_dim,chunk", [
    ("bf16", 72, 64, 64, 2, 32, 7), ("bf16", 104, 128, 64, 4, 16, 24), ("f32", 40, 32, 16, 2, 16, 5)])
@pytest.mark.parametrize("dim", [0, 1])
def test_pair(B, dtype, n, c_z, c_hidden, heads, head_dim, chunk, dim):
    cfg = I.PairConfig("psh", 72, n, c_z, c_hidden, heads, head_dim, 2, dtype)
    kinds = range(B.AC_REGION_TRIMUL_OUT, B.AC_REGION_PAIR_TRANSITION + 1)
    # (columns of the bf16 cases' incoming update find no room for a second segment)
    share = [k for k in kinds if not (dim == 1 and dtype == "bf16" and k == B.AC_REGION_TRIMUL_IN)]
    compare(B, lambda f: B.pair_desc(cfg, flags=f), [s for _, s in I.pair_tensor_shapes(cfg)], (n, n, c_z), dtype,
            [(k, dim, chunk) for k in kinds], share, 72)


@pytest.mark.parametrize("n,heads,head_dim,chunk", [(1032, 1, 32, 7), (1088, 2, 32, 23)])
def test_pair_with_key_splits(B, n, heads, head_dim, chunk):
    """Rows of more than 1024 keys: launches of few rows cut them and hold partial results, beside tensors that share their launch."""
    cfg = I.PairConfig("psk", 74, n, 64, 64, heads, head_dim, 2, "bf16")
    kind = B.AC_REGION_TRIATT_START
    compare(B, lambda f: B.pair_desc(cfg, flags=f | B.AC_FLAG_LISTED_REGIONS_ONLY), [s for _, s in I.pair_tensor_shapes(cfg)], (n, n, 64), "bf16",
            [(kind, B.AC_DIM_ROW, chunk)], [kind], 74, exact=False)


def unet(B, layers, batch, h, w, c, heads, f, context, gated, chunks, share, exact=True):
    cfg = I.ResStackConfig("ush", 73, layers, batch, h, w, c, 16, heads=heads, d_ffn=f, context_tokens=context, context_dim=24 if context else 0,
                           gated=gated)
    up = 2 if gated else 1
    special = {"w1": (c, 9 * c), "w2": (c, 9 * c), "temb": (batch, c), "w_in": (c, c), "w_qkv": (3 * c, c), "b_qkv": (3 * c,),
               "w_o": (c, c), "w_1": (up * f, c), "b_1": (up * f,), "w_2": (c, f), "w_out": (c, c), "w_qc": (c, c),
               "w_kvc": (2 * c, 24), "w_oc": (c, c), "context": (batch * context, 24)}
    names = list(I.RES_BLOCK_TENSORS) + list(I.attn_block_tensors(cfg))
    kinds = [B.AC_REGION_RES_BLOCK, B.AC_REGION_UNET_ATTN][:1 + (heads > 0)]
    compare(B, lambda fl: B.res_stack_desc(cfg, flags=fl), [special.get(n, (c,)) for _ in range(layers) for n in names],
            (batch, h, w, c), "bf16", [(k, B.AC_DIM_BATCH, n) for k, n in zip(kinds, chunks)], kinds[:share], 73, exact)


@pytest.mark.parametrize("layers,batch,chunk,heads,context,gated", [
    (1, 7, 2, 0, 0, False), (3, 5, 1, 0, 0, False), (1, 8, 2, 2, 0, False), (2, 7, 1, 2, 13, True)])
def test_unet(B, layers, batch, chunk, heads, context, gated):
    unet(B, layers, batch, 8, 16, 64, heads, 128 if heads else 0, context, gated, (chunk, chunk), 2)


@pytest.mark.parametrize("batch,h,w,c,heads,f,gated,chunks,share,exact", [
    (9, 32, 40, 128, 4, 512, False, (2, 2), 2, True),       # two runs of keys whatever a launch's images
    (9, 32, 40, 128, 4, 512, True, (2, 2), 2, True),
    (18, 80, 16, 128, 4, 192, False, (4, 11), 1, False),    # two runs in a launch of the last seven images, which then has no room
    (14, 72, 16, 320, 5, 320, True, (9, 9), 2, False)])
def test_unet_with_key_splits(B, batch, h, w, c, heads, f, gated, chunks, share, exact):
    unet(B, 1, batch, h, w, c, heads, f, 0, gated, chunks, share, exact)
