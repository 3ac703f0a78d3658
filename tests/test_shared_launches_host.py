"""Plans whose segments share launches run to their end: the walk of ac_execute with the kernel launches stubbed out, so that no GPU
is needed and no pointer is followed."""
import pytest

import launch_stub

WALK = """
def walk(what, desc, regions):
    plan = B.Plan(desc, regions)
    info = plan.ac_plan_query()
    ptrs = (B.VP * info.n_weights)(*[(1 << 44) + 256 * i for i in range(info.n_weights)])
    assert L.ac_plan_bind_weights(plan._h, ptrs, info.n_weights) == 0
    peak = B.U64(0)
    status = L.ac_execute(plan._h, X, Y, W, info.workspace_bytes, None, ctypes.byref(peak))
    assert status == 0, (what, L.ac_last_error())
    assert peak.value <= info.peak_bytes_planned, what
    assert all(r.launches <= r.n_segments for r in info.regions[:info.n_regions]), what

def unet(batch, h, w, c, heads, f, c_res, c_attn, gated=False, context=0, layers=1):
    cfg = I.ResStackConfig("plan", 1, layers, batch, h, w, c, 16, heads=heads, d_ffn=f, gated=gated,
                           context_tokens=context, context_dim=64 if context else 0)
    walk(("unet", batch, h, w, c, heads, f, c_res, c_attn, gated, context, layers), B.res_stack_desc(cfg),
         [(B.AC_REGION_RES_BLOCK, B.AC_DIM_BATCH, c_res), (B.AC_REGION_UNET_ATTN, B.AC_DIM_BATCH, c_attn)])

def pair(n, c_z, heads, dh, settings):
    cfg = I.PairConfig("plan", 1, n, c_z, 64, heads, dh, 2, "bf16")
    walk(("pair", n, c_z, heads, dh, settings), B.pair_desc(cfg, flags=B.AC_FLAG_LISTED_REGIONS_ONLY), [(k, B.AC_DIM_ROW, c) for k, c in settings])
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    lib = launch_stub.build(str(tmp_path_factory.mktemp("stub")))
    return lambda calls: launch_stub.run(lib, WALK + calls)


@pytest.mark.parametrize("call", [
    "unet(14, 72, 16, 320, 5, 320, 9, 9)", "unet(16, 72, 16, 320, 5, 64, 9, 9)", "unet(17, 64, 24, 640, 10, 320, 4, 4)",
    "unet(21, 64, 24, 192, 3, 192, 13, 13)", "unet(18, 80, 16, 128, 4, 192, 4, 11)", "unet(48, 40, 96, 128, 1, 256, 22, 9)",
    "unet(35, 72, 48, 64, 2, 64, 23, 8)", "pair(1088, 64, 2, 32, [(B.AC_REGION_TRIATT_START, 23)])"])
def test_a_short_run_needs_more_scratch_than_a_long_one(walk, call):
    """A launch of few problems cuts their keys into more runs, each with partial results, and the last run of a region has no rows of
    the result left to borrow: such a run must not be taken for one that fits."""
    walk(call)


def test_drawn_plans(walk):
    walk("""
rng = random.Random(2)
for i in range(12000):
    if i % 2:
        n, listed = 8 * rng.randint(3, 225), sorted(rng.sample(range(B.AC_REGION_TRIMUL_OUT, B.AC_REGION_PAIR_TRANSITION + 1), rng.randint(1, 5)))
        pair(n, 64, rng.choice([1, 2, 4]), rng.choice([16, 32, 64]), [(k, rng.randint(1, rng.choice([n, 1 + n // 20]))) for k in listed])
    else:
        batch, c, dh = rng.randint(1, 50), rng.choice([64, 128, 192, 320, 640]), rng.choice([32, 64])
        unet(batch, 8 * rng.randint(1, 12), 8 * rng.randint(1, 12), c, c // dh, 64 * rng.randint(1, max(1, c // 16)), rng.randint(1, batch),
             rng.randint(1, batch), rng.random() < 0.3, rng.choice([0, 0, 13]), rng.choice([1, 1, 2, 3]))
""")


def test_a_transition_of_few_rows_takes_two_launches(walk):
    """One block walks the hidden columns of its rows by itself; where rows are few, the two launches share the columns out."""
    walk("""
def kernels_of(n, c_z, factor, activation, chunk=None, flags=0):
    kernels()
    cfg = I.PairConfig("plan", 1, n, c_z, 64, 2, 32, factor, "bf16", activation=activation)
    walk((n, c_z, factor, activation, chunk), B.pair_desc(cfg, flags=B.AC_FLAG_LISTED_REGIONS_ONLY), [(B.AC_REGION_PAIR_TRANSITION, B.AC_DIM_ROW, chunk or n)])
    return kernels()

def one_kernel(*args):
    names = kernels_of(*args)
    ours = ["pair_transition" in k for k in names]
    assert all(ours) or (not any(ours) and len(names) % 2 == 0), names
    return ours[0]

for n, c_z, factor, activation, one in (
        (8, 128, 8, "gelu_erf", False), (96, 128, 8, "gelu_tanh", False), (112, 128, 8, "gelu_erf", True), (8, 128, 4, "relu", False), (64, 128, 4, "relu", False),
        (72, 128, 4, "relu", True), (200, 128, 4, "relu", True), (8, 128, 2, "relu", True), (8, 128, 1, "gelu_erf", True), (8, 64, 4, "gelu_erf", True),
        (8, 64, 8, "gelu_erf", False), (96, 64, 8, "gelu_erf", True), (8, 64, 8, "relu", True), (64, 64, 12, "relu", False)):
    for chunk in (n, (n + 2) // 3, 1):
        assert one_kernel(n, c_z, factor, activation, chunk) == one, (n, c_z, factor, activation, chunk)
""")


def test_layers_of_128_channels_take_their_tail_apart_where_rows_are_few_or_many(walk):
    """fp32 layers: the kernel of all that follows the attention core where it is ahead of its four launches."""
    walk("""
def tail(batch, seq, d, chunk, dim=B.AC_DIM_SEQ):
    kernels()
    cfg = I.TransformerConfig("plan", 1, 1, seq, d, 2, 4 * d, False, "f32", None, batch=batch)
    kinds = (B.AC_REGION_QKV, B.AC_REGION_ATTENTION, B.AC_REGION_OUT_PROJ, B.AC_REGION_FFN)
    plan = B.Plan(B.transformer_desc(cfg), [(k, dim, chunk) for k in kinds])
    info = plan.ac_plan_query()
    assert L.ac_plan_bind_weights(plan._h, (B.VP * info.n_weights)(*[(1 << 44) + 256 * i for i in range(info.n_weights)]), info.n_weights) == 0
    assert L.ac_execute(plan._h, X, Y, W, info.workspace_bytes, None, None) == 0, L.ac_last_error()
    names = kernels()
    fused = any("layer_tail" in k for k in names)
    assert fused != any("layernorm" in k for k in names[1:]), names
    return fused

for d in (32, 64):
    for batch, seq in ((1, 16), (1, 2048), (128, 128), (512, 128)):
        assert tail(batch, seq, d, seq)
for batch, seq, chunk, one in ((1, 16, 16, False), (1, 256, 64, False), (8, 128, 128, False), (1, 4096, 4096, False), (1, 5000, 5000, True), (48, 128, 128, True),
                               (2, 5000, 5000, True), (2, 5000, 2000, True), (1, 20480, 20480, True), (160, 128, 128, True), (256, 128, 128, False), (1, 20496, 20496, False)):
    assert tail(batch, seq, 128, chunk) == one, (batch, seq, chunk)
assert tail(2, 3000, 128, 1, B.AC_DIM_BATCH) == False and tail(2, 3000, 128, 2, B.AC_DIM_BATCH) == True
""")
