"""Which kernel and tile a product takes: the rule runs on the host, so it is checked without a GPU."""
import pytest

from paper_2401_10652_amd import binding as B
from paper_2401_10652_amd.build import ensure_built

THREADS = {"fma": 256, "f32": 256, "f32-ring": 256, "f32-ring-deep": 256, "staged 32x64": 128, "staged": 256, "quad": 512, "ring 256x128": 512, "ring 128x128": 512, "ring": 256,
           "ragged 256x128": 512, "ragged": 256, "conv 128x128": 512, "conv": 256,
           "conv-wide": 256}


@pytest.fixture(scope="module", autouse=True)
def built():
    ensure_built()


def grid_threads(name, m, n):
    """Threads in the first dimension of the launch."""
    kind, tile = name.split()
    bm, bn = (int(t) for t in tile.split("x"))
    per_block = THREADS.get(name, THREADS[kind])
    return -(-n // bn) * per_block if kind == "fma" else -(-m // bm) * -(-n // bn) * per_block


@pytest.mark.parametrize("dtype,m,n,k", [
    ("f32", 65537, 65536, 64), ("f32", 66000, 70000, 512), ("f32", 1 << 20, 1 << 15, 64), ("f32", (1 << 30) + 1, 16, 4),
    ("bf16", 1 << 21, 1 << 16, 72), ("bf16", 1 << 21, 1 << 15, 8), ("bf16", 1 << 21, 1 << 16, 64), ("bf16", (1 << 30) - 1, 64, 200),
])
def test_large_products_fit_a_grid_dimension(dtype, m, n, k):
    assert grid_threads(B.ac_linear_kernel(m, n, k, dtype), m, n) < 1 << 32


@pytest.mark.parametrize("c", [64, 128, 256])
def test_many_pixels_fit_a_grid_dimension(c):
    """8 output channels of a little under 2^30 pixels."""
    m = (1 << 30) - 64
    assert grid_threads(B.ac_linear_kernel(m, 8, 9 * c, "bf16", lda=c, conv=True), m, 8) < 1 << 32


@pytest.mark.parametrize("m,n,k", [(1000, 1024, 1024), (100, 768, 768), (8192, 4096, 64), (16, 64, 1 << 22)])
@pytest.mark.parametrize("side", ["lda", "ldw"])
def test_long_row_strides_keep_the_matrix_cores(m, n, k, side):
    """Rows 2^22 elements apart and more: the loops with 64-bit addresses, not the FMA kernel."""
    for stride in (1 << 22, 1 << 33):
        assert B.ac_linear_kernel(m, n, k, "bf16", **{side: stride}).startswith("staged")
    assert not B.ac_linear_kernel(m, n, min(k, 1024), "bf16", **{side: (1 << 22) - 8}).startswith("fma")


@pytest.mark.parametrize("m,n,k", [(1024, 2048, 512), (1024, 1536, 512), (768, 512, 512), (1500, 2048, 512), (200, 1536, 512)])
def test_a_row_more_does_not_send_an_fp32_product_to_the_smallest_tile(m, n, k):
    for rows in (m, m + 1, m + 9):
        assert B.ac_linear_kernel(rows, n, k, "f32").split()[1] in ("32x64", "32x32")


def test_near_ties_of_fp32_tiles_go_to_the_larger():
    """(Depths of whole tiles in each part of a sum have prices of their own, fitted closely enough for no preference.)"""
    for m, n, k in ((1024, 1536, 500), (4000, 2048, 124), (4000, 2048, 96)):
        assert B.ac_linear_kernel(m, n, k, "f32") == "f32 32x64"
    for m, n, k in ((1024, 1536, 512), (4000, 2048, 128)):
        assert B.ac_linear_kernel(m, n, k, "f32") == "f32-ring 32x64"


def test_short_fp32_sums_of_many_columns_take_one_kernel_whatever_the_rows():
    for m in (1, 100, 1000, 20000):
        assert B.ac_linear_kernel(m, 1024, 64, "f32") == "fma 64x64"
        assert B.ac_linear_kernel(m, 1020, 64, "f32").startswith("f32") and B.ac_linear_kernel(m, 4096, 68, "f32").startswith("f32")


def test_ragged_depths_are_priced_among_the_tiles_that_exist():
    """(2000 x 2100 and 720 x 616 are fastest on the 128x128 tile by estimate, which ragged depths do not have.)"""
    for m, n, k, batch in ((2000, 2100, 1000, 4), (720, 616, 280, 128), (200, 200, 200, 128)):
        assert B.ac_linear_kernel(m, n, k, "bf16", batch=batch) == "ragged 256x128"
    for m, n, k, batch in ((40, 200, 200, 128), (64, 328, 328, 128), (24, 208, 3048, 1)):
        assert B.ac_linear_kernel(m, n, k, "bf16", batch=batch) == "ragged 64x64"


@pytest.mark.parametrize("m,n,k", [(128, 2048, 512), (128, 1536, 384), (96, 2048, 512), (128, 3072, 768), (256, 512, 2048), (512, 768, 3072)])
def test_launches_of_one_round_of_small_tiles_take_the_smallest(m, n, k):
    assert B.ac_linear_kernel(m, n, k, "bf16") == "staged 32x64"


def test_the_gated_product_takes_small_tiles_where_it_is_small(tmp_path):
    """The tile of the gated feed-forward's first product, by the kernels that one image's plan launches: of 64 rows and 2 * 5120 weight rows, 256-row
    tiles would leave three quarters of the work as padding."""
    import launch_stub
    launch_stub.run(launch_stub.build(str(tmp_path)), """
def gated_kernel(h, w, c, f):
    cfg = I.ResStackConfig("plan", 1, 1, 1, h, w, c, 32, heads=c // 64, d_ffn=f, gated=True)
    plan = B.Plan(B.res_stack_desc(cfg), [])
    info = plan.ac_plan_query()
    assert L.ac_plan_bind_weights(plan._h, (B.VP * info.n_weights)(*[(1 << 44) + 256 * i for i in range(info.n_weights)]), info.n_weights) == 0
    assert L.ac_execute(plan._h, X, Y, W, info.workspace_bytes, None, None) == 0, L.ac_last_error()
    (name,) = [k for k in kernels() if "linear_quad_bf16ILb1E" in k or ("linear_ring_bf16" in k and "ELb0ELb0ELb0ELb1E" in k)]
    return "256x256" if "quad" in name else "x".join(name[name.index("ILi") + 3:].split("ELi")[:2])

assert gated_kernel(8, 8, 1280, 5120) == "64x128"
assert gated_kernel(16, 16, 1280, 5120) == "64x128"
assert gated_kernel(16, 32, 1280, 5120) == "256x128"
assert gated_kernel(32, 32, 1280, 5120) == "256x256"
assert gated_kernel(32, 32, 320, 1280) == "64x128"
assert gated_kernel(64, 64, 320, 1280) == "256x256"
""")


def test_projections_of_few_rows_share_out_their_columns(tmp_path):
    """Beside the kernel that keeps weights in registers, a block per CU, the one of 64-column tiles: where rows are few its launch has more blocks."""
    import launch_stub
    launch_stub.run(launch_stub.build(str(tmp_path)), """
def part(i, n, rows, strided=False, gated=False):
    p = B.ac_proj_part()
    p.w, p.n = (1 << 43) + (i << 20), n
    if gated: p.w_gate, p.gated = (1 << 43) + (i << 20) + 65536, 1
    if strided: p.out_t, p.t_s2, p.t_s3 = Y + (i << 36), 1, rows
    else: p.out, p.ldo = Y + (i << 36), n
    return p

def slices(rows, k, kind):
    parts = {"four": lambda: [part(i, 128, rows, i == 3) for i in range(4)], "two": lambda: [part(i, 128, rows) for i in range(2)],
             "pairs": lambda: [part(i, 128, rows, True, True) for i in range(2)],
             "narrow": lambda: [part(2, 4, rows, True), part(0, 128, rows), part(1, 128, rows, True)]}[kind]()
    kernels()
    assert L.ac_op_ln_linear(X, k, W, W + 4096, 1e-5, rows, k, (B.ac_proj_part * len(parts))(*parts), len(parts), B.AC_BF16, None) == 0
    (name,) = kernels()
    assert "ln_proj_slices" in name or "ln_multi_proj" in name
    return "ln_proj_slices" in name

assert [slices(rows, 64, "two") for rows in (8, 8192, 8200, 13312, 13320, 1 << 20)] == [True, True, False, False, True, True]
for k, kind, line in ((64, "four", 8192), (128, "four", 8192), (128, "two", 0), (64, "pairs", 32768), (128, "pairs", 16384), (64, "narrow", 13312),
                      (128, "narrow", 4096)):
    assert [slices(rows, k, kind) for rows in (8, 1024, line, line + 8, 40000, 1 << 20) if rows > 0] == [rows > line for rows in (8, 1024, line, line + 8, 40000, 1 << 20) if rows > 0], (k, kind)
""")


def test_an_fp32_products_name_is_the_kernel_that_is_launched(tmp_path):
    """Every fp32 kernel, by the launch that the call makes."""
    import launch_stub
    launch_stub.run(launch_stub.build(str(tmp_path)), """
import re
SHARED = {"2, 4": "f32 32x64", "2, 2": "f32 32x32", "2, 1": "f32 32x16", "1, 1": "f32 16x16"}
RING = {"32, 64, 1, 4, 32": "f32-ring 32x64", "32, 32, 2, 2, 32": "f32-ring 32x32", "32, 32, 2, 2, 64": "f32-ring-deep 32x32"}
def launched(m, n, k, batch):
    kernels()
    if batch == 1: status = L.ac_op_linear(X, k, W, k, None, None, 0, None, 0, Y, n, None, n, 0, 0, 0, 0, m, n, k, 0, B.AC_F32, None)
    else: status = L.ac_op_triangle_contract(X, k, m * k, W, k, n * k, Y, n, m * n, m, n, k, batch, B.AC_F32, None)
    assert status == 0, L.ac_last_error()
    (name,) = kernels()
    numbers = ", ".join(re.findall(r"ELi(\\d+)|ILi(\\d+)", name) and [a or b for a, b in re.findall(r"ELi(\\d+)|ILi(\\d+)", name)])
    return "fma 64x64" if "linear_fma" in name else SHARED[numbers] if "linear_mfma_f32" in name else RING[numbers] if "linear_ring_f32" in name else name

seen = set()
rng = random.Random(3)
sizes = [(rng.choice([1, 33, 200, 260, 700, 1024, 2066, 5000]), 4 * rng.randint(1, 500), rng.choice([64, 100, 128, 256, 384, 500, 640, 1024, 2048]), rng.choice([1, 1, 1, 16, 128])) for _ in range(600)]
for m, n, k, batch in sizes + [(1000, 1024, 64, 1)]:
    name = B.ac_linear_kernel(m, n, k, "f32", batch=batch)
    assert name == launched(m, n, k, batch), (m, n, k, batch, name)
    seen.add(name)
assert len(seen) == 8, seen
""")
