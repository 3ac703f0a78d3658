"""Which loop of the attention kernel a call takes, on the host."""
import pytest

import launch_stub

CALL = """
def loop(sq, sk, dh, ldk, ldv, causal):
    r = L.ac_op_attention(X, dh, 0, Y, ldk, 0, W, ldv, 0, 1, None, 0, 0, None, 0, 0, 1 << 43, dh, 0, 1, sq, sk, 1, dh, causal, 0, 1, None, 0,
                          B.AC_BF16, None)
    assert r == 0, L.ac_last_error()
    (name,) = kernels()
    return name[name.index("KeysE") + 5]        # 0 whole tiles, 1 whole chunks (pipelined, a buffer of 2^31 bytes), 2 any keys
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return launch_stub.build(str(tmp_path_factory.mktemp("stub")))


@pytest.mark.parametrize("dh,ldv,route", [
    (128, 4096, 1), (128, 8454656, 1), (128, 8454664, 2), (128, 9000000, 2), (128, (1 << 24) - 8, 2), (64, (1 << 24) - 8, 1)])
@pytest.mark.parametrize("causal", [0, 1])
def test_a_ragged_last_tile_keeps_all_rows_of_the_values_in_the_buffers_range(lib, dh, ldv, route, causal):
    """The loop whose last tile gets its zeros from the buffer's range check would get them for far rows of V^T too."""
    assert (dh - 1) * ldv * 2 + 128 < 1 << 31 or route == 2
    launch_stub.run(lib, CALL + f"""
assert loop(200, 1000, {dh}, {dh}, {ldv}, {causal}) == "{route}"
assert loop(200, 1000, {dh}, (1 << 24) - 8, {ldv}, {causal}) == "{route}"
assert loop(200, 1024, {dh}, {dh}, {ldv}, {causal}) == "0"
""")


@pytest.mark.parametrize("dh,sk,causal", [(64, 1024, 1), (64, 1000, 0), (64, 1000, 1), (128, 1024, 0), (128, 1000, 1)])
def test_rows_in_descending_order_take_addresses_of_64_bits(lib, dh, sk, causal):
    launch_stub.run(lib, CALL + f"""
assert loop(200, {sk}, {dh}, -{dh}, 4096, {causal}) == "2" and loop(200, {sk}, {dh}, {dh}, -4096, {causal}) == "2"
""")
