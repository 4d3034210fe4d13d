"""Host-only checks of the workspace sizes."""
import ctypes as C

import pytest

import paper_2507_16099_amd as fp8


@pytest.mark.parametrize("limit", [1 << 22, 1 << 23])
@pytest.mark.parametrize("axis", ["M", "K", "N"])
def test_row_padding_does_not_reach_the_limits_of_the_products(limit, axis):
    """Rows of fp8 operands are padded to 128 bytes, but not up to 2^22 or 2^23 bytes, from where on the products' 32-bit
    offsets do not reach: the last length below (a multiple of 16) keeps its own rows, as do the lengths from the limit on."""
    r = fp8.Recipe(gran=fp8.FP8_TENSOR)
    size = lambda v: fp8.fp8_linear_workspace_bytes(**{**dict(M=16, K=16, N=16), axis: v}, recipe=r, bwd=axis != "K")      # noqa: E731
    others = 0 if axis == "K" else 16 * 16   # an operand that has the axis as its rows
    assert size(limit) - size(limit - 16) == others + 2 * 16 * 16            # two operands of 16 rows contract over the axis
    assert size(limit - 128) - size(limit - 144) == others                   # padded
    assert size(limit + 128) - size(limit + 112) == others


@pytest.mark.parametrize("M,K,N", [(1008, 640, 528), (256, 512, 128), (384, 1152, 2432)])
def test_one_byte_less_than_asked_for_is_refused(M, K, N):
    """On the host, before anything is launched."""
    L = fp8.load_library()
    buf = (C.c_char * 8192)()
    p = (C.addressof(buf) + 255) // 256 * 256
    refused = lambda rc: rc == -5 and "workspace" in fp8.fp8_last_error()      # noqa: E731
    for gran in (fp8.FP8_TENSOR, fp8.FP8_ROW):
        for flags in (0, fp8.FP8_SAVE_FOR_BWD, fp8.FP8_GRAD_WEIGHT_HP):
            r = fp8.Recipe(gran=gran, flags=flags)
            fwd, bwd = (fp8.fp8_linear_workspace_bytes(M, K, N, r, b) - 1 for b in (False, True))
            sig = fp8.fp8_linear_bwd_sigmoid_workspace_bytes(M, K, N, r) - 1
            assert refused(L.fp8_linear_fwd(p, p, M, K, N, C.byref(r.c()), p, p, fwd, None))
            assert refused(L.fp8_linear_bwd(p, p, p, M, K, N, C.byref(r.c()), p, p, p, bwd, None))
            assert refused(L.fp8_linear_bwd_sigmoid(p, p, p, p, M, K, N, C.byref(r.c()), p, p, p, sig, None))
    if K % 128 == 0:
        assert refused(L.fp8_mx_linear_fwd(p, p, M, K, N, 0, 0, p, p, fp8.fp8_mx_linear_workspace_bytes(M, K, N) - 1, None))
        assert refused(L.fp8_block_linear_fwd(p, p, M, K, N, 0, 0, p, p, fp8.fp8_block_linear_workspace_bytes(M, K, N) - 1, None))
    if M % 128 == 0 and N % 128 == 0:
        assert refused(L.fp8_mx_linear_bwd(p, p, p, M, K, N, 1, 0, 0, p, p, p, fp8.fp8_mx_linear_bwd_workspace_bytes(M, K, N) - 1, None))
        assert refused(L.fp8_block_linear_bwd(p, p, p, M, K, N, 1, 0, 0, p, p, p, fp8.fp8_block_linear_bwd_workspace_bytes(M, K, N) - 1, None))
    assert refused(L.fp8_linear_fwd_prequantized(p, M, K, 0, 1, 0, p, K, 0, p, 1, N, p, N, p, fp8.fp8_linear_prequantized_workspace_bytes(M, K) - 1, None))
