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
