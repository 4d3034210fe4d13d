"""Two-pass quantizations around 64 Mi elements, where the stores of the codes change: ragged rows and columns above the
line, both sides of it, public outputs with padded rows and the workspaces of the linear calls.  Bit for bit against the
untransposed codes, and against the single-tensor calls."""
import pytest
import torch

from tests.gpu_util import knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


def _tensor(rows, cols):
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    return torch.randn((rows, cols), device="cuda", generator=g).to(torch.bfloat16)


@pytest.mark.parametrize("rows,cols", [(8192, 8192), (8192, 8200), (8201, 8208), (16400, 4104)])
@pytest.mark.parametrize("gran", [fp8.FP8_TENSOR, fp8.FP8_COL])
def test_transposed_codes_equal_the_untransposed_ones(rows, cols, gran):
    x = _tensor(rows, cols)
    want, want_s = fp8.fp8_quantize(x, gran, fp8.FP8_E4M3FN)
    ld = (rows + 15) // 16 * 16 + 16
    out = torch.full((cols, ld), 0x5A, dtype=torch.uint8, device="cuda")
    q, s = fp8.fp8_quantize(x, gran, fp8.FP8_E4M3FN, fp8.FP8_TRANSPOSE_OUT, out=out[:, :rows])
    assert torch.equal(s, want_s) and torch.equal(q, want.t())
    assert bool((out[:, rows:] == 0x5A).all())                    # the bytes between the rows are the caller's


@pytest.mark.parametrize("rows,cols", [(8192, 8192), (8201, 8208)])
def test_both_orientations_equal_the_single_ones(rows, cols):
    x = _tensor(rows, cols)
    q_row, s_row, q_col_t, s_col = fp8.fp8_quantize_row_col(x, fp8.FP8_E5M2)
    want_row, want_sr = fp8.fp8_quantize(x, fp8.FP8_ROW, fp8.FP8_E5M2)
    want_col, want_sc = fp8.fp8_quantize(x, fp8.FP8_COL, fp8.FP8_E5M2)
    assert torch.equal(s_row, want_sr) and torch.equal(s_col, want_sc)
    assert torch.equal(q_row, want_row) and torch.equal(q_col_t, want_col.t())


@pytest.mark.parametrize("recipe", ["tensorwise", "rowwise"])
def test_ragged_step_in_a_workspace_of_nan_codes(recipe):
    M, K, N = 8201, 8208, 64
    x, w, dy = _tensor(M, K), _tensor(N, K), _tensor(M, N)
    r = fp8.Recipe(gran=fp8.FP8_TENSOR if recipe == "tensorwise" else fp8.FP8_ROW, flags=fp8.FP8_SAVE_FOR_BWD)

    def run():
        ws = torch.full((fp8.fp8_linear_workspace_bytes(M, K, N, r, True),), 0x7F, dtype=torch.uint8, device="cuda")
        outs = [fp8.fp8_linear_fwd(x, w, r, workspace=ws)]
        outs += list(fp8.fp8_linear_bwd(dy, x, w, r, workspace=ws))
        return [o.view(torch.int16).clone() for o in outs]

    shared = run()
    with knobs(PAIRS=0):
        single = run()
    assert all(torch.equal(a, b) for a, b in zip(shared, single))


@pytest.mark.parametrize("rows,cols", [(12288, 16384), (12416, 16384)])
@pytest.mark.parametrize("scheme", ["mx", "block"])
def test_block_codes_of_both_orientations_equal_the_single_ones(rows, cols, scheme):
    """192 Mi elements, and a tile row more: the other kind of store."""
    x = _tensor(rows, cols)
    both = getattr(fp8, f"fp8_{scheme}_quantize_row_col")(x, fp8.FP8_E4M3FN)
    args = () if scheme == "mx" else (1,)
    row = getattr(fp8, f"fp8_{scheme}_quantize")(x, *args, fp8.FP8_E4M3FN)
    col = getattr(fp8, f"fp8_{scheme}_quantize_t")(x, *args, fp8.FP8_E4M3FN)
    for a, b in zip(both, (*row, *col)):
        assert torch.equal(a, b)
