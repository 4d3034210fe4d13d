"""Routes of the quantizations inside the linear entry points that depend on sizes: per-column scales of tensors with few
rows, token counts off the 16-byte grid, and the per-tensor activations of a quantized weight's forward."""
import numpy as np
import pytest
import torch

import synthetic_inputs as si
from oracle import fp8_oracle as orc
from tests.gpu_util import dev_bf16, knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


@pytest.mark.parametrize("rows", [240, 256, 272, 1008, 4080, 4096, 4112])
@pytest.mark.parametrize("cols", [24, 512, 1032])
def test_column_scales_at_every_count_of_first_level_blocks(rows, cols):
    """64 blocks from 256 rows on, 1024 from 4096 on; below that the general path."""
    x = si.normal_bf16((rows, cols), 1.0, 3, rows + cols)
    x[rows - 1, cols - 1] = x[0, 0] = si.f32_to_bf16_bits(np.array([37.0], np.float32))[0]
    for fmt, flags in ((orc.E4M3FN, 0), (orc.E5M2, fp8.FP8_POW2_SCALE)):
        want_q, want_s = orc.quantize(x, orc.COL, fmt, bool(flags))
        q, s = fp8.fp8_quantize(dev_bf16(x), fp8.FP8_COL, fmt, flags | fp8.FP8_TRANSPOSE_OUT)
        assert (s.cpu().numpy() == want_s).all()
        assert (q.cpu().numpy() == want_q.T).all()


@pytest.mark.parametrize("M,K,N", [(257, 528, 512), (1001, 1024, 1040), (2057, 2048, 528), (4111, 1040, 4112)])
@pytest.mark.parametrize("recipe", ["tensorwise", "rowwise", "rowwise_gw_hp"])
def test_ragged_token_counts_share_launches_and_change_no_bit(M, K, N, recipe):
    """The shared launches keep the first-level maxima in the padded transposed outputs and fill the padding themselves: the
    same bits as the single-tensor calls, in a workspace full of NaN codes."""
    rng = np.random.default_rng(M)
    x, w, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    gran = fp8.FP8_TENSOR if recipe == "tensorwise" else fp8.FP8_ROW
    hp = fp8.FP8_GRAD_WEIGHT_HP if recipe.endswith("hp") else 0

    def run():
        outs = []
        for save in (0, fp8.FP8_SAVE_FOR_BWD):
            r = fp8.Recipe(gran=gran, flags=hp | save)
            ws = torch.full((fp8.fp8_linear_workspace_bytes(M, K, N, r, True),), 0x7F, dtype=torch.uint8, device="cuda")
            wf = ws if save else torch.empty(fp8.fp8_linear_workspace_bytes(M, K, N, r, False), dtype=torch.uint8, device="cuda")
            outs.append(fp8.fp8_linear_fwd(x, w, r, workspace=wf))
            outs += list(fp8.fp8_linear_bwd(dy, x, w, r, workspace=ws))
        return [o.view(torch.int16).clone() for o in outs]

    shared = run()
    with knobs(PAIRS=0):
        single = run()
    for a, b in zip(shared, single):
        assert torch.equal(a, b)


@pytest.mark.parametrize("M,K,N", [(2, 16, 8), (33, 28672, 64), (64, 16400, 72), (65, 528, 1000), (513, 8208, 256)])
@pytest.mark.parametrize("flags", [0, fp8.FP8_POW2_SCALE])
def test_per_tensor_activations_of_a_quantized_weight(M, K, N, flags):
    """Per-block maxima in what room the workspace has behind the scale (64 to 512 of them): the codes, and so the product,
    of the separate calls; nothing outside the workspace is touched."""
    x = dev_bf16(si.normal_bf16((M, K), 1.0, 5, M))
    x[M - 1, K - 1] = 50.0
    wq, sw = fp8.fp8_quantize(dev_bf16(si.normal_bf16((N, K), 0.02, 5, N)), fp8.FP8_ROW, fp8.FP8_E4M3FN)
    need = fp8.fp8_linear_prequantized_workspace_bytes(M, K)
    guard = torch.full((need + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    y = fp8.fp8_linear_fwd_prequantized(x, wq, fp8.FP8_E4M3FN, sw, fp8.FP8_ROW, fp8.FP8_E4M3FN, fp8.FP8_TENSOR, flags, workspace=guard[:need])
    xq, sx = fp8.fp8_quantize(x, fp8.FP8_TENSOR, fp8.FP8_E4M3FN, flags)
    want = fp8.fp8_scaled_mm(xq, fp8.FP8_E4M3FN, sx, fp8.FP8_TENSOR, wq, fp8.FP8_E4M3FN, sw, fp8.FP8_ROW)
    assert torch.equal(y.view(torch.int16), want.view(torch.int16))
    assert bool((guard[need:] == 0xA5).all())
    if need <= 8 << 20:        # what the static scratch holds
        ys = torch.empty_like(y)
        fp8.fp8_linear_fwd_prequantized_static(x, wq, fp8.FP8_E4M3FN, sw, fp8.FP8_ROW, ys, fp8.FP8_E4M3FN, fp8.FP8_TENSOR, flags)
        assert torch.equal(ys.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("M,K,N", [(1001, 1040, 1200), (600, 2000, 528), (513, 528, 1008)])
@pytest.mark.parametrize("recipe", ["tensorwise", "rowwise"])
@pytest.mark.parametrize("save", [0, fp8.FP8_SAVE_FOR_BWD])
def test_padded_operand_rows_give_the_products_of_dense_ones(M, K, N, recipe, save):
    """Operands in the workspace whose contracted length is no multiple of 128 have padded rows; the products are those of
    the public quantizers' dense operands, bit for bit, and what lies in the padding (NaN codes here) does not matter."""
    rng = np.random.default_rng(K)
    x, w, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    row, col = (fp8.FP8_TENSOR,) * 2 if recipe == "tensorwise" else (fp8.FP8_ROW, fp8.FP8_COL)
    g = fp8.FP8_TENSOR if recipe == "tensorwise" else fp8.FP8_ROW
    r = fp8.Recipe(gran=g, flags=save)
    full = lambda n: torch.full((n,), 0x7F, dtype=torch.uint8, device="cuda")      # noqa: E731
    wb = full(fp8.fp8_linear_workspace_bytes(M, K, N, r, True))
    y = fp8.fp8_linear_fwd(x, w, r, workspace=wb if save else full(fp8.fp8_linear_workspace_bytes(M, K, N, r, False)))
    dx, dw = fp8.fp8_linear_bwd(dy, x, w, r, workspace=wb)
    T, E4, E5 = fp8.FP8_TRANSPOSE_OUT, fp8.FP8_E4M3FN, fp8.FP8_E5M2

    def product(a, ga, fa, ta, b, gb, fb, tb):
        (qa, sa), (qb, sb) = fp8.fp8_quantize(a, ga, fa, ta), fp8.fp8_quantize(b, gb, fb, tb)
        k16 = (qa.shape[1] + 15) // 16 * 16
        if k16 != qa.shape[1]:      # the product contracts over multiples of 16: zero codes
            pa, pb = (torch.zeros((q.shape[0], k16), dtype=torch.uint8, device="cuda") for q in (qa, qb))
            pa[:, :qa.shape[1]], pb[:, :qb.shape[1]] = qa, qb
            qa, qb = pa, pb
        return fp8.fp8_scaled_mm(qa, fa, sa, g, qb, fb, sb, g)

    assert torch.equal(y, product(x, row, E4, 0, w, row, E4, 0))
    assert torch.equal(dx, product(dy, row, E5, 0, w, col, E4, T))
    assert torch.equal(dw, product(dy, col, E5, T, x, col, E4, T))


@pytest.mark.parametrize("rows,cols", [(1, 8), (128, 4096), (129, 4096), (64, 8200), (1023, 512), (17, 32768), (3, 130), (4097, 128)])
def test_rowwise_codes_on_both_sides_of_the_store_rule(rows, cols):
    """Up to 512 Ki elements another form of the rowwise kernel stores the codes; rows with a tail, padded input and output."""
    x = si.normal_bf16((rows, cols), 1.0, 3, rows + cols)
    ld = (cols + 7) // 8 * 8 + 8
    xd = dev_bf16(x, ld)
    for fmt, flags in ((orc.E4M3FN, 0), (orc.E5M2, fp8.FP8_POW2_SCALE)):
        want_q, want_s = orc.quantize(x, orc.ROW, fmt, bool(flags))
        out = torch.full((rows, (cols + 15) // 16 * 16 + 16), 0x5A, dtype=torch.uint8, device="cuda")
        q, s = fp8.fp8_quantize(xd, fp8.FP8_ROW, fmt, flags, out=out[:, :cols])
        assert (s.cpu().numpy() == want_s).all() and (q.cpu().numpy() == want_q).all()
        assert bool((out[:, cols:] == 0x5A).all())
