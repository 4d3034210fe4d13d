"""Both sides of the lines beyond which the quantizers read their input with the streaming hint (2 Mi elements alone, 24 Mi for a pair): the
codes and scales of plain arithmetic on the same tensors."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402

E4 = fp8.FP8_E4M3FN


def _expected(x, dim):
    f = x.float()
    amax = f.abs().amax() if dim is None else f.abs().amax(dim, keepdim=True)
    s = (448.0 / amax.double().clamp(min=1e-12)).float()
    return (f * s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8), s


def _tensor(rows, cols):
    gen = torch.Generator(device="cuda").manual_seed(rows)
    return torch.randn((rows, cols), device="cuda", generator=gen).to(torch.bfloat16)


@pytest.mark.parametrize("rows", [512, 513, 2048, 2049])
def test_rows_and_tensor_scaled_products_at_the_line(rows):
    x = _tensor(rows, 4096)
    wq, sw = fp8.fp8_quantize(_tensor(64, 4096), fp8.FP8_ROW, E4)
    for gran, dim in ((fp8.FP8_ROW, 1), (fp8.FP8_TENSOR, None)):
        want, s = _expected(x, dim)
        if gran == fp8.FP8_ROW:
            q, sq = fp8.fp8_quantize(x, gran, E4)
            assert torch.equal(q, want) and torch.equal(sq.view(-1), s.view(-1))
        y = fp8.fp8_linear_fwd_prequantized(x, wq, E4, sw, fp8.FP8_ROW, E4, gran)
        ref = fp8.fp8_scaled_mm(want, E4, s.reshape(-1).contiguous(), gran, wq, E4, sw, fp8.FP8_ROW)
        assert torch.equal(y.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("M,N", [(2048, 4096), (2064, 4096)])
@pytest.mark.parametrize("gran,dim", [(fp8.FP8_ROW, 1), (fp8.FP8_TENSOR, None)])
def test_pairs_at_the_line(M, N, gran, dim):
    x, w = _tensor(M, 4096), _tensor(N, 4096)
    y = fp8.fp8_linear_fwd(x, w, fp8.Recipe(gran=gran))
    (xq, sx), (wq, sw) = _expected(x, dim), _expected(w, dim)
    ref = fp8.fp8_scaled_mm(xq, E4, sx.reshape(-1).contiguous(), gran, wq, E4, sw.reshape(-1).contiguous(), gran)
    assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
