"""Rowwise quantization of a decode batch (up to 512 Ki elements, a wider block per row): the bits that the same rows get in a larger tensor."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


@pytest.mark.parametrize("cols", [513, 520, 1000, 2047, 2048, 2056, 4095, 4096, 4104, 8192, 8200, 12000, 16384, 16392, 32765, 32768])
@pytest.mark.parametrize("rows", [1, 5, 16])
def test_as_in_a_larger_tensor(rows, cols):
    gen = torch.Generator(device="cuda").manual_seed(rows * cols)
    ld = (cols + 15) // 8 * 8
    more = (1 << 19) // cols + 2
    x = (torch.randn((rows + more, ld), device="cuda", generator=gen) * torch.logspace(-4, 4, rows + more, device="cuda")[:, None]).to(torch.bfloat16)[:, :cols]
    if rows >= 5:
        x[1] = 0
        x[2, cols - 1] = float("inf")
        x[3, 0] = float("nan")
        x[4, cols // 2] = -3.0e38
    for fmt in (fp8.FP8_E4M3FN, fp8.FP8_E5M2):
        for flags in (0, fp8.FP8_POW2_SCALE):
            want, scale = fp8.fp8_quantize(x, fp8.FP8_ROW, fmt, flags)
            out = torch.full((rows + 1, want.stride(0)), 0x55, dtype=torch.uint8, device="cuda")
            s = torch.full((rows + 1,), -1.0, device="cuda")
            fp8.fp8_quantize(x[:rows], fp8.FP8_ROW, fmt, flags, out=out[:rows, :cols], scale_out=s[:rows])
            assert torch.equal(out[:rows, :cols], want[:rows]) and torch.equal(s[:rows], scale[:rows]), (fmt, flags)
            assert bool((out[rows] == 0x55).all() and (out[:, cols:] == 0x55).all()) and s[rows] == -1.0
