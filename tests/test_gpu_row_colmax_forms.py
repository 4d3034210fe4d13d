"""Codes along both axes from a pass that gathers column maxima: blocks of 512 threads for rows of 4097 to 16384 elements, fewer rows
in flight in tall tensors, with a sigmoid's output or without: the bits of the separate passes."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402
from tests.gpu_util import knobs  # noqa: E402

SIZES = [(300, 4104), (1000, 8192), (1030, 8200), (2050, 12296), (520, 16384), (264, 16392), (6143, 2048), (6144, 520), (6150, 2056), (8200, 4096)]


@pytest.mark.parametrize("rows,cols", SIZES)
@pytest.mark.parametrize("fmt", [fp8.FP8_E4M3FN, fp8.FP8_E5M2])
def test_both_axes(rows, cols, fmt):
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn((rows, cols), device="cuda", generator=gen) * torch.logspace(-3, 3, cols, device="cuda")
    x = x.to(torch.bfloat16)
    x[1] = 0
    x[2, cols - 1] = float("inf")
    x[3, 0] = float("nan")
    x[rows - 1, cols // 2] = -3.0e38
    xt = torch.zeros((cols, (rows + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")[:, :rows]
    xt.copy_(x.t())
    for flags in (0, fp8.FP8_POW2_SCALE):
        with knobs(STRIPS=0):
            q, s, qt, st = fp8.fp8_quantize_row_col(x, fmt, flags)
        want, scale = fp8.fp8_quantize(x, fp8.FP8_ROW, fmt, flags)
        want_t, scale_t = fp8.fp8_quantize(xt, fp8.FP8_ROW, fmt, flags)
        assert torch.equal(q, want) and torch.equal(s.view(torch.int32), scale.view(torch.int32)), flags
        assert torch.equal(qt, want_t) and torch.equal(st.view(torch.int32), scale_t.view(torch.int32)), flags


@pytest.mark.parametrize("M,N", [(1024, 4112), (1040, 8192), (1104, 12304), (1024, 16384), (6144, 2048), (6208, 4096)])
def test_sigmoid_gradient(M, N):
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    K = 128
    dy, x, w = (torch.randn(s, device="cuda", generator=gen).to(torch.bfloat16) for s in ((M, N), (M, K), (N, K)))
    y = torch.sigmoid(2 * torch.randn((M, N), device="cuda", generator=gen)).to(torch.bfloat16)
    dz = ((dy.float() * y.float()) * (1 - y.float())).to(torch.bfloat16)       # one rounding per operation, as in the kernel
    r = fp8.Recipe(gran=fp8.FP8_ROW)
    dx0, dw0 = fp8.fp8_linear_bwd(dz, x, w, r)
    dx1, dw1 = fp8.fp8_linear_bwd_sigmoid(dy, y, x, w, r)
    assert torch.equal(dx0, dx1) and torch.equal(dw0, dw1)
