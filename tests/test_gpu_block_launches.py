"""MX and blockwise steps quantize their tensors in one launch per direction: the bits of the single-tensor launches, at sizes where
tensors end inside a tile or a patch of tiles, for every mix of formats and every gradient wanted."""
import numpy as np
import pytest
import torch

from tests.gpu_util import knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


@pytest.mark.parametrize("M,K,N", [(32, 128, 32), (160, 256, 2112), (2080, 384, 96), (128, 2176, 128), (2176, 128, 2304), (384, 640, 512),
                                   (2048, 2048, 2048), (2048, 2048, 2176)])      # (the last two: on and beyond the 8 Mi elements of plain loads)
@pytest.mark.parametrize("kind", ["mx", "block"])
def test_one_launch_changes_no_bit(M, K, N, kind):
    if kind == "block" and (M % 128 or N % 128):
        M, N = (M + 127) // 128 * 128, (N + 127) // 128 * 128
    rng = np.random.default_rng(M + N)
    x, w, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    x[0, :] = 0
    w[:, 1] = 0
    fwd, bwd = (fp8.fp8_mx_linear_fwd, fp8.fp8_mx_linear_bwd) if kind == "mx" else (fp8.fp8_block_linear_fwd, fp8.fp8_block_linear_bwd)
    fws, bws = (fp8.fp8_mx_linear_workspace_bytes, fp8.fp8_mx_linear_bwd_workspace_bytes) if kind == "mx" else \
        (fp8.fp8_block_linear_workspace_bytes, fp8.fp8_block_linear_bwd_workspace_bytes)
    ff = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")      # noqa: E731

    def run():
        outs = []
        for fmt_w, fmt_dy in ((0, 0), (1, 1), (0, 1)):
            outs.append(fwd(x, w, fmt_w, fmt_w, workspace=ff(fws(M, K, N))))
            outs += [o for o in bwd(dy, x, w, fmt_dy, fmt_w, fmt_w, workspace=ff(bws(M, K, N)))]
        return [o.view(torch.int16).clone() for o in outs]

    got = run()
    with knobs(PAIRS=0):
        want = run()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("block_rows", [1, 128])
def test_blocks_with_infinities_and_nan_are_clamped(fmt, block_rows):
    """The cast without a clamp only where the block's maximum is finite: infinities become the largest normal value, NaN stays NaN, in
    either direction, and blocks beside them are as ever."""
    rng = np.random.default_rng(fmt)
    x = torch.from_numpy(rng.standard_normal((256, 384)).astype(np.float32)).to(torch.bfloat16)
    x[3, 5], x[130, 200], x[131, 380], x[255, 0], x[7, 300] = float("inf"), float("-inf"), float("nan"), 3e38, 0.0
    xd = x.cuda()
    t8, top = ((torch.float8_e4m3fn, 448.0), (torch.float8_e5m2, 57344.0))[fmt]

    def check(q, e, v):                          # q [r, c] codes, e [r, c / 32] scale bytes
        s = torch.exp2(127.0 - e.cpu().float()).repeat_interleave(32, 1)
        p = v.float() * s
        want = torch.where(p.isnan(), p, p.clamp(-top, top)).to(t8).view(torch.uint8)
        got = q.cpu()
        same = torch.where(p.isnan(), (got & 0x7F) > (0x7E, 0x7C)[fmt], got == want)      # any code of the NaN class
        assert bool(same.all())

    check(*fp8.fp8_block_quantize(xd, block_rows, fmt), x)
    check(*fp8.fp8_block_quantize_t(xd, block_rows, fmt), x.t().contiguous())
    if block_rows == 1:
        q, e, qt, et = fp8.fp8_block_quantize_row_col(xd, fmt)
        check(q, e, x)
        check(qt, et, x.t().contiguous())
