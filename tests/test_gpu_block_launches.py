"""MX and blockwise steps quantize their tensors in one launch per direction: the bits of the single-tensor launches, at sizes where
tensors end inside a tile or a patch of tiles, for every mix of formats and every gradient wanted."""
import numpy as np
import pytest
import torch

from tests.gpu_util import knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


@pytest.mark.parametrize("M,K,N", [(32, 128, 32), (160, 256, 2112), (2080, 384, 96), (128, 2176, 128), (2176, 128, 2304), (384, 640, 512)])
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
