"""Block-scaled products on the persistent kernel: bit for bit the tile-per-workgroup kernel's result (the same order of sums), with one and
several tiles per workgroup, every tile height, odd and even counts of K steps, contractions that end inside a group of four steps."""
import pytest
import torch

import synthetic_inputs as si
from tests.gpu_util import dev_bf16, knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


@pytest.mark.parametrize("height", [256, 224, 192])
@pytest.mark.parametrize("M,N,K", [(256, 256, 1024), (192, 264, 1536), (700, 520, 1024), (1345, 1032, 2048), (449, 3000, 2560), (1, 8, 4096)])
def test_as_the_tile_per_workgroup_kernel(height, M, N, K):
    x, w = dev_bf16(si.normal_bf16((M, K), 1.0, 1, M)), dev_bf16(si.normal_bf16((N, K), 0.02, 2, N))
    for fa, fb in ((0, 0), (1, 0), (0, 1), (1, 1)):
        (qa, ea), (qb, eb) = fp8.fp8_mx_quantize(x, fa, slabs=True), fp8.fp8_mx_quantize(w, fb, slabs=True)
        with knobs(MX_VARIANT=1):
            want = fp8.fp8_mx_scaled_mm(qa, fa, ea, qb, fb, eb)
        for grid in (8, 16, 256):
            out = torch.full((M + 2, (N + 15) // 8 * 8), -7.0, dtype=torch.bfloat16, device="cuda")
            with knobs(GEMM_STREAM=grid, GEMM_RING=0, GEMM_TILE_M=height):
                fp8.fp8_mx_scaled_mm(qa, fa, ea, qb, fb, eb, out=out[1:M + 1, :N])
            assert torch.equal(out[1:M + 1, :N], want), (fa, fb, grid)
            assert bool((out[0] == -7.0).all() and (out[M + 1] == -7.0).all() and (out[:, N:] == -7.0).all())


@pytest.mark.parametrize("height", [256, 224, 192])
@pytest.mark.parametrize("M,K,N", [(640, 640, 768), (512, 768, 896), (896, 1152, 1664), (1280, 1408, 640)])
def test_partly_filled_groups(height, M, K, N):
    """Contractions of 5 to 13 steps (one step of zeros where odd; two, four or no steps in the last group), scale bytes past their end NaN."""
    gen = torch.Generator(device="cuda").manual_seed(K)
    x, w, dy = (torch.randn(s, device="cuda", generator=gen).to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    ff = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")      # noqa: E731

    def run():
        outs = [fp8.fp8_mx_linear_fwd(x, w, workspace=ff(fp8.fp8_mx_linear_workspace_bytes(M, K, N))),
                fp8.fp8_block_linear_fwd(x, w, workspace=ff(fp8.fp8_block_linear_workspace_bytes(M, K, N)))]
        outs += list(fp8.fp8_mx_linear_bwd(dy, x, w, workspace=ff(fp8.fp8_mx_linear_bwd_workspace_bytes(M, K, N))))
        outs += list(fp8.fp8_block_linear_bwd(dy, x, w, workspace=ff(fp8.fp8_block_linear_bwd_workspace_bytes(M, K, N))))
        return [o.view(torch.int16).clone() for o in outs]

    with knobs(MX_SLAB=0, MX_VARIANT=1):
        want = run()
    for grid in (8, 256):
        with knobs(GEMM_STREAM=grid, GEMM_RING=0, GEMM_TILE_M=height):
            got = run()
        for a, b in zip(got, want):
            assert torch.equal(a, b), grid
