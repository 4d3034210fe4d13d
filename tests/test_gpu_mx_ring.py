"""The ring kernel's block-scaled form: every tile, plain scale rows and slabs, bit for bit the 256 x 256 kernel's result
(the same order of sums), at the edges of tiles and of the ring of K steps."""
import numpy as np
import pytest
import torch

import synthetic_inputs as si
from oracle import fp8_oracle as orc
from tests.gpu_util import dev_bf16, host_bf16_bits, knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402

TILES = {"64x64": 1, "128x64": 2, "64x128": 3, "128x128": 4, "128x256": 5, "256x128": 6}


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,K", [(1, 8, 128), (64, 64, 512), (65, 72, 640), (257, 264, 1024), (130, 520, 384), (300, 1000, 2048)])
def test_every_tile_and_scale_layout(tile, M, N, K):
    x, w = si.normal_bf16((M, K), 1.0, 1, M), si.normal_bf16((N, K), 0.02, 2, N)
    xd, wd = dev_bf16(x), dev_bf16(w)
    for fa, fb in ((0, 0), (1, 0), (0, 1), (1, 1)):
        for slabs in (False, True) if K % 512 == 0 else (False,):
            qa, ea = fp8.fp8_mx_quantize(xd, fa, slabs=slabs)
            qb, eb = fp8.fp8_mx_quantize(wd, fb, slabs=slabs)
            for flags in (0, fp8.FP8_OUT_FP32):
                with knobs(MX_VARIANT=1):
                    want = fp8.fp8_mx_scaled_mm(qa, fa, ea, qb, fb, eb, flags)
                with knobs(GEMM_RING=TILES[tile]):
                    got = fp8.fp8_mx_scaled_mm(qa, fa, ea, qb, fb, eb, flags)
                assert torch.equal(got, want), (fa, fb, slabs, flags)
    with knobs(GEMM_RING=TILES[tile]):
        y = fp8.fp8_mx_linear_fwd(xd, wd)
    want = orc.mx_linear_fwd(x, w)
    assert orc.rel_frobenius(si.bf16_bits_to_f32(host_bf16_bits(y)), si.bf16_bits_to_f32(want.out16)) <= 1e-3


@pytest.mark.parametrize("M,K,N", [(96, 64, 160), (512, 1024, 512), (1024, 2048, 1536)])
def test_linear_steps_on_every_path(M, K, N):
    """MX and blockwise steps whose products the dispatch sends to the ring kernel, in slabs and plain rows, against the
    256 x 256 kernel."""
    rng = np.random.default_rng(M)
    x, w, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))

    def run():
        outs = list(fp8.fp8_mx_linear_bwd(dy, x, w))
        if K % 128 == 0:
            outs.append(fp8.fp8_mx_linear_fwd(x, w))
        if M % 128 == 0 and N % 128 == 0 and K % 128 == 0:
            outs += [fp8.fp8_block_linear_fwd(x, w)] + list(fp8.fp8_block_linear_bwd(dy, x, w))
        return [o.view(torch.int16).clone() for o in outs]

    with knobs(MX_VARIANT=1):
        want = run()
    for k in ({}, {"MX_SLAB": 0}, {"GEMM_RING": 1}, {"GEMM_RING": 5}):
        with knobs(**k):
            got = run()
        for a, b in zip(got, want):
            assert torch.equal(a, b), k


@pytest.mark.parametrize("M,K,N", [(256, 640, 384), (1408, 896, 1664), (384, 1152, 2432)])
@pytest.mark.parametrize("variant", [None, 1])
def test_partly_filled_slabs(M, K, N, variant):
    """Contractions that are no multiple of 512 (odd and even step counts): inside the linear calls the last slab of scales is
    partly filled; in a workspace full of NaN scale bytes, the bits of plain scale rows."""
    rng = np.random.default_rng(K)
    x, w, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    ff = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")      # noqa: E731

    def run():
        outs = [fp8.fp8_mx_linear_fwd(x, w, workspace=ff(fp8.fp8_mx_linear_workspace_bytes(M, K, N))),
                fp8.fp8_block_linear_fwd(x, w, workspace=ff(fp8.fp8_block_linear_workspace_bytes(M, K, N)))]
        outs += list(fp8.fp8_mx_linear_bwd(dy, x, w, workspace=ff(fp8.fp8_mx_linear_bwd_workspace_bytes(M, K, N))))
        outs += list(fp8.fp8_block_linear_bwd(dy, x, w, workspace=ff(fp8.fp8_block_linear_bwd_workspace_bytes(M, K, N))))
        return [o.view(torch.int16).clone() for o in outs]

    with knobs(MX_VARIANT=variant):
        got = run()
    with knobs(MX_SLAB=0, MX_VARIANT=1):
        want = run()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("tile", ["128x256", "256x128"])
@pytest.mark.parametrize("M,N,K", [(70, 72, 3072), (130, 264, 3200), (257, 520, 6144), (65, 264, 6272), (300, 392, 6656)])
def test_widest_tiles_on_either_side_of_their_short_contractions(tile, M, N, K):
    """Eight wavefronts up to K = 3072 with plain scale rows and 6144 with slabs, four beyond: bit for bit the 256 x 256 kernel's result."""
    x, w = dev_bf16(si.normal_bf16((M, K), 1.0, 1, M)), dev_bf16(si.normal_bf16((N, K), 0.02, 2, N))
    for fa, fb in ((0, 0), (1, 0), (0, 1), (1, 1)):
        for slabs in (False, True) if K % 512 == 0 else (False,):
            args = (fp8.fp8_mx_quantize(x, fa, slabs=slabs), fp8.fp8_mx_quantize(w, fb, slabs=slabs))
            for flags in (0, fp8.FP8_OUT_FP32):
                run = lambda: fp8.fp8_mx_scaled_mm(args[0][0], fa, args[0][1], args[1][0], fb, args[1][1], flags)      # noqa: E731
                with knobs(MX_VARIANT=1):
                    want = run()
                with knobs(GEMM_RING=TILES[tile]):
                    assert torch.equal(run(), want), (fa, fb, slabs, flags)
