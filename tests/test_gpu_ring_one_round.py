"""Tiles that only products of one round take (between the sizes that the others come in), and the lower 256-column tiles of the persistent
kernel in one round: exact integer products at the edges of tiles and of the ring of K steps, the 256 x 256 kernel's bits elsewhere."""
import numpy as np
import pytest
import torch

import synthetic_inputs as si
from oracle import fp8_oracle as orc
from tests.gpu_util import dev_bf16, dev_f32, dev_u8, host_bf16_bits, host_f32, knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402

TILES = {(96, 64): 7, (64, 192): 8, (160, 64): 9, (96, 128): 10, (160, 128): 11, (192, 128): 12, (128, 192): 13, (160, 192): 14, (192, 192): 15,
         (160, 256): 16, (224, 192): 17}


def _ints(shape, rng):
    return rng.integers(-2, 3, size=shape).astype(np.float32)


@pytest.mark.parametrize("tile", TILES, ids=str)
@pytest.mark.parametrize("extra_m,extra_n,K", [(0, 0, 128), (1, 8, 16), (-1, -8, 400), (33, 40, 528), (0, 72, 1040), (130, 200, 640), (0, 0, 4240)])
def test_exact_on_small_integers(tile, extra_m, extra_n, K):
    """Around one tile, and one more row or column of tiles; all formats, scales and outputs, inside a padded output."""
    M, N = tile[0] + extra_m, tile[1] + extra_n
    rng = np.random.default_rng(M * 7 + N + K)
    ai, bi = _ints((M, K), rng), _ints((N, K), rng)
    sa, sb = (2.0 ** rng.integers(-3, 4, size=M)).astype(np.float32), (2.0 ** rng.integers(-3, 4, size=N)).astype(np.float32)
    want = (ai @ bi.T).astype(np.float32) / sa[:, None] / sb[None, :]
    with knobs(GEMM_RING=TILES[tile]):
        for fa, fb in ((0, 0), (1, 0), (0, 1), (1, 1)):
            a, b = dev_u8(orc.encode_array(ai, fa), (K + 31) // 16 * 16), dev_u8(orc.encode_array(bi, fb))
            args = (a, fa, dev_f32(sa), fp8.FP8_ROW, b, fb, dev_f32(sb), fp8.FP8_ROW)
            assert (host_f32(fp8.fp8_scaled_mm(*args, fp8.FP8_OUT_FP32)) == want).all(), (fa, fb)
            out = torch.full((M + 2, (N + 15) // 8 * 8), -7.0, dtype=torch.bfloat16, device="cuda")
            fp8.fp8_scaled_mm(*args, 0, out=out[1:M + 1, :N])
            got = host_bf16_bits(out)
            assert (got[1:M + 1, :N] == orc.f32_to_bf16(want)).all(), (fa, fb)
            assert bool((out[0] == -7.0).all() and (out[M + 1] == -7.0).all() and (out[:, N:] == -7.0).all())
        one = (a, 1, dev_f32(sa[:1]), fp8.FP8_TENSOR, b, 1, dev_f32(sb[:1]), fp8.FP8_TENSOR)
        assert (host_f32(fp8.fp8_scaled_mm(*one, fp8.FP8_OUT_FP32)) == (ai @ bi.T) / sa[0] / sb[0]).all()
        sig = host_bf16_bits(fp8.fp8_scaled_mm(*args, fp8.FP8_EPILOGUE_SIGMOID))
    with knobs(GEMM_VARIANT=4):
        assert (sig == host_bf16_bits(fp8.fp8_scaled_mm(*args, fp8.FP8_EPILOGUE_SIGMOID))).all()


@pytest.mark.parametrize("tile", TILES, ids=str)
def test_every_count_of_steps_around_the_depth_of_the_ring(tile):
    one = dev_f32(np.ones(1, np.float32))
    for steps in range(10):
        rng = np.random.default_rng(steps)
        M, N, K = tile[0] + 3, tile[1] - 8, max(0, 128 * steps - 16)
        ai, bi = _ints((M, K), rng), _ints((N, K), rng)
        a, b = (dev_u8(orc.encode_array(v, 0)) if K else torch.empty((len(v), 0), dtype=torch.uint8, device="cuda") for v in (ai, bi))
        with knobs(GEMM_RING=TILES[tile]):
            got = host_f32(fp8.fp8_scaled_mm(a, 0, one, 0, b, 0, one, 0, fp8.FP8_OUT_FP32))
        assert (got == ai @ bi.T).all(), steps


@pytest.mark.parametrize("tile", [t for t, i in TILES.items() if i <= 15], ids=str)
@pytest.mark.parametrize("extra_m,extra_n,K", [(0, 0, 128), (1, 8, 512), (-31, 72, 640), (65, 200, 1536), (0, 0, 1664)])
def test_block_scaled_as_the_large_product_kernel(tile, extra_m, extra_n, K):
    M, N = tile[0] + extra_m, tile[1] + extra_n
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


@pytest.mark.parametrize("M,N,K", [(3001, 4096, 400), (3072, 4088, 528), (3300, 4096, 1040), (2305, 3600, 272), (1400, 4096, 256), (3072, 3072, 256), (702, 11264, 384),
                                   (2500, 2048, 640), (8200, 1000, 384), (1500, 2048, 272)])
def test_one_round_as_the_tile_per_workgroup_kernel(M, N, K):
    """Whatever form the choice takes: the same order of sums, hence the same bits."""
    x, w = (torch.randn(s, device="cuda", generator=torch.Generator(device="cuda").manual_seed(K)).to(torch.bfloat16) for s in ((M, K), (N, K)))
    a, b = fp8.fp8_quantize(x, fp8.FP8_ROW, 0, 0), fp8.fp8_quantize(w, fp8.FP8_ROW, 0, 0)
    for flags in (0, fp8.FP8_OUT_FP32, fp8.FP8_EPILOGUE_SIGMOID):
        run = lambda: fp8.fp8_scaled_mm(a[0], 0, a[1], fp8.FP8_ROW, b[0], 0, b[1], fp8.FP8_ROW, flags)      # noqa: E731
        with knobs(GEMM_VARIANT=4, GEMM_STREAM=0, GEMM_RING=0):
            want = run()
        assert torch.equal(run(), want), flags
