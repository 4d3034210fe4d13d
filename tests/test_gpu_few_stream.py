"""Persistent few-row products: exact integer products for every count of K steps per wavefront, partly filled steps, tiles and lists of
tiles, both orders of tiles, all formats, scales and outputs; and the choice on either side of its line."""
import numpy as np
import pytest
import torch

from oracle import fp8_oracle as orc
from tests.gpu_util import dev_f32, dev_u8, host_bf16_bits, host_f32, knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


def _ints(shape, rng):
    return rng.integers(-2, 3, size=shape).astype(np.float32)


@pytest.mark.parametrize("order", [2, 3])
@pytest.mark.parametrize("M,N,K", [(1, 8, 16), (5, 16, 128), (16, 24, 1024), (3, 264, 1040), (16, 4096, 528), (9, 4104, 1168), (16, 8200, 400), (2, 12400, 144),
                                   (16, 40, 4096), (7, 72, 4112), (16, 56, 8192), (4, 300, 8208), (16, 24, 12304), (11, 40, 16384)])
def test_exact_on_small_integers(order, M, N, K):
    rng = np.random.default_rng(M + N + K)
    ai, bi = _ints((M, K), rng), _ints((N, K), rng)
    sa, sb = (2.0 ** rng.integers(-3, 4, size=M)).astype(np.float32), (2.0 ** rng.integers(-3, 4, size=N)).astype(np.float32)
    want = (ai @ bi.T).astype(np.float32) / sa[:, None] / sb[None, :]
    with knobs(GEMM_VARIANT=5, SKINNY_DMA=order):
        for fa, fb in ((0, 0), (1, 0), (0, 1), (1, 1)):
            a, b = dev_u8(orc.encode_array(ai, fa), (K + 31) // 16 * 16), dev_u8(orc.encode_array(bi, fb), (K + 47) // 16 * 16)
            args = (a, fa, dev_f32(sa), fp8.FP8_ROW, b, fb, dev_f32(sb), fp8.FP8_ROW)
            assert (host_f32(fp8.fp8_scaled_mm(*args, fp8.FP8_OUT_FP32)) == want).all(), (fa, fb)
            out = torch.full((M + 2, (N + 15) // 8 * 8), -7.0, dtype=torch.bfloat16, device="cuda")
            fp8.fp8_scaled_mm(*args, 0, out=out[1:M + 1, :N])
            assert (host_bf16_bits(out)[1:M + 1, :N] == orc.f32_to_bf16(want)).all(), (fa, fb)
            assert bool((out[0] == -7.0).all() and (out[M + 1] == -7.0).all() and (out[:, N:] == -7.0).all())
        one = (a, 1, dev_f32(sa[:1]), fp8.FP8_TENSOR, b, 1, dev_f32(sb[:1]), fp8.FP8_TENSOR)
        assert (host_f32(fp8.fp8_scaled_mm(*one, fp8.FP8_OUT_FP32)) == (ai @ bi.T) / sa[0] / sb[0]).all()


@pytest.mark.parametrize("N,K", [(16384, 6144), (6144, 16384), (16392, 6144), (28672, 4096), (32776, 4096), (6144, 16400), (16400, 6160), (7680, 13120)])
def test_large_weights_on_either_side_of_the_line(N, K):
    """Small integers in e4m3: the choice may take either kernel, both are exact."""
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    codes = torch.tensor([0x00, 0x38, 0x40, 0xB8, 0xC0], dtype=torch.uint8, device="cuda")      # 0, 1, 2, -1, -2
    b = codes[torch.randint(0, 5, (N, K), generator=gen, device="cuda")]
    sb = torch.exp2(torch.randint(-3, 4, (N,), generator=gen, device="cuda").float())
    for M in (1, 9, 16, 17):
        a = codes[torch.randint(0, 5, (M, K), generator=gen, device="cuda")]
        sa = torch.exp2(torch.randint(-3, 4, (M,), generator=gen, device="cuda").float())
        run = lambda: fp8.fp8_scaled_mm(a, 0, sa, fp8.FP8_ROW, b, 0, sb, fp8.FP8_ROW, fp8.FP8_OUT_FP32)      # noqa: E731
        with knobs(GEMM_VARIANT=4):
            want = run()
        assert torch.equal(run(), want), M
