"""Products of few rows on both sides of the rule for the streaming hint (a weight of 96 MiB), on every kernel that has it, and on both
sides of the rule that sends 17-32 rows to the ring kernel: exact integer products, against the 256 x 256 kernel."""
import pytest
import torch

from tests.gpu_util import knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402

ROW, E4, E5 = fp8.FP8_ROW, fp8.FP8_E4M3FN, fp8.FP8_E5M2


def _ints(rows, cols, seed, fmt):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.randint(-2, 3, (rows, cols), device="cuda", generator=gen, dtype=torch.int8)
    t = torch.float8_e4m3fn if fmt == E4 else torch.float8_e5m2
    return v.to(torch.float32).to(t).view(torch.uint8)


def _mm(a, fa, b, fb):
    sa = torch.full((a.shape[0],), 0.5, device="cuda")
    sb = torch.exp2((torch.arange(b.shape[0], device="cuda") % 3).float())
    return fp8.fp8_scaled_mm(a, fa, sa, ROW, b, fb, sb, ROW).view(torch.int16)


@pytest.mark.parametrize("N,K", [(16384, 6144), (16376, 6144), (16400, 6160), (16128, 6400)])      # 96 MiB exactly, less, ragged, a longer contraction
@pytest.mark.parametrize("fb", [E4, E5])
def test_both_sides_of_the_size_of_a_streamed_weight(N, K, fb):
    b = _ints(N, K, 1, fb)
    for M in (3, 16, 31, 64, 65, 128, 129, 192, 255):
        a = _ints(M, K, M, E4)
        with knobs(GEMM_VARIANT=4):
            want = _mm(a, E4, b, fb)
        assert torch.equal(_mm(a, E4, b, fb), want), M
        for tile in (1, 3, 4, 5, 6):
            with knobs(GEMM_RING=tile):
                assert torch.equal(_mm(a, E4, b, fb), want), (M, tile)


@pytest.mark.parametrize("N,K", [(16384, 6144), (6144, 16384), (16376, 6144)])
def test_one_launch_decode_of_a_streamed_weight(N, K):
    gen = torch.Generator(device="cuda").manual_seed(N)
    w = torch.randn((N, K), device="cuda", generator=gen).to(torch.bfloat16)
    wq, sw = fp8.fp8_quantize(w, ROW, E4)
    del w
    for M in (1, 2):
        x = torch.randn((M, K), device="cuda", generator=gen).to(torch.bfloat16)
        run = lambda: fp8.fp8_linear_fwd_prequantized(x, wq, E4, sw, ROW).view(torch.int16)      # noqa: E731
        got = run()
        with knobs(DECODE_FUSED=0, SKINNY_DMA=1):      # (the persistent few-row kernel adds the parts of K in another order)
            assert torch.equal(got, run())


@pytest.mark.parametrize("M", [16, 17, 32, 33])
@pytest.mark.parametrize("N", [10176, 10232, 10240, 11008])
def test_rows_between_the_few_row_and_the_ring_kernel(M, N):
    for K in (16, 528, 2064):
        a, b = _ints(M, K, M, E5), _ints(N, K, 2, E4)
        with knobs(GEMM_VARIANT=4):
            want = _mm(a, E5, b, E4)
        assert torch.equal(_mm(a, E5, b, E4), want), K


@pytest.mark.parametrize("M", [1, 4, 5, 8, 9])
@pytest.mark.parametrize("N,K", [(1024, 10240), (1024, 10256), (2048, 11024), (2056, 11024), (3072, 11024), (3080, 10256), (24, 28672)])
def test_both_sides_of_the_longer_ring_of_few_rows(M, N, K):
    a, b = _ints(M, K, M, E4), _ints(N, K, 2, E5)
    with knobs(GEMM_VARIANT=4):
        want = _mm(a, E4, b, E5)
    assert torch.equal(_mm(a, E4, b, E5), want)
