"""The one-launch decode linear holds X as pieces of 512 elements, a count per wavefront that depends on M * K: every count, rows that start
inside a wavefront's pieces, rows of zeros, infinities and NaN; the bits of the two-launch form, its product on the few-row kernel
(SKINNY_DMA = 1: the persistent one adds eight parts of K where that and the one-launch kernel add four)."""
import pytest
import torch

from tests.gpu_util import knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


@pytest.mark.parametrize("N", [40, 1024, 3072, 6152])
@pytest.mark.parametrize("K", [512, 1536, 2560, 4096, 5120, 6656, 10752, 16384, 32768])
def test_as_two_launches(N, K):
    gen = torch.Generator(device="cuda").manual_seed(K + N)
    w = torch.randn((N, K), device="cuda", generator=gen).to(torch.bfloat16)
    wq, sw = fp8.fp8_quantize(w, fp8.FP8_ROW, fp8.FP8_E4M3FN)
    for M in range(1, 9):
        if M * K > 32768:
            break
        x = torch.randn((M, K), device="cuda", generator=gen) * torch.logspace(-3, 3, M, device="cuda")[:, None]
        x[torch.arange(M), torch.randint(0, K, (M,), generator=gen, device="cuda")] *= 20.0      # the row's maximum, in any of its pieces
        x = x.to(torch.bfloat16)
        odd = x.clone()
        odd[M // 2] = 0
        odd[M - 1, K - 1] = float("inf")
        odd[0, K // 2] = float("nan")
        for v in (x, odd):
            for gran, flags in ((fp8.FP8_ROW, 0), (fp8.FP8_ROW, fp8.FP8_POW2_SCALE), (fp8.FP8_TENSOR, 0)):
                run = lambda: fp8.fp8_linear_fwd_prequantized(v, wq, fp8.FP8_E4M3FN, sw, fp8.FP8_ROW, fp8.FP8_E4M3FN, gran, flags).view(torch.int16)      # noqa: E731
                with knobs(DECODE_FUSED=0, SKINNY_DMA=1):
                    want = run()
                with knobs(DECODE_FUSED=2):
                    assert torch.equal(run(), want), (M, gran, flags)
                with knobs(SKINNY_DMA=1):
                    assert torch.equal(run(), want), (M, gran, flags)


@pytest.mark.parametrize("M,N,K", [(1, 40, 512), (1, 4096, 4096), (1, 6152, 31744), (1, 16384, 32256), (1, 16384, 32768), (1, 28672, 32768), (2, 6152, 8192), (4, 28672, 4096),
                                   (3, 1024, 5120)])
def test_the_workspace_is_not_written(M, N, K):
    """One token, and up to four of 16384 activations together: programs may hand the same workspace, or none of their own, to
    calls on several streams."""
    gen = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn((M, K), device="cuda", generator=gen).to(torch.bfloat16)
    wq = torch.randint(0, 0x70, (N, K), dtype=torch.uint8, device="cuda", generator=gen)
    sw = torch.ones(N, device="cuda")
    ws = torch.full((fp8.fp8_linear_prequantized_workspace_bytes(M, K),), 0x5A, dtype=torch.uint8, device="cuda")
    for gran in (fp8.FP8_ROW, fp8.FP8_TENSOR):
        fp8.fp8_linear_fwd_prequantized(x, wq, fp8.FP8_E4M3FN, sw, fp8.FP8_ROW, fp8.FP8_E4M3FN, gran, workspace=ws)
        assert bool((ws == 0x5A).all())


@pytest.mark.parametrize("one,M,N,K", [(True, 4, 1024, 4096), (False, 5, 1024, 4096), (False, 4, 1024, 5120), (False, 4, 8184, 5120), (True, 4, 8192, 5120), (False, 3, 4088, 5632),
                                       (True, 3, 4096, 5632), (True, 3, 2048, 5120), (False, 3, 3064, 9216), (True, 3, 3072, 9216), (True, 3, 1024, 8192), (True, 2, 1024, 12288),
                                       (True, 2, 1024, 10752), (True, 2, 1024, 9216), (True, 3, 1024, 10752), (False, 8, 8184, 4096), (True, 8, 8192, 4096), (False, 5, 32776, 1024), (False, 8, 28672, 4096),
                                       (False, 8, 12280, 2560), (True, 8, 12288, 2560), (False, 7, 8192, 2560), (True, 6, 8192, 2560), (True, 6, 8192, 3072)])
def test_one_launch_or_two(one, M, N, K):
    """Both sides of the lines of the choice: two launches write the workspace."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("lines for 256 CUs")
    gen = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn((M, K), device="cuda", generator=gen).to(torch.bfloat16)
    wq = torch.randint(0, 0x70, (N, K), dtype=torch.uint8, device="cuda", generator=gen)
    ws = torch.full((fp8.fp8_linear_prequantized_workspace_bytes(M, K),), 0x5A, dtype=torch.uint8, device="cuda")
    sw = torch.ones(N, device="cuda")
    fp8.fp8_linear_fwd_prequantized(x, wq, fp8.FP8_E4M3FN, sw, fp8.FP8_ROW, workspace=ws)
    assert bool((ws == 0x5A).all()) == one
    if M <= 4:      # one scale for all tokens, whose two launches are three: always one
        ws.fill_(0x5A)
        fp8.fp8_linear_fwd_prequantized(x, wq, fp8.FP8_E4M3FN, sw, fp8.FP8_ROW, fp8.FP8_E4M3FN, fp8.FP8_TENSOR, workspace=ws)
        assert bool((ws == 0x5A).all())
