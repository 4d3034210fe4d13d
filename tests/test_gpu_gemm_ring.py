"""The ring kernel (products of few to middling size): every tile of it, at the edges of its tiles and of its ring of
K steps, against exact integer products; two products in one launch; the sigmoid in its epilogue."""
import numpy as np
import pytest
import torch

import synthetic_inputs as si
from oracle import fp8_oracle as orc
from tests.gpu_util import dev_f32, dev_u8, host_bf16_bits, host_f32, knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402

TILES = {"64x64": 1, "128x64": 2, "64x128": 3, "128x128": 4, "128x256": 5, "256x128": 6}
# one tile, tiles plus one row / column, ragged rows and columns, fewer K steps than the ring, a K that ends inside a step
SHAPES = [(1, 8, 16), (64, 64, 128), (65, 72, 144), (257, 264, 1040), (130, 520, 528), (1100, 392, 640), (300, 1000, 2064)]


def _ints(shape, rng):
    return rng.integers(-2, 3, size=shape).astype(np.float32)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_every_tile_exact_on_small_integers(tile, M, N, K):
    rng = np.random.default_rng(M * 13 + N + K)
    ai, bi = _ints((M, K), rng), _ints((N, K), rng)
    sa, sb = (2.0 ** rng.integers(-3, 4, size=M)).astype(np.float32), (2.0 ** rng.integers(-3, 4, size=N)).astype(np.float32)
    exact = (ai @ bi.T).astype(np.float32)
    lda, ldb = (K + 15) // 16 * 16 + 16, (K + 15) // 16 * 16
    with knobs(GEMM_RING=TILES[tile]):
        for fa in (orc.E4M3FN, orc.E5M2):
            for fb in (orc.E4M3FN, orc.E5M2):
                a, b = dev_u8(orc.encode_array(ai, fa), lda), dev_u8(orc.encode_array(bi, fb), ldb)
                want = exact / sa[:, None] / sb[None, :]
                row = (a, fa, dev_f32(sa), fp8.FP8_ROW, b, fb, dev_f32(sb), fp8.FP8_ROW)
                assert (host_f32(fp8.fp8_scaled_mm(*row, fp8.FP8_OUT_FP32)) == want).all(), (fa, fb)
                assert (host_bf16_bits(fp8.fp8_scaled_mm(*row)) == orc.f32_to_bf16(want)).all(), (fa, fb)
                one = (a, fa, dev_f32(sa[:1]), fp8.FP8_TENSOR, b, fb, dev_f32(sb[:1]), fp8.FP8_TENSOR)
                assert (host_f32(fp8.fp8_scaled_mm(*one, fp8.FP8_OUT_FP32)) == exact / sa[0] / sb[0]).all(), (fa, fb)


@pytest.mark.parametrize("tile", TILES)
def test_writes_stay_inside_a_padded_output(tile):
    rng = np.random.default_rng(5)
    M, N, K = 70, 88, 160
    ai, bi = _ints((M, K), rng), _ints((N, K), rng)
    out = torch.full((M + 2, 128), -7.0, dtype=torch.bfloat16, device="cuda")
    one = dev_f32(np.ones(1, np.float32))
    with knobs(GEMM_RING=TILES[tile]):
        fp8.fp8_scaled_mm(dev_u8(orc.encode_array(ai, 0)), 0, one, 0, dev_u8(orc.encode_array(bi, 0)), 0, one, 0, 0, out=out[1:M + 1, :N])
    got = si.bf16_bits_to_f32(host_bf16_bits(out))
    assert (got[1:M + 1, :N] == ai @ bi.T).all()
    assert (got[:, N:] == -7.0).all() and (got[0] == -7.0).all() and (got[M + 1] == -7.0).all()


@pytest.mark.parametrize("M,N,K", [(16, 24, 128), (200, 304, 400), (1024, 768, 512)])
def test_sigmoid_matches_the_large_product_kernel(M, N, K):
    """The same accumulation order and the same epilogue arithmetic: bit for bit."""
    rng = np.random.default_rng(M)
    x, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    a, b = dev_u8(orc.encode_array(x, 0)), dev_u8(orc.encode_array(w, 0))
    sa, sb = dev_f32(rng.uniform(2, 8, M).astype(np.float32)), dev_f32(rng.uniform(2, 8, N).astype(np.float32))
    outs = []
    for k in ({"GEMM_VARIANT": 4}, {"GEMM_RING": 1}, {"GEMM_RING": 4}, {"GEMM_RING": 6}):
        with knobs(**k):
            outs.append(host_bf16_bits(fp8.fp8_scaled_mm(a, 0, sa, 1, b, 0, sb, 1, fp8.FP8_EPILOGUE_SIGMOID)))
    for o in outs[1:]:
        assert (o == outs[0]).all()


@pytest.mark.parametrize("tile", TILES)
def test_two_products_in_one_launch(tile):
    """The backward's products share a launch where that pays; forced here for every tile, the larger one first or second."""
    for M, K, N in ((272, 144, 528), (528, 656, 80)):
        rng = np.random.default_rng(M)
        dy, x, w = (torch.from_numpy(_ints(s, rng)).cuda().to(torch.bfloat16) for s in ((M, N), (M, K), (N, K)))
        r = fp8.Recipe(gran=fp8.FP8_ROW, flags=fp8.FP8_POW2_SCALE)
        with knobs(GEMM_RING=TILES[tile]):
            dx, dw = fp8.fp8_linear_bwd(dy, x, w, r)
        with knobs(GEMM_RING=0, PAIRS=0, GEMM_VARIANT=4):
            dx0, dw0 = fp8.fp8_linear_bwd(dy, x, w, r)
        assert torch.equal(dx.view(torch.int16), dx0.view(torch.int16)) and torch.equal(dw.view(torch.int16), dw0.view(torch.int16))


@pytest.mark.parametrize("tile", TILES)
def test_empty_contraction(tile):
    """K = 0: zeros, 0.5 behind the sigmoid, whatever the scales."""
    M, N = 70, 72
    a, b = (torch.empty((r, 0), dtype=torch.uint8, device="cuda") for r in (M, N))
    sa, sb = torch.full((M,), 3.0, device="cuda"), torch.full((N,), 0.25, device="cuda")
    with knobs(GEMM_RING=TILES[tile]):
        for flags, value in ((0, 0.0), (fp8.FP8_OUT_FP32, 0.0), (fp8.FP8_EPILOGUE_SIGMOID, 0.5)):
            out = torch.full((M, N), 7.0, dtype=torch.float32 if flags & fp8.FP8_OUT_FP32 else torch.bfloat16, device="cuda")
            fp8.fp8_scaled_mm(a, 0, sa, fp8.FP8_ROW, b, 1, sb, fp8.FP8_ROW, flags, out=out)
            assert bool((out == value).all())


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_every_count_of_steps_around_the_depth_of_the_ring(tile, steps):
    """Odd and even counts, fewer and more steps than stages: exact integer products."""
    rng = np.random.default_rng(steps)
    M, N, K = 140, 136, 128 * steps - 16
    ai, bi = _ints((M, K), rng), _ints((N, K), rng)
    one = dev_f32(np.ones(1, np.float32))
    a, b = dev_u8(orc.encode_array(ai, 0), (K + 15) // 16 * 16), dev_u8(orc.encode_array(bi, 0), (K + 15) // 16 * 16)
    with knobs(GEMM_RING=TILES[tile]):
        got = host_f32(fp8.fp8_scaled_mm(a, 0, one, 0, b, 0, one, 0, fp8.FP8_OUT_FP32))
    assert (got == ai @ bi.T).all()


@pytest.mark.parametrize("M", [17, 32])
@pytest.mark.parametrize("K,N", [(10192, 128), (11008, 64), (11008, 256), (14336, 512), (10240, 1024), (28672, 192)])
def test_backward_of_few_tokens_in_one_launch(M, K, N):
    """dX of 17 to 32 rows beside the weight gradient, together or apart as estimated: the bits of one product at a time."""
    rng = np.random.default_rng(K + N)
    dy, x, w = (torch.from_numpy(_ints(s, rng)).cuda().to(torch.bfloat16) for s in ((M, N), (M, K), (N, K)))
    r = fp8.Recipe(gran=fp8.FP8_ROW, flags=fp8.FP8_POW2_SCALE)
    dx, dw = fp8.fp8_linear_bwd(dy, x, w, r)
    with knobs(PAIRS=0):
        dx0, dw0 = fp8.fp8_linear_bwd(dy, x, w, r)
    assert torch.equal(dx.view(torch.int16), dx0.view(torch.int16)) and torch.equal(dw.view(torch.int16), dw0.view(torch.int16))


@pytest.mark.parametrize("tile", ["128x256", "256x128"])
@pytest.mark.parametrize("M,N,K", [(1, 8, 6160), (130, 264, 6272), (257, 520, 6400), (300, 392, 6144)])
def test_widest_tiles_on_either_side_of_their_short_contractions(tile, M, N, K):
    """Eight wavefronts up to K = 6144, four beyond: odd and even counts of steps, a K that ends inside a step, ragged rows and columns; all
    outputs, and the sigmoid as the large-product kernel gives it."""
    rng = np.random.default_rng(K + M)
    ai, bi = _ints((M, K), rng), _ints((N, K), rng)
    sa, sb = (2.0 ** rng.integers(-3, 4, size=M)).astype(np.float32), (2.0 ** rng.integers(-3, 4, size=N)).astype(np.float32)
    want = (ai @ bi.T).astype(np.float32) / sa[:, None] / sb[None, :]
    with knobs(GEMM_RING=TILES[tile]):
        for fa, fb in ((0, 0), (0, 1), (1, 0), (1, 1)):
            args = (dev_u8(orc.encode_array(ai, fa)), fa, dev_f32(sa), fp8.FP8_ROW, dev_u8(orc.encode_array(bi, fb)), fb, dev_f32(sb), fp8.FP8_ROW)
            assert (host_f32(fp8.fp8_scaled_mm(*args, fp8.FP8_OUT_FP32)) == want).all(), (fa, fb)
            assert (host_bf16_bits(fp8.fp8_scaled_mm(*args)) == orc.f32_to_bf16(want)).all(), (fa, fb)
        got = host_bf16_bits(fp8.fp8_scaled_mm(*args, fp8.FP8_EPILOGUE_SIGMOID))
    with knobs(GEMM_VARIANT=4):
        assert (got == host_bf16_bits(fp8.fp8_scaled_mm(*args, fp8.FP8_EPILOGUE_SIGMOID))).all()


@pytest.mark.parametrize("tile", ["128x256", "256x128"])
@pytest.mark.parametrize("M,K,N", [(272, 144, 6272), (6272, 144, 272), (6160, 80, 6400)])
def test_two_products_of_which_one_or_both_are_long(tile, M, K, N):
    rng = np.random.default_rng(M)
    dy, x, w = (torch.from_numpy(_ints(s, rng)).cuda().to(torch.bfloat16) for s in ((M, N), (M, K), (N, K)))
    r = fp8.Recipe(gran=fp8.FP8_ROW, flags=fp8.FP8_POW2_SCALE)
    with knobs(GEMM_RING=TILES[tile]):
        dx, dw = fp8.fp8_linear_bwd(dy, x, w, r)
    with knobs(GEMM_RING=0, PAIRS=0, GEMM_VARIANT=4):
        dx0, dw0 = fp8.fp8_linear_bwd(dy, x, w, r)
    assert torch.equal(dx.view(torch.int16), dx0.view(torch.int16)) and torch.equal(dw.view(torch.int16), dw0.view(torch.int16))
