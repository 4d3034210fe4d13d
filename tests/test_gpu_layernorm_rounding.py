"""LayerNorm's rounding to bfloat16 where the binary32 value in between is a bfloat16 tie, which the kernel leaves to a path of its own:
rows whose results lie on a tie, a hair above and a hair below it, in every position of a thread's eight elements."""
import numpy as np
import pytest
import torch

import synthetic_inputs as si
from oracle import fp8_oracle as orc
from tests.gpu_util import dev_bf16, host_bf16_bits, host_u8

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


@pytest.mark.parametrize("cols", [8, 72, 512, 1000, 2048, 2056, 4096, 8200])
def test_ties_of_the_intermediate_rounding(cols):
    rng = np.random.default_rng(cols)
    rows = 37
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    # h = (x - mean) rstd gamma + beta: gamma of 2^-18 .. 2^-30 under a beta that is no power of two leaves the binary64 sum next to beta
    gamma = np.exp2(rng.integers(-30, -6, cols)).astype(np.float32)
    beta = rng.standard_normal(cols).astype(np.float32)
    # and rows of +-1, whose mean is 0 and rstd nearly 1: results gamma + beta with bits of gamma at the tie of beta's last place
    x[::2] = np.where(np.arange(cols) % 2 == 0, 1.0, -1.0)
    beta[::3] = 1.0 + 2.0 ** -7 * rng.integers(0, 127, beta[::3].size)
    gamma[::3] = 2.0 ** -8
    xb, gb, bb = si.f32_to_bf16_bits(x), si.f32_to_bf16_bits(gamma), si.f32_to_bf16_bits(beta)
    for eps in (0.0, 1e-5):
        want = orc.layernorm(xb, gb, bb, eps)
        wh = want[0] if isinstance(want, tuple) else want.h
        h, q, s, _, _ = fp8.fp8_layernorm_quantize(dev_bf16(xb), dev_bf16(gb[None])[0], dev_bf16(bb[None])[0], eps, fp8.FP8_E4M3FN)
        assert (host_bf16_bits(h) == wh).all()
        wq, ws = orc.quantize(wh, orc.ROW, orc.E4M3FN)
        assert (host_u8(q) == wq).all() and (s.cpu().numpy() == ws).all()
