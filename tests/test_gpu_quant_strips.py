"""Column strips: all tensors of a rowwise step quantized in one launch.  Strips of both widths, at the edges of their rows and columns
and of the workgroups that hold them, against the single-tensor calls: the same bits."""
import numpy as np
import pytest
import torch

from tests.gpu_util import knobs

pytestmark = pytest.mark.gpu

import paper_2507_16099_amd as fp8  # noqa: E402


def _step(M, K, N, x, w, dy, flags):
    outs = []
    for save in (0, fp8.FP8_SAVE_FOR_BWD):
        r = fp8.Recipe(gran=fp8.FP8_ROW, flags=flags | save)
        ws = torch.full((fp8.fp8_linear_workspace_bytes(M, K, N, r, True),), 0x7F, dtype=torch.uint8, device="cuda")
        wf = ws if save else torch.full((fp8.fp8_linear_workspace_bytes(M, K, N, r, False),), 0x7F, dtype=torch.uint8, device="cuda")
        outs.append(fp8.fp8_linear_fwd(x, w, r, workspace=wf))
        outs += list(fp8.fp8_linear_bwd(dy, x, w, r, workspace=ws))
    return [o.view(torch.int16).clone() for o in outs]


def _inputs(M, K, N, hard):
    rng = np.random.default_rng(M + K + N)
    x, w, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda().to(torch.bfloat16) for s in ((M, K), (N, K), (M, N)))
    if hard:      # groups of zeros, below the clamp, infinite and NaN, with finite values beside them
        for t in (x, w, dy):
            t[:, 0] = 0
            t[t.shape[0] // 2] = 0
            t[:, 1] *= 1e-20
            t[t.shape[0] - 1, 3] = float("inf")
            t[0, 5] = float("nan")
            t[t.shape[0] - 1, t.shape[1] - 1] = 300.0
    return x, w, dy


@pytest.mark.parametrize("M,K,N", [(1, 16, 16), (15, 48, 1040), (17, 2064, 32), (1000, 1040, 528), (1024, 4112, 1024), (1025, 272, 2048),
                                   (2049, 528, 4096), (4095, 144, 272), (4097, 272, 1040), (8192, 64, 8192), (64, 8208, 48), (33, 16384, 64)])
def test_strips_change_no_bit(M, K, N):
    x, w, dy = _inputs(M, K, N, False)
    for flags in (0, fp8.FP8_POW2_SCALE, fp8.FP8_GRAD_WEIGHT_HP):
        with knobs(PAIRS=0):
            want = _step(M, K, N, x, w, dy, flags)
        for strips in (None, 2, 4, 0):
            with knobs(STRIPS=strips):
                got = _step(M, K, N, x, w, dy, flags)
            for a, b in zip(got, want):
                assert torch.equal(a, b), (strips, flags)


@pytest.mark.parametrize("strips", [2, 4])
@pytest.mark.parametrize("flags", [0, fp8.FP8_POW2_SCALE])
def test_zero_tiny_and_non_finite_groups(strips, flags):
    """The conversion without a clamp only where no group's maximum is NaN."""
    M, K, N = 96, 272, 160
    x, w, dy = _inputs(M, K, N, True)
    with knobs(PAIRS=0):
        want = _step(M, K, N, x, w, dy, flags)
    with knobs(STRIPS=strips):
        got = _step(M, K, N, x, w, dy, flags)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("M,K,N", [(1024, 256, 512), (1040, 528, 1040), (4096, 128, 2064)])
def test_weight_and_input_of_the_sigmoid_backward(M, K, N):
    x, w, dy = _inputs(M, K, N, False)
    y = torch.sigmoid(dy.float()).to(torch.bfloat16)
    r = fp8.Recipe(gran=fp8.FP8_ROW)
    with knobs(PAIRS=0):
        want = fp8.fp8_linear_bwd_sigmoid(dy, y, x, w, r)
    for strips in (None, 2, 4):
        with knobs(STRIPS=strips):
            got = fp8.fp8_linear_bwd_sigmoid(dy, y, x, w, r)
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("M,K,N", [(144, 272, 528), (2064, 528, 1040)])
@pytest.mark.parametrize("want", ["dx", "dw"])
def test_one_gradient_wanted(M, K, N, want):
    """The tensors of one product only."""
    x, w, dy = _inputs(M, K, N, False)
    r = fp8.Recipe(gran=fp8.FP8_ROW)
    run = lambda: fp8.fp8_linear_bwd(dy, x, w, r, need_dx=want == "dx", need_dw=want == "dw")[want == "dw"].view(torch.int16)      # noqa: E731
    with knobs(PAIRS=0):
        ref = run()
    for strips in (None, 2, 4):
        with knobs(STRIPS=strips):
            assert torch.equal(run(), ref)


@pytest.mark.parametrize("M,K,N", [(2048, 4096, 4096), (2064, 4096, 4096), (4096, 2056 * 2, 2048), (592, 16384, 1008)])
def test_rows_of_large_steps_are_read_with_the_hint(M, K, N):
    """Both sides of 24 Mi elements by rows, whose loads carry the streaming hint beyond."""
    x, w, dy = _inputs(M, K, N, False)
    for flags in (0, fp8.FP8_GRAD_WEIGHT_HP):
        r = fp8.Recipe(gran=fp8.FP8_ROW, flags=flags | fp8.FP8_SAVE_FOR_BWD)

        def run():
            ws = torch.full((fp8.fp8_linear_workspace_bytes(M, K, N, r, True),), 0x7F, dtype=torch.uint8, device="cuda")
            outs = [fp8.fp8_linear_fwd(x, w, r, workspace=ws)]
            outs += list(fp8.fp8_linear_bwd(dy, x, w, r, workspace=ws))
            return [o.view(torch.int16).clone() for o in outs]

        with knobs(PAIRS=0):
            want = run()
        for strips in (None, 2, 4):
            with knobs(STRIPS=strips):
                got = run()
            for a, b in zip(got, want):
                assert torch.equal(a, b), (strips, flags)
