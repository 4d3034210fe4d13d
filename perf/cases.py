"""The work that a user of this framework has it do, as cases that can be timed and compared.

Five kinds of pass, each through the public entry points of ``paper_2507_16099_amd.fp8``:

  infer   a linear layer of a served model: the weight quantized once, the activations per call
          (``fp8_linear_fwd_prequantized``).  One token is a single user's decode step, 2..64 tokens a batch of
          users, hundreds to thousands a prompt or a chunk of one (whatever length the prompts have).
  train   a training step of one linear layer: ``fp8_linear_fwd`` and ``fp8_linear_bwd``, per tensor or per row, with
          power-of-two scales or not, with the workspace shared between the two calls or not, the weight gradient in
          fp8 or kept in bfloat16 (``rowwise_gw_hp``).
  mx      the same step with MX block scaling (blocks of 32).
  block   the same step with blockwise scaling (tiles of 1 x 128, blocks of 128 x 128).
  lnsig   LayerNorm + Linear + Sigmoid, forward and backward, with the fused entry points.

Sizes are those of the Llama-3 8B and 70B linear layers and of the shape sweep, and sizes beside them: token counts of
every parity, feature counts of every multiple that the entry points take.  Activations are N(0, 1) (or heavy-tailed
with a few hot columns), weights N(0, 0.02), output gradients N(0, 1e-3), as in training.
"""
from __future__ import annotations

import math

import torch

from paper_2507_16099_amd import fp8

E4, E5, TENSOR, ROW = fp8.FP8_E4M3FN, fp8.FP8_E5M2, fp8.FP8_TENSOR, fp8.FP8_ROW
FMAX = {E4: 448.0, E5: 57344.0}


def _case(kind, M, K, N, *, gran="row", pow2=False, save=True, hp=False, outliers=False):
    return {"kind": kind, "M": M, "K": K, "N": N, "gran": gran, "pow2": pow2, "save": save, "hp": hp, "outliers": outliers}


def listed():
    return [
        # serving -------------------------------------------------------------------------------------------------
        # the smallest call: one user's token through the output projection of the 8B model
        {"name": "decode_8b_o_1_token", **_case("infer", 1, 4096, 4096)},
        # a decode batch through the up projection of the 70B model: the weight stream decides
        {"name": "decode_70b_up_16_tokens", **_case("infer", 16, 8192, 28672, pow2=True)},
        # a larger decode batch (or a short prompt) through the up projection of the 8B model
        {"name": "batch_8b_up_72_tokens", **_case("infer", 72, 4096, 14336)},
        # a prompt of an odd length through the down projection of the 8B model, activations per tensor
        {"name": "prefill_8b_down_777_tokens", **_case("infer", 777, 14336, 4096, gran="tensor")},
        # training ------------------------------------------------------------------------------------------------
        # a small model's layer: launches count
        {"name": "train_row_1024_2048_1024", **_case("train", 1024, 2048, 1024)},
        # a mid-size layer, stateless calls, a token count that is no multiple of anything
        {"name": "train_row_ragged_3001_4096_2048", **_case("train", 3001, 4096, 2048, save=False)},
        # the 8B model's fused QKV projection, one scale per tensor
        {"name": "train_tensor_8b_qkv", **_case("train", 8192, 4096, 6144, gran="tensor")},
        # the 8B model's FFN layer, rowwise: the benchmark shape and the largest case
        {"name": "train_row_8b_ffn", **_case("train", 16384, 4096, 14336)},
        # rowwise with the weight gradient in bfloat16, at the few thousand tokens where that recipe is chosen
        {"name": "train_gw_hp_2048_4096_4096", **_case("train", 2048, 4096, 4096, hp=True)},
        # the finer-grained recipes
        {"name": "mx_4096_4096_14336", **_case("mx", 4096, 4096, 14336)},
        {"name": "block_2048_4096_4096", **_case("block", 2048, 4096, 4096)},
        # the microbenchmark block of the paper
        {"name": "lnsig_8192_4096_4096", **_case("lnsig", 8192, 4096, 4096)},
    ]


# feature counts that occur in the models and the sweep
_DIMS = (1024, 2048, 4096, 6144, 8192, 11008, 14336, 16384, 28672)


def _cost(case):
    """Rough cost in fp8 operations: the bfloat16 weight gradient takes about three times as long as the fp8 one."""
    f = 2.0 * case["M"] * case["K"] * case["N"]
    return f if case["kind"] == "infer" else (5.0 if case["hp"] else 3.4 if case["kind"] == "lnsig" else 3.0) * f


def draw(rng):
    """One more case of the ranges above: M, K and N over their logarithm, feature counts half of the time from the
    models' list and otherwise any multiple that the entry points take."""
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    def dim(lo, hi, multiple):
        if rng.random() < 0.5:
            return rng.choice([d for d in _DIMS if lo <= d <= hi])
        return max(multiple, int(log(lo, hi)) // multiple * multiple)

    limit = 0.9 * _cost(_case("train", 16384, 4096, 14336))
    while True:
        kind = rng.choice(("infer", "infer", "infer", "train", "train", "train", "train", "mx", "block", "lnsig"))
        if kind == "infer":
            M = int(log(1, 4097))
            c = _case(kind, M, dim(1024, 28672, 16), dim(1024, 28672, 8), gran=rng.choice(("row", "row", "tensor")),
                      pow2=rng.random() < 0.3, outliers=rng.random() < 0.2)
        elif kind == "train":
            M = int(log(512, 16385))
            if rng.random() < 0.6:                      # most batches are whole sequences
                M = max(512, M // 256 * 256)
            gran = rng.choice(("row", "row", "tensor"))
            c = _case(kind, M, dim(1024, 16384, 16), dim(1024, 16384, 16), gran=gran, pow2=rng.random() < 0.3,
                      save=rng.random() < 0.7, hp=gran == "row" and rng.random() < 0.25, outliers=rng.random() < 0.2)
        elif kind == "lnsig":
            c = _case(kind, max(512, int(log(512, 16385)) // 64 * 64), dim(1024, 8192, 128), dim(1024, 16384, 128),
                      pow2=rng.random() < 0.3)
        else:
            c = _case(kind, max(512, int(log(512, 16385)) // 128 * 128), dim(1024, 16384, 128), dim(1024, 16384, 128))
        if _cost(c) <= limit:
            return c


# ---------------------------------------------------------------------------------------------------------------------
# inputs


def _activations(case, rows, cols, gen):
    x = torch.randn((rows, cols), device="cuda", generator=gen)
    if case["outliers"]:      # Student-t with three degrees of freedom, 0.1 % of the columns a hundred times larger
        chi = torch.zeros((rows, cols), device="cuda")
        for _ in range(3):
            chi += torch.randn((rows, cols), device="cuda", generator=gen).square_()
        x /= (chi / 3.0).sqrt_()
        hot = torch.randperm(cols, device="cuda", generator=gen)[: max(1, round(0.001 * cols))]
        x[:, hot] *= 100.0
    return x.to(torch.bfloat16)


def _tensors(case, seed):
    """The bfloat16 tensors of a case, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    M, K, N = case["M"], case["K"], case["N"]
    t = {"x": _activations(case, M, K, gen), "w": torch.randn((N, K), device="cuda", generator=gen).mul_(0.02).to(torch.bfloat16)}
    if case["kind"] != "infer":
        t["dy"] = torch.randn((M, N), device="cuda", generator=gen).mul_(1e-3).to(torch.bfloat16)
    if case["kind"] == "lnsig":
        t["gamma"] = (torch.rand(K, device="cuda", generator=gen) + 0.5).to(torch.bfloat16)
        t["beta"] = (torch.rand(K, device="cuda", generator=gen) - 0.5).to(torch.bfloat16)
    return t


def _recipe(case):
    fl = (fp8.FP8_POW2_SCALE if case["pow2"] else 0) | (fp8.FP8_SAVE_FOR_BWD if case["save"] else 0) \
        | (fp8.FP8_GRAD_WEIGHT_HP if case["hp"] else 0)
    return fp8.Recipe(gran=TENSOR if case["gran"] == "tensor" else ROW, flags=fl)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _bf16(*shape):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda")


def prepare(case, seed):
    """Inputs, and the buffers, workspace and quantized weight that a program keeps from call to call."""
    kind, M, K, N = case["kind"], case["M"], case["K"], case["N"]
    s = {"case": case, **_tensors(case, seed), "y": _bf16(M, (N + 7) // 8 * 8)[:, :N]}
    if kind == "infer":
        s["wq"], s["sw"] = fp8.fp8_quantize(s.pop("w"), ROW, E4, fp8.FP8_POW2_SCALE if case["pow2"] else 0)
        s["ws"] = _bytes(fp8.fp8_linear_prequantized_workspace_bytes(M, K))
        return s
    s["dx"], s["dw"] = _bf16(M, K), _bf16(N, K)
    if kind == "train":
        s["recipe"] = r = _recipe(case)
        s["ws_bwd"] = _bytes(fp8.fp8_linear_workspace_bytes(M, K, N, r, True))
        s["ws_fwd"] = s["ws_bwd"] if case["save"] else _bytes(fp8.fp8_linear_workspace_bytes(M, K, N, r, False))
    elif kind == "mx":
        s["ws_fwd"] = _bytes(fp8.fp8_mx_linear_workspace_bytes(M, K, N))
        s["ws_bwd"] = _bytes(fp8.fp8_mx_linear_bwd_workspace_bytes(M, K, N))
    elif kind == "block":
        s["ws_fwd"] = _bytes(fp8.fp8_block_linear_workspace_bytes(M, K, N))
        s["ws_bwd"] = _bytes(fp8.fp8_block_linear_bwd_workspace_bytes(M, K, N))
    else:
        s["recipe"] = r = fp8.Recipe(gran=ROW, flags=fp8.FP8_POW2_SCALE if case["pow2"] else 0)
        s["ws_bwd"] = _bytes(fp8.fp8_linear_bwd_sigmoid_workspace_bytes(M, K, N, r))
        f32 = dict(dtype=torch.float32, device="cuda")
        s["ln"] = (_bf16(M, K), torch.empty((M, K), dtype=torch.uint8, device="cuda"), torch.empty(M, **f32),
                   torch.empty(M, **f32), torch.empty(M, **f32))
        s["wq"], s["sw"] = torch.empty((N, K), dtype=torch.uint8, device="cuda"), torch.empty(N, **f32)
    return s


# ---------------------------------------------------------------------------------------------------------------------
# one pass


def run(s):
    case = s["case"]
    kind = case["kind"]
    pow2 = fp8.FP8_POW2_SCALE if case["pow2"] else 0
    if kind == "infer":
        gran = TENSOR if case["gran"] == "tensor" else ROW
        fp8.fp8_linear_fwd_prequantized(s["x"], s["wq"], E4, s["sw"], ROW, E4, gran, pow2, y=s["y"], workspace=s["ws"])
        return s["y"]
    if kind == "train":
        fp8.fp8_linear_fwd(s["x"], s["w"], s["recipe"], y=s["y"], workspace=s["ws_fwd"])
        fp8.fp8_linear_bwd(s["dy"], s["x"], s["w"], s["recipe"], dx=s["dx"], dw=s["dw"], workspace=s["ws_bwd"])
    elif kind == "mx":
        fp8.fp8_mx_linear_fwd(s["x"], s["w"], y=s["y"], workspace=s["ws_fwd"])
        fp8.fp8_mx_linear_bwd(s["dy"], s["x"], s["w"], dx=s["dx"], dw=s["dw"], workspace=s["ws_bwd"])
    elif kind == "block":
        fp8.fp8_block_linear_fwd(s["x"], s["w"], y=s["y"], workspace=s["ws_fwd"])
        fp8.fp8_block_linear_bwd(s["dy"], s["x"], s["w"], dx=s["dx"], dw=s["dw"], workspace=s["ws_bwd"])
    else:
        h, hq, sh, mean, rstd = fp8.fp8_layernorm_quantize(s["x"], s["gamma"], s["beta"], 1e-5, E4, pow2, out=s["ln"])
        fp8.fp8_quantize(s["w"], ROW, E4, pow2, out=s["wq"], scale_out=s["sw"])
        fp8.fp8_scaled_mm(hq, E4, sh, ROW, s["wq"], E4, s["sw"], ROW, fp8.FP8_EPILOGUE_SIGMOID, out=s["y"])
        fp8.fp8_linear_bwd_sigmoid(s["dy"], s["y"], h, s["w"], s["recipe"], dx=s["dx"], dw=s["dw"], workspace=s["ws_bwd"])
        return {"h": h, "mean": mean, "rstd": rstd, "y": s["y"], "dx": s["dx"], "dw": s["dw"]}
    return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}


def work(case):
    M, K, N = case["M"], case["K"], case["N"]
    if case["kind"] == "infer":
        return {"bytes": 2.0 * M * K + N * K + 4.0 * N + 2.0 * M * N, "flops": 2.0 * M * K * N}
    # X, W, dY in; Y, dX, dW out
    b = 2.0 * (M * K + N * K + M * N) * 2
    if case["kind"] == "lnsig":
        b += 2.0 * M * K + 8.0 * M + 4.0 * K      # the normalised activations and their statistics
    return {"bytes": b, "flops": 6.0 * M * K * N}


def tolerance(case):
    # Codes and scales are decided bit for bit; the products' fp32 sums may be taken in any order, which turns about one
    # bfloat16 result in a hundred to its neighbour.  Seen between this path and 64-bit sums rounded to bfloat16: 2.3e-4
    # (largest single difference 7.8e-3, one bfloat16 step); 5.4e-4 with heavy-tailed activations, whose few large
    # products decide a sum; and in lnsig, where a turned bfloat16 y also enters the gradient's quantization and can
    # move a group's scale, 1.6e-3 (0.14).
    if case["kind"] == "lnsig":
        return {"rel": 6e-3, "max": 0.5}
    return {"rel": 2e-3 if case["outliers"] else 1e-3, "max": 0.04}


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits


def _cast(v, fmt):
    """fp32 values -> fp8 (saturating, nearest even) -> fp64."""
    t = torch.float8_e4m3fn if fmt == E4 else torch.float8_e5m2
    return v.clamp(-FMAX[fmt], FMAX[fmt]).to(t).to(torch.float64)


def _scale(amax, fmt, pow2):
    s = (FMAX[fmt] / amax.double().clamp(min=1e-12)).float()
    return (s.view(torch.int32) & -0x800000).view(torch.float32) if pow2 else s


def _q(x, fmt, dim, pow2=False):
    """Dequantized values of x with one scale per tensor (dim None) or per group along `dim`."""
    f = x.float()
    amax = f.abs().amax() if dim is None else f.abs().amax(dim, keepdim=True)
    s = _scale(amax, fmt, pow2)
    return _cast(f * s, fmt) / s.double()


def _q_mx(x):
    """MX blocks of 32 along the last axis, e4m3 elements."""
    f = x.float().reshape(x.shape[0], -1, 32)
    e = torch.frexp(f.abs().amax(2, keepdim=True))[1] - 1 - 8
    e = torch.where(f.abs().amax(2, keepdim=True) > 0, e, torch.full_like(e, -127)).clamp(-127, 127)
    p = torch.exp2(e.double())
    return (_cast((f.double() / p).float(), E4) * p).reshape(x.shape)


def _q_block(x, square):
    """Tiles of 1 x 128 (blocks of 128 x 128) with power-of-two scales, e4m3 elements."""
    R, C = x.shape
    f = x.float()
    if square:
        f = f.reshape(R // 128, 128, C // 128, 128)
        s = _scale(f.abs().amax((1, 3), keepdim=True), E4, True)
    else:
        f = f.reshape(R, C // 128, 128)
        s = _scale(f.abs().amax(2, keepdim=True), E4, True)
    return (_cast(f * s, E4) / s.double()).reshape(R, C)


def exact(case, seed):
    kind, t, pow2 = case["kind"], _tensors(case, seed), case["pow2"]
    x, w, dy = t["x"], t["w"], t.get("dy")
    if kind == "infer":
        return _q(x, E4, None if case["gran"] == "tensor" else 1, pow2) @ _q(w, E4, 1, pow2).T
    if kind == "train":
        row = case["gran"] == "row"
        a, b = (0, 1) if row else (None, None)
        y = _q(x, E4, b, pow2) @ _q(w, E4, b, pow2).T
        dx = _q(dy, E5, b, pow2) @ _q(w, E4, a, pow2)
        dw = dy.double().T @ x.double() if case["hp"] else _q(dy, E5, a, pow2).T @ _q(x, E4, a, pow2)
        return {"y": y, "dx": dx, "dw": dw}
    if kind == "mx":
        along = lambda v: _q_mx(v)                                     # noqa: E731
        down = lambda v: _q_mx(v.T.contiguous()).T                     # noqa: E731
        return {"y": along(x) @ along(w).T, "dx": along(dy) @ down(w), "dw": down(dy).T @ down(x)}
    if kind == "block":
        down = lambda v: _q_block(v.T.contiguous(), False).T           # noqa: E731
        wb = _q_block(w, True)
        return {"y": _q_block(x, False) @ wb.T, "dx": _q_block(dy, False) @ wb, "dw": down(dy).T @ down(x)}
    xd = x.double()
    mean = xd.mean(1, keepdim=True)
    rstd = 1.0 / ((xd - mean).square().mean(1, keepdim=True) + 1e-5).sqrt()
    h = (xd - mean) * rstd * t["gamma"].double() + t["beta"].double()
    hb = h.to(torch.bfloat16)
    y = torch.sigmoid(_q(hb, E4, 1, pow2) @ _q(w, E4, 1, pow2).T)
    yb, g = y.to(torch.bfloat16).float(), dy.float()
    dz = (g * yb * (1.0 - yb)).to(torch.bfloat16)
    return {"h": h, "mean": mean[:, 0], "rstd": rstd[:, 0], "y": y, "dx": _q(dz, E5, 1, pow2) @ _q(w, E4, 0, pow2),
            "dw": _q(dz, E5, 0, pow2).T @ _q(hb, E4, 0, pow2)}
