"""What this library is timed on: the calls that its users make, one pass of a case = one or a few `ucl_*` calls.

Every case is a layer or an operator of a network, called through the public binding with buffers that the caller owns
(outputs included, as the library allocates nothing).  `tune` is left out except where the option itself is what is
used (split-K), so the library's own choice of kernel is part of what is timed.

The families, with the sizes that their drawn cases cover:

  tiny          a small fused GEMM on row-major operands (64..512 each way): the 256^3 problem of the benchmark; latency
  decode        a linear layer on a few tokens (1..64 rows) against a weight stored [N][K]: reading the weight is the work
  ragged        a linear layer with a residual on sizes that fit no tile, odd N included (a vocabulary or class head)
  linear        a linear layer on a full batch of tokens, bias + GELU: the 4096^3 problem of the benchmark
  weight_grad   a linear layer's weight gradient dY^T X into fp32: both operands contiguous along M / N
  deep_k        a small output over a deep reduction with parallel split-K and the caller's workspace
  batched       attention-score like batched GEMM, scaled, the 64 x 512 x 512 x 128 problem of the benchmark
  grouped       mixture-of-experts layer on a prefill batch, ragged groups of 64-row multiples, SiLU
  grouped_decode  the same while decoding: 8-bit operands, many experts with a few rows each, some with none
  conv          3x3 convolution forward, bias + residual + ReLU, the four stages of a residual network
  conv_pipeline an NCHW fp32 tensor through transform -> convolution (1x1 or 3x3, stride 1 or 2) -> transform back
  conv_backward both gradients of a convolution (1x1 or 3x3, stride 1 or 2), the filter's through split-K
"""
import math

import torch
import torch.nn.functional as F

import paper_2603_29010_amd as ucl

TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32, "e4m3": torch.float8_e4m3fn,
         "e5m2": torch.float8_e5m2}
SIZE = {"bf16": 2, "f16": 2, "f32": 4, "e4m3": 1, "e5m2": 1}


def listed():
    return [
        # the smallest call of the benchmark: launch and latency
        {"name": "tiny_256", "family": "tiny", "M": 256, "N": 256, "K": 256, "dt": "bf16"},
        # sixteen sequences decoding one token each through a 4096 x 4096 linear layer
        {"name": "decode_16x4096x4096", "family": "decode", "M": 16, "N": 4096, "K": 4096, "dt": "bf16", "act": "silu"},
        # an odd head on a ragged batch: no extent but K is a multiple of anything
        {"name": "ragged_1000x1001x1992", "family": "ragged", "M": 1000, "N": 1001, "K": 1992, "dt": "f16"},
        # the headline problem: a full batch through a linear layer with GELU
        {"name": "linear_4096", "family": "linear", "M": 4096, "N": 4096, "K": 4096, "dt": "bf16"},
        # training: gradient of a 1024 -> 4096 linear layer's weight over 8192 tokens
        {"name": "weight_grad_4096x1024x8192", "family": "weight_grad", "M": 4096, "N": 1024, "K": 8192, "dt": "bf16"},
        # a projection with a deep reduction, split along K in the caller's workspace
        {"name": "deep_k_256x256x16384", "family": "deep_k", "M": 256, "N": 256, "K": 16384, "dt": "bf16"},
        # batched scores of 64 heads
        {"name": "batched_64x512x512x128", "family": "batched", "batch": 64, "M": 512, "N": 512, "K": 128, "dt": "f16", "out": "f32"},
        # sixteen experts on a prefill batch
        {"name": "grouped_16x4096x1024", "family": "grouped", "groups": 16, "rows": "prefill", "mix": 4, "N": 4096, "K": 1024,
         "dt": "bf16"},
        # sixty-four experts while decoding: 0..32 rows each, 8-bit weights and activations
        {"name": "grouped_decode_64x2048x1024", "family": "grouped_decode", "groups": 64, "rows": "decode", "mix": 7, "N": 2048,
         "K": 1024, "dt": "e4m3"},
        # the 56 x 56 stage of a residual network
        {"name": "conv_32x56x56x64_128", "family": "conv", "n": 32, "hw": 56, "C": 64, "Ko": 128, "dt": "bf16"},
        # the strided 3x3 convolution that opens the next stage, in a program that keeps NCHW fp32 outside
        {"name": "conv_pipeline_32x56x56x128_s2", "family": "conv_pipeline", "n": 32, "hw": 56, "C": 128, "Ko": 128, "ker": 3,
         "stride": 2, "dt": "bf16"},
        # training: both gradients of the 28 x 28 stage's convolution
        {"name": "conv_backward_32x28x28x128", "family": "conv_backward", "n": 32, "hw": 28, "C": 128, "Ko": 128, "ker": 3,
         "stride": 1, "dt": "bf16"},
    ]


# ---- drawn cases ---------------------------------------------------------------------------------------------------
LARGEST_FLOPS = 2.0 * 4096 ** 3


def _log(rng, lo, hi, step=1):
    """A whole number in lo..hi, even over the logarithm, a multiple of `step`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi // step * step, max(-(-lo // step) * step, int(round(v / step)) * step))


def draw(rng):
    while True:
        case = _draw(rng, rng.choice(("tiny", "decode", "ragged", "linear", "weight_grad", "deep_k", "batched", "grouped",
                                      "grouped_decode", "conv", "conv_pipeline", "conv_backward")))
        w = work(case)
        if w["flops"] <= LARGEST_FLOPS and w["bytes"] <= 290e6:
            return case


def _draw(rng, family):
    c = {"family": family, "dt": rng.choice(("bf16", "f16"))}
    if family == "tiny":
        c.update(M=_log(rng, 64, 512), N=_log(rng, 64, 512, 8), K=_log(rng, 64, 512, 8))
    elif family == "decode":
        c.update(M=_log(rng, 1, 64), N=_log(rng, 1024, 16384, 8), K=_log(rng, 1024, 8192, 64), act=rng.choice(("none", "silu", "gelu_tanh")),
                 dt=rng.choice(("bf16", "f16", "e4m3")))
    elif family == "ragged":
        c.update(M=_log(rng, 200, 4000), N=_log(rng, 200, 4000), K=_log(rng, 256, 4096, 8))
    elif family == "linear":
        c.update(M=_log(rng, 512, 8192), N=_log(rng, 512, 8192, 8), K=_log(rng, 512, 8192, 16), dt=rng.choice(("bf16", "f16", "e4m3", "e5m2")))
    elif family == "weight_grad":
        c.update(M=_log(rng, 512, 4096, 8), N=_log(rng, 512, 4096, 8), K=_log(rng, 512, 16384))
    elif family == "deep_k":
        c.update(M=_log(rng, 32, 512), N=_log(rng, 32, 512), K=_log(rng, 4096, 65536, 8))
    elif family == "batched":
        c.update(batch=_log(rng, 4, 128), M=_log(rng, 64, 1024), N=_log(rng, 64, 1024), K=rng.choice((32, 64, 80, 96, 128, 256)),
                 out=rng.choice(("f32", "same")))
    elif family == "grouped":
        c.update(groups=_log(rng, 4, 32), rows="prefill", mix=rng.randrange(1 << 16), N=_log(rng, 512, 4096, 8), K=_log(rng, 512, 4096, 64))
    elif family == "grouped_decode":
        c.update(groups=_log(rng, 8, 128), rows="decode", mix=rng.randrange(1 << 16), N=_log(rng, 512, 4096, 8), K=_log(rng, 512, 4096, 64),
                 dt=rng.choice(("bf16", "e4m3")))
    else:
        hw, width = rng.choice(((56, 64), (28, 128), (14, 256), (7, 512)))
        # (network inputs other than 224 x 224 give other, odd, map sizes)
        hw = max(7, hw + rng.choice((0, 0, -3, 1, 4)))
        c.update(n=_log(rng, 1, 48), hw=hw, C=rng.choice((width // 2, width, width)), Ko=rng.choice((width, width, 2 * width)))
        if family != "conv":
            c.update(ker=rng.choice((1, 3, 3)), stride=rng.choice((1, 2)))
    return c


def group_rows(case):
    """Rows of each group, from the case alone: 128 + 64 j (prefill) or 0..32 with every eighth expert unused (decode)."""
    x, rows = case["mix"] * 2654435761 % (1 << 32), []
    for g in range(case["groups"]):
        x = (x * 1664525 + 1013904223) % (1 << 32)
        if case["rows"] == "prefill":
            rows.append(128 + 64 * ((x >> 16) % 31))
        else:
            rows.append(0 if g % 8 == 5 else (x >> 16) % 33)
    if not sum(rows):
        rows[0] = 1
    return rows


# ---- sizes ---------------------------------------------------------------------------------------------------------
def _conv_geom(c):
    ker, stride = c.get("ker", 3), c.get("stride", 1)
    pad = ker // 2
    return ker, stride, pad, (c["hw"] + 2 * pad - ker) // stride + 1


def work(case):
    f, e = case["family"], SIZE[case["dt"]]
    if f in ("tiny", "decode", "ragged", "linear", "weight_grad", "deep_k", "batched"):
        b, M, N, K = case.get("batch", 1), case["M"], case["N"], case["K"]
        out = 4 if f == "weight_grad" or case.get("out") == "f32" else 2
        extra = {"ragged": N * 2 + M * N * 2, "weight_grad": 0, "batched": 0}.get(f, N * 2)
        return {"bytes": b * ((M + N) * K * e + M * N * out) + extra, "flops": 2.0 * b * M * N * K}
    if f in ("grouped", "grouped_decode"):
        rows, N, K = group_rows(case), case["N"], case["K"]
        used = sum(1 for r in rows if r)
        return {"bytes": sum(rows) * K * e + used * N * K * e + sum(rows) * N * 2, "flops": 2.0 * sum(rows) * N * K}
    ker, _, _, P = _conv_geom(case)
    n, hw, C, Ko = case["n"], case["hw"], case["C"], case["Ko"]
    n_x, n_y, n_w = n * hw * hw * C, n * P * P * Ko, Ko * ker * ker * C
    flops = 2.0 * n_y * ker * ker * C
    if f == "conv":
        return {"bytes": 2 * (n_x + n_w + Ko + 2 * n_y), "flops": flops}
    if f == "conv_pipeline":      # the fp32 input read and the fp32 output written; what passes between is the program's own
        return {"bytes": 4 * n_x + 2 * n_w + 2 * Ko + 4 * n_y, "flops": flops}
    return {"bytes": 2 * (n_y + n_w + n_x) + 2 * n_x + 4 * n_w, "flops": 2 * flops}


def tolerance(case):
    """About four times the distance of one correct result from the 64-bit one, measured over listed and drawn cases: the
    rounding of the stored type, or for fp32 outputs the sums'."""
    f = case["family"]
    out = "f32" if f == "weight_grad" or case.get("out") == "f32" else "f16" if case["dt"] == "f16" else "bf16"
    if f == "conv_backward":
        out = "f16" if case["dt"] == "f16" else "bf16"
    if out == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 7e-3, "max": 1.6e-2} if out == "bf16" else {"rel": 9e-4, "max": 2e-3}


# ---- inputs --------------------------------------------------------------------------------------------------------
class _Rng:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, shape, dt, scale=1.0):
        x = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)
        return (x * scale).to(TORCH[dt])


def _aux(dt):
    """Type of biases, residuals and outputs beside operands of type dt."""
    return "f16" if dt == "f16" else "bf16"


def _inputs(case, seed):
    r, f, dt = _Rng(seed), case["family"], case["dt"]
    if f in ("tiny", "decode", "ragged", "linear", "deep_k", "weight_grad", "batched"):
        b, M, N, K = case.get("batch", 1), case["M"], case["N"], case["K"]
        s = K ** -0.25
        lead = (b,) if f == "batched" else ()
        a = r.normal(lead + ((K, M) if f == "weight_grad" else (M, K)), dt, s)
        w = r.normal(lead + ((K, N) if f in ("tiny", "weight_grad") else (N, K)), dt, s)
        i = {"a": a, "w": w}
        if f not in ("weight_grad", "batched"):
            i["bias"] = r.normal((N,), _aux(dt), 0.5)
        if f == "ragged":
            i["res"] = r.normal((M, N), _aux(dt))
        return i
    if f in ("grouped", "grouped_decode"):
        rows, N, K = group_rows(case), case["N"], case["K"]
        s = K ** -0.25
        return {"a": r.normal((sum(rows), K), dt, s), "w": r.normal((case["groups"], N, K), dt, s)}
    ker, _, _, P = _conv_geom(case)
    n, hw, C, Ko = case["n"], case["hw"], case["C"], case["Ko"]
    s = (ker * ker * C) ** -0.25
    w = r.normal((Ko, ker, ker, C), dt, s)
    if f == "conv":
        return {"x": r.normal((n, hw, hw, C), dt, s), "w": w, "bias": r.normal((Ko,), dt, 0.5), "res": r.normal((n, P, P, Ko), dt)}
    if f == "conv_pipeline":
        return {"x": r.normal((n, C, hw, hw), "f32", s), "w": w, "bias": r.normal((Ko,), dt, 0.5)}
    # gradients arrive small: the loss is averaged over the batch
    return {"x": r.normal((n, hw, hw, C), dt, 1.0), "w": w, "dy": r.normal((n, P, P, Ko), dt, (n * P * P) ** -0.5)}


def prepare(case, seed):
    s = dict(case)
    s.update(_inputs(case, seed))
    f, dt = case["family"], case["dt"]
    aux = _aux(dt)
    new = lambda shape, d: torch.empty(shape, dtype=TORCH[d], device="cuda")  # noqa: E731
    ptr = lambda k: s[k].data_ptr()  # noqa: E731
    s["stream"] = torch.cuda.current_stream().cuda_stream
    if f in ("tiny", "decode", "ragged", "linear", "deep_k"):
        M, N, K = case["M"], case["N"], case["K"]
        s["out"] = new((M, N), aux)
        steps = [("bias", ptr("bias"), aux)]
        if f == "ragged":
            steps.append(("aux_load", ptr("res"), aux, N, 0, 1.0))
        act = {"linear": "gelu_tanh", "decode": case.get("act")}.get(f, "relu")
        s["epi"] = ucl.Epilogue(steps + ([(act,)] if act != "none" else []))
        if f == "deep_k":
            s["tune"] = _split_tuning(s, "gemm", dt, aux, M=M, N=N, K=K)
    elif f == "weight_grad":
        s["out_t"] = new((case["M"], case["N"]), "f32")
    elif f == "batched":
        s["out_dt"] = "f32" if case["out"] == "f32" else dt
        s["out_t"] = new((case["batch"], case["M"], case["N"]), s["out_dt"])
        s["epi"] = ucl.Epilogue([("scale", case["K"] ** -0.5)])
    elif f in ("grouped", "grouped_decode"):
        rows, N, K = group_rows(case), case["N"], case["K"]
        s["M_g"], s["out"] = rows, new((sum(rows), N), aux)
        first, at = [], 0
        for m in rows:
            first.append(at)
            at += m
        table = lambda v: torch.tensor(v, dtype=torch.int64, device="cuda")  # noqa: E731
        s["tab_a"] = table([ptr("a") + o * K * SIZE[dt] for o in first])
        s["tab_w"] = table([ptr("w") + g * N * K * SIZE[dt] for g in range(case["groups"])])
        s["tab_d"] = table([ptr("out") + o * N * 2 for o in first])
        s["epi"] = ucl.Epilogue([("silu",)])
    else:
        ker, stride, pad, P = _conv_geom(case)
        n, hw, C, Ko = case["n"], case["hw"], case["C"], case["Ko"]
        s["geom"] = (n, hw, hw, C, Ko, ker, ker, pad, pad, stride, stride, 1, 1)
        if f == "conv":
            s["out"] = new((n, P, P, Ko), dt)
            s["epi"] = ucl.Epilogue([("bias", ptr("bias"), dt), ("aux_load", ptr("res"), dt, Ko, 0, 1.0), ("relu",)])
        elif f == "conv_pipeline":
            s["P"] = P
            s["x_nhwc"], s["y_nhwc"] = new((n, hw, hw, C), dt), new((n, P, P, Ko), dt)
            s["out"] = new((n, Ko, P, P), "f32")
            s["epi"] = ucl.Epilogue([("bias", ptr("bias"), dt), ("relu",)])
        else:
            s["dx"], s["dw"] = new((n, hw, hw, C), dt), new((Ko, ker, ker, C), "f32")
            s["tune"] = _split_tuning(s, "conv2d_wgrad", dt, "f32", conv=s["geom"])
    return s


def _split_tuning(s, op, dt_in, dt_out, **problem):
    """Parallel split-K with the library's own choice of slices, in a workspace that the program keeps."""
    nbytes, _ = ucl.ucl_workspace_size(op, dt_in, dt_out, tune=ucl.Tuning(split_k="parallel"), **problem)
    nbytes = max(nbytes, 1 << 16)
    s["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    ucl.ucl_workspace_init(s["workspace"].data_ptr(), nbytes, s["stream"])
    return ucl.Tuning(split_k="parallel", workspace=s["workspace"].data_ptr(), workspace_bytes=nbytes)


# ---- one pass ------------------------------------------------------------------------------------------------------
def run(s):
    f, dt, st = s["family"], s["dt"], torch.cuda.current_stream().cuda_stream
    aux = _aux(dt)
    if f in ("tiny", "decode", "ragged", "linear", "deep_k"):
        M, N, K = s["M"], s["N"], s["K"]
        w_rs, w_cs = (N, 1) if f == "tiny" else (1, K)
        ucl.ucl_gemm(M, N, K, s["a"].data_ptr(), dt, K, 1, s["w"].data_ptr(), dt, w_rs, w_cs, s["out"].data_ptr(), aux, N, 1,
                     s["epi"], s.get("tune"), st)
        return s["out"]
    if f == "weight_grad":        # dW[m, n] = sum over tokens of dY[k, m] X[k, n]
        M, N, K = s["M"], s["N"], s["K"]
        ucl.ucl_gemm(M, N, K, s["a"].data_ptr(), dt, 1, M, s["w"].data_ptr(), dt, N, 1, s["out_t"].data_ptr(), "f32", N, 1,
                     None, None, st)
        return s["out_t"]
    if f == "batched":
        M, N, K = s["M"], s["N"], s["K"]
        ucl.ucl_batched_gemm(s["batch"], M, N, K, s["a"].data_ptr(), dt, K, 1, M * K, s["w"].data_ptr(), dt, 1, K, N * K,
                             s["out_t"].data_ptr(), s["out_dt"], N, 1, M * N, s["epi"], None, st)
        return s["out_t"]
    if f in ("grouped", "grouped_decode"):
        N, K = s["N"], s["K"]
        ucl.ucl_grouped_gemm(s["M_g"], N, K, s["tab_a"].data_ptr(), dt, K, 1, s["tab_w"].data_ptr(), dt, 1, K,
                             s["tab_d"].data_ptr(), aux, N, 1, s["epi"], None, st)
        return s["out"]
    if f == "conv":
        ucl.ucl_conv2d_fprop(*s["geom"], s["x"].data_ptr(), dt, s["w"].data_ptr(), dt, s["out"].data_ptr(), dt, s["epi"], None, st)
        return s["out"]
    if f == "conv_pipeline":
        n, hw, C, Ko, P = s["n"], s["hw"], s["C"], s["Ko"], s["P"]
        ucl.ucl_transpose(n, C, hw * hw, s["x"].data_ptr(), "f32", s["x_nhwc"].data_ptr(), dt, st)
        ucl.ucl_conv2d_fprop(*s["geom"], s["x_nhwc"].data_ptr(), dt, s["w"].data_ptr(), dt, s["y_nhwc"].data_ptr(), dt, s["epi"], None, st)
        ucl.ucl_transpose(n, P * P, Ko, s["y_nhwc"].data_ptr(), dt, s["out"].data_ptr(), "f32", st)
        return s["out"]
    ucl.ucl_conv2d_dgrad(*s["geom"], s["dy"].data_ptr(), dt, s["w"].data_ptr(), dt, s["dx"].data_ptr(), dt, None, None, st)
    ucl.ucl_conv2d_wgrad(*s["geom"], s["dy"].data_ptr(), dt, s["x"].data_ptr(), dt, s["dw"].data_ptr(), "f32", None, s["tune"], st)
    return {"dx": s["dx"], "dw": s["dw"]}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------
def _f64(x):
    return x.float().double()


def _act64(name, v):
    return {"none": lambda t: t, "relu": torch.relu, "silu": F.silu, "gelu_tanh": lambda t: F.gelu(t, approximate="tanh")}[name](v)


def _taps(x, ker, stride, pad, P):
    """(r, s, the pixels that tap reads as an [n*P*P, C] matrix) of an NHWC tensor."""
    xp = F.pad(x, (0, 0, pad, pad, pad, pad))
    for r in range(ker):
        for t in range(ker):
            v = xp[:, r:r + (P - 1) * stride + 1:stride, t:t + (P - 1) * stride + 1:stride, :]
            yield r, t, v.reshape(-1, x.shape[-1])


def exact(case, seed):
    i, f = _inputs(case, seed), case["family"]
    if f in ("tiny", "decode", "ragged", "linear", "deep_k"):
        w = _f64(i["w"])
        v = _f64(i["a"]) @ (w if f == "tiny" else w.t().contiguous()) + _f64(i["bias"])
        if f == "ragged":
            v = v + _f64(i["res"])
        return _act64({"linear": "gelu_tanh", "decode": case.get("act")}.get(f, "relu"), v)
    if f == "weight_grad":
        return _f64(i["a"]).t().contiguous() @ _f64(i["w"])
    if f == "batched":
        scale = float(torch.tensor(case["K"] ** -0.5, dtype=torch.float32))
        return torch.stack([_f64(a) @ _f64(w).t().contiguous() * scale for a, w in zip(i["a"], i["w"])])
    if f in ("grouped", "grouped_decode"):
        parts, at = [], 0
        for g, m in enumerate(group_rows(case)):
            parts.append(F.silu(_f64(i["a"][at:at + m]) @ _f64(i["w"][g]).t().contiguous()))
            at += m
        return torch.cat(parts)
    ker, stride, pad, P = _conv_geom(case)
    n, hw, C, Ko = case["n"], case["hw"], case["C"], case["Ko"]
    w = _f64(i["w"])
    if f in ("conv", "conv_pipeline"):
        x = _f64(i["x"]) if f == "conv" else _f64(i["x"].to(TORCH[case["dt"]])).permute(0, 2, 3, 1).contiguous()
        v = torch.zeros(n * P * P, Ko, dtype=torch.float64, device="cuda")
        for r, t, px in _taps(x, ker, stride, pad, P):
            v += px @ w[:, r, t, :].t().contiguous()
        v += _f64(i["bias"])
        if f == "conv":
            return torch.relu(v.view(n, P, P, Ko) + _f64(i["res"]))
        return torch.relu(v).view(n, P * P, Ko).transpose(1, 2).reshape(n, Ko, P, P)
    dy, x = _f64(i["dy"]), _f64(i["x"])
    dy2 = dy.view(-1, Ko)
    dw = torch.empty(Ko, ker, ker, C, dtype=torch.float64, device="cuda")
    for r, t, px in _taps(x, ker, stride, pad, P):
        dw[:, r, t, :] = dy2.t().contiguous() @ px
    dxp = torch.zeros(n, hw + 2 * pad, hw + 2 * pad, C, dtype=torch.float64, device="cuda")
    for r in range(ker):
        for t in range(ker):
            dxp[:, r:r + (P - 1) * stride + 1:stride, t:t + (P - 1) * stride + 1:stride, :] += (dy2 @ w[:, r, t, :].contiguous()).view(n, P, P, C)
    return {"dx": dxp[:, pad:pad + hw, pad:pad + hw, :].contiguous(), "dw": dw}
