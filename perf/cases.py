"""What the speed of this library is judged by: the calls a program makes that trains or evaluates
linear layers in FP4, through ``paper_2505_19115_amd.binding``.

Kinds of case
  eval      Eq. 4 alone on weights that were quantized once (``linear_fwd`` with ``w_operands``) or,
            with ``weights = "tensor"``, on the weight tensor itself.
  train     one linear layer of a training step, forward and backward (Eqs. 4-6).
            hand_over "saved":  the forward call leaves the transposed operands for the backward call;
            hand_over "scales": only the tensor scales are handed over, X and W are quantized again;
            hand_over "reuse":  as "saved", with W's operands written once per optimizer step.
  mlp       the three linear layers of a SwiGLU MLP, each forward and backward.
  swiglu    SwiGLU backward fused with the quantizers of dG and dU, then the gate and up layers'
            backward calls on those operands.
  quantize  one tensor quantized along one axis (optionally a view with a larger row pitch).
  monitor   a gradient quantized and its quantization-noise sums taken (the noise monitor of Sec. 4).
"""
import ctypes
import math

import torch

from paper_2505_19115_amd import binding as nv

FORMATS = {
    "nvfp4": nv.NVFP4,
    "mxfp4": nv.MXFP4,
    "e4m3_32": nv.Format(32, nv.SCALE_E4M3, 1),
    "e4m3_64": nv.Format(64, nv.SCALE_E4M3, 1),
    "e4m3_128": nv.Format(128, nv.SCALE_E4M3, 1),
}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
ROUNDING = {"rtn": nv.RTN, "sr": nv.SR}


def listed():
    return [
        # the smallest training call: a layer of a test-sized network, where launches and host work are everything
        dict(name="train_tiny", kind="train", M=64, N=256, K=128, fmt="nvfp4", dtype="f32", out="f32", hand_over="saved"),
        # generation with a 7B gate projection: 16 sequences, one token each, against packed weights
        dict(name="eval_decode", kind="eval", M=16, N=11008, K=4096, fmt="nvfp4", dtype="bf16", out="bf16", weights="packed"),
        # the same for the down projection in MXFP4, with a batch of 64
        dict(name="eval_decode_mx", kind="eval", M=64, N=4096, K=11008, fmt="mxfp4", dtype="bf16", out="bf16", weights="packed"),
        # a prompt of odd length through the 7B QKV projection
        dict(name="eval_prompt", kind="eval", M=777, N=12288, K=4096, fmt="nvfp4", dtype="bf16", out="bf16", weights="packed"),
        # the 7B attention output projection on one sequence of 2048 tokens
        dict(name="train_out", kind="train", M=2048, N=4096, K=4096, fmt="nvfp4", dtype="bf16", out="bf16", hand_over="saved"),
        # sizes that are multiples of 32 and of nothing larger, binary32 in and out, no saved operands
        dict(name="train_ragged", kind="train", M=1056, N=2080, K=2784, fmt="nvfp4", dtype="f32", out="f32", hand_over="scales"),
        # block-size study (Sec. 3.1): the 7B down projection with E4M3 scales per 64 elements
        dict(name="train_block64", kind="train", M=4096, N=4096, K=11008, fmt="e4m3_64", dtype="bf16", out="bf16", hand_over="scales"),
        # the 7B MLP's three linear layers at 4096 tokens, the benchmark's workload
        dict(name="mlp_nvfp4", kind="mlp", M=4096, D=4096, F=11008, fmt="nvfp4", dtype="bf16", out="bf16", hand_over="saved"),
        # the same in MXFP4, for a later micro-batch of the optimizer step
        dict(name="mlp_mxfp4", kind="mlp", M=4096, D=4096, F=11008, fmt="mxfp4", dtype="bf16", out="bf16", hand_over="reuse"),
        # the backward half of that MLP from the down layer's input gradient on, at 2048 tokens
        dict(name="swiglu_bwd", kind="swiglu", M=2048, D=4096, F=11008, fmt="nvfp4", dtype="bf16", out="bf16"),
        # a weight-gradient-sized tensor quantized down its columns, stochastic rounding, rows of a wider buffer
        dict(name="quantize_cols", kind="quantize", rows=8192, cols=8192, pad=64, axis=0, rounding="sr", fmt="nvfp4", dtype="bf16"),
        # the noise monitor on an output gradient of the 7B MLP
        dict(name="monitor", kind="monitor", rows=4096, cols=11008, axis=1, rounding="sr", fmt="nvfp4", dtype="bf16"),
    ]


def _size(rng, lo, hi, step=1):
    """Log-uniform between lo and hi, a multiple of step."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(step, int(round(v / step)) * step)


MOST_PRODUCTS = 3 * 4096 * 4096 * 11008  # multiply-adds of each of Eqs. 4-6 in the largest listed case


def draw(rng):
    kind = rng.choice(["eval", "eval", "train", "train", "train", "mlp", "swiglu", "quantize", "monitor"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    out = rng.choice(["bf16", "bf16", "f32"])
    while True:
        if kind == "eval":
            fmt = rng.choice(["nvfp4", "nvfp4", "mxfp4"])
            c = dict(kind=kind, M=_size(rng, 1, 4096), N=_size(rng, 256, 12288, 32), K=_size(rng, 256, 12288, 32), fmt=fmt,
                     dtype=dtype, out=out, weights=rng.choice(["packed", "packed", "packed", "tensor"]))
            products = c["M"] * c["N"] * c["K"]
        elif kind == "train":
            fmt = rng.choice(["nvfp4", "nvfp4", "nvfp4", "mxfp4", "mxfp4", "e4m3_32", "e4m3_64", "e4m3_128"])
            step = max(32, FORMATS[fmt].block)
            c = dict(kind=kind, M=_size(rng, 64, 8192, step), N=_size(rng, 128, 12288, step), K=_size(rng, 128, 12288, step), fmt=fmt,
                     dtype=dtype, out=out, hand_over=rng.choice(["saved", "saved", "reuse", "scales"]))
            products = c["M"] * c["N"] * c["K"]
        elif kind in ("mlp", "swiglu"):
            fmt = rng.choice(["nvfp4", "nvfp4", "mxfp4"])
            step = rng.choice([32, 128])
            c = dict(kind=kind, M=_size(rng, 128, 4096, step), D=_size(rng, 256, 4096, step), F=_size(rng, 512, 11008, step), fmt=fmt,
                     dtype=dtype, out=out)
            if kind == "mlp":
                c["hand_over"] = rng.choice(["saved", "reuse"])
            products = 3 * c["M"] * c["D"] * c["F"]
        else:
            fmt = rng.choice(["nvfp4", "nvfp4", "mxfp4", "e4m3_32", "e4m3_64", "e4m3_128"])
            b = FORMATS[fmt].block
            axis = rng.choice([0, 1])
            c = dict(kind=kind, rows=_size(rng, 128, 16384, b if axis == 0 else 1), cols=_size(rng, 128, 16384, b if axis == 1 else 1),
                     axis=axis, rounding=rng.choice(["rtn", "sr"]), fmt=fmt, dtype=dtype)
            if kind == "quantize":
                c["pad"] = rng.choice([0, 0, 64])
            products = 0 if c["rows"] * c["cols"] <= 8192 * 8192 else MOST_PRODUCTS + 1
        if products <= MOST_PRODUCTS:
            return c


# ---- inputs: activations N(0, 1), weights N(0, 0.02), output gradients N(0, 1e-3) with 0.05 % of entries 50 times larger

def _normal(g, rows, cols, std, dtype, pitch=None):
    pitch = cols if pitch is None else pitch
    return torch.randn((rows, pitch), generator=g, device="cuda").mul_(std).to(dtype)[:, :cols]


def _gradient(g, rows, cols, dtype, pitch=None):
    pitch = cols if pitch is None else pitch
    x = torch.randn((rows, pitch), generator=g, device="cuda").mul_(1e-3)
    x.mul_(torch.rand((rows, pitch), generator=g, device="cuda").lt_(5e-4).mul_(49.0).add_(1.0))
    return x.to(dtype)[:, :cols]


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def _layer(g, M, N, K, case, seed):
    """Tensors and kept buffers of one linear layer of a training program."""
    fmt, dtype, out = FORMATS[case["fmt"]], DTYPES[case["dtype"]], DTYPES[case["out"]]
    f = fmt.c()
    L = dict(M=M, N=N, K=K, fmt=fmt, seed=seed, hand_over=case["hand_over"],
             X=_normal(g, M, K, 1.0, dtype), W=_normal(g, N, K, 0.02, dtype), dY=_gradient(g, M, N, dtype),
             Y=torch.empty((M, N), dtype=out, device="cuda"), dX=torch.empty((M, K), dtype=out, device="cuda"),
             dW=torch.empty((N, K), dtype=out, device="cuda"),
             wf=_bytes(nv.lib.nvfp4_linear_fwd_workspace_bytes(M, N, K, ctypes.byref(f))),
             wb=_bytes(nv.lib.nvfp4_linear_bwd_workspace_bytes(M, N, K, ctypes.byref(f))))
    if L["hand_over"] == "scales":
        L["scales"] = torch.empty(2, dtype=torch.float32, device="cuda")
    else:
        L["saved"] = _bytes(nv.linear_saved_bytes(M, N, K, fmt))
    if L["hand_over"] == "reuse":
        L["w_operands"] = nv.quantize_weight(L["W"], M, fmt)
    return L


def _layer_step(L):
    if L["hand_over"] == "scales":
        nv.linear_fwd(L["X"], L["W"], L["fmt"], workspace=L["wf"], out=L["Y"], scales_out=L["scales"])
        nv.linear_bwd(L["dY"], L["X"], L["W"], L["seed"], L["fmt"], workspace=L["wb"], out=(L["dX"], L["dW"]), xw_scales=L["scales"])
    elif L["hand_over"] == "saved":
        nv.linear_fwd(L["X"], L["W"], L["fmt"], workspace=L["wf"], out=L["Y"], saved=L["saved"], bwd_seed=L["seed"])
        nv.linear_bwd(L["dY"], None, None, L["seed"], L["fmt"], workspace=L["wb"], out=(L["dX"], L["dW"]), saved=L["saved"], K=L["K"])
    else:
        nv.linear_fwd(L["X"], None, L["fmt"], workspace=L["wf"], out=L["Y"], saved=L["saved"], bwd_seed=L["seed"],
                      w_operands=L["w_operands"], N=L["N"])
        nv.linear_bwd(L["dY"], None, None, L["seed"], L["fmt"], workspace=L["wb"], out=(L["dX"], L["dW"]), saved=L["saved"],
                      K=L["K"], w_operands=L["w_operands"])
    return L["Y"], L["dX"], L["dW"]


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind, fmt, dtype = case["kind"], FORMATS[case["fmt"]], DTYPES[case["dtype"]]
    S = dict(case=case, fmt=fmt, seed=seed)
    if kind == "eval":
        M, N, K = case["M"], case["N"], case["K"]
        S.update(X=_normal(g, M, K, 1.0, dtype), W=_normal(g, N, K, 0.02, dtype), out=DTYPES[case["out"]])
        if case["weights"] == "packed":
            S["w_operands"] = nv.quantize_weight(S.pop("W"), M, fmt)
    elif kind == "train":
        S["layers"] = [_layer(g, case["M"], case["N"], case["K"], case, seed)]
    elif kind == "mlp":
        M, D, F = case["M"], case["D"], case["F"]
        S["layers"] = [_layer(g, M, N, K, case, seed + 3 * i) for i, (N, K) in enumerate(((F, D), (F, D), (D, F)))]
    elif kind == "swiglu":
        M, D, F = case["M"], case["D"], case["F"]
        f = fmt.c()
        S.update(dH=_gradient(g, M, F, dtype), G=_normal(g, M, F, 1.0, dtype), U=_normal(g, M, F, 1.0, dtype))
        S["store"] = (torch.empty_like(S["dH"]), torch.empty_like(S["dH"]))
        takes = [bool(nv.lib.nvfp4_gemm_takes_slabs(*s, ctypes.byref(f))) for s in ((M, D, F), (F, D, M))]
        slabs = dict(slab_rows=takes[0] and F % 128 == 0, slab_cols=takes[1] and M % 128 == 0)
        S["operands"] = tuple(nv.empty_dual_operands(M, F, fmt, **slabs) for _ in range(2))
        S["workspace"] = _bytes(nv.lib.nvfp4_linear_bwd_workspace_bytes(M, F, D, ctypes.byref(f)))
        S["saved"], S["grads"] = [], []
        X = _normal(g, M, D, 1.0, dtype)
        for i in range(2):  # the forward calls of the gate and up layers, whose saved operands the backward calls read
            saved = _bytes(nv.linear_saved_bytes(M, F, D, fmt))
            nv.linear_fwd(X, _normal(g, F, D, 0.02, dtype), fmt, out_dtype=dtype, saved=saved, bwd_seed=seed + 3 * i)
            S["saved"].append(saved)
            S["grads"].append((torch.empty((M, D), dtype=DTYPES[case["out"]], device="cuda"), torch.empty((F, D), dtype=DTYPES[case["out"]], device="cuda")))
    else:
        rows, cols = case["rows"], case["cols"]
        pitch = -(-cols // 8) * 8 + case.get("pad", 0)
        S["x"] = _gradient(g, rows, cols, dtype, pitch)
    return S


def run(S):
    case, fmt, seed = S["case"], S["fmt"], S["seed"]
    kind = case["kind"]
    if kind == "eval":
        if case["weights"] == "packed":
            return nv.linear_fwd(S["X"], None, fmt, out_dtype=S["out"], w_operands=S["w_operands"], N=case["N"])
        return nv.linear_fwd(S["X"], S["W"], fmt, out_dtype=S["out"])
    if kind in ("train", "mlp"):
        return [_layer_step(L) for L in S["layers"]]
    if kind == "swiglu":
        M, D, F = case["M"], case["D"], case["F"]
        both = nv.swiglu_bwd_quantize(S["dH"], S["G"], S["U"], seed, seed + 3, fmt, out=S["operands"], store=S["store"])
        grads = [nv.linear_bwd_dyq(q, None, None, seed + 3 * i, M, F, D, fmt, in_dtype=S["dH"].dtype, workspace=S["workspace"],
                                   out=S["grads"][i], saved=S["saved"][i]) for i, q in enumerate(both)]
        return list(S["store"]), grads
    q = nv.quantize(S["x"], case["axis"], ROUNDING[case["rounding"]], seed, fmt)
    if kind == "quantize":
        return q
    return q, nv.quant_noise(S["x"], q, case["axis"], fmt)


def work(case):
    b = FORMATS[case["fmt"]].block
    e = 2 if case["dtype"] == "bf16" else 4
    kind = case["kind"]
    packed = 0.5 + 1.0 / b  # bytes per element of a quantized tensor
    if kind in ("quantize", "monitor"):
        return {"bytes": case["rows"] * case["cols"] * (e + packed), "flops": 0}
    o = 2 if case["out"] == "bf16" else 4
    M = case["M"]
    if kind == "eval":
        N, K = case["N"], case["K"]
        return {"bytes": M * K * e + N * K * (packed if case["weights"] == "packed" else e) + M * N * o, "flops": 2 * M * N * K}
    if kind == "swiglu":
        D, F = case["D"], case["F"]
        return {"bytes": M * F * 5 * e + 2 * ((M + F) * D * packed + (M + F) * D * o), "flops": 8 * M * D * F}
    shapes = [(case["N"], case["K"])] if kind == "train" else [(case["F"], case["D"])] * 2 + [(case["D"], case["F"])]
    total = flops = 0
    for N, K in shapes:
        w = 2 * packed if case["hand_over"] == "reuse" else e  # W itself, or its two packed operands
        total += M * K * e + N * K * w + M * N * e + (M * N + M * K + N * K) * o
        flops += 6 * M * N * K
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"
    # measured against binary64 at 128 to 11008 summands, times four
    if case["kind"] == "monitor":
        return {"rel": 1e-7}  # codes exact; squares summed in binary32 over 8 elements, above that in binary64
    if case["out"] == "f32":
        return {"rel": 3e-7, "max": 3e-6}  # exact products summed in binary32
    return {"rel": 1e-4, "max": 1e-2}  # the same sums, a few of which round to the other bf16 neighbour
