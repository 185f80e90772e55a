"""The work that users of the library have it do, as cases that can be timed and compared.

Every case goes through the public entry points (the names of include/tweo.h, by way of the
package's binding) on inputs made from a seed.  Families, each over the range of sizes that the
package's own workloads (`synth.CONFIGS`), tests and benchmark span:

  train     one linear layer of a training step: forward from bf16 operands with the TWEO penalty,
            then backward; current or delayed scaling, E4M3 or E5M2 gradients, with and without the
            residual stream and the penalty's gradient
  block     the linear layers of a Transformer block: all forwards, then all backwards in reverse
  layernorm residual add + LayerNorm + per-tensor cast in front of the next linear
  infer     FP8 linear on quantised weights: amax and cast of the activation, then the GEMM
  w8a8      INT8 linear: quantise the activation (static per-tensor or per token), then the GEMM
"""
import math

import torch

import paper_2511_23225_amd as tw

DEV = "cuda:0"
PEN = (3.0, 1e-6, 4)  # tau, eps, p: the paper's setting in every experiment


def listed():
    return [
        # The smallest training call, the one the smoke run and the parity tests use: a 512-wide
        # layer over 256 tokens.  Latency and the number of launches decide.
        dict(name="train-256x512x512", family="train", M=256, K=512, N=512, outliers="sparse", top=1e4, penalty=True,
             residual=False, inject=False, scaling="current", dy="e4m3"),
        # A GPT-2-small block (qkv, proj, fc1, fc2; 8192 tokens), forward and backward: a whole call
        # made of many middling launches.
        dict(name="block-gpt2-8192", family="block", tokens=8192, width=768, outliers="sparse", top=5e3),
        # The first MLP projection of a ViT-B/16 block, 256 images of 197 tokens (not a multiple of a
        # GEMM tile), channel outliers.
        dict(name="train-vit-fc1", family="train", M=50432, K=768, N=3072, outliers="channel", top=2e3, penalty=True,
             residual=False, inject=False, scaling="current", dy="e4m3"),
        # The last linear of the same block as the TWEO loss uses it: the output with the residual
        # stream added is what is penalised, and the penalty's gradient joins the incoming one.
        dict(name="train-vit-fc2-tweo", family="train", M=50432, K=3072, N=768, outliers="none", top=20.0, penalty=True,
             residual=True, inject=True, scaling="current", dy="e4m3"),
        # The widest projection of a LLaMA-1B block over 16384 tokens, current scaling: the largest
        # GEMMs of the package's benchmark.
        dict(name="train-llama-qkv", family="train", M=16384, K=2048, N=6144, outliers="sparse", top=1e4, penalty=True,
             residual=False, inject=False, scaling="current", dy="e4m3"),
        # The down projection of the same block under the recipe the paper trained with: delayed
        # scaling (history of 16), E5M2 gradients, residual stream.
        dict(name="train-llama-down-delayed", family="train", M=16384, K=5632, N=2048, outliers="none", top=20.0,
             penalty=True, residual=True, inject=False, scaling="delayed", dy="e5m2"),
        # Residual add + LayerNorm + cast of a LLaMA-1B-wide stream, in front of the block's linears.
        dict(name="layernorm-16384x2048", family="layernorm", rows=16384, cols=2048, residual=True, delayed=False),
        # Evaluation on a batch of whole sequences, whose token count fits no tile: amax, cast and
        # the gate projection of a LLaMA-1B block on weights quantised once.
        dict(name="infer-12345x2048x5632", family="infer", M=12345, K=2048, N=5632),
        # W8A8 at the 7B shapes.  Decoding one sequence: the weight stream.
        dict(name="w8a8-decode-1", family="w8a8", M=1, K=4096, N=12288, steps="tensor"),
        # Decoding a batch of 64 with per-token activations and per-channel weights.
        dict(name="w8a8-decode-64-rows", family="w8a8", M=64, K=4096, N=11008, steps="rows"),
        # A chunk of a prompt beside the decoding batch (chunked prefill), into the narrow projection.
        dict(name="w8a8-chunk-384", family="w8a8", M=384, K=11008, N=4096, steps="tensor"),
        # Prefill of 4096 tokens.
        dict(name="w8a8-prefill-4096", family="w8a8", M=4096, K=4096, N=11008, steps="tensor"),
    ]


def _log_int(rng, lo, hi, step):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(step, min(hi // step, max(1, round(v / step))) * step)


# what the largest listed case multiplies and holds
_MAX_MNK = 16384 * 2048 * 6144
_MAX_ELEMENTS = 16384 * (2048 + 6144)


def draw(rng):
    family = rng.choice(["train", "train", "train", "block", "layernorm", "infer", "w8a8", "w8a8", "w8a8"])
    if family == "train":
        while True:  # the entry points take multiples of 16 on every side
            M, K, N = _log_int(rng, 64, 50432, 16), _log_int(rng, 256, 6144, 16), _log_int(rng, 256, 6144, 16)
            if rng.random() < 0.5:
                K, N = (K + 255) // 256 * 256, (N + 255) // 256 * 256
            if M * K * N <= _MAX_MNK and M * (K + N) <= _MAX_ELEMENTS:
                break
        scaling = rng.choice(["current", "current", "delayed"])
        outliers = rng.choice(["sparse", "channel", "none"])
        residual = rng.random() < 0.3
        return dict(family="train", M=M, K=K, N=N, outliers=outliers, top={"sparse": 1e4, "channel": 2e3, "none": 20.0}[outliers],
                    penalty=rng.random() < 0.8, residual=residual, inject=residual and scaling == "current" and rng.random() < 0.5,
                    scaling=scaling, dy=rng.choice(["e4m3", "e5m2"]))
    if family == "block":
        return dict(family="block", tokens=_log_int(rng, 512, 8192, 16), width=rng.choice([512, 640, 768]),
                    outliers="sparse", top=5e3)
    if family == "layernorm":
        cols = _log_int(rng, 256, 8192, 16)
        return dict(family="layernorm", rows=_log_int(rng, 128, min(32768, (1 << 25) // cols), 16), cols=cols,
                    residual=rng.random() < 0.5, delayed=rng.random() < 0.5)
    if family == "infer":
        return dict(family="infer", M=_log_int(rng, 16, 16384, 1), K=_log_int(rng, 512, 4096, 16), N=_log_int(rng, 512, 6144, 8))
    K, N = rng.choice([(4096, 12288), (4096, 11008), (11008, 4096), (2048, 5632), (5632, 2048), (3072, 776), (1000 // 16 * 16, 3072)])
    return dict(family="w8a8", M=_log_int(rng, 1, 4096, 1), K=K, N=N, steps=rng.choice(["tensor", "tensor", "rows", "rows_i8"]))


# ------------------------------------------------------------------------------------ inputs
def _gen(seed, index):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1009 + index) & 0x7FFFFFFFFFFF)
    return g


def _normal(shape, std, seed, index):
    return (torch.randn(shape, generator=_gen(seed, index), device=DEV) * std).bfloat16()


def _activation(M, K, outliers, top, seed, index):
    """N(0,1) with the outlier statistics of synth: sparse +-U(top/10, top) in 0.01 % of the places,
    three channels times `top`, or none (clipped at `top`: a TWEO-trained model)."""
    x = torch.randn((M, K), generator=_gen(seed, index), device=DEV)
    if outliers == "sparse":
        g = _gen(seed, index + 500)
        k = max(1, round(1e-4 * M * K))
        at = torch.randint(0, M * K, (k,), generator=g, device=DEV)
        mag = torch.rand(k, generator=g, device=DEV) * (0.9 * top) + 0.1 * top
        sign = torch.randint(0, 2, (k,), generator=g, device=DEV) * 2 - 1
        # repeated places: the first value of a place wins on every run
        at, first = torch.unique(at, return_inverse=True)
        val = torch.full((at.numel(),), -1e30, device=DEV).scatter_reduce_(0, first, mag * sign, "amax")
        x.view(-1)[at] = val
    elif outliers == "channel":
        cols = torch.randperm(K, generator=_gen(seed, index + 500), device=DEV)[:3]
        x[:, cols] *= top
    else:
        x.clamp_(-top, top)
    return x.bfloat16()


def _u8(*shape):
    return torch.empty(shape, dtype=torch.uint8, device=DEV)


def _bf(*shape):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV)


def _f32(n):
    return torch.zeros(n, dtype=torch.float32, device=DEV)


def _workspace(M, N, K, *ops):
    return _u8(max(tw.tweo_workspace_bytes(op, M, N, K) for op in ops))


def _gradient_factor(M, N):
    """lambda / (L * numel) of the TWEO loss (lambda = 0.01, 12 layers)."""
    return 0.01 / (12 * M * N)


def _train_inputs(case, seed, index=0):
    M, K, N = case["M"], case["K"], case["N"]
    t = dict(x=_activation(M, K, case["outliers"], case["top"], seed, index), w=_normal((N, K), 0.02, seed, index + 1),
             dy=_normal((M, N), 1.0, seed, index + 2))
    if case["residual"]:
        t["residual"] = _normal((M, N), 1.0, seed, index + 3)
    return t


def _train_buffers(case):
    M, K, N = case["M"], case["K"], case["N"]
    s = dict(case=case, y=_bf(M, N), dx=_bf(M, K), dw=_bf(N, K), xq=_u8(M, K), xqT=_u8(K, M), wq=_u8(N, K), wqT=_u8(K, N),
             dyq=_u8(M, N), dyqT=_u8(N, M), scalars=_f32(16), penalty=torch.zeros(1, dtype=torch.float64, device=DEV),
             workspace=_workspace(M, N, K, tw.TWEO_OP_FP8_LINEAR_FWD_BF16, tw.TWEO_OP_FP8_LINEAR_BWD_BF16))
    s["saved"] = tw.make_saved(s["xq"], s["xqT"], s["wq"], s["wqT"], s["scalars"])
    return s


def _train_state(case, seed, index=0):
    s = _train_buffers(case)
    s.update(_train_inputs(case, seed, index))
    if case["scaling"] == "delayed":
        # one step on another batch has gone before: the histories hold its maxima
        words = tw.tweo_delayed_state_bytes() // 4
        s["states"] = [torch.zeros(words, dtype=torch.int32, device=DEV) for _ in range(3)]
        for st in s["states"]:
            tw.tweo_delayed_state_init(st)
        before = _train_inputs(case, seed, index + 100)
        _train_forward(s, before, True)
        _train_backward(s, before, True)
    return s


def _train_forward(s, t, bootstrap=False):
    c = s["case"]
    pen = dict(pen=PEN, penalty_sum=s["penalty"]) if c["penalty"] else {}
    if c["scaling"] == "delayed":
        tw.tweo_fp8_linear_fwd_bf16_delayed(t["x"], t["w"], s["y"], s["saved"], s["states"][0], s["states"][1],
                                            bootstrap=bootstrap, residual_bf16=t.get("residual"),
                                            workspace=s["workspace"], **pen)
    else:
        tw.tweo_fp8_linear_fwd_bf16(t["x"], t["w"], s["y"], s["saved"], residual_bf16=t.get("residual"),
                                    workspace=s["workspace"], **pen)


def _train_backward(s, t, bootstrap=False):
    c = s["case"]
    args = (s["saved"], c["K"], s["dyq"], s["dyqT"], s["dx"], s["dw"], s["workspace"])
    if c["scaling"] == "delayed":
        tw.tweo_fp8_linear_bwd_bf16_delayed(t["dy"], s["saved"], s["states"][2], c["K"], s["dyq"], s["dyqT"], s["dx"],
                                            s["dw"], s["workspace"], bootstrap=bootstrap, dy_e5m2=c["dy"] == "e5m2")
    elif c["inject"]:
        tw.tweo_fp8_linear_bwd_bf16_inject(t["dy"], s["y"], PEN, _gradient_factor(c["M"], c["N"]), *args,
                                           dy_e5m2=c["dy"] == "e5m2")
    elif c["dy"] == "e5m2":
        tw.tweo_fp8_linear_bwd_bf16_hybrid(t["dy"], *args)
    else:
        tw.tweo_fp8_linear_bwd_bf16(t["dy"], *args)


def _block_layers(case):
    M, w = case["tokens"], case["width"]
    return [dict(family="train", M=M, K=K, N=N, outliers=case["outliers"], top=case["top"], penalty=True, residual=False,
                 inject=False, scaling="current", dy="e4m3") for K, N in ((w, 3 * w), (w, w), (w, 4 * w), (4 * w, w))]


def _layernorm_inputs(case, seed, index=0):
    R, C = case["rows"], case["cols"]
    t = dict(x=_activation(R, C, "none", 20.0, seed, index),
             gamma=(1 + 0.1 * torch.randn(C, generator=_gen(seed, index + 1), device=DEV)).bfloat16(),
             beta=_normal((C,), 0.1, seed, index + 2))
    if case["residual"]:
        t["residual"] = _normal((R, C), 1.0, seed, index + 3)
    return t


def _layernorm_run(s, t, bootstrap=False):
    more = dict(residual_bf16=t["residual"], h_out_bf16=s["h"]) if s["case"]["residual"] else {}
    if s["case"]["delayed"]:
        tw.tweo_layernorm_quantize_e4m3_delayed(t["x"], t["gamma"], s["state"], s["q"], s["workspace"], bootstrap=bootstrap,
                                                beta_bf16=t["beta"], eps=1e-5, qT=s["qT"], **more)
    else:
        tw.tweo_layernorm_quantize_e4m3(t["x"], t["gamma"], s["q"], s["workspace"], beta_bf16=t["beta"], eps=1e-5,
                                        amax_out=s["amax"], qT=s["qT"], scale_out=s["scale"], scale_inv_out=s["scale_inv"],
                                        **more)


def _w8a8_inputs(case, seed):
    M, K, N = case["M"], case["K"], case["N"]
    return _activation(M, K, "none", 20.0, seed, 0), _normal((N, K), 0.02, seed, 1)


# the calibration of a static per-tensor step: 4.5 standard deviations of the activation's body (the
# few values beyond saturate), the weight's own maximum
_X_CALIBRATED = 4.5


def prepare(case, seed):
    """What a program has in hand before the call."""
    f = case["family"]
    if f == "train":
        return _train_state(case, seed)
    if f == "block":
        return dict(case=case, layers=[_train_state(c, seed, 1000 * (i + 1)) for i, c in enumerate(_block_layers(case))])
    if f == "layernorm":
        R, C = case["rows"], case["cols"]
        s = dict(case=case, q=_u8(R, C), qT=_u8(C, R), amax=_f32(1), scale=_f32(1), scale_inv=_f32(1),
                 workspace=_workspace(R, 1, 1, tw.TWEO_OP_LAYERNORM_QUANTIZE))
        s.update(_layernorm_inputs(case, seed))
        if case["residual"]:
            s["h"] = _bf(R, C)
        if case["delayed"]:
            s["state"] = torch.zeros(tw.tweo_delayed_state_bytes() // 4, dtype=torch.int32, device=DEV)
            tw.tweo_delayed_state_init(s["state"])
            _layernorm_run(s, _layernorm_inputs(case, seed, 100), True)
        return s
    if f == "infer":
        M, K, N = case["M"], case["K"], case["N"]
        s = dict(case=case, x=_activation(M, K, "sparse", 1e4, seed, 0), wq=_u8(N, K), sw_inv=_f32(1), xq=_u8(M, K),
                 amax=_f32(1), sx_inv=_f32(1), y=_bf(M, N), workspace=_workspace(M, N, K, tw.TWEO_OP_FP8_LINEAR_FWD))
        w = _normal((N, K), 0.02, seed, 1)
        tw.tweo_amax(w, s["amax"])
        tw.tweo_quantize_e4m3(w, s["amax"], s["wq"], scale_inv_out=s["sw_inv"])
        return s
    M, K, N = case["M"], case["K"], case["N"]
    x, w = _w8a8_inputs(case, seed)
    i8 = lambda *shape: torch.empty(shape, dtype=torch.int8, device=DEV)
    s = dict(case=case, x=x, xq=i8(M, K), wq=i8(N, K), y=i8(M, N) if case["steps"] == "rows_i8" else _bf(M, N))
    if case["steps"] == "tensor":
        sx, sw = _X_CALIBRATED, float(w.abs().max())
        tw.tweo_quantize_i8(w, 127.0 / sw, s["wq"])
        s.update(inv_step=127.0 / sx, alpha=sx / 127.0 * (sw / 127.0), workspace=_workspace(M, N, K, tw.TWEO_OP_W8A8_LINEAR))
    else:
        s.update(x_step=_f32(M), w_step=_f32(N))
        tw.tweo_quantize_i8_rows(w, 1e-6, s["wq"], s["w_step"])
        if case["steps"] == "rows_i8":
            # the output's calibrated maximum: 4.5 standard deviations of the product
            s["inv_step_out"] = 127.0 / (4.5 * 0.02 * math.sqrt(K))
    return s


def run(state):
    """One pass."""
    s, c = state, state["case"]
    f = c["family"]
    if f == "train":
        _train_forward(s, s)
        _train_backward(s, s)
        out = {k: s[k] for k in ("y", "dx", "dw", "scalars", "xq", "xqT", "wq", "wqT")}
        if not c["inject"]:
            # (with the penalty's gradient the codes of dy' follow y's last bit)
            out.update(dyq=s["dyq"], dyqT=s["dyqT"])
        if c["penalty"]:
            out["penalty"] = s["penalty"]
        if c["scaling"] == "delayed":
            out["states"] = s["states"]
        return out
    if f == "block":
        for t in s["layers"]:
            _train_forward(t, t)
        for t in reversed(s["layers"]):
            _train_backward(t, t)
        return [{k: t[k] for k in ("y", "dx", "dw", "scalars", "penalty")} for t in s["layers"]]
    if f == "layernorm":
        _layernorm_run(s, s)
        out = dict(q=s["q"], qT=s["qT"])
        if c["residual"]:
            out["h"] = s["h"]
        if c["delayed"]:
            out["state"] = s["state"]
        else:
            out.update(amax=s["amax"], scale=s["scale"], scale_inv=s["scale_inv"])
        return out
    if f == "infer":
        tw.tweo_amax(s["x"], s["amax"])
        tw.tweo_quantize_e4m3(s["x"], s["amax"], s["xq"], scale_inv_out=s["sx_inv"])
        tw.tweo_fp8_linear_fwd(s["xq"], s["sx_inv"], s["wq"], s["sw_inv"], s["y"], workspace=s["workspace"])
        return dict(y=s["y"], xq=s["xq"], sx_inv=s["sx_inv"])
    if c["steps"] == "tensor":
        tw.tweo_quantize_i8(s["x"], s["inv_step"], s["xq"])
        tw.tweo_w8a8_linear(s["xq"], s["wq"], s["alpha"], s["y"], s["workspace"])
        return dict(y=s["y"], xq=s["xq"])
    tw.tweo_quantize_i8_rows(s["x"], 1e-6, s["xq"], s["x_step"])
    if c["steps"] == "rows_i8":
        tw.tweo_w8a8_linear_scaled_i8out(s["xq"], s["wq"], s["x_step"], s["w_step"], s["inv_step_out"], s["y"])
    else:
        tw.tweo_w8a8_linear_scaled(s["xq"], s["wq"], s["x_step"], s["w_step"], s["y"])
    return dict(y=s["y"], xq=s["xq"], x_step=s["x_step"])


def work(case):
    f = case["family"]
    if f == "train":
        M, K, N = case["M"], case["K"], case["N"]
        # bf16 x, w, dy (and the residual) in; y, dx, dw and the operands' codes with their transposes out
        n = 2 * (M * K + N * K + M * N) + 2 * (M * N + M * K + N * K) + 2 * (M * K + N * K + M * N)
        return dict(bytes=n + (2 * M * N if case["residual"] else 0), flops=6.0 * M * N * K)
    if f == "block":
        ws = [work(c) for c in _block_layers(case)]
        return dict(bytes=sum(w["bytes"] for w in ws), flops=sum(w["flops"] for w in ws))
    if f == "layernorm":
        n = case["rows"] * case["cols"]
        return dict(bytes=n * (2 + 2 + (4 if case["residual"] else 0)), flops=8.0 * n)
    M, K, N = case["M"], case["K"], case["N"]
    if f == "infer":
        return dict(bytes=2 * M * K + M * K + N * K + 2 * M * N, flops=2.0 * M * N * K)
    y_bytes = 1 if case["steps"] == "rows_i8" else 2
    return dict(bytes=2 * M * K + M * K + N * K + y_bytes * M * N, flops=2.0 * M * N * K)


def tolerance(case):
    if case["family"] in ("train", "block", "infer"):
        return {"rel": 7e-3, "max": 4e-2}
    return "exact"  # whole numbers, and floats that are one rounding of an exact value


# -------------------------------------------------------------------------- the same in 64 bits
_TOP = {"e4m3": 448.0, "e5m2": 57344.0}
_TYPE = {"e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}


def _quantise(x, amax, fmt):
    """Per-tensor codes of a bf16 tensor as fp64 values, and the two scales: scale = top / amax as one
    fp32 division, round to nearest even, saturating."""
    scale = torch.tensor(_TOP[fmt], dtype=torch.float32, device=DEV) / amax
    v = (x.float() * scale).clamp(-_TOP[fmt], _TOP[fmt])
    return v.to(_TYPE[fmt]).double(), scale, 1.0 / scale


def _amax(x):
    return x.float().abs().max()


def _layer_exact(case, seed, index=0):
    c, t = case, _train_inputs(case, seed, index)
    before = _train_inputs(case, seed, index + 100) if c["scaling"] == "delayed" else t
    ax, aw = _amax(before["x"]), _amax(before["w"])
    xq, sx, sxi = _quantise(t["x"], ax, "e4m3")
    wq, sw, swi = _quantise(t["w"], aw, "e4m3")
    y = xq @ wq.t() * (sxi.double() * swi.double())
    if c["residual"]:
        y += t["residual"].double()
    out = dict(y=y)
    stored = y.bfloat16()
    denom = PEN[0] + PEN[1]
    if c["penalty"]:
        out["penalty"] = ((stored.double().abs() / denom) ** PEN[2]).sum().reshape(1)
    dy = t["dy"]
    if c["inject"]:
        a = stored.double()
        g = _gradient_factor(c["M"], c["N"])
        dy = (dy.double() + g * PEN[2] * torch.sign(a) * (a.abs() / denom) ** (PEN[2] - 1) / denom).bfloat16()
    ady = _amax(before["dy"] if c["scaling"] == "delayed" else dy)
    dyq, sdy, sdyi = _quantise(dy, ady, c["dy"])
    out["dx"] = dyq @ wq * (sdyi.double() * swi.double())
    out["dw"] = dyq.t() @ xq * (sdyi.double() * sxi.double())
    amaxes = (_amax(t["x"]), _amax(t["w"]), _amax(dy))
    words = [amaxes[0], sx, sxi, amaxes[1], sw, swi, amaxes[2], sdy, sdyi]
    out["scalars"] = torch.stack([v.double() for v in words] + [torch.zeros((), dtype=torch.float64, device=DEV)] * 7)
    return out


def exact(case, seed):
    f = case["family"]
    if f == "train":
        return _layer_exact(case, seed)
    if f == "block":
        return [_layer_exact(c, seed, 1000 * (i + 1)) for i, c in enumerate(_block_layers(case))]
    if f == "layernorm":
        t = _layernorm_inputs(case, seed)
        h = t["x"].double()
        out = {}
        if case["residual"]:
            out["h"] = h + t["residual"].double()
            h = out["h"].bfloat16().double()
        if not case["delayed"]:
            mean = h.mean(1, keepdim=True)
            var = ((h - mean) ** 2).mean(1, keepdim=True)
            y = ((h - mean) / torch.sqrt(var + float(torch.tensor(1e-5, dtype=torch.float32))) * t["gamma"].double()
                 + t["beta"].double()).bfloat16()
            amax = _amax(y)
            scale = torch.tensor(448.0, device=DEV) / amax
            out.update(amax=amax.double().reshape(1), scale=scale.double().reshape(1), scale_inv=(1.0 / scale).double().reshape(1))
        return out or None
    M, K, N = case["M"], case["K"], case["N"]
    if f == "infer":
        x, w = _activation(M, K, "sparse", 1e4, seed, 0), _normal((N, K), 0.02, seed, 1)
        xq, _, sxi = _quantise(x, _amax(x), "e4m3")
        wq, _, swi = _quantise(w, _amax(w), "e4m3")
        return dict(y=xq @ wq.t() * (sxi.double() * swi.double()), sx_inv=sxi.double().reshape(1))
    x, w = _w8a8_inputs(case, seed)
    q8 = lambda v, inv: torch.round(v.float() * inv).clamp(-127, 127).double()
    if case["steps"] == "tensor":
        sx, sw = _X_CALIBRATED, float(w.abs().max())
        f32 = lambda v: torch.tensor(v, dtype=torch.float32, device=DEV)
        return dict(y=q8(x, f32(127.0 / sx)) @ q8(w, f32(127.0 / sw)).t() * (sx / 127.0 * (sw / 127.0)))
    rows = lambda v: v.float().abs().amax(1, keepdim=True) + 1e-6
    rx, rw = rows(x), rows(w)
    step = (rx / 127.0).double()
    out = dict(x_step=step.reshape(-1))
    if case["steps"] == "rows":
        out["y"] = q8(x, 127.0 / rx) @ q8(w, 127.0 / rw).t() * step * (rw / 127.0).double().t()
    return out
