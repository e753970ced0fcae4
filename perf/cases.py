"""The calls this library is used for, at the sizes of its own benchmark and tests.

Shapes are the Llama-2-7B linears (fused QKV, output projection, gate+up, down) and the 16384 x 8192
quantizer tensor, with ragged ones beside them; inputs are seeded Gaussian stimulus with outlier channels,
lognormal sensitivities and thresholds calibrated for a target share of FP8 blocks.  Every call goes
through the Python binding with the buffers that a serving program keeps: workspace, result, packed weights.

`exact` restates the method in plain torch: block decisions and codes in the FP32 steps that define
them, then products and scores in 64 bits.
"""
from __future__ import annotations

import math

import torch

from paper_2504_14152_amd import fgmp

LINEARS = {"qkv": (4096, 12288), "o": (4096, 4096), "fc1": (4096, 22016), "fc2": (11008, 4096)}   # K, N
BLOCK = 16


def _fused(name, M, linear=None, N=0, K=0, dtype="bf16", fp8=0.1, score="nvfp4_error"):
    if linear is not None:
        K, N = LINEARS[linear]
    return {"name": name, "op": "fused", "M": M, "N": N, "K": K, "dtype": dtype, "fp8": fp8, "score": score}


def listed():
    return [
        # one token of one sequence through the smallest linear: latency
        _fused("decode_o_m1", 1, "o"),
        # a small decode batch
        _fused("decode_qkv_m8", 8, "qkv"),
        # the largest batch that counts as a decode step, over the longest dot product
        _fused("decode_fc2_m32", 32, "fc2"),
        # a well-filled decode batch, or a handful of speculative tokens for eight sequences
        _fused("batch_qkv_m64", 64, "qkv"),
        # a short prompt of no particular length, or a large decode batch
        _fused("prompt_fc1_m200", 200, "fc1"),
        # nothing aligned: FP32 activations, a vocabulary-like row count, a K that ends inside a tile, and the
        # score of the error increase
        _fused("ragged_f32_m77", 77, N=5003, K=2064, dtype="f32", fp8=0.2, score="delta"),
        # one chunk of a chunked prefill
        _fused("chunk_fc2_m512", 512, "fc2"),
        # a 4096-token prompt: the headline workload
        _fused("prefill_qkv_m4096", 4096, "qkv"),
        # the gated MLP: FC1, gate and output quantizer, then FC2 from the packed result
        {"name": "gated_mlp_m2048", "op": "mlp", "M": 2048, "N": 22016, "K": 4096, "dtype": "bf16", "fp8": 0.1},
        # activations packed on their own
        {"name": "quantize_16384x8192", "op": "quantize", "M": 16384, "K": 8192, "dtype": "bf16", "fp8": 0.1,
         "score": "nvfp4_error"},
        # preparing one weight tensor: scores, threshold, packing
        {"name": "calibrate_fc1", "op": "calibrate", "N": 22016, "K": 4096, "dtype": "bf16", "fp8": 0.1, "fisher": "element"},
        # the same with the block scales searched for
        {"name": "clip_qkv", "op": "clip", "N": 12288, "K": 4096, "dtype": "bf16", "fp8": 0.1, "fisher": "element"},
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choices(["fused", "mlp", "quantize", "calibrate", "clip"], [12, 2, 2, 1.5, 1.5])[0]
    dtype = rng.choices(["bf16", "f32"], [3, 1])[0]
    fp8 = rng.choices([0.0, 0.05, 0.1, 0.2, 0.3, 1.0], [1, 2, 6, 2, 2, 1])[0]
    score = rng.choices(["nvfp4_error", "delta"], [6, 1])[0]
    if kind == "fused":
        if rng.random() < 0.5:
            K, N = LINEARS[rng.choice(sorted(LINEARS))]
        else:
            K, N = _log_int(rng, 256, 11008, 16), _log_int(rng, 256, 22016)
        most = min(4096, 4096 * 4096 * 12288 // (N * K))
        return {"op": "fused", "M": _log_int(rng, 1, most), "N": N, "K": K, "dtype": dtype, "fp8": fp8, "score": score}
    if kind == "mlp":
        hidden, K = _log_int(rng, 512, 11008, 32), _log_int(rng, 512, 4096, 16)
        return {"op": "mlp", "M": _log_int(rng, 1, 2048), "N": 2 * hidden, "K": K, "dtype": dtype, "fp8": max(fp8, 0.05)}
    if kind == "quantize":
        K = _log_int(rng, 256, 16384, 16)
        return {"op": "quantize", "M": _log_int(rng, 16, 16384 * 4096 // K), "K": K, "dtype": dtype, "fp8": fp8, "score": score}
    most = 22016 * 4096 if kind == "calibrate" else 12288 * 4096
    K = _log_int(rng, 512, 8192, 16)
    return {"op": kind, "N": _log_int(rng, 512, most // K), "K": K, "dtype": dtype, "fp8": max(fp8, 0.05),
            "fisher": rng.choice(["element", "channel"])}


# ---- inputs (no code of the library) ----

_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


def _generator(seed, part):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + part)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _scale(x):
    """The tensor scale amax / 448 in FP32, as a Python number."""
    return float((x.abs().max().float() / 448.0).item())


def _activations(case, seed):
    g = _generator(seed, 1)
    x = _randn(g, case["M"], case["K"])
    outliers = torch.randperm(case["K"], generator=g, device="cuda")[: max(1, case["K"] // 100)]
    x[:, outliers] *= 20.0
    return x.to(_TORCH[case["dtype"]]), torch.exp(_randn(g, case["K"]))


def _weights(N, K, dtype, per_element, seed, part):
    g = _generator(seed, part)
    w = (_randn(g, N, K) * 0.02).to(_TORCH[dtype])
    return w, torch.exp(_randn(g, *((N, K) if per_element else (K,))))


def _hidden_inputs(case, seed):
    """Sensitivities, threshold and scale of the hidden activations: constants of a calibration elsewhere."""
    g = _generator(seed, 4)
    hidden = case["N"] // 2
    size = case["K"] * 4e-4 * 5.0                     # about the mean square of a gate or up value
    return torch.exp(_randn(g, hidden)), 0.2 * size * size, 24.0 * size / 448.0   # a tenth of the blocks in FP8


def _linear_inputs(case, seed):
    x, f = _activations(case, seed)
    w, fw = _weights(case["N"], case["K"], "bf16", False, seed, 2)
    return x, f, w, fw


# ---- the calls ----

def _pack(w, fw, fraction):
    s = _scale(w)
    _, scores = fgmp.quantize_weights(w, fw, math.inf, s, want_scores=True)
    return fgmp.quantize_weights(w, fw, fgmp.threshold_for_fraction(scores, fraction), s)


def _calibrated(x, f, fraction, score="nvfp4_error"):
    s = _scale(x)
    _, scores = fgmp.quantize_activations(x, f, math.inf, s, want_scores=True, score_mode=score)
    return fgmp.threshold_for_fraction(scores, fraction), s


def _mode(case):
    return None if case["score"] == "nvfp4_error" else case["score"]


def _zeroed(rows, K):
    return fgmp.Packed(torch.zeros(fgmp.packed_bytes(rows, K), dtype=torch.uint8, device="cuda"), rows, K)


def prepare(case, seed):
    op = case["op"]
    st = {"op": op}
    if op == "fused":
        x, f, w, fw = _linear_inputs(case, seed)
        T, s = _calibrated(x, f, case["fp8"], case["score"])
        st.update(x=x, f=f, T=T, s=s, mode=_mode(case), pw=_pack(w, fw, case["fp8"]),
                  y=torch.empty(case["M"], case["N"], device="cuda"),
                  ws=fgmp.new_workspace(fgmp.workspace_bytes(case["M"], case["N"], case["K"]), x.device))
    elif op == "mlp":
        M, N, K = case["M"], case["N"], case["K"]
        x, f, w, fw = _linear_inputs(case, seed)
        T, s = _calibrated(x, f, case["fp8"])
        w2, fw2 = _weights(K, N // 2, "bf16", False, seed, 3)
        fh, Th, sh = _hidden_inputs(case, seed)
        gate = fgmp.EPILOGUE_SILU_GATE
        st.update(x=x, f=f, T=T, s=s, pw=_pack(w, fw, case["fp8"]), pw2=_pack(w2, fw2, case["fp8"]), fh=fh, Th=Th, sh=sh,
                  ph=_zeroed(M, N // 2), z=torch.empty(M, K, device="cuda"),
                  ws=fgmp.new_workspace(fgmp.workspace_bytes_packed_out(M, N, K, gate), x.device),
                  ws2=fgmp.new_workspace(fgmp.workspace_bytes(M, K, N // 2), x.device))
    elif op == "quantize":
        x, f = _activations(case, seed)
        T, s = _calibrated(x, f, case["fp8"], case["score"])
        st.update(x=x, f=f, T=T, s=s, mode=_mode(case), p=_zeroed(case["M"], case["K"]))
    else:
        w, fw = _weights(case["N"], case["K"], case["dtype"], case["fisher"] == "element", seed, 2)
        st.update(w=w, fw=fw, s=_scale(w), fp8=case["fp8"], p=_zeroed(case["N"], case["K"]))
        if op == "clip":
            _, scores = fgmp.quantize_weights(w, fw, math.inf, st["s"], want_scores=True)
            st["T"] = fgmp.threshold_for_fraction(scores, case["fp8"])
    return st


def run(st):
    op = st["op"]
    if op == "fused":
        return fgmp.quant_gemm_fused(st["x"], st["f"], st["T"], st["s"], st["pw"], out=st["y"], workspace=st["ws"],
                                     score_mode=st["mode"])
    if op == "mlp":
        ph = fgmp.quant_gemm_fused_packed_out(st["x"], st["f"], st["T"], st["s"], st["pw"], st["fh"], st["Th"], st["sh"],
                                              out=st["ph"], workspace=st["ws"], epilogue=fgmp.EPILOGUE_SILU_GATE)
        return fgmp.gemm(ph, st["pw2"], out=st["z"], workspace=st["ws2"])
    if op == "quantize":
        return fgmp.quantize_activations(st["x"], st["f"], st["T"], st["s"], out=st["p"], score_mode=st["mode"]).buf
    if op == "calibrate":
        _, scores = fgmp.quantize_weights(st["w"], st["fw"], math.inf, st["s"], want_scores=True, out=st["p"])
        T = fgmp.threshold_for_fraction(scores, st["fp8"])
        p = fgmp.quantize_weights(st["w"], st["fw"], T, st["s"], out=st["p"])
        return {"packed": p.buf, "scores": scores, "threshold": T}
    p, scores = fgmp.quantize_weights_clip(st["w"], st["fw"], st["T"], st["s"], want_scores=True, out=st["p"])
    return {"packed": p.buf, "scores": scores}


# ---- what a pass cannot do without ----

def _packed_size(rows, K, fp8):
    """9 bytes per 4-bit block, 16 per 8-bit block, one bit of metadata per block."""
    return rows * (K // BLOCK) * (9.0 * (1.0 - fp8) + 16.0 * fp8 + 0.125)


def work(case):
    op, K = case["op"], case["K"]
    size = 2 if case["dtype"] == "bf16" else 4
    if op == "fused":
        M, N = case["M"], case["N"]
        return {"bytes": M * K * size + 4.0 * K + _packed_size(N, K, case["fp8"]) + 4.0 * M * N, "flops": 2.0 * M * N * K}
    if op == "mlp":
        M, N = case["M"], case["N"]
        return {"bytes": M * K * size + _packed_size(N, K, case["fp8"]) + 2 * _packed_size(M, N // 2, 0.1) +
                _packed_size(K, N // 2, case["fp8"]) + 4.0 * M * K, "flops": 3.0 * M * N * K}
    if op == "quantize":
        return {"bytes": case["M"] * K * size + 4.0 * K + _packed_size(case["M"], K, case["fp8"]),
                "flops": 10.0 * case["M"] * K}
    N = case["N"]
    fisher = 4.0 * N * K if case["fisher"] == "element" else 4.0 * K
    moved = N * K * size + fisher + _packed_size(N, K, case["fp8"]) + N * (K // BLOCK) * 4.0
    # the threshold separates the pass that scores from the pass that packs, so W and its sensitivities are read twice
    if op == "calibrate":
        moved += N * K * size + fisher + N * (K // BLOCK) * 4.0
    return {"bytes": moved, "flops": 10.0 * N * K}


def tolerance(case):
    if case["op"] == "fused":
        return {"rel": 1e-6, "max": 1e-5}       # FP32 sums of the same exact products in another order (4e-8 .. 7e-8 off)
    if case["op"] == "mlp":
        # a last-bit difference in h moves a code or a decision now and then (8.5e-5 off the 64-bit chain)
        return {"rel": 4e-4, "max": 0.02}
    return "exact"                              # codes, decisions and scores are defined bit for bit


# ---- the same in plain torch, 64 bits where numbers are summed ----

def _e4m3(v):
    """Nearest E4M3 value (ties to even, saturating) of FP32 numbers, as FP32."""
    return v.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).float()


def _e2m1(v):
    """Nearest E2M1 value (ties to even, saturating) of FP32 numbers, as FP32."""
    a = v.abs().clamp(max=6.0)
    r = torch.where(a < 2.0, torch.round(a * 2.0) * 0.5, torch.where(a < 4.0, torch.round(a), torch.round(a * 0.5) * 2.0))
    return torch.where(v < 0, -r, r)


def _tree(t):
    while t.shape[-1] > 1:
        t = t[..., 0::2] + t[..., 1::2]
    return t[..., 0]


def _f32(value):
    return torch.tensor(value, dtype=torch.float32, device="cuda")


def _nvfp4(xb, sc, S):
    """(E2M1 values, reconstruction) of blocks [..., 16] under E4M3 scales sc [...]."""
    d = sc * S
    inv = torch.where(sc != 0, 1.0 / d, torch.zeros_like(d))
    q = _e2m1(xb * inv[..., None])
    return q, q * d[..., None]


def _clip_scale(xb, fb, S):
    codes = torch.arange(127, dtype=torch.uint8, device="cuda").view(torch.float8_e4m3fn).float()
    best = torch.zeros(xb.shape[:-1], device="cuda")
    least = None
    for value in codes:
        e = xb - _nvfp4(xb, value.expand(xb.shape[:-1]), S)[1]
        err = _tree((e * e) * fb)
        if least is None:
            least = err
            continue
        better = err < least
        least = torch.where(better, err, least)
        best = torch.where(better, value, best)
    return best


def _quantized(x, f, scale, fraction, mode="nvfp4_error", threshold=None, clip=False):
    """(stored values in 64 bits without the tensor scale, scores in FP32 steps, scores in 64 bits)."""
    rows, K = x.shape
    S = _f32(scale)
    xb = x.float().view(rows, K // BLOCK, BLOCK)
    fb = f.view(-1, K // BLOCK, BLOCK)
    amax = xb.abs().amax(-1)
    sc = _clip_scale(xb, fb, S) if clip else _e4m3(amax / (6.0 * S))
    q, xh = _nvfp4(xb, sc, S)
    c8 = _e4m3(xb * (1.0 / S))
    q64 = q.double()
    if mode == "delta":
        e = xh - c8 * S
        e64 = q64 * (sc * S).double()[..., None] - c8.double() * S.double()
    else:
        e = xb - xh
        e64 = xb.double() - q64 * (sc * S).double()[..., None]
    scores = _tree((e * e) * fb)
    scores64 = (e64 * e64 * fb.double()).sum(-1)
    if threshold is None:
        n = scores.numel()
        above = int(math.floor(fraction * n + 0.5))
        if above == 0:
            threshold = math.inf
        elif above >= n:
            threshold = -math.inf
        else:
            threshold = float(torch.sort(scores.flatten())[0][n - above - 1].item())
    stored = torch.where((scores > threshold)[..., None], c8.double(), q64 * sc.double()[..., None])
    return stored.view(rows, K), scores, scores64


def _silu_gate(y, N):
    """SiLU(gate) * up of the 32 + 32 column groups."""
    v = y.view(y.shape[0], N // 64, 2, 32)
    g, u = v[:, :, 0], v[:, :, 1]
    return (g / (1.0 + torch.exp(-g)) * u).reshape(y.shape[0], N // 2)


def exact(case, seed):
    op = case["op"]
    if op == "quantize":
        return None
    if op in ("fused", "mlp"):
        x, f, w, fw = _linear_inputs(case, seed)
        sx, sw = _scale(x), _scale(w)
        xs = _quantized(x, f, sx, case["fp8"], case.get("score", "nvfp4_error"))[0]
        ws = _quantized(w, fw, sw, case["fp8"])[0]
        y = (xs @ ws.t()) * (_f32(sx).double() * _f32(sw).double())
        if op == "fused":
            return y
        fh, Th, sh = _hidden_inputs(case, seed)
        hs = _quantized(_silu_gate(y, case["N"]).float(), fh, sh, 0.0, threshold=float(_f32(Th)))[0]
        w2, fw2 = _weights(case["K"], case["N"] // 2, "bf16", False, seed, 3)
        s2 = _scale(w2)
        w2s = _quantized(w2, fw2, s2, case["fp8"])[0]
        return (hs @ w2s.t()) * (_f32(sh).double() * _f32(s2).double())
    w, fw = _weights(case["N"], case["K"], case["dtype"], case["fisher"] == "element", seed, 2)
    scores64 = _quantized(w, fw, _scale(w), case["fp8"], clip=op == "clip")[2]
    return {"packed": None, "scores": scores64} if op == "clip" else {"packed": None, "scores": scores64, "threshold": None}
