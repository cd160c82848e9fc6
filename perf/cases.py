"""The work a user of this library has it do, as measurable cases.

Each case is one pass through the public entry points of `paper_2604_04701_amd.binding`, with
what a serving program keeps between calls (quantised weights, calibrated channel lists,
workspaces, output buffers) made beforehand.  Four kinds:

  linear   one quantised projection Y = X W + b: any number of tokens from one (decode) to
           16384 (prefill), per-tensor or per-token activation scales, per-tensor or per-channel
           weight scales, outlier channels found at run time or fixed offline
  mlp      c_fc, GELU, c_proj of a GPT-2 block as one call
  weight   the offline weight quantiser, what loading a model runs once per projection
  stages   the activation side by itself: outlier detection, then Body and Aux codes

Shapes are those of the GPT-2 projections that `synth.config_cases` lists, the same with the few
tokens of a decode step, and generic odd ones.  Activations are normal with a few channels
20 to 100 times larger, weights 0.02 times normal (the distributions of `synth`), drawn on the
GPU from the seed.
"""
import math

import torch

from paper_2604_04701_amd import binding as B

DEV = "cuda"
THRESHOLD = 6.0
EXP = 2


def _linear(name, M, K, N, *, r, w_gran="tensor", x_gran="tensor", bias=True, static=False,
            noalloc=False):
    case = {"kind": "linear", "M": M, "K": K, "N": N, "r": r, "w_gran": w_gran, "x_gran": x_gran,
            "bias": bias, "static": static, "noalloc": noalloc}
    return _named(case, name)


def _mlp(name, M, K, N1, N2, *, r, w_gran="tensor", x_gran="tensor"):
    case = {"kind": "mlp", "M": M, "K": K, "N1": N1, "N2": N2, "r": r, "w_gran": w_gran,
            "x_gran": x_gran}
    return _named(case, name)


def _weight(name, K, N, *, w_gran):
    return _named({"kind": "weight", "K": K, "N": N, "w_gran": w_gran}, name)


def _stages(name, M, K, *, r):
    return _named({"kind": "stages", "M": M, "K": K, "r": r}, name)


def _named(case, name):
    return case if name is None else {"name": name, **case}


def listed():
    return [
        # one token of one sequence through c_attn of GPT-2 small: the smallest call, all latency
        # (the entry point for serving loops that carry no workspace)
        _linear("decode_1x768x2304", 1, 768, 2304, r=6, noalloc=True),
        # a decode step of 24 sequences through the MLP's c_proj of GPT-2 large, the per-vector
        # setting with calibrated outlier channels: few rows, a long K
        _linear("decode_24x5120x1280_vector_static", 24, 5120, 1280, r=16, w_gran="channel",
                x_gran="token", static=True),
        # a decode step of 8 sequences through a whole MLP of GPT-2 large
        _mlp("decode_mlp_8x1280", 8, 1280, 5120, 1280, r=8),
        # a chunk of 512 prompt tokens through c_proj of GPT-2 medium's MLP
        _linear("chunk_512x4096x1024_channel", 512, 4096, 1024, r=12, w_gran="channel"),
        # one full context of GPT-2 small through c_fc
        _linear("context_1024x768x3072", 1024, 768, 3072, r=8),
        # eight contexts of GPT-2 medium through the attention's c_proj
        _linear("prefill_8192x1024x1024_channel", 8192, 1024, 1024, r=12, w_gran="channel"),
        # packed prompts of odd total length, no dimension a multiple of a tile, per-vector setting
        _linear("ragged_3001x1592x4808_vector", 3001, 1592, 4808, r=10, w_gran="channel",
                x_gran="token"),
        # sixteen contexts of GPT-2 large through c_attn, per-vector setting
        _linear("prefill_16384x1280x3840_vector", 16384, 1280, 3840, r=16, w_gran="channel",
                x_gran="token"),
        # eight contexts of GPT-2 medium through a whole MLP
        _mlp("prefill_mlp_8192x1024", 8192, 1024, 4096, 1024, r=12),
        # the benchmark's layer, the largest product
        _linear("large_8192x4096x16384", 8192, 4096, 16384, r=32, bias=False),
        # the weight of that layer quantised when a model is loaded
        _weight("weight_4096x16384_channel", 4096, 16384, w_gran="channel"),
        # the activation side alone on an X larger than half of the memory-side cache
        _stages("stages_16384x5120", 16384, 5120, r=16),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choices(["linear", "mlp", "weight", "stages"], [10, 3, 2, 2])[0]
    w_gran = rng.choice(["tensor", "channel"])
    x_gran = rng.choices(["tensor", "token"], [3, 2])[0]
    K = _log_int(rng, 256, 5120, 8)
    if kind == "weight":
        # (whole blocks of 16 output channels: the packed buffer then has no unwritten rows)
        return _weight(None, K, _log_int(rng, 512, 16384, 16), w_gran=w_gran)
    M = _log_int(rng, 1, 16384)
    r = rng.randint(1, 24)
    if kind == "stages":
        return _stages(None, max(M, 64), K, r=r)
    if kind == "mlp":
        # hidden width about four times the model's; no more work than the largest listed case
        K = min(K, 1600)
        return _mlp(None, M, K, 4 * K, K, r=r, w_gran=w_gran, x_gran=x_gran)
    N = _log_int(rng, 256, 16384, 8)
    while M * K * N > 8192 * 4096 * 16384:
        M = (M + 1) // 2
    static = rng.random() < 0.25
    noalloc = M <= 64 and not static and x_gran == "tensor" and rng.random() < 0.5
    return _linear(None, M, K, N, r=r, w_gran=w_gran, x_gran=x_gran, bias=rng.random() < 0.8,
                   static=static, noalloc=noalloc)


# ---- inputs --------------------------------------------------------------------------------


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)


def _make_x(g, M, K, r):
    """X fp16 [M, K] and its r loud channels (int64, ascending)."""
    x = _normal(g, M, K)
    ch = torch.randperm(K, generator=g, device=DEV)[:r].sort().values
    gain = 20.0 + 80.0 * torch.rand(r, generator=g, device=DEV, dtype=torch.float32)
    x[:, ch] *= gain
    return x.half(), ch


def _make_w(g, K, N):
    return (0.02 * _normal(g, K, N)).half()


def _make_bias(g, N):
    return (0.1 * _normal(g, N)).half()


def _inputs(case, seed):
    """The raw fp16 inputs, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kind = case["kind"]
    if kind == "weight":
        return {"W": _make_w(g, case["K"], case["N"])}
    X, ch = _make_x(g, case["M"], case["K"], case["r"])
    if kind == "stages":
        return {"X": X}
    if kind == "mlp":
        K, N1, N2 = case["K"], case["N1"], case["N2"]
        return {"X": X, "W1": _make_w(g, K, N1), "b1": _make_bias(g, N1), "W2": _make_w(g, N1, N2),
                "b2": _make_bias(g, N2)}
    W = _make_w(g, case["K"], case["N"])
    b = _make_bias(g, case["N"]) if case["bias"] else None
    return {"X": X, "W": W, "b": b, "channels": ch}


R_CAP = 64


def prepare(case, seed):
    i = _inputs(case, seed)
    kind = case["kind"]
    s = {"case": case}
    if kind == "weight":
        s["W"] = i["W"]
    elif kind == "stages":
        s["X"] = i["X"]
    elif kind == "mlp":
        M, K, N1, N2 = case["M"], case["K"], case["N1"], case["N2"]
        s["X"], s["b1"], s["b2"] = i["X"], i["b1"], i["b2"]
        s["w1"] = B.muxq_quantize_weight(i["W1"], case["w_gran"])
        s["w2"] = B.muxq_quantize_weight(i["W2"], case["w_gran"])
        s["H"] = torch.empty((M, N1), dtype=torch.float16, device=DEV)
        s["Y"] = torch.empty((M, N2), dtype=torch.float16, device=DEV)
        s["ws"] = torch.empty(B.lib().muxq_mlp_workspace_bytes(M, K, N1, N2, R_CAP),
                              dtype=torch.uint8, device=DEV)
    else:
        M, K, N = case["M"], case["K"], case["N"]
        s["X"], s["b"] = i["X"], i["b"]
        s["w_q"], s["w_scale"] = B.muxq_quantize_weight(i["W"], case["w_gran"])
        s["Y"] = torch.empty((M, N), dtype=torch.float16, device=DEV)
        # a shape too large for the static array has a workspace like any other
        s["noalloc"] = case["noalloc"] and B.workspace_bytes(M, K, N, R_CAP) <= B.lib().muxq_noalloc_max_bytes()
        if not s["noalloc"]:
            s["ws"] = B.alloc_workspace(M, K, N, R_CAP)
        if case["static"]:
            s["block"] = B.muxq_prepare_static(i["channels"].int(), K, s["w_q"], N, R_CAP)
    return s


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "linear":
        if c["static"]:
            return B.muxq_linear_static(state["X"], state["w_q"], state["w_scale"], c["N"], state["block"],
                                        c["w_gran"], bias=state["b"], out=state["Y"], workspace=state["ws"],
                                        x_gran=c["x_gran"])
        if state["noalloc"]:
            return B.muxq_linear_noalloc(state["X"], state["w_q"], state["w_scale"], c["N"], c["w_gran"],
                                         bias=state["b"], out=state["Y"])
        return B.muxq_linear(state["X"], state["w_q"], state["w_scale"], c["N"], c["w_gran"], bias=state["b"],
                             out=state["Y"], workspace=state["ws"], x_gran=c["x_gran"])
    if kind == "mlp":
        H, Y, _ = B.muxq_mlp(state["X"], *state["w1"], c["N1"], *state["w2"], c["N2"], c["w_gran"],
                             bias1=state["b1"], bias2=state["b2"], x_gran=c["x_gran"],
                             workspace=state["ws"], out_h=state["H"], out=state["Y"])
        return H, Y
    if kind == "weight":
        w_q, w_scale = B.muxq_quantize_weight(state["W"], c["w_gran"])
        codes = w_q[:B.packed_bytes(c["N"], B.k_pad(c["K"]))]
        return codes, B.wq_row_sums(w_q, c["K"], c["N"]), w_scale
    col_absmax, idx, n_out = B.muxq_detect_outliers(state["X"], THRESHOLD, R_CAP)
    body_q, aux_q, x_scale = B.muxq_build_aux(state["X"], col_absmax, idx, n_out, R_CAP, EXP)
    M, K = c["M"], c["K"]
    if M % 16:      # rows past M of the packed buffers are never written: whole blocks of 16 rows,
        m16, kp = M // 16 * 16, B.k_pad(K)      # then the rows of the last, partial one
        body_q = [body_q[:m16 * kp], body_q[m16 * kp:].view(-1, 16, 64)[:, :M - m16]]
        aux_q = [aux_q[:m16 * R_CAP], aux_q[m16 * R_CAP:].view(-1, 16, 64)[:, :M - m16]]
    return col_absmax, idx, n_out, body_q, aux_q, x_scale


# ---- what a pass cannot do without -----------------------------------------------------------


def _layer_work(M, K, N, w_gran, bias):
    weight = K * N + 4 * (N if w_gran == "channel" else 1) + (2 * N if bias else 0)
    return 2 * M * K, weight, 2 * M * N, 2 * M * K * N


def work(case):
    kind = case["kind"]
    if kind == "linear":
        x, w, y, ops = _layer_work(case["M"], case["K"], case["N"], case["w_gran"], case["bias"])
        return {"bytes": x + w + y, "flops": ops}
    if kind == "mlp":
        x, w1, h, ops1 = _layer_work(case["M"], case["K"], case["N1"], case["w_gran"], True)
        _, w2, y, ops2 = _layer_work(case["M"], case["N1"], case["N2"], case["w_gran"], True)
        return {"bytes": x + w1 + h + w2 + y, "flops": ops1 + ops2}
    if kind == "weight":
        K, N = case["K"], case["N"]
        return {"bytes": 2 * K * N + K * N + 4 * N + 4 * (N if case["w_gran"] == "channel" else 1),
                "flops": 2 * K * N}
    M, K = case["M"], case["K"]
    return {"bytes": 2 * M * K + M * K + M * R_CAP + 4 * K, "flops": 2 * M * K}


def tolerance(case):
    """Codes, sums and scales are whole numbers and correctly rounded quotients: exact.  A layer's
    output is an exact integer times a scale, rounded to fp16: against 64-bit arithmetic that
    rounding shows 2e-4 (2-norm), and codes that fall the other way at near-ties up to 6e-4; in
    the MLP the last place of H moves codes of the second layer, up to 1e-3.  Four times that."""
    if case["kind"] in ("weight", "stages"):
        return "exact"
    if case["kind"] == "linear":
        return {"rel": 2.4e-3}
    return {"rel": 4e-3}


# ---- the same in 64 bits ---------------------------------------------------------------------


def _codes(v, amax):
    """Eq. 1-2 codes (float64) and scale of v on the abs-max `amax` (broadcast)."""
    inv = torch.where(amax > 0, 127.0 / amax, torch.zeros_like(amax))
    return (v * inv).round_().clamp_(-127.0, 127.0), amax / 127.0


def _quant_w64(W, w_gran):
    W = W.double()
    amax = W.abs().amax(0) if w_gran == "channel" else W.abs().amax().reshape(1)
    return _codes(W, amax)


def _listed(colmax, r_cap=R_CAP):
    return (colmax > THRESHOLD).nonzero().flatten()[:r_cap]


def _linear64(X, w_codes, w_scale, bias, x_gran, channels=None):
    """The layer of Eq. 1-7 in float64 on fp16 inputs."""
    X = X.double()
    idx = _listed(X.abs().amax(0)) if channels is None else channels[:R_CAP]
    X[:, idx] *= 2.0 ** -EXP
    amax = X.abs().amax(1, keepdim=True) if x_gran == "token" else X.abs().amax().reshape(1)
    q, s = _codes(X, amax)
    q[:, idx] *= 2.0 ** EXP                   # Body + (2^e - 1) Aux
    y = (q @ w_codes) * (s * w_scale)
    return y if bias is None else y + bias.double()


def _pack64(mat):
    """Row-major [rows, cols] -> the packed order of 16 x 64 blocks; rows a multiple of 16."""
    r, c = mat.shape
    return mat.view(r // 16, 16, c // 64, 64).permute(0, 2, 1, 3).contiguous().reshape(-1)


def _pad_cols(mat, to):
    return torch.nn.functional.pad(mat, (0, to - mat.shape[1]))


def _packed_like_run(mat):
    """A code matrix laid out as `run` returns it: packed, a partial last block by itself."""
    M = mat.shape[0]
    m16 = M // 16 * 16
    if m16 == M:
        return _pack64(mat)
    tail = mat[m16:].view(M - m16, -1, 64).permute(1, 0, 2)
    return [_pack64(mat[:m16]), tail]


def exact(case, seed):
    i = _inputs(case, seed)
    kind = case["kind"]
    if kind == "weight":
        q, s = _quant_w64(i["W"], case["w_gran"])
        kp = (case["K"] + 63) // 64 * 64
        return _pack64(_pad_cols(q.t(), kp)), q.sum(0), s
    if kind == "stages":
        X = i["X"].double()
        kp = (case["K"] + 63) // 64 * 64
        colmax = X.abs().amax(0)
        found = (colmax > THRESHOLD).nonzero().flatten()
        idx = found[:R_CAP]
        X[:, idx] *= 2.0 ** -EXP
        amax = X.abs().amax().reshape(1)
        q, s = _codes(X, amax)
        idx_out = torch.full((R_CAP,), -1.0, dtype=torch.float64, device=DEV)
        idx_out[:len(idx)] = idx.double()
        n_out = torch.tensor([float(len(idx)), float(len(found))], dtype=torch.float64, device=DEV)
        aux = _pad_cols(q[:, idx], R_CAP)
        return (colmax, idx_out, n_out, _packed_like_run(_pad_cols(q, kp)), _packed_like_run(aux),
                torch.cat([s, 127.0 / amax]))
    if kind == "mlp":
        y1 = _linear64(i["X"], *_quant_w64(i["W1"], case["w_gran"]), i["b1"], case["x_gran"])
        y1 = y1.half().double()               # the GELU's and the second layer's inputs are fp16
        H = torch.nn.functional.gelu(y1, approximate="tanh")
        Y = _linear64(H.half(), *_quant_w64(i["W2"], case["w_gran"]), i["b2"], case["x_gran"])
        return H, Y
    channels = i["channels"] if case["static"] else None
    return _linear64(i["X"], *_quant_w64(i["W"], case["w_gran"]), i["b"], case["x_gran"], channels)
