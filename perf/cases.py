"""The work that a program built on this library has it do, for timing and for comparing outputs.

Each case is one pass of a path of a LLaMA-style transformer block through paper_2605_19269_amd.coda, called the way a
training or serving program calls it: weights prepared once (gamma folded, gate and up columns interleaved), outputs and
scratch buffers kept between passes, the epilogue programs built anew for every call.  The paths:

  linear        RMSNorm statistic -> one GEMM with row scale, residual and row sum of squares -> combine
  block         serving, one non-attention block chain: RMSNorm statistic -> QKV projection with RoPE -> up-projection
                with SwiGLU -> down-projection with residual and row sum of squares -> combine (next layer's statistic)
  mlp           the MLP half of a block, forward; with save, the pre-activation is kept for a backward pass
  mlp_backward  dY -> SwiGLU backward with its row statistic -> both weight gradients, added up in fp32, and RMSNorm
                backward with the residual gradient and dgamma
  lm_head       logits with log-sum-exp partials -> loss per token

Operands are bf16, or with f8 the two GEMM operands are OCP E4M3 bytes (the program's own quantised copies).  In f8 cases
weight_layout says how the weight bytes lie: "out_in" [out x in], "in_out" [in x out].
"""
import math

import torch

from paper_2605_19269_amd import coda

EPS = 1e-6


def listed():
    return [
        # the library's smallest configuration: five short launches, all latency
        {"name": "tiny-linear", "path": "linear", "tokens": 256, "hidden": 256, "out": 512},
        # one sequence decoding on 8B-style weights: every weight is read for a single row
        {"name": "decode-8b-1", "path": "block", "tokens": 1, "hidden": 4096, "inter": 14336, "qkv": 6144},
        # a small serving batch: 32 sequences, one token each
        {"name": "decode-8b-32", "path": "block", "tokens": 32, "hidden": 4096, "inter": 14336, "qkv": 6144},
        # a fuller serving batch with 8-bit weights and activations
        {"name": "decode-8b-96-f8", "path": "mlp", "tokens": 96, "hidden": 4096, "inter": 14336, "save": False, "f8": True,
         "weight_layout": "out_in"},
        # one short prompt of an odd length on 1B-style weights
        {"name": "prompt-1b-509", "path": "mlp", "tokens": 509, "hidden": 2048, "inter": 8192, "save": False, "f8": False},
        # an ordinary prompt (or a chunk of a long one) on 8B-style weights
        {"name": "prompt-8b-2048", "path": "block", "tokens": 2048, "hidden": 4096, "inter": 14336, "qkv": 6144},
        # a small training batch: token count not a multiple of the tile, FFN width 8/3 hidden
        {"name": "train-small-bwd", "path": "mlp_backward", "tokens": 1000, "hidden": 2048, "inter": 5632},
        # the 1B-style training step, forward and backward
        {"name": "train-1b-fwd", "path": "mlp", "tokens": 8192, "hidden": 2048, "inter": 8192, "save": True, "f8": False},
        {"name": "train-1b-bwd", "path": "mlp_backward", "tokens": 8192, "hidden": 2048, "inter": 8192},
        # the same forward pass on 8-bit operands, weights kept [in x out]
        {"name": "train-1b-fwd-f8", "path": "mlp", "tokens": 8192, "hidden": 2048, "inter": 8192, "save": False, "f8": True,
         "weight_layout": "in_out"},
        # cross-entropy over a 32768-word vocabulary in training
        {"name": "lm-head-8192", "path": "lm_head", "tokens": 8192, "hidden": 4096, "vocab": 32768},
        # the largest: a full batch of prompts through an 8B-style block
        {"name": "prefill-8b-16384", "path": "block", "tokens": 16384, "hidden": 4096, "inter": 14336, "qkv": 6144},
    ]


_LARGEST_FLOPS = 2.0 * 16384 * 4096 * (6144 + 2 * 14336 + 14336)


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, round(v / step) * step)))


def draw(rng):
    path = rng.choice(["linear", "block", "block", "mlp", "mlp", "mlp_backward", "mlp_backward", "lm_head"])
    f8 = path == "mlp" and rng.random() < 0.4
    step = 16 if f8 else 8
    # half of the draws take a model-like width, the others any width the path takes
    if rng.random() < 0.5:
        hidden = rng.choice([2048, 4096])
        inter = {2048: rng.choice([8192, 5632]), 4096: rng.choice([14336, 11008])}[hidden]
    else:
        hidden = _log_int(rng, 512, 5120, step)
        inter = _log_int(rng, 2 * hidden, 4 * hidden, step)
    # backward contracts over the tokens, which come in eights there
    tokens = _log_int(rng, 256, 16384, 8) if path == "mlp_backward" else _log_int(rng, 1, 16384)
    if path == "linear":
        case = {"path": path, "tokens": tokens, "hidden": hidden, "out": _log_int(rng, 256, 8192, 8)}
    elif path == "block":
        qkv = 128 * rng.randint(hidden // 128 + 2, 3 * hidden // 128)
        case = {"path": path, "tokens": tokens, "hidden": hidden, "inter": inter, "qkv": qkv}
    elif path == "mlp":
        case = {"path": path, "tokens": tokens, "hidden": hidden, "inter": inter, "save": not f8 and rng.random() < 0.5, "f8": f8}
        if f8:
            case["weight_layout"] = rng.choice(["out_in", "in_out"])
    elif path == "mlp_backward":
        case = {"path": path, "tokens": tokens, "hidden": hidden, "inter": inter}
    else:
        case = {"path": path, "tokens": tokens, "hidden": hidden, "vocab": _log_int(rng, 8192, 65536, 8)}
    while work(case)["flops"] > _LARGEST_FLOPS or case["tokens"] > 16384:
        case["tokens"] = max(8, case["tokens"] // 16 * 8)
    return case


# ---------------------------------------------------------------- inputs and buffers
class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, shape, std=1.0):
        return torch.randn(shape, device="cuda", dtype=torch.float32, generator=self.g) * std

    def bf16(self, shape, std=1.0):
        return torch.randn(shape, device="cuda", dtype=torch.bfloat16, generator=self.g).mul_(std)

    def f8(self, shape):
        return torch.randn(shape, device="cuda", dtype=torch.bfloat16, generator=self.g).to(torch.float8_e4m3fn).view(torch.uint8)

    def uniform(self, n, lo=0.5, hi=1.5):
        return torch.rand(n, device="cuda", dtype=torch.float32, generator=self.g) * (hi - lo) + lo

    def ints(self, n, high):
        return torch.randint(0, high, (n,), device="cuda", dtype=torch.int32, generator=self.g)


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def _b16(*shape):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda")


def _workspace(*shapes):
    """One scratch buffer that serves all GEMMs of the program, or None where none of them asks for any."""
    need = max(coda.coda_gemm_workspace_bytes(M, N, K, []) for M, N, K in shapes)
    return torch.empty(need, dtype=torch.uint8, device="cuda") if need else None


def _partials(tokens, width):
    return _f32(coda.coda_row_partial_blocks(width), tokens)


def prepare(case, seed):
    rnd = _Draws(seed)
    T, d, path = case["tokens"], case["hidden"], case["path"]
    s = {"case": dict(case)}
    if path == "linear":
        N = case["out"]
        s.update(X=rnd.bf16((T, d)), R=rnd.bf16((T, N)), ss=_f32(1, T), rstd=_f32(T), Y=_b16(T, N), part=_partials(T, N), ssy=_f32(T))
        W = rnd.bf16((d, N), 1.0 / math.sqrt(d))
        s["W"] = torch.empty_like(W)
        coda.coda_fold_gamma(W, rnd.uniform(d), s["W"])
        s["ws"] = _workspace((T, N, d))
    elif path in ("block", "mlp"):
        F = case["inter"]
        f8 = case.get("f8", False)
        s.update(X=rnd.bf16((T, d)), ss=_f32(1, T), rstd=_f32(T), H=_b16(T, F), Y=_b16(T, d), part=_partials(T, d), rnext=_f32(T))
        shapes = [(T, 2 * F, d), (T, d, F)]
        if f8:
            # the program's quantised copies; the quantisation scales of both operands fold into the row scales
            out_in = case["weight_layout"] == "out_in"
            s.update(X8=rnd.f8((T, d)), H8=rnd.f8((T, F)), xscale=rnd.uniform(T, 0.01, 0.03), hscale=rnd.uniform(T, 0.01, 0.03),
                     Wup=rnd.f8((2 * F, d) if out_in else (d, 2 * F)), Wdown=rnd.f8((d, F) if out_in else (F, d)), out_in=out_in)
        else:
            s["Wup"], s["Wdown"] = rnd.bf16((d, 2 * F), 0.02), rnd.bf16((F, d), 0.02)
        if case.get("save"):
            s["Z"] = _b16(T, 2 * F)
        if path == "block":
            N, half, rows = case["qkv"], 64, 4096
            freq = 10000.0 ** (-torch.arange(half, device="cuda", dtype=torch.float64) / half)
            angle = torch.arange(rows, device="cuda", dtype=torch.float64)[:, None] * freq
            s.update(Wqkv=rnd.bf16((d, N), 0.02), Q=_b16(T, N), cos=angle.cos().float().contiguous(), sin=angle.sin().float().contiguous(),
                     # prompts follow one another; decoding tokens stand at any position
                     pos=rnd.ints(T, rows) if T <= 256 else (torch.arange(T, device="cuda") % 2048).to(torch.int32),
                     rope_cols=(d + (N - d) // 2) // 128 * 128)
            shapes.append((T, N, d))
        s["ws"] = _workspace(*shapes)
    elif path == "mlp_backward":
        F = case["inter"]
        X = rnd.bf16((T, d))
        s.update(X=X, dY=rnd.bf16((T, d), 1e-2), Z=rnd.bf16((T, 2 * F)), H=rnd.bf16((T, F)), Wup=rnd.bf16((d, 2 * F), 0.02), Wdown=rnd.bf16((F, d), 0.02),
                 gamma=rnd.uniform(d), rstd=(X.float().square().mean(1) + EPS).rsqrt(), dWdown=rnd.normal((F, d), 1e-3), dWup=rnd.normal((d, 2 * F), 1e-3),
                 dZ=_b16(T, 2 * F), part=_partials(T, F), stat=_f32(T), Xn=_b16(T, d), dX=_b16(T, d), dgpart=_f32(coda.coda_col_partial_blocks(T), d), dgamma=_f32(d))
        s["ws"] = _workspace((T, F, d), (F, d, T), (T, d, 2 * F), (d, 2 * F, T))
    else:
        V = case["vocab"]
        s.update(X=rnd.bf16((T, d)), W=rnd.bf16((d, V), 0.02), rstd=rnd.uniform(T), y=rnd.ints(T, V), logits=_b16(T, V), pmax=_partials(T, V),
                 psum=_partials(T, V), ztgt=_f32(T), loss=_f32(T))
        s["ws"] = _workspace((T, V, d))
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    return _RUN[s["case"]["path"]](s)


def _statistic(s):
    T, d = s["X"].shape
    coda.coda_row_sumsq(s["X"], s["ss"])
    coda.coda_row_finalize(s["ss"], T, 1, rstd_out=s["rstd"], d=d, eps=EPS)


def _linear(s):
    T, N = s["Y"].shape
    _statistic(s)
    coda.coda_gemm(s["X"], s["W"], [coda.row_scale(s["rstd"]), coda.add_tile(s["R"]), coda.row_sumsq(s["part"]), coda.store(s["Y"])], workspace=s["ws"])
    coda.coda_row_finalize(s["part"], T, s["part"].shape[0], sum_out=s["ssy"], d=N)
    return {"Y": s["Y"], "ssy": s["ssy"]}


def _mlp(s):
    T, d = s["Y"].shape
    f8, ws = s["case"].get("f8", False), s["ws"]
    out = {"Y": s["Y"], "H": s["H"], "rnext": s["rnext"]}
    if f8:
        # the row scales carry the quantisation scales and come with the quantised activations, those of X with its rstd
        trans = s["out_in"]
        coda.coda_gemm(s["X8"], s["Wup"], [coda.row_scale(s["xscale"]), coda.swiglu_fwd(), coda.store(s["H"])], transB=trans, workspace=ws)
        coda.coda_gemm(s["H8"], s["Wdown"], [coda.row_scale(s["hscale"]), coda.add_tile(s["X"]), coda.row_sumsq(s["part"]), coda.store(s["Y"])],
                       transB=trans, workspace=ws)
    else:
        if "Q" not in s:
            _statistic(s)
        up = coda.swiglu_fwd(s["Z"]) if "Z" in s else coda.swiglu_fwd()
        coda.coda_gemm(s["X"], s["Wup"], [coda.row_scale(s["rstd"]), up, coda.store(s["H"])], workspace=ws)
        coda.coda_gemm(s["H"], s["Wdown"], [coda.add_tile(s["X"]), coda.row_sumsq(s["part"]), coda.store(s["Y"])], workspace=ws)
        if "Z" in s:
            out["Z"] = s["Z"]
    coda.coda_row_finalize(s["part"], T, s["part"].shape[0], rstd_out=s["rnext"], d=d, eps=EPS)
    return out


def _block(s):
    _statistic(s)
    coda.coda_gemm(s["X"], s["Wqkv"], [coda.row_scale(s["rstd"]), coda.rope(s["cos"], s["sin"], s["pos"], 128, s["rope_cols"]), coda.store(s["Q"])],
                   workspace=s["ws"])
    return dict(_mlp(s), Q=s["Q"])


def _mlp_backward(s):
    T, d = s["X"].shape
    F = s["H"].shape[1]
    ws = s["ws"]
    coda.coda_gemm(s["dY"], s["Wdown"], [coda.swiglu_bwd(s["Z"], stat_out=s["part"]), coda.store(s["dZ"])], transB=True, workspace=ws)
    coda.coda_row_finalize(s["part"], T, s["part"].shape[0], sum_out=s["stat"], d=d)
    coda.coda_gemm(s["H"], s["dY"], [coda.accum_f32(s["dWdown"])], transA=True, workspace=ws)
    coda.coda_gemm(s["dZ"], s["Wup"], [coda.rmsnorm_bwd(s["X"], s["rstd"], s["stat"], s["gamma"], c_out=s["Xn"], dgamma_out=s["dgpart"], z_sum_over=d),
                                       coda.add_tile(s["dY"]), coda.store(s["dX"])], transB=True, workspace=ws)
    coda.coda_col_finalize(s["dgpart"], d, s["dgpart"].shape[0], s["dgamma"])
    coda.coda_gemm(s["Xn"], s["dZ"], [coda.accum_f32(s["dWup"])], transA=True, workspace=ws)
    return {"dX": s["dX"], "dZ": s["dZ"], "dWdown": s["dWdown"], "dWup": s["dWup"], "dgamma": s["dgamma"], "stat": s["stat"], "Xn": s["Xn"]}


def _lm_head(s):
    T = s["X"].shape[0]
    coda.coda_gemm(s["X"], s["W"], [coda.row_scale(s["rstd"]), coda.lse_partial(s["y"], s["pmax"], s["psum"], s["ztgt"]), coda.store(s["logits"])],
                   workspace=s["ws"])
    coda.coda_lse_finalize(s["pmax"], s["psum"], T, s["pmax"].shape[0], ztgt=s["ztgt"], loss_out=s["loss"])
    return {"logits": s["logits"], "loss": s["loss"]}


_RUN = {"linear": _linear, "block": _block, "mlp": _mlp, "mlp_backward": _mlp_backward, "lm_head": _lm_head}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Every input read once, every output written once; operations of the matrix products only."""
    T, d, path = case["tokens"], case["hidden"], case["path"]
    if path == "linear":
        N = case["out"]
        return {"bytes": 2.0 * (T * d + d * N + 2 * T * N) + 4.0 * T, "flops": 2.0 * T * d * N}
    if path in ("block", "mlp"):
        F, q = case["inter"], case.get("qkv", 0)
        w = 1 if case.get("f8") else 2
        nbytes = w * (3.0 * d * F + d * q) + 2.0 * T * d + 2.0 * T * (F + d + q) + 4.0 * T
        if case.get("f8"):
            nbytes += T * (d + F)          # the quantised activations
        if case.get("save"):
            nbytes += 4.0 * T * F
        return {"bytes": nbytes, "flops": 2.0 * T * d * (3 * F + q)}
    if path == "mlp_backward":
        F = case["inter"]
        return {"bytes": 2.0 * T * (2 * d + 3 * F) + 2.0 * 3 * d * F + 2.0 * T * (2 * F + 2 * d) + 2 * 4.0 * 3 * d * F, "flops": 2.0 * T * d * 6 * F}
    V = case["vocab"]
    return {"bytes": 2.0 * (T * d + d * V + T * V) + 16.0 * T, "flops": 2.0 * T * d * V}


def tolerance(case):
    # Against the same chains in 64 bits with the same bf16 roundings of what is stored, the outputs are off by up to
    # rel 3.2e-4 and by one bf16 step, 2^-7 of the value, at the worst element; four times that.
    return {"rel": 1.3e-3, "max": 0.032}
