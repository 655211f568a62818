"""The calls whose speed counts, as a training program makes them through the public entry points.

Six kinds of call:

  step       tm_stage_fwd + tm_stage_bwd_adam: the last micro-batch of an iteration on one rank's transformer layers
  accum      tm_stage_fwd + tm_stage_bwd in TM_GRAD_ADD mode: a middle micro-batch of such an iteration
  attn       tm_op_attn_fwd + tm_op_attn_bwd
  linear     the products of one linear map: forward, input gradient, weight gradient, bias gradient
  ends       what the first and the last pipeline stage have: embedding and output layer, forward and backward
  moe        the mixture-of-experts MLP shard, forward and backward
  optimizer  squared gradient norm and Adam on a flat slice (a distributed optimizer's rank)

Sizes are LOCAL to a rank and come from the presets in synth_inputs.py, from the tests, or are generic (head sizes 32
to 128, sequences and widths that are no multiple of a tile).  Values follow synth_inputs.py's recipe: matrices and
biases N(0, 0.02^2), gains 1 + N(0, 0.02^2), activations N(0, 1), output gradients N(0, 1e-4).
"""
from __future__ import annotations

import math

import torch

import paper_2412_12636_amd as tm

LN, RMS = tm.TM_NORM_LAYERNORM, tm.TM_NORM_RMSNORM
TANH, ERF, SWIGLU = tm.TM_ACT_GELU_TANH, tm.TM_ACT_GELU_ERF, tm.TM_ACT_SWIGLU
EPS, THETA = 1e-5, 10000.0
LR, BETA1, BETA2, ADAM_EPS = 1e-5, 0.9, 0.999, 1e-8
FIRST_STEP = 1000   # a run that is under way: the bias corrections are near 1


# ---- the cases -----------------------------------------------------------------------------------------------------
def _stage(kind, layers, hidden, nq, nkv, d, ffn, seq, batch, dtype="bf16", norm=LN, act=TANH, rotary=False, bias=True,
           tune=False):
    return dict(kind=kind, layers=layers, hidden=hidden, nq=nq, nkv=nkv, d=d, ffn=ffn, seq=seq, batch=batch, dtype=dtype,
                norm=norm, act=act, rotary=rotary, bias=bias, tune=tune)


def _attn(seq, batch, nq, nkv, d, dtype="bf16"):
    return dict(kind="attn", seq=seq, batch=batch, nq=nq, nkv=nkv, d=d, dtype=dtype)


def _linear(T, N, K, dtype="bf16", bias=True, residual=True, accumulate=True):
    return dict(kind="linear", T=T, N=N, K=K, dtype=dtype, bias=bias, residual=residual, accumulate=accumulate)


def _ends(seq, batch, hidden, vocab, dtype="bf16", norm=LN, positions=True):
    return dict(kind="ends", seq=seq, batch=batch, hidden=hidden, vocab=vocab, dtype=dtype, norm=norm, positions=positions)


def _moe(tokens, hidden, ffn, experts, ep, top_k, capacity, dtype="bf16", act=TANH, bias=True):
    return dict(kind="moe", tokens=tokens, hidden=hidden, ffn=ffn, experts=experts, ep=ep, top_k=top_k, capacity=capacity,
                dtype=dtype, act=act, bias=bias)


def _optimizer(n, dtype="bf16"):
    return dict(kind="optimizer", n=n, dtype=dtype)


def listed():
    cases = {
        # the "tiny" preset, fp32 end to end: what a functional run of the training loop calls; launch latency
        "step_tiny_fp32": _stage("step", 2, 256, 4, 4, 64, 1024, 128, 2, dtype="fp32"),
        # a small model trained in fp32 (a reference run beside a bf16 one)
        "step_small_fp32": _stage("step", 1, 1024, 16, 16, 64, 4096, 512, 2, dtype="fp32", norm=RMS, act=SWIGLU, rotary=True,
                                  bias=False),
        # a small GPT on one GPU: 16 heads of 64, several sequences of ragged length per micro-batch
        "step_small_bf16": _stage("step", 1, 1024, 16, 16, 64, 4096, 1000, 4, act=ERF),
        # the "gpt6p7b" shard (two of its four layers), untuned as most callers run it
        "step_gpt6p7b": _stage("step", 2, 4096, 4, 4, 128, 2048, 2048, 1),
        # one layer of the "gpt175b" shard, the benchmark's workload, after tm_stage_tune as the benchmark runs it
        "step_gpt175b": _stage("step", 1, 12288, 12, 12, 128, 6144, 2048, 1, tune=True),
        # one layer of the "llama70b" shard in the middle of an iteration of several micro-batches
        "accum_llama70b": _stage("accum", 1, 8192, 8, 1, 128, 3584, 4096, 1, norm=RMS, act=SWIGLU, rotary=True, bias=False),
        # the "longctx" shard's attention
        "attn_longctx": _attn(16384, 1, 8, 1, 128),
        # attention of a small grouped-query model: head size 64, ragged sequence
        "attn_gqa_d64": _attn(1500, 2, 16, 4, 64),
        # a linear map of generic ragged sizes: no dimension a multiple of 64
        "linear_ragged": _linear(1000, 5128, 3080),
        # both ends of the pipeline at the "gpt175b" shard: 51200 / 8 vocabulary rows
        "ends_gpt175b": _ends(2048, 1, 12288, 6400),
        # the "moe5t" shard: top-2 of 16 experts, one local expert, capacity factor 1
        "moe_moe5t": _moe(2048, 20480, 10240, 16, 16, 2, 256),
        # the Adam sweep over 1.2e9 elements, after the gradient norm
        "optimizer_1p2b": _optimizer(1_200_000_000),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log(rng, low, high, multiple=1):
    v = math.exp(rng.uniform(math.log(low), math.log(high)))
    return max(multiple, int(round(v / multiple)) * multiple)


def _draw(rng):
    kind = rng.choices(["step", "accum", "attn", "linear", "ends", "moe", "optimizer"], [28, 12, 22, 16, 8, 6, 8])[0]
    dtype = "fp32" if rng.random() < 0.25 else "bf16"
    small = dtype == "fp32"
    if kind in ("step", "accum"):
        d = rng.choice([32, 64, 64, 80, 96, 128, 128, 128])
        hidden = _log(rng, 256, 2048 if small else 12288, rng.choice([8, 64, 256]))
        nq = rng.choice([n for n in (2, 4, 8, 12, 16) if n * d <= hidden])
        nkv = rng.choice([n for n in (1, 2, 4, 8, 12, 16) if nq % n == 0])
        llama = rng.random() < 0.5
        return _stage(kind, rng.choice([1, 1, 2]), hidden, nq, nkv, d,
                      _log(rng, 256, 4096 if small else 8192, rng.choice([8, 64, 256])), _log(rng, 64, 1024 if small else 4096),
                      rng.choice([1, 1, 2, 4]), dtype=dtype, norm=RMS if llama else LN,
                      act=SWIGLU if llama else rng.choice([TANH, ERF]), rotary=llama, bias=not llama)
    if kind == "attn":
        d = rng.choice([32, 64, 64, 80, 96, 128, 128, 128])
        nq = rng.choice([2, 4, 8, 12, 16, 32])
        nkv = rng.choice([n for n in (1, 2, 4, 8, 12, 16, 32) if nq % n == 0])
        return _attn(_log(rng, 64, 12288 if d == 128 and not small else 1536 if not small else 1024), rng.choice([1, 1, 2, 4]), nq,
                     nkv, d, dtype)
    if kind == "linear":
        m = rng.choice([8, 8, 64, 128])
        top = 2048 if small else 12288
        return _linear(_log(rng, 16, 2048 if small else 8192), _log(rng, 128, top, m), _log(rng, 128, top, m), dtype,
                       rng.random() < 0.5, rng.random() < 0.5, rng.random() < 0.5)
    if kind == "ends":
        return _ends(_log(rng, 64, 512 if small else 4096), rng.choice([1, 2]), _log(rng, 256, 1024 if small else 12288, 64),
                     _log(rng, 1000, 8000, 8), dtype, rng.choice([LN, RMS]), rng.random() < 0.5)
    if kind == "moe":
        ep = rng.choice([2, 4, 8])
        tokens, experts, top_k = _log(rng, 128, 512 if small else 4096), ep * rng.choice([1, 2]), rng.choice([1, 2])
        return _moe(tokens, _log(rng, 256, 1024 if small else 8192, 64), _log(rng, 256, 1024 if small else 8192, 64), experts, ep, top_k,
                    max(1, int(1.25 * tokens * top_k / experts)), dtype, rng.choice([TANH, ERF]), rng.random() < 0.5)
    return _optimizer(_log(rng, 100_000, 1_000_000_000, 8), dtype)


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        if w["flops"] <= (8e10 if c["dtype"] == "fp32" else 5e12) and w["bytes"] <= 3.6e10:
            return c


# ---- inputs (plain torch; made on the GPU from the seed alone) ------------------------------------------------------
def _td(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _dtype(case):
    return tm.TM_DTYPE_BF16 if case["dtype"] == "bf16" else tm.TM_DTYPE_FP32


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, std, td, mean=0.0):
    t = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(mean, std, generator=g)
    return t.to(td)


def _stage_layout(c):
    """Tensors of one layer in flat-buffer order."""
    h, A, f = c["hidden"], c["nq"] * c["d"], c["ffn"]
    qkv, f1 = A + 2 * c["nkv"] * c["d"], 2 * f if c["act"] == SWIGLU else f
    ln, b = c["norm"] == LN, c["bias"]
    out = [("norm1_gain", (h,)), ("norm1_offset", (h,) if ln else None), ("w_qkv", (qkv, h)), ("b_qkv", (qkv,) if b else None),
           ("w_out", (h, A)), ("b_out", (h,) if b else None), ("norm2_gain", (h,)), ("norm2_offset", (h,) if ln else None),
           ("w_fc1", (f1, h)), ("b_fc1", (f1,) if b else None), ("w_fc2", (h, f)), ("b_fc2", (h,) if b else None)]
    return [(n, s) for n, s in out if s is not None]


def _moe_layout(c):
    out = [("w_router", (c["experts"], c["hidden"]))]
    for j in range(c["experts"] // c["ep"]):
        out += [("w_fc1.%d" % j, (c["ffn"], c["hidden"])), ("b_fc1.%d" % j, (c["ffn"],) if c["bias"] else None),
                ("w_fc2.%d" % j, (c["hidden"], c["ffn"])), ("b_fc2.%d" % j, (c["hidden"],) if c["bias"] else None)]
    return [(n, s) for n, s in out if s is not None]


def _count(layout):
    return sum(math.prod(s) for _, s in layout)


def _adam_state(g, n):
    """Moments of a run that is under way, for gradients of the size these inputs give."""
    m = _normal(g, (n,), 1e-4, torch.float32)
    v = torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, 1e-3, generator=g)
    return m, v.mul_(v).mul_(1e-1)


def _inputs(c, seed):
    g, td, k = _gen(seed), _td(c), c["kind"]
    if k in ("step", "accum"):
        lay = _stage_layout(c)
        n1 = _count(lay)
        params = _normal(g, (c["layers"] * n1,), 0.02, td)
        off = 0
        for _ in range(c["layers"]):
            for name, shape in lay:
                n = math.prod(shape)
                if name.endswith("_gain"):
                    params[off:off + n] += 1.0
                off += n
        shape = (c["seq"], c["batch"], c["hidden"])
        s = dict(params=params, x=_normal(g, shape, 1.0, td), dy=_normal(g, shape, 1e-2, td))
        if k == "accum":
            s["grads"] = _normal(g, (params.numel(),), 1e-2, torch.float32)   # the micro-batches before
        else:
            s["m"], s["v"] = _adam_state(g, params.numel())
        return s
    if k == "attn":
        rows = (c["seq"], c["batch"])
        return dict(qkv=_normal(g, rows + ((c["nq"] + 2 * c["nkv"]) * c["d"],), 1.0, td),
                    dctx=_normal(g, rows + (c["nq"] * c["d"],), 1e-2, td))
    if k == "linear":
        T, N, K = c["T"], c["N"], c["K"]
        return dict(x=_normal(g, (T, K), 1.0, td), w=_normal(g, (N, K), 0.02, td), bias=_normal(g, (N,), 0.02, td) if c["bias"] else None,
                    residual=_normal(g, (T, N), 1.0, td) if c["residual"] else None, dy=_normal(g, (T, N), 1e-2, td),
                    dw=_normal(g, (N, K), 1e-2, torch.float32), db=_normal(g, (N,), 1e-2, torch.float32))
    if k == "ends":
        s, b, h, V = c["seq"], c["batch"], c["hidden"], c["vocab"]
        ids = lambda: torch.randint(0, 8 * V, (s, b), generator=g, device="cuda", dtype=torch.int32)  # one of 8 shards is local
        return dict(tokens=ids(), targets=ids(), w=_normal(g, (V, h), 0.02, td), pos=_normal(g, (s, h), 0.02, td) if c["positions"] else None,
                    y=_normal(g, (s, b, h), 1.0, td), gain=_normal(g, (h,), 0.02, td, 1.0),
                    offset=_normal(g, (h,), 0.02, td) if c["norm"] == LN else None, dx0=_normal(g, (s, b, h), 1e-2, td))
    if k == "moe":
        lay = _moe_layout(c)
        params = _normal(g, (_count(lay),), 0.02, td)
        rows = (c["tokens"], c["hidden"])
        return dict(params=params, c=_normal(g, rows, 1.0, td), dout=_normal(g, rows, 1e-2, td))
    n = c["n"]
    p = _normal(g, (n,), 0.02, torch.float32)
    s = dict(p=p, g=_normal(g, (n,), 1e-3, torch.float32))
    s["m"], s["v"] = _adam_state(g, n)
    return s


# ---- prepare and run ------------------------------------------------------------------------------------------------
class _Stage:
    """A stage handle with the attributes of the public configuration."""

    def __init__(self, c, params, master, grads, m, v, stream):
        self.n_layers, self.hidden, self.n_q_heads, self.n_kv_heads = c["layers"], c["hidden"], c["nq"], c["nkv"]
        self.head_dim, self.ffn, self.seq, self.micro_batch, self.dtype = c["d"], c["ffn"], c["seq"], c["batch"], _dtype(c)
        self.norm, self.act, self.pos, self.has_bias = c["norm"], c["act"], int(c["rotary"]), int(c["bias"])
        self.norm_eps, self.rope_theta = EPS, THETA
        self.ws = torch.empty(tm.tm_stage_workspace_bytes(self), dtype=torch.uint8, device="cuda")
        self.handle = tm.tm_stage_init(self, params, master, grads, m, v, self.ws)
        if c["tune"]:
            tm.tm_stage_tune(self.handle, stream)

    def __del__(self):
        if getattr(self, "handle", None):
            tm.tm_stage_destroy(self.handle)


class _Moe:
    def __init__(self, c):
        self.tokens, self.hidden, self.ffn, self.n_experts, self.ep = c["tokens"], c["hidden"], c["ffn"], c["experts"], c["ep"]
        self.top_k, self.capacity, self.dtype, self.act, self.has_bias = c["top_k"], c["capacity"], _dtype(c), c["act"], int(c["bias"])


def _bytes(n):
    return torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    td, k = _td(c), c["kind"]
    s["case"], s["stream"] = c, int(torch.cuda.current_stream().cuda_stream)
    new32 = lambda *shape: torch.empty(shape, dtype=torch.float32, device="cuda")
    if k in ("step", "accum"):
        n = s["params"].numel()
        s["master"] = s["params"].float() if td == torch.bfloat16 else None
        if k == "step":
            s["grads"] = torch.zeros(n, dtype=torch.float32, device="cuda")
        else:
            s["m"], s["v"] = (torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(2))
        s["stage"] = _Stage(c, s["params"], s["master"], s["grads"], s["m"], s["v"], s["stream"])
        tm.tm_stage_grad_mode(s["stage"].handle, tm.TM_GRAD_TRANSIENT if k == "step" else tm.TM_GRAD_ADD)
        s["hp"], s["step"] = tm.make_hparams(LR, BETA1, BETA2, ADAM_EPS), FIRST_STEP
        s["y"], s["dx"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
    elif k == "attn":
        s["ctx"], s["dqkv"] = torch.empty_like(s["dctx"]), torch.empty_like(s["qkv"])
        s["lse"] = new32(c["batch"], c["nq"], c["seq"])
        s["scratch"] = _bytes(tm.tm_op_attn_bwd_scratch_bytes(_dtype(c), c["seq"], c["batch"], c["nq"], c["nkv"], c["d"]))
    elif k == "linear":
        s["y"], s["dx"] = torch.empty_like(s["dy"]), torch.empty_like(s["x"])
        s["split"] = tm.tm_op_linear_dgrad_scratch_bytes(_dtype(c), c["T"], c["N"], c["K"])
        s["scratch"] = _bytes(max(s["split"], tm.tm_op_reduce_scratch_bytes(c["T"], c["N"])))
    elif k == "ends":
        h, V = c["hidden"], c["vocab"]
        s["ws"] = _bytes(tm.tm_head_workspace_bytes(_dtype(c), c["seq"], c["batch"], h, V))
        s["x0"], s["out"] = torch.empty_like(s["dx0"]), torch.empty_like(s["y"])
        s["dw"], s["loss"], s["dgain"] = new32(V, h), new32(1), new32(h)
        s["doffset"] = new32(h) if c["norm"] == LN else None
        s["dpos"] = new32(c["seq"], h).zero_() if c["positions"] else None
    elif k == "moe":
        s["cfg"] = _Moe(c)
        s["ws"] = _bytes(tm.tm_moe_workspace_bytes(s["cfg"]))
        s["out"], s["dc"], s["grads"] = torch.empty_like(s["c"]), torch.empty_like(s["c"]), new32(s["params"].numel())
    else:
        s["p16"] = s["p"].to(torch.bfloat16) if td == torch.bfloat16 else None
        s["scratch"] = _bytes(tm.tm_sq_sum_scratch_bytes(c["n"]))
        s["norm2"] = torch.empty(1, dtype=torch.float64, device="cuda")
        s["hp"], s["step"] = tm.make_hparams(LR, BETA1, BETA2, ADAM_EPS), FIRST_STEP
    return s


def run(s):
    c, st = s["case"], s["stream"]
    k, dt = c["kind"], _dtype(c)
    if k in ("step", "accum"):
        h = s["stage"].handle
        tm.tm_stage_fwd(h, s["x"], s["y"], st)
        if k == "accum":
            tm.tm_stage_bwd(h, s["dy"], s["dx"], st)
            return dict(y=s["y"], dx=s["dx"], grads=s["grads"])
        tm.tm_stage_bwd_adam(h, s["dy"], s["dx"], s["hp"], s["step"], st)
        s["step"] += 1
        return dict(y=s["y"], dx=s["dx"], params=s["params"], master=s["master"], m=s["m"], v=s["v"])
    if k == "attn":
        dims = (dt, c["seq"], c["batch"], c["nq"], c["nkv"], c["d"])
        tm.tm_op_attn_fwd(*dims, s["qkv"], s["ctx"], s["lse"], st)
        tm.tm_op_attn_bwd(*dims, s["qkv"], s["ctx"], s["dctx"], s["lse"], s["scratch"], s["dqkv"], st)
        return dict(ctx=s["ctx"], lse=s["lse"], dqkv=s["dqkv"])
    if k == "linear":
        dims, acc = (dt, c["T"], c["N"], c["K"]), int(c["accumulate"])
        tm.tm_op_linear_fwd(*dims, s["x"], s["w"], s["bias"], s["residual"], s["y"], st)
        tm.tm_op_linear_dgrad_ws(*dims, s["dy"], s["w"], s["dx"], s["scratch"], s["split"], st)
        tm.tm_op_linear_wgrad(*dims, s["dy"], s["x"], s["dw"], acc, st)
        if c["bias"]:
            tm.tm_op_bias_grad(dt, c["T"], c["N"], s["dy"], s["db"], s["scratch"], acc, st)
        return dict(y=s["y"], dx=s["dx"], dw=s["dw"], db=s["db"])
    if k == "ends":
        sq, b, hd, V = c["seq"], c["batch"], c["hidden"], c["vocab"]
        tm.tm_op_embed_fwd(dt, sq, b, hd, V, 0, s["tokens"], s["w"], s["pos"], s["x0"], st)
        tm.tm_head_fwd_bwd(dt, c["norm"], EPS, sq, b, hd, V, 0, s["y"], s["targets"], s["gain"], s["offset"], s["w"], 1.0, s["ws"],
                           s["loss"], s["out"], s["dgain"], s["doffset"], s["dw"], 0, st)
        # the two layers share their weights, so their gradients add up
        tm.tm_op_embed_bwd(dt, sq, b, hd, V, 0, s["tokens"], s["dx0"], s["dw"], s["dpos"], sq, 1, st)
        return dict(x0=s["x0"], loss=s["loss"], dy=s["out"], dgain=s["dgain"], doffset=s["doffset"], dw=s["dw"], dpos=s["dpos"])
    if k == "moe":
        tm.tm_moe_fwd(s["cfg"], s["params"], s["c"], s["out"], s["ws"], st)
        tm.tm_moe_bwd(s["cfg"], s["params"], s["c"], s["dout"], s["dc"], s["grads"], 0, s["ws"], st)
        return dict(out=s["out"], dc=s["dc"], grads=s["grads"])
    tm.tm_sq_sum(c["n"], s["g"], s["scratch"], s["norm2"], st)
    tm.tm_adam_step_flat(c["n"], s["p"], s["g"], s["m"], s["v"], s["p16"], s["hp"], s["step"], st)
    s["step"] += 1
    return dict(norm2=s["norm2"], p=s["p"], m=s["m"], v=s["v"], p16=s["p16"])


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def work(case):
    c = case
    es, k = (2 if c["dtype"] == "bf16" else 4), c["kind"]
    if k in ("step", "accum"):
        n = c["layers"] * _count(_stage_layout(c))
        weights = c["layers"] * sum(math.prod(s) for _, s in _stage_layout(c) if len(s) == 2)
        T = c["seq"] * c["batch"]
        # weights and optimizer state in and out (accum: the gradient buffer in and out); x, dy in, y, dx out
        state = n * (es + (es + 24 if es == 2 else 24)) if k == "step" else n * (es + 8)
        return dict(bytes=state + 4 * T * c["hidden"] * es,
                    flops=6 * T * weights + 6 * c["layers"] * c["batch"] * c["nq"] * c["seq"] ** 2 * c["d"])
    if k == "attn":
        rows = c["seq"] * c["batch"]
        return dict(bytes=rows * c["d"] * es * (2 * (c["nq"] + 2 * c["nkv"]) + 2 * c["nq"]) + rows * c["nq"] * 4,
                    flops=6 * c["batch"] * c["nq"] * c["seq"] ** 2 * c["d"])
    if k == "linear":
        T, N, K = c["T"], c["N"], c["K"]
        return dict(bytes=es * (2 * T * K + N * K + T * N * (3 if c["residual"] else 2)) + N * K * (8 if c["accumulate"] else 4),
                    flops=6 * T * N * K)
    if k == "ends":
        T, h, V = c["seq"] * c["batch"], c["hidden"], c["vocab"]
        return dict(bytes=es * (4 * T * h + V * h) + 4 * V * h, flops=6 * T * h * V)
    if k == "moe":
        n, rows = _count(_moe_layout(c)), c["experts"] * c["capacity"]
        return dict(bytes=n * (es + 4) + 4 * c["tokens"] * c["hidden"] * es,
                    flops=12 * rows * c["hidden"] * c["ffn"] + 6 * c["tokens"] * c["hidden"] * c["experts"])
    return dict(bytes=c["n"] * (28 + (2 if es == 2 else 0)), flops=16 * c["n"])


def tolerance(case):
    """About four times what the calls are off exact() on their first pass: 1.4e-6 in fp32; in bf16 2.4e-3 for attention and
    products, 4.8e-3 at the ends, and 1.6e-2 for a layer at hidden 12288, whose attention scores amplify its roundings."""
    if case["kind"] == "optimizer":
        return dict(rel=1e-5) if case["dtype"] == "fp32" else dict(rel=1e-4, max=1e-2)   # a flipped rounding of the bf16 copy
    if case["dtype"] == "fp32":
        return dict(rel=1e-5, max=1e-3)
    if case["kind"] in ("step", "accum"):
        return dict(rel=3e-2, max=0.9)
    return dict(rel=2e-2 if case["kind"] == "ends" else 1e-2, max=0.4)


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------
def _d(t):
    return None if t is None else t.double()


def _norm64(x, gain, offset, kind):
    if kind == LN:
        x = x - x.mean(-1, keepdim=True)
    xh = x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS)
    return xh * gain + offset if offset is not None else xh * gain


def _gelu64(u, act):
    if act == ERF:
        return 0.5 * u * (1.0 + torch.erf(u / math.sqrt(2.0)))
    return 0.5 * u * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (u + 0.044715 * u ** 3)))


def _rotate64(z):
    s, d = z.shape[0], z.shape[-1]
    a = torch.arange(s, dtype=torch.float64, device=z.device)[:, None] * THETA ** (
        -2.0 * torch.arange(d // 2, dtype=torch.float64, device=z.device) / d)[None, :]
    cos, sin = torch.cos(a)[:, None, None, :], torch.sin(a)[:, None, None, :]
    lo, hi = z[..., :d // 2], z[..., d // 2:]
    return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)


class _Attn64(torch.autograd.Function):
    """Causal attention of [s, b, heads, d] tensors, one head at a time; probabilities are formed again for the gradient."""

    @staticmethod
    def _probs(q, k):
        s = q.shape[0]
        sc = (q @ k.t()).div_(math.sqrt(q.shape[1]))
        sc.masked_fill_(torch.ones((s, s), dtype=torch.bool, device=q.device).triu_(1), -math.inf)
        lse = torch.logsumexp(sc, 1)
        return sc.sub_(lse[:, None]).exp_(), lse

    @staticmethod
    def forward(ctx, q, k, v):
        ctx.save_for_backward(q, k, v)
        group, out = q.shape[2] // k.shape[2], torch.empty_like(q)
        lse = torch.empty((q.shape[1], q.shape[2], q.shape[0]), dtype=torch.float64, device=q.device)
        for n in range(q.shape[1]):
            for h in range(q.shape[2]):
                p, lse[n, h] = _Attn64._probs(q[:, n, h], k[:, n, h // group])
                out[:, n, h] = p @ v[:, n, h // group]
        ctx.mark_non_differentiable(lse)
        return out, lse

    @staticmethod
    def backward(ctx, do, _):
        q, k, v = ctx.saved_tensors
        group = q.shape[2] // k.shape[2]
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        for n in range(q.shape[1]):
            for h in range(q.shape[2]):
                j = h // group
                p, _ = _Attn64._probs(q[:, n, h], k[:, n, j])
                dv[:, n, j] += p.t() @ do[:, n, h]
                dp = do[:, n, h] @ v[:, n, j].t()
                ds = p.mul_(dp - (dp * p).sum(1, keepdim=True)).div_(math.sqrt(q.shape[3]))
                dq[:, n, h] = ds @ k[:, n, j]
                dk[:, n, j] += ds.t() @ q[:, n, h]
        return dq, dk, dv


def _split_heads(c, qkv):
    s, b, A, B = c["seq"], c["batch"], c["nq"] * c["d"], c["nkv"] * c["d"]
    return (qkv[..., :A].reshape(s, b, c["nq"], c["d"]), qkv[..., A:A + B].reshape(s, b, c["nkv"], c["d"]),
            qkv[..., A + B:].reshape(s, b, c["nkv"], c["d"]))


def _layer64(c, p, x):
    q, k, v = _split_heads(c, torch.nn.functional.linear(_norm64(x, p["norm1_gain"], p.get("norm1_offset"), c["norm"]), p["w_qkv"],
                                                         p.get("b_qkv")))
    if c["rotary"]:
        q, k = _rotate64(q), _rotate64(k)
    a = _Attn64.apply(q.contiguous(), k.contiguous(), v.contiguous())[0]
    x = x + torch.nn.functional.linear(a.reshape(c["seq"], c["batch"], -1), p["w_out"], p.get("b_out"))
    u = torch.nn.functional.linear(_norm64(x, p["norm2_gain"], p.get("norm2_offset"), c["norm"]), p["w_fc1"], p.get("b_fc1"))
    if c["act"] == SWIGLU:
        f = c["ffn"]
        g = u[..., :f] * torch.sigmoid(u[..., :f]) * u[..., f:]
    else:
        g = _gelu64(u, c["act"])
    return x + torch.nn.functional.linear(g, p["w_fc2"], p.get("b_fc2"))


def _adam64(p, g, m, v):
    m = BETA1 * m.double() + (1 - BETA1) * g
    v = BETA2 * v.double() + (1 - BETA2) * g * g
    return p.double() - LR * (m / (1 - BETA1 ** FIRST_STEP)) / (torch.sqrt(v / (1 - BETA2 ** FIRST_STEP)) + ADAM_EPS), m, v


def exact(case, seed):
    c, k = case, case["kind"]
    s = _inputs(c, seed)
    if k in ("step", "accum"):
        flat = s["params"].double().requires_grad_()
        x = s["x"].double().requires_grad_()
        y, off = x, 0
        for _ in range(c["layers"]):
            p = {}
            for name, shape in _stage_layout(c):
                n = math.prod(shape)
                p[name] = flat[off:off + n].view(shape)
                off += n
            y = _layer64(c, p, y)
        y.backward(s["dy"].double())
        y = y.detach()
        if k == "accum":
            return dict(y=y, dx=x.grad, grads=flat.grad.add_(s["grads"]))
        p, m, v = _adam64(flat.detach(), flat.grad, s["m"], s["v"])
        return dict(y=y, dx=x.grad, params=p, master=p if c["dtype"] == "bf16" else None, m=m, v=v)
    if k == "attn":
        qkv = s["qkv"].double().requires_grad_()
        ctx, lse = _Attn64.apply(*[t.contiguous() for t in _split_heads(c, qkv)])
        ctx = ctx.reshape(s["dctx"].shape)
        ctx.backward(s["dctx"].double())
        return dict(ctx=ctx.detach(), lse=lse, dqkv=qkv.grad)
    if k == "linear":
        x, w, dy = _d(s["x"]), _d(s["w"]), _d(s["dy"])
        y = x @ w.t()
        if c["bias"]:
            y = y + _d(s["bias"])
        if c["residual"]:
            y = y + _d(s["residual"])
        acc = 1.0 if c["accumulate"] else 0.0
        return dict(y=y, dx=dy @ w, dw=dy.t() @ x + acc * _d(s["dw"]), db=dy.sum(0) + acc * _d(s["db"]) if c["bias"] else _d(s["db"]))
    if k == "ends":
        sq, b, h, V = c["seq"], c["batch"], c["hidden"], c["vocab"]
        w, y, gain = (s[n].double().requires_grad_() for n in ("w", "y", "gain"))
        offset = None if s["offset"] is None else s["offset"].double().requires_grad_()
        rows = lambda ids: (ids.reshape(-1).long(), ids.reshape(-1) < V)
        logits = _norm64(y, gain, offset, c["norm"]).reshape(sq * b, h) @ w.t()
        t, here = rows(s["targets"])
        loss = (torch.logsumexp(logits, 1) - torch.where(here, logits.gather(1, t.clamp(max=V - 1)[:, None])[:, 0], 0.0)).mean()
        loss.backward()
        t, here = rows(s["tokens"])
        x0 = torch.where(here[:, None], w.detach()[t.clamp(max=V - 1)], 0.0).reshape(sq, b, h)
        dx0 = s["dx0"].double()
        dw = w.grad.index_add_(0, t[here], dx0.reshape(sq * b, h)[here])
        if c["positions"]:
            x0 = x0 + s["pos"].double()[:, None, :]
        return dict(x0=x0, loss=loss.detach().reshape(1), dy=y.grad, dgain=gain.grad, doffset=None if offset is None else offset.grad, dw=dw,
                    dpos=dx0.sum(1) if c["positions"] else None)
    if k == "moe":
        T, E, C, el = c["tokens"], c["experts"], c["capacity"], c["experts"] // c["ep"]
        flat, x = s["params"].double().requires_grad_(), s["c"].double().requires_grad_()
        p, off = {}, 0
        for name, shape in _moe_layout(c):
            n = math.prod(shape)
            p[name] = flat[off:off + n].view(shape)
            off += n
        chosen, idx = torch.topk(x @ p["w_router"].t(), c["top_k"], dim=1)
        gates = torch.softmax(chosen, 1)
        taken = torch.nn.functional.one_hot(idx.reshape(-1), E)              # assignments in token order
        place = (taken.cumsum(0) - taken).gather(1, idx.reshape(-1, 1)).reshape(T, -1)
        out = torch.zeros_like(x)
        for e in range(E):
            t, i = torch.nonzero((idx == e) & (place < C), as_tuple=True)
            j = e % el
            u = torch.nn.functional.linear(x[t], p["w_fc1.%d" % j], p.get("b_fc1.%d" % j))
            o = torch.nn.functional.linear(_gelu64(u, c["act"]), p["w_fc2.%d" % j], p.get("b_fc2.%d" % j))
            out = out.index_add(0, t, gates[t, i][:, None] * o)
        out.backward(s["dout"].double())
        return dict(out=out.detach(), dc=x.grad, grads=flat.grad)
    g = s["g"].double()
    p, m, v = _adam64(s["p"], g, s["m"], s["v"])
    return dict(norm2=(g * g).sum().reshape(1), p=p, m=m, v=v, p16=p if c["dtype"] == "bf16" else None)
