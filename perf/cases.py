"""Performance cases of the framework: the work that a training program has it do, through its public entry points.

Most cases are single layers and blocks (a Linear layer forward and backward with the parameter update, attention, a
LayerNorm, the output head with its loss) called through paper_2107_06469_amd.ops for a group of models; two are whole
training epochs through paper_2107_06469_amd.hydra.  Sizes are those of the workload configurations and of the scaled
replicas that the tests train.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, weights, optimizer state and buffers on the device
    run(state)           one pass; returns its outputs
    work(case)           bytes and flops that one pass cannot do without
    tolerance(case)      how far another correct implementation at the same precision may be off
    exact(case, seed)    the same outputs from plain torch in 64 bits
"""
from __future__ import annotations

import math

import numpy as np
import torch

BF16, F32 = "bf16", "f32"
ADAM_T = 10                                   # optimizer steps taken before a layer's backward pass is timed
B1, B2, EPS = 0.9, 0.999, 1e-8


# ---- the cases --------------------------------------------------------------------------------------------------------

def _linear_fwd(name, G, rows, d_in, d_out, dtype, epi, act="gelu"):
    return dict(name=name, kind="linear_fwd", G=G, rows=rows, d_in=d_in, d_out=d_out, dtype=dtype, epi=epi, act=act)


def _linear_bwd(name, G, rows, d_in, d_out, dtype, gate, act, opt):
    return dict(name=name, kind="linear_bwd", G=G, rows=rows, d_in=d_in, d_out=d_out, dtype=dtype, gate=gate, act=act, opt=opt)


def _attention(name, G, B, S, H, DH, causal):
    return dict(name=name, kind="attention", G=G, B=B, S=S, H=H, DH=DH, causal=causal)


def _layernorm(name, G, rows, d, dtype):
    return dict(name=name, kind="layernorm", G=G, rows=rows, d=d, dtype=dtype)


def _head(name, G, rows, d, V):
    return dict(name=name, kind="head", G=G, rows=rows, d=d, V=V)


def _train_mlp(name, K, layers, d_in, d, out, batch, steps, act, opt, dtype):
    return dict(name=name, kind="train_mlp", K=K, layers=layers, d_in=d_in, d=d, out=out, batch=batch, steps=steps, act=act,
                opt=opt, dtype=dtype)


def _train_encoder(name, K, layers, d, H, ffn, V, S, batch, targets, steps):
    return dict(name=name, kind="train_encoder", K=K, layers=layers, d=d, H=H, ffn=ffn, V=V, S=S, batch=batch, targets=targets,
                steps=steps)


def listed():
    return [
        # one epoch of 4 small fp32 MLPs trained side by side with SGD: launches and latency are all it costs
        _train_mlp("train_mlp256_f32", 4, 4, 256, 256, 10, 32, 10, "relu", "sgd", F32),
        # one epoch of 4 small bf16 encoders trained with Adam: every kind of kernel, at sizes far from filling the chip
        _train_encoder("train_encoder256_bf16", 4, 4, 256, 4, 1024, 512, 128, 8, 19, 20),
        # a hidden layer of the smallest bf16 MLPs, forward: a few hundred thousand multiplications per model
        _linear_fwd("fwd_mlp320_bf16", 3, 96, 320, 320, BF16, "act"),
        # the first FFN layer of the 12-block encoders at 32 x 512 tokens, forward with the pre-activation kept
        _linear_fwd("fwd_ffn768_bf16", 4, 16384, 768, 3072, BF16, "act"),
        # a layer of the 1.2 M-parameter fp32 feed-forward net, backward with the SGD update
        _linear_bwd("bwd_ffn784_f32", 4, 64, 784, 768, F32, True, "gelu", "sgd"),
        # the second FFN layer of a BERT-Large-shaped encoder at 8 x 384 tokens, backward with the Adam update
        _linear_bwd("bwd_bert4096_bf16", 4, 3072, 4096, 1024, BF16, True, "gelu", "adam"),
        # a hidden layer of the 8 wide MLPs at batch 512, backward with the Adam update: optimizer state is the traffic
        _linear_bwd("bwd_mlp4096_bf16", 8, 512, 4096, 4096, BF16, True, "gelu", "adam"),
        # attention of the 12-block encoders, forward and backward
        _attention("attn_encoder_dh64", 4, 32, 512, 12, 64, False),
        # attention of the BERT-Large-shaped encoders at 384 tokens
        _attention("attn_bert384_dh64", 4, 8, 384, 16, 64, False),
        # causal attention of one large decoder at 2048 tokens and heads of 128
        _attention("attn_decoder_dh128", 1, 8, 2048, 32, 128, True),
        # a LayerNorm of the 12-block encoders, forward and backward with the residual gradient
        _layernorm("layernorm768_bf16", 4, 16384, 768, BF16),
        # the output head of the 12-block encoders on the masked positions: logits, loss, gradients, Adam update
        _head("head30522_bf16", 4, 2432, 768, 30522),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, odd=0.0):
    """A layer width: a multiple of 8 as a rule, any number now and then."""
    w = min(max(_log(rng, lo, hi), lo), hi)
    return w if rng.random() < odd else max(8, (w + 4) // 8 * 8)


def draw(rng):
    kind = rng.choice(["linear_fwd", "linear_fwd", "linear_bwd", "linear_bwd", "attention", "attention", "attention",
                       "layernorm", "head", "train_mlp", "train_encoder"])
    dtype = F32 if rng.random() < 0.2 else BF16
    while True:
        if kind == "linear_fwd":
            c = _linear_fwd("", rng.randint(1, 8), _log(rng, 24, 16384), _width(rng, 64, 4096, 0.1), _width(rng, 64, 4096, 0.2),
                            dtype, rng.choice(["act", "bias", "resid"]), rng.choice(["gelu", "gelu", "relu"]))
            top = 3.2e11 if dtype == BF16 else 1.5e10
        elif kind == "linear_bwd":
            c = _linear_bwd("", rng.randint(1, 8), _log(rng, 24, 16384), _width(rng, 64, 4096), _width(rng, 64, 4096, 0.2), dtype,
                            rng.random() < 0.5, rng.choice(["gelu", "gelu", "relu"]), rng.choice(["adam", "adam", "sgd"]))
            top = 3.2e11 if dtype == BF16 else 1.5e10
        elif kind == "attention":
            DH = rng.choice([64, 64, 128])
            c = _attention("", rng.randint(1, 6), _log(rng, 1, 32), _log(rng, 40, 2048), rng.randint(2, 2048 // DH), DH,
                           rng.random() < 0.4)
            top = 9e11
        elif kind == "layernorm":
            c = _layernorm("", rng.randint(1, 8), _log(rng, 96, 16384), _width(rng, 128, 4096), dtype)
            top = 1e12
        elif kind == "head":
            c = _head("", rng.randint(1, 4), _log(rng, 16, 4096), _width(rng, 64, 1024), _log(rng, 72, 32000))
            top = 1.3e12
        elif kind == "train_mlp":
            d = _width(rng, 48, 512)
            c = _train_mlp("", rng.randint(1, 6), rng.randint(1, 6), d, d, rng.randint(5, 80), _log(rng, 8, 128), rng.randint(5, 10),
                           rng.choice(["gelu", "relu"]), rng.choice(["adam", "sgd"]), F32 if rng.random() < 0.6 else BF16)
            top = 2e11
        else:
            H = rng.randint(1, 4)
            d = 64 * H
            c = _train_encoder("", rng.randint(1, 4), rng.randint(1, 4), d, H, _width(rng, 2 * d, 4 * d), rng.randint(64, 600),
                               _log(rng, 24, 160), rng.randint(2, 8), 4, rng.randint(5, 20))
            c["targets"] = max(1, int(0.15 * c["S"]))
            top = 1e12
        w = work(c)
        if w["flops"] <= top and w["bytes"] <= 4.0e9:
            del c["name"]
            return c


# ---- work and tolerance ------------------------------------------------------------------------------------------------

def _esz(dtype):
    return 2 if dtype == BF16 else 4


def _mlp_params(c):
    n, prev = 0, c["d_in"]
    for _ in range(c["layers"]):
        n, prev = n + prev * c["d"] + c["d"], c["d"]
    return n + prev * c["out"] + c["out"]


def _state_bytes(opt, dtype):
    """Bytes per parameter of an update: state read and written, the bf16 copy written."""
    return (24 if opt == "adam" else 8) + (2 if dtype == BF16 else 0)


def work(c):
    k = c["kind"]
    if k == "linear_fwd":
        G, m, i, o, e = c["G"], c["rows"], c["d_in"], c["d_out"], _esz(c["dtype"])
        extra = {"act": 1, "resid": 1, "bias": 0}[c["epi"]]
        return dict(bytes=G * (e * (m * i + i * o + m * o * (1 + extra)) + 4 * o), flops=2.0 * G * m * i * o)
    if k == "linear_bwd":
        G, m, i, o, e = c["G"], c["rows"], c["d_in"], c["d_out"], _esz(c["dtype"])
        n = i * o
        return dict(bytes=G * (e * (m * o + m * i * (2 + (1 if c["gate"] else 0)) + (n if c["dtype"] == BF16 else 0))
                               + n * _state_bytes(c["opt"], c["dtype"]) + 4 * o), flops=4.0 * G * m * i * o)
    if k == "attention":
        t, d = c["G"] * c["B"] * c["S"], c["H"] * c["DH"]
        f = 4.0 * t * c["S"] * d * (0.5 if c["causal"] else 1.0)
        return dict(bytes=2.0 * t * d * (3 + 1 + 1 + 3) + 4.0 * t * c["H"], flops=3.5 * f)
    if k == "layernorm":
        n = c["G"] * c["rows"] * c["d"]
        return dict(bytes=_esz(c["dtype"]) * 5.0 * n + 8.0 * c["G"] * c["rows"], flops=20.0 * n)
    if k == "head":
        G, m, d, V = c["G"], c["rows"], c["d"], c["V"]
        return dict(bytes=G * (2.0 * 2 * m * d + 2.0 * d * V + 6.0 * m * V + 26.0 * d * V + 4.0 * V), flops=6.0 * G * m * d * V)
    if k == "train_mlp":
        n = _mlp_params(c)
        return dict(bytes=c["K"] * c["steps"] * (n * (2.0 * _esz(c["dtype"]) + _state_bytes(c["opt"], c["dtype"]))
                                                 + 4.0 * c["batch"] * c["d_in"]), flops=6.0 * c["K"] * c["steps"] * c["batch"] * n)
    n, t, d = _enc_params(c), c["batch"] * c["S"], c["d"]
    blk = c["layers"] * (4 * d * d + 2 * d * c["ffn"])
    per = 6.0 * t * blk + 6.0 * c["batch"] * c["targets"] * d * c["V"] + 14.0 * t * c["S"] * d * c["layers"]
    return dict(bytes=c["K"] * c["steps"] * (n * 30.0 + 2.0 * t * d * (c["layers"] + 1)), flops=c["K"] * c["steps"] * per)


def tolerance(c):
    """About four times the distance from the 64-bit results.  bf16 outputs carry their own rounding (measured 2e-3 over a
    tensor, 2.6e-3 behind a second rounding); fp32 sums differ by their order (5e-7, bias gradients 1.2e-6).  A trained model
    adds what a changed last bit does to the steps that follow: bf16 encoders 2.1e-3, fp32 with SGD 2.6e-7 unless a ReLU
    input lies within rounding of its kink (then 1e-5 to 1e-4 in ten steps); with Adam an element whose gradient is smaller than
    its own rounding may step the other way, 2 lr a step."""
    k = c["kind"]
    if k == "train_mlp":
        if c["dtype"] == F32:
            return dict(rel=1e-5, max=1e-2) if c["opt"] == "sgd" and c["act"] == "gelu" else dict(rel=1e-4, max=2e-2)
        return dict(rel=1e-2, max=0.5)
    if k == "train_encoder":
        return dict(rel=1e-2, max=0.5)
    if c.get("dtype", BF16) == F32:
        return dict(rel=1e-5, max=1e-3)
    return dict(rel=1e-2, max=0.2)


# ---- inputs ------------------------------------------------------------------------------------------------------------

class _Draws:
    """Seeded tensors on the device."""

    def __init__(self, seed, dev="cuda"):
        self.g = torch.Generator(device=dev)
        self.g.manual_seed(int(seed) * 1000003 + 17)
        self.dev = dev

    def normal(self, shape, std=1.0, dtype=torch.float32):
        return (torch.randn(shape, generator=self.g, device=self.dev) * std).to(dtype)

    def rows(self, m, n, ld, std=1.0, dtype=torch.bfloat16):
        """[m, ld] with n drawn columns and zeros behind them."""
        t = torch.zeros(m, ld, device=self.dev, dtype=dtype)
        t[:, :n] = self.normal((m, n), std, dtype)
        return t

    def ints(self, shape, hi):
        return torch.randint(0, hi, shape, generator=self.g, device=self.dev, dtype=torch.int32)


def _up8(n):
    return (n + 7) // 8 * 8


def _tt(dtype):
    return torch.bfloat16 if dtype == BF16 else torch.float32


def _hp(G):
    lrs = [1e-4 * (1 + g) for g in range(G)]
    return [(lr, B1, B2, EPS, 1.0 / (1.0 - B1 ** ADAM_T), 1.0 / (1.0 - B2 ** ADAM_T)) for lr in lrs]


def _linear_fwd_inputs(c, seed):
    D, t = _Draws(seed), _tt(c["dtype"])
    G, m, i, o = c["G"], c["rows"], c["d_in"], c["d_out"]
    li, lo = _up8(i), _up8(o)
    s = dict(x=[D.rows(m, i, li, 1.0, t) for _ in range(G)], w=[D.rows(o, i, li, i ** -0.5, t) for _ in range(G)],
             b=[D.normal((lo,), 0.1) for _ in range(G)])
    if c["epi"] == "resid":
        s["resid"] = [D.rows(m, o, lo, 1.0, t) for _ in range(G)]
    return s


def _linear_bwd_inputs(c, seed):
    D, t = _Draws(seed), _tt(c["dtype"])
    G, m, i, o = c["G"], c["rows"], c["d_in"], c["d_out"]
    lo = _up8(o)
    s = dict(dy=[D.rows(m, o, lo, 1e-2, t) for _ in range(G)], x=[D.normal((m, i), 1.0, t) for _ in range(G)],
             p=[D.normal((o, i), i ** -0.5) for _ in range(G)])
    s["w"] = [p.to(t) for p in s["p"]] if t == torch.bfloat16 else s["p"]
    if c["gate"]:
        s["gate"] = [D.normal((m, i), 1.0, t) for _ in range(G)]
    if c["opt"] == "adam":
        g = 1e-2 * m ** 0.5                      # size of a weight's gradient
        s["m"] = [D.normal((o, i), 0.3 * g) for _ in range(G)]
        s["v"] = [D.normal((o, i), 0.1 * g).square_() for _ in range(G)]
    return s


def _attention_inputs(c, seed):
    D = _Draws(seed)
    t, d = c["B"] * c["S"], c["H"] * c["DH"]
    bf = torch.bfloat16
    return dict(qkv=[D.normal((t, 3 * d), 0.7, bf) for _ in range(c["G"])], dout=[D.normal((t, d), 1.0, bf) for _ in range(c["G"])])


def _layernorm_inputs(c, seed):
    D, t = _Draws(seed), _tt(c["dtype"])
    sh, G = (c["rows"], c["d"]), c["G"]
    return dict(x=[D.normal(sh, 1.3, t) for _ in range(G)], dy=[D.normal(sh, 1.0, t) for _ in range(G)],
                add=[D.normal(sh, 1.0, t) for _ in range(G)], gamma=[1.0 + D.normal((c["d"],), 0.1) for _ in range(G)],
                beta=[D.normal((c["d"],), 0.1) for _ in range(G)])


def _head_inputs(c, seed):
    D, bf = _Draws(seed), torch.bfloat16
    G, m, d, V = c["G"], c["rows"], c["d"], c["V"]
    s = dict(x=[D.normal((m, d), 1.0, bf) for _ in range(G)], p=[D.normal((V, d), 0.02) for _ in range(G)],
             b=[D.normal((_up8(V),), 0.01) for _ in range(G)], y=D.ints((m,), V))
    s["w"] = [p.to(bf) for p in s["p"]]
    s["m"] = [D.normal((V, d), 1e-4) for _ in range(G)]
    s["v"] = [D.normal((V, d), 1e-4).square_() for _ in range(G)]
    return s


def _mlp_inputs(c, seed):
    """Initial weights [out, in] and biases in canonical order per model, and the epoch's batches (host arrays: that is what
    the trainer takes)."""
    r = np.random.default_rng(seed)
    models = []
    for _ in range(c["K"]):
        ts, prev = [], c["d_in"]
        for width in [c["d"]] * c["layers"] + [c["out"]]:
            a = math.sqrt(6.0 / prev)
            ts += [r.uniform(-a, a, (width, prev)).astype(np.float32), np.zeros(width, np.float32)]
            prev = width
        models.append(ts)
    x = r.standard_normal((c["steps"], c["batch"], c["d_in"]), dtype=np.float32)
    y = r.integers(0, c["out"], (c["steps"], c["batch"]), dtype=np.int32)
    return models, x, y


def _mlp_lr(c, k):
    return (0.02 if c["opt"] == "sgd" else 1e-4) / (1 + k)


def _enc_shapes(c):
    d, F, V = c["d"], c["ffn"], c["V"]
    blk = [(d,), (d,), (3 * d, d), (3 * d,), (d, d), (d,), (d,), (d,), (F, d), (F,), (d, F), (d,)]
    return [(V, d), (c["S"], d)] + blk * c["layers"] + [(d,), (d,), (V, d), (V,)]


def _enc_params(c):
    return sum(int(np.prod(s)) for s in _enc_shapes(c))


def _enc_inputs(c, seed):
    r = np.random.default_rng(seed)
    shapes = _enc_shapes(c)
    gains = {2 + 12 * l + j for l in range(c["layers"]) for j in (0, 6)} | {2 + 12 * c["layers"]}
    models = []
    for _ in range(c["K"]):
        a = 0.02 * math.sqrt(3.0)
        models.append([np.ones(s, np.float32) if i in gains else r.uniform(-a, a, s).astype(np.float32) if len(s) == 2
                       else np.zeros(s, np.float32) for i, s in enumerate(shapes)])
    ids = r.integers(0, c["V"], (c["steps"], c["batch"], c["S"]), dtype=np.int32)
    pos = np.sort(np.argsort(r.random((c["steps"], c["batch"], c["S"])), axis=2)[:, :, :c["targets"]], axis=2).astype(np.int32)
    y = np.take_along_axis(ids, pos, axis=2)
    np.put_along_axis(ids, pos, 0, axis=2)                  # masked positions
    return models, ids, pos, y


def _enc_lr(k):
    return 1e-4 * (1 + k)


# ---- prepare and run -----------------------------------------------------------------------------------------------------

class _Trainer:
    """A context with its models and data, as a training program holds it between epochs."""

    def __init__(self, archs, hparams, models, inputs, pos, targets, cuts):
        from paper_2107_06469_amd import hydra
        self.h, self.ctx, self.K, self.steps = hydra, hydra.hydra_create(), len(models), inputs.shape[0]
        hydra.hydra_define_models(self.ctx, archs, hparams, 42)
        for k in range(self.K):
            hydra.hydra_shard(self.ctx, k, cuts)
        hydra.hydra_set_data(self.ctx, inputs, pos, targets)
        for k, ts in enumerate(models):
            hydra.hydra_write_params(self.ctx, k, -1, ts)

    def epoch(self):
        h = self.h
        h.hydra_train_epoch(self.ctx)
        loss = [h.hydra_read_loss(self.ctx, k)[-self.steps:] for k in range(self.K)]
        return dict(loss=np.stack(loss), params=[np.concatenate([t.reshape(-1) for t in h.hydra_read_params(self.ctx, k)])
                                                 for k in range(self.K)])

    def __del__(self):
        if getattr(self, "ctx", None) is not None:
            self.h.hydra_destroy(self.ctx)


def prepare(c, seed):
    from hydra_workloads import configs as W
    from paper_2107_06469_amd import ops
    k = c["kind"]
    dev, bf = "cuda", torch.bfloat16
    f32 = lambda *sh: torch.zeros(*sh, device=dev)  # noqa: E731
    if k == "linear_fwd":
        s, t, lo = _linear_fwd_inputs(c, seed), _tt(c["dtype"]), _up8(c["d_out"])
        s["out"] = [torch.zeros(c["rows"], lo, device=dev, dtype=t) for _ in range(c["G"])]
        if c["epi"] == "act":
            s["pre"] = [torch.zeros(c["rows"], lo, device=dev, dtype=t) for _ in range(c["G"])]
    elif k == "linear_bwd":
        s, t = _linear_bwd_inputs(c, seed), _tt(c["dtype"])
        s["dx"] = [torch.zeros(c["rows"], c["d_in"], device=dev, dtype=t) for _ in range(c["G"])]
        s["db"] = [f32(c["d_out"]) for _ in range(c["G"])]
        if c["opt"] == "sgd":
            s["m"] = s["v"] = None
        nb = ops.hydra_op_gemm_split_ws_bytes(c["d_out"], c["d_in"], c["rows"], c["d_in"]) if c["dtype"] == BF16 else 0
        s["ws"] = [torch.zeros(nb, device=dev, dtype=torch.uint8) for _ in range(c["G"])] if nb else None
        s["hp"] = _hp(c["G"])
    elif k == "attention":
        s, t, d = _attention_inputs(c, seed), c["B"] * c["S"], c["H"] * c["DH"]
        s["o"] = [torch.zeros(t, d, device=dev, dtype=bf) for _ in range(c["G"])]
        s["lse"], s["delta"] = ([f32(t * c["H"]) for _ in range(c["G"])] for _ in range(2))
        s["dqkv"] = [torch.zeros(t, 3 * d, device=dev, dtype=bf) for _ in range(c["G"])]
    elif k == "layernorm":
        s, t, sh = _layernorm_inputs(c, seed), _tt(c["dtype"]), (c["rows"], c["d"])
        s["y"], s["dx"] = ([torch.zeros(sh, device=dev, dtype=t) for _ in range(c["G"])] for _ in range(2))
        s["mean"], s["rstd"] = ([f32(c["rows"]) for _ in range(c["G"])] for _ in range(2))
        s["dgamma"], s["dbeta"] = ([f32(c["d"]) for _ in range(c["G"])] for _ in range(2))
        s["part"] = [f32(ops.hydra_op_layernorm_part_floats(*sh)) for _ in range(c["G"])]
    elif k == "head":
        s, lv, m = _head_inputs(c, seed), _up8(c["V"]), c["rows"]
        G = range(c["G"])
        s["z"], s["dz"] = [f32(m, lv) for _ in G], [torch.zeros(m, lv, device=dev, dtype=bf) for _ in G]
        s["rowloss"], s["loss"], s["db"] = [f32(m) for _ in G], [f32(1) for _ in G], [f32(c["V"]) for _ in G]
        s["dx"] = [torch.zeros(m, c["d"], device=dev, dtype=bf) for _ in G]
        nb = ops.hydra_op_gemm_split_ws_bytes(c["V"], c["d"], m, c["d"])
        s["ws"] = [torch.zeros(nb, device=dev, dtype=torch.uint8) for _ in G] if nb else None
        s["hp"] = _hp(c["G"])
    elif k == "train_mlp":
        models, x, y = _mlp_inputs(c, seed)
        a = W.mlp_arch(c["layers"], c["d_in"], c["d"], c["out"], W.ACT_RELU if c["act"] == "relu" else W.ACT_GELU,
                       W.DTYPE_F32 if c["dtype"] == F32 else W.DTYPE_BF16)
        hps = [W.hparams(W.OPT_SGD if c["opt"] == "sgd" else W.OPT_ADAM, _mlp_lr(c, i)) for i in range(c["K"])]
        s = dict(trainer=_Trainer([a] * c["K"], hps, models, x, None, y, [c["layers"] // 2] if c["layers"] > 1 else []))
    else:
        models, ids, pos, y = _enc_inputs(c, seed)
        a = W.transformer_arch(W.KIND_ENCODER, c["layers"], c["d"], c["H"], c["ffn"], c["V"], c["S"], 0, W.DTYPE_BF16)
        hps = [W.hparams(W.OPT_ADAM, _enc_lr(i)) for i in range(c["K"])]
        s = dict(trainer=_Trainer([a] * c["K"], hps, models, ids, pos, y, [c["layers"] // 2] if c["layers"] > 1 else []))
    s["case"] = c
    return s


def run(s):
    from paper_2107_06469_amd import ops
    c = s["case"]
    k = c["kind"]
    if k.startswith("train"):
        return s["trainer"].epoch()
    dt = ops.F32 if c.get("dtype") == F32 else ops.BF16
    act = ops.EPI_RELU if c.get("act") == "relu" else ops.EPI_GELU
    if k == "linear_fwd":
        m, i, o = c["rows"], c["d_in"], c["d_out"]
        li, lo = _up8(i), _up8(o)
        kw = {}
        if c["epi"] == "act":
            kw = dict(pre=s["pre"], act=act)
        elif c["epi"] == "resid":
            kw = dict(resid=s["resid"], ldr=lo)
        ops.hydra_op_gemm(dt, m, o, i, s["x"], s["w"], s["out"], x_kmajor=True, w_kmajor=True, ldx=li, ldw=li, ldo=lo, bias=s["b"],
                          **kw)
        return dict(out=[t[:, :o] for t in s["out"]], pre=[t[:, :o] for t in s.get("pre", [])])
    if k == "linear_bwd":
        m, i, o = c["rows"], c["d_in"], c["d_out"]
        lo = _up8(o)
        kw = dict(gate=s["gate"], ldg=i, act=act) if c["gate"] else {}
        ops.hydra_op_gemm(dt, m, i, o, s["dy"], s["w"], s["dx"], x_kmajor=True, w_kmajor=False, ldx=lo, ldw=i, ldo=i, **kw)
        w16 = s["w"] if dt == ops.BF16 else None
        ops.hydra_op_gemm_update(dt, o, i, m, s["dy"], s["x"], 1 if c["opt"] == "adam" else 0, s["p"], s["m"], s["v"], w16, s["hp"],
                                 ldx=lo, ldw=i, ldo=i, rowsum=s["db"], ws=s["ws"])
        return dict(dx=s["dx"], db=s["db"], p=s["p"], w=w16, m=s["m"], v=s["v"])
    if k == "attention":
        d, sc = c["H"] * c["DH"], c["DH"] ** -0.5
        ops.hydra_op_attention_fwd(c["B"], c["S"], c["H"], c["DH"], 3 * d, d, c["causal"], sc, s["qkv"], s["o"], s["lse"])
        ops.hydra_op_attention_bwd(c["B"], c["S"], c["H"], c["DH"], 3 * d, d, c["causal"], sc, s["qkv"], s["o"], s["dout"], s["lse"],
                                   s["delta"], s["dqkv"])
        return dict(o=s["o"], lse=s["lse"], dqkv=s["dqkv"])
    if k == "layernorm":
        m, d = c["rows"], c["d"]
        ops.hydra_op_layernorm_fwd(dt, m, d, d, 1e-5, s["x"], s["y"], s["gamma"], s["beta"], s["mean"], s["rstd"])
        ops.hydra_op_layernorm_bwd(dt, m, d, d, s["x"], s["dy"], s["add"], s["dx"], s["gamma"], s["mean"], s["rstd"], s["part"],
                                   s["dgamma"], s["dbeta"])
        return dict(y=s["y"], mean=s["mean"], rstd=s["rstd"], dx=s["dx"], dgamma=s["dgamma"], dbeta=s["dbeta"])
    m, d, V = c["rows"], c["d"], c["V"]
    lv = _up8(V)
    ops.hydra_op_gemm(ops.BF16, m, V, d, s["x"], s["w"], s["z"], x_kmajor=True, w_kmajor=True, ldx=d, ldw=d, ldo=lv, bias=s["b"],
                      out_f32=True)
    ops.hydra_op_softmax_ce(ops.BF16, m, V, lv, lv, 1.0 / m, s["z"], s["y"], s["dz"], s["rowloss"], s["loss"])
    ops.hydra_op_gemm(ops.BF16, m, d, V, s["dz"], s["w"], s["dx"], x_kmajor=True, w_kmajor=False, ldx=lv, ldw=d, ldo=d)
    ops.hydra_op_gemm_update(ops.BF16, V, d, m, s["dz"], s["x"], 1, s["p"], s["m"], s["v"], s["w"], s["hp"], ldx=lv, ldw=d, ldo=d,
                             rowsum=s["db"], ws=s["ws"])
    return dict(logits=[t[:, :V] for t in s["z"]], loss=s["loss"], dz=[t[:, :V] for t in s["dz"]], dx=s["dx"], db=s["db"], p=s["p"],
                w=s["w"], m=s["m"], v=s["v"])


# ---- the same in 64 bits --------------------------------------------------------------------------------------------------

def _gelu(z):
    return 0.5 * z * (1.0 + torch.erf(z * math.sqrt(0.5)))


def _gelu_grad(z):
    return 0.5 * (1.0 + torch.erf(z * math.sqrt(0.5))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def _updated(p, g, m, v, opt, hp):
    lr, b1, b2, eps, bc1, bc2 = hp
    if opt == "sgd":
        return p - lr * g, None, None
    m = b1 * m + (1.0 - b1) * g
    v = b2 * v + (1.0 - b2) * g * g
    return p - lr * (m * bc1) / (torch.sqrt(v * bc2) + eps), m, v


def _attention_exact(c, seed):
    s = _attention_inputs(c, seed)
    B, S, H, DH = c["B"], c["S"], c["H"], c["DH"]
    d, sc, out = H * DH, DH ** -0.5, dict(o=[], lse=[], dqkv=[])
    mask = torch.ones(S, S, device="cuda", dtype=torch.bool).triu(1) if c["causal"] else None
    for qkv, dout in zip(s["qkv"], s["dout"]):
        o, lse = torch.empty(B * S, d, device="cuda", dtype=torch.float64), torch.empty(B, H, S, device="cuda", dtype=torch.float64)
        dq = torch.empty(B * S, 3 * d, device="cuda", dtype=torch.float64)
        for b in range(B):
            r = slice(b * S, (b + 1) * S)
            for h in range(H):
                q, k, v = (qkv[r, j * d + h * DH:j * d + (h + 1) * DH].double().contiguous() for j in range(3))
                do = dout[r, h * DH:(h + 1) * DH].double().contiguous()
                z = torch.mm(q, k.t().contiguous()) * sc
                if mask is not None:
                    z = z.masked_fill(mask, -math.inf)
                ls = torch.logsumexp(z, 1)
                p = torch.exp(z - ls[:, None])
                oh = torch.mm(p, v)
                dp = torch.mm(do, v.t().contiguous())
                ds = p * (dp - (do * oh).sum(1, keepdim=True)) * sc
                o[r, h * DH:(h + 1) * DH], lse[b, h] = oh, ls
                for j, g in enumerate((torch.mm(ds, k), torch.mm(ds.t().contiguous(), q), torch.mm(p.t().contiguous(), do))):
                    dq[r, j * d + h * DH:j * d + (h + 1) * DH] = g
        out["o"].append(o)
        out["lse"].append(lse.reshape(-1))
        out["dqkv"].append(dq)
    return out


def _adam(opt, ts, grads, st, lr, t):
    with torch.no_grad():
        for i, (p, g) in enumerate(zip(ts, grads)):
            hp = (lr, B1, B2, EPS, 1.0 / (1.0 - B1 ** t), 1.0 / (1.0 - B2 ** t))
            p1, m1, v1 = _updated(p, g, *st[i], opt, hp)
            p.copy_(p1)
            st[i] = (m1, v1)


def _trained(models, opt, lrs, steps, loss_of):
    out = dict(loss=[], params=[])
    for k, ts in enumerate(models):
        ts = [torch.tensor(t, dtype=torch.float64).requires_grad_() for t in ts]
        st, losses = [(torch.zeros_like(t), torch.zeros_like(t)) for t in ts], []
        for t in range(steps):
            loss = loss_of(ts, t)
            losses.append(float(loss.detach()))
            _adam(opt, ts, torch.autograd.grad(loss, ts), st, lrs[k], t + 1)
        out["loss"].append(losses)
        out["params"].append(torch.cat([t.detach().reshape(-1) for t in ts]))
    out["loss"] = np.array(out["loss"], dtype=np.float64)
    return out


def _mlp_exact(c, seed):
    models, x, y = _mlp_inputs(c, seed)
    x, y = torch.tensor(x).double(), torch.tensor(y).long()

    def loss_of(ts, t):
        h = x[t]
        for l in range(c["layers"]):
            h = h @ ts[2 * l].t() + ts[2 * l + 1]
            h = torch.relu(h) if c["act"] == "relu" else _gelu(h)
        return torch.nn.functional.cross_entropy(h @ ts[-2].t() + ts[-1], y[t])

    return _trained(models, c["opt"], [_mlp_lr(c, k) for k in range(c["K"])], c["steps"], loss_of)


def _enc_exact(c, seed):
    models, ids, pos, y = _enc_inputs(c, seed)
    ids, pos, y = (torch.tensor(a).long() for a in (ids, pos, y))
    B, S, d, H = c["batch"], c["S"], c["d"], c["H"]
    dh = d // H
    ln = torch.nn.functional.layer_norm

    def loss_of(ts, t):
        x = (ts[0][ids[t]] + ts[1][None]).reshape(B * S, d)
        for l in range(c["layers"]):
            g1, b1, wq, bq, wo, bo, g2, b2, w1, c1, w2, c2 = ts[2 + 12 * l:14 + 12 * l]
            qkv = ln(x, (d,), g1, b1, 1e-5) @ wq.t() + bq
            q, k, v = (u.reshape(B, S, H, dh).transpose(1, 2) for u in qkv.split(d, 1))
            p = torch.softmax(q @ k.transpose(2, 3) * dh ** -0.5, -1)
            x = x + (p @ v).transpose(1, 2).reshape(B * S, d) @ wo.t() + bo
            x = x + _gelu(ln(x, (d,), g2, b2, 1e-5) @ w1.t() + c1) @ w2.t() + c2
        g, b, wh, bh = ts[-4:]
        rows = (torch.arange(B)[:, None] * S + pos[t]).reshape(-1)
        return torch.nn.functional.cross_entropy(ln(x[rows], (d,), g, b, 1e-5) @ wh.t() + bh, y[t].reshape(-1))

    return _trained(models, "adam", [_enc_lr(k) for k in range(c["K"])], c["steps"], loss_of)


def exact(c, seed):
    k = c["kind"]
    if k == "train_mlp":
        return _mlp_exact(c, seed)
    if k == "train_encoder":
        return _enc_exact(c, seed)
    if k == "attention":
        return _attention_exact(c, seed) if c["G"] * c["B"] * c["H"] <= 4000 else None
    if k == "linear_fwd":
        s, i, o, out = _linear_fwd_inputs(c, seed), c["d_in"], c["d_out"], dict(out=[], pre=[])
        for g in range(c["G"]):
            z = torch.mm(s["x"][g][:, :i].double(), s["w"][g][:, :i].double().t().contiguous()) + s["b"][g][:o].double()
            if c["epi"] == "act":
                out["pre"].append(z)
                z = torch.relu(z) if c["act"] == "relu" else _gelu(z)
            elif c["epi"] == "resid":
                z = z + s["resid"][g][:, :o].double()
            out["out"].append(z)
        return out
    if k == "linear_bwd":
        s, o, hp = _linear_bwd_inputs(c, seed), c["d_out"], _hp(c["G"])
        out = dict(dx=[], db=[], p=[], w=[], m=[], v=[])
        for g in range(c["G"]):
            dy = s["dy"][g][:, :o].double()
            dx = torch.mm(dy, s["w"][g].double())
            if c["gate"]:
                z = s["gate"][g].double()
                dx = dx * ((z > 0).double() if c["act"] == "relu" else _gelu_grad(z))
            gw = torch.mm(dy.t().contiguous(), s["x"][g].double())
            st = [s[n][g].double() if c["opt"] == "adam" else None for n in ("m", "v")]
            p, m, v = _updated(s["p"][g].double(), gw, *st, c["opt"], hp[g])
            for n, t in zip(("dx", "db", "p", "w", "m", "v"), (dx, dy.sum(0), p, p if c["dtype"] == BF16 else None, m, v)):
                out[n].append(t)
        return out
    if k == "layernorm":
        s = _layernorm_inputs(c, seed)
        out = {n: [] for n in ("y", "mean", "rstd", "dx", "dgamma", "dbeta")}
        for g in range(c["G"]):
            x, dy, ga = s["x"][g].double(), s["dy"][g].double(), s["gamma"][g].double()
            mu = x.mean(1, keepdim=True)
            rs = torch.rsqrt((x - mu).square().mean(1, keepdim=True) + 1e-5)
            xh, gy = (x - mu) * rs, dy * ga
            dx = rs * (gy - gy.mean(1, keepdim=True) - xh * (gy * xh).mean(1, keepdim=True)) + s["add"][g].double()
            for n, t in zip(out, (xh * ga + s["beta"][g].double(), mu[:, 0], rs[:, 0], dx, (dy * xh).sum(0), dy.sum(0))):
                out[n].append(t)
        return out
    s, hp, V, m = _head_inputs(c, seed), _hp(c["G"]), c["V"], c["rows"]
    out = {n: [] for n in ("logits", "loss", "dz", "dx", "db", "p", "w", "m", "v")}
    for g in range(c["G"]):
        x, w = s["x"][g].double(), s["w"][g].double()
        z = torch.mm(x, w.t().contiguous()) + s["b"][g][:V].double()
        lp = torch.log_softmax(z, 1)
        y = s["y"].long()[:, None]
        dz = torch.exp(lp)
        dz.scatter_add_(1, y, torch.full_like(lp[:, :1], -1.0))
        dz /= m
        dw = torch.mm(dz.t().contiguous(), x)
        p, mm, vv = _updated(s["p"][g].double(), dw, s["m"][g].double(), s["v"][g].double(), "adam", hp[g])
        for n, t in zip(out, (z, -lp.gather(1, y).mean().reshape(1), dz, torch.mm(dz, w), dz.sum(0), p, p, mm, vv)):
            out[n].append(t)
    return out
