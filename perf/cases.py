"""The layer calls whose speed is measured: one dict per case, how its inputs are made, one pass through the public
entry points, the work of a pass and the tolerance between two correct implementations.

Layer shapes are those of workloads.py (Switch-base, Switch-large and NLLB-MoE sized layers and the fp32 preset), token
counts run from one decoder token to the largest prefill preset.  Inputs follow the same recipe as workloads.py
(x ~ N(0, 1), gate ~ N(0, gate_std^2), W ~ N(0, 1 / fan_in), rounded to the storage type; skewed layers add a gate bias
of log Zipf weights), drawn on the GPU because the largest layer holds 8.6 GB of weights.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2405_18832_amd as moe

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name=None, *, call="layer", T, d, f, E, k, dtype="bf16", renorm=True, act="relu", expert_bias=False, zipf=0.0,
          gate_std=0.02, H=-1):
    c = dict(call=call, T=T, d=d, f=f, E=E, k=k, dtype=dtype, renorm=renorm, act=act, expert_bias=expert_bias, zipf=zipf,
             gate_std=gate_std, H=H)
    if name is not None:
        c["name"] = name
    return c


NLLB = dict(d=2048, f=8192, E=128, k=2)
SWITCH_LARGE = dict(d=1024, f=4096, E=128, k=1, renorm=False)
SWITCH_BASE = dict(d=768, f=3072, k=1, renorm=False)


def listed():
    return [
        # one sentence being generated: a token per step in a loop that allocates nothing
        _case("decoder_1_token_noalloc", call="noalloc", T=1, **NLLB),
        # generation for a batch of sentences, one token each per step
        _case("decoder_32_tokens", T=32, **NLLB),
        # a larger generation batch with beams, not a multiple of anything
        _case("decoder_93_tokens", T=93, **NLLB),
        # encoder pass over a few short sequences, tokens spread over all experts
        _case("switch_base_2048_tokens", T=2048, E=64, **SWITCH_BASE),
        # few experts, ragged token count, experts with biases and GeLU
        _case("switch_base_8_gelu_bias", T=1501, E=8, act="gelu", expert_bias=True, **SWITCH_BASE),
        # encoder pass with skewed routing: a handful of hot experts and a tail of cold ones
        _case("switch_large_4096_skewed", T=4096, zipf=1.1, **SWITCH_LARGE),
        # the largest single-GPU pass: a long prefill batch, skewed routing
        _case("prefill_16384_skewed", T=16384, zipf=1.2, **NLLB),
        # the hot side of a split layer, ragged prefill batch, most experts reached; with the counts, the mask and the
        # routing that the other side needs
        _case("prefill_5003_hot_share", call="share", T=5003, zipf=1.2, gate_std=1.28 / math.sqrt(2048), H=32, **NLLB),
        # the layer step by step (a host program that works on the dispatched rows), hot share of a small encoder batch
        _case("steps_777_tokens_hot_share", call="steps", T=777, zipf=1.1, gate_std=1.28 / math.sqrt(1024), H=16,
              **SWITCH_LARGE),
        # the fp32 preset: latency of a tiny layer
        _case("f32_tiny", T=64, d=64, f=256, E=8, k=2, dtype="f32"),
        # fp32 run of a Switch-base layer with few experts (numerics checks against a bf16 deployment)
        _case("f32_switch_base_8", T=500, E=8, dtype="f32", **SWITCH_BASE),
        # loading a layer: weights as a checkpoint holds them into the layout the kernels read
        _case("pack_switch_base_64", call="pack", T=1, E=64, **SWITCH_BASE),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "layer", "layer", "layer", "share", "steps", "f32", "pack"])
    dims = rng.choice([NLLB, SWITCH_LARGE, dict(SWITCH_BASE, E=rng.choice([8, 64, 128]))])
    if rng.random() < 0.3:       # a layer of none of the presets' widths
        d = 32 * rng.randint(12, 64)
        dims = dict(d=d, f=32 * rng.randint(2 * d // 32, 4 * d // 32), E=rng.randint(8, 128), k=rng.choice([1, 2]))
    extra = dict(act=rng.choice(["relu", "relu", "gelu"]), expert_bias=rng.random() < 0.3)
    zipf = rng.choice([0.0, 1.1, 1.2])
    gate_std = rng.choice([0.02, 1.28 / math.sqrt(dims["d"])]) if zipf else 0.02
    if kind == "decode":
        T = _log_int(rng, 1, 127)
        if rng.random() < 0.5:
            return _case(call="noalloc", T=T, **dims)
        return _case(T=T, **dims, **extra)
    if kind == "layer":
        T = _log_int(rng, 128, 12000 if zipf else 6000)
        return _case(T=T, zipf=zipf, gate_std=gate_std, **dims, **extra)
    if kind == "share":
        T = _log_int(rng, 64, 8000)
        return _case(call="share", T=T, zipf=zipf, gate_std=gate_std, H=rng.randint(1, max(1, dims["E"] // 4)), **dims)
    if kind == "steps":
        T = _log_int(rng, 16, 3000)
        return _case(call="steps", T=T, zipf=zipf, gate_std=gate_std, H=rng.choice([-1, rng.randint(1, max(1, dims["E"] // 4))]),
                     **dims)
    if kind == "f32":
        d = rng.choice([64, 256, 512, 768])
        return _case(T=_log_int(rng, 16, 600), d=d + rng.choice([0, 2, 32]), f=4 * d, E=rng.randint(2, 16), k=rng.choice([1, 2]),
                     dtype="f32", **extra)
    E = rng.randint(4, 64)
    return _case(call="pack", T=1, d=dims["d"], f=dims["f"], E=E, k=1, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))


def _shape(c):
    return moe.make_shape(c["T"], c["d"], c["f"], c["E"], c["k"], c["dtype"], c["renorm"], {"relu": 0, "gelu": 1}[c["act"]])


def _normal(gen, shape, scale, dtype):
    return torch.randn(shape, dtype=dtype, device="cuda", generator=gen).mul_(scale)


def prepare(case, seed):
    c = case
    T, d, f, E, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    dt = DTYPES[c["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = _shape(c)
    s = {"case": c, "shape": shape}
    packed = moe.moe_packed_weight_bytes(shape) // dt.itemsize // E

    if c["call"] == "pack":
        s["src"] = [_normal(gen, (E, f, d), d ** -0.5, dt), _normal(gen, (E, d, f), f ** -0.5, dt)]
        s["dst"] = [torch.empty((E, packed), dtype=dt, device="cuda") for _ in range(2)]
        return s

    # a few experts' plain weights at a time: the packed layer is what stays
    s["w1"], s["w2"] = (torch.empty((E, packed), dtype=dt, device="cuda") for _ in range(2))
    step = max(1, min(E, (1 << 28) // (d * f)))
    for e in range(0, E, step):
        n = min(step, E - e)
        some = moe.make_shape(T, d, f, n, 1, c["dtype"], c["renorm"])
        moe.moe_pack_weights(some, 1, _normal(gen, (n, f, d), d ** -0.5, dt), s["w1"][e:e + n])
        moe.moe_pack_weights(some, 2, _normal(gen, (n, d, f), f ** -0.5, dt), s["w2"][e:e + n])

    s["x"] = _normal(gen, (T, d), 1.0, dt)
    s["wg"] = _normal(gen, (E, d), c["gate_std"], dt)
    s["bg"] = s["b1"] = s["b2"] = None
    if c["zipf"]:
        rank = torch.randperm(E, generator=torch.Generator().manual_seed(seed))
        s["bg"] = torch.log_softmax(-c["zipf"] * torch.log1p(rank.double()), 0).float().cuda()
    if c["expert_bias"]:
        s["b1"], s["b2"] = _normal(gen, (E, f), 0.25, torch.float32), _normal(gen, (E, d), 0.25, torch.float32)

    A, i32, f32 = T * k, torch.int32, torch.float32
    new = lambda size, dtype: torch.empty(size, dtype=dtype, device="cuda")
    s["out"] = new((T, d), dt)
    if c["call"] != "noalloc":
        s["ws"] = new((max(256, moe.moe_workspace_bytes(shape)),), torch.uint8)
    if c["call"] in ("share", "steps"):
        s.update(idx=new((T, k), i32), w=new((T, k), f32), counts=new((E,), i32), perm=new((A,), i32), mask=new((E,), torch.uint8))
    if c["call"] == "steps":
        # rows of experts outside the share stay as they are: zeros
        s.update(offsets=new((E + 1,), i32), inv=new((A,), i32), x_perm=new((A, d), dt),
                 y_perm=torch.zeros((A, d), dtype=f32, device="cuda"))
    return s


def run(s):
    c, shape = s["case"], s["shape"]
    if c["call"] == "pack":
        for i in range(2):
            moe.moe_pack_weights(shape, i + 1, s["src"][i], s["dst"][i])
        return s["dst"]
    if c["call"] == "noalloc":
        moe.moe_layer_forward_noalloc(shape, s["x"], s["wg"], s["bg"], s["w1"], s["w2"], None, c["H"], s["out"])
        return s["out"]
    if c["call"] == "layer":
        if c["expert_bias"]:
            moe.moe_layer_forward_biased(shape, s["x"], s["wg"], s["bg"], s["w1"], s["b1"], s["w2"], s["b2"], None, c["H"],
                                         s["out"], ws=s["ws"])
        else:
            moe.moe_layer_forward(shape, s["x"], s["wg"], s["bg"], s["w1"], s["w2"], None, c["H"], s["out"], ws=s["ws"])
        return s["out"]
    if c["call"] == "share":
        moe.moe_layer_forward(shape, s["x"], s["wg"], s["bg"], s["w1"], s["w2"], None, c["H"], s["out"], s["idx"], s["w"],
                              s["counts"], s["perm"], s["mask"], ws=s["ws"])
        return {n: s[n] for n in ("out", "idx", "w", "counts", "perm", "mask")}
    hot = s["mask"] if c["H"] >= 0 else None
    moe.moe_route(shape, s["x"], s["wg"], s["bg"], s["idx"], s["w"], None, s["counts"], s["offsets"], c["H"], hot, s["ws"])
    moe.moe_permute(shape, s["x"], s["idx"], s["offsets"], s["perm"], s["inv"], s["x_perm"], s["ws"])
    moe.moe_expert_ffn(shape, s["x_perm"], s["w1"], s["w2"], s["offsets"], hot, s["y_perm"], s["ws"])
    moe.moe_combine(shape, s["y_perm"], s["inv"], s["idx"], s["w"], hot, s["out"])
    names = ["out", "idx", "w", "counts", "offsets", "perm", "inv", "x_perm", "y_perm"] + (["mask"] if c["H"] >= 0 else [])
    return {n: s[n] for n in names}


def _expert_shares(c):
    """Expected share of the assignments per expert, largest first: the routing of 4096 random tokens."""
    rng = np.random.default_rng(0)
    logits = rng.standard_normal((4096, c["E"])) * c["gate_std"] * math.sqrt(c["d"])
    if c["zipf"]:
        logits -= c["zipf"] * np.log(np.arange(1, c["E"] + 1))
    top = np.argpartition(-logits, c["k"] - 1, axis=1)[:, :c["k"]]
    return np.sort(np.bincount(top.ravel(), minlength=c["E"]) / top.size)[::-1]


def work(case):
    c = case
    T, d, f, E, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    es = DTYPES[c["dtype"]].itemsize
    if c["call"] == "pack":
        return {"bytes": 4 * E * d * f * es, "flops": 0}
    A = T * k
    p = _expert_shares(c)
    if c["H"] >= 0:
        p = p[:c["H"]]
    active = float(np.sum(1.0 - (1.0 - np.minimum(1.0, p * k)) ** T))     # experts of the share that receive a token
    rows = A * float(np.sum(p))
    # weights of the active experts, tokens in and out, the gate
    bytes_ = 2 * active * d * f * es + 2 * T * d * es + E * d * es
    if c["call"] == "steps":
        bytes_ += A * d * es + rows * d * 4           # x_perm and y_perm are outputs
    return {"bytes": bytes_, "flops": 4 * rows * d * f + 2 * T * d * E}


def tolerance(case):
    c = case
    if c["call"] == "pack":
        return "exact"
    # Four times the largest error of these paths against the same layer computed in 64 bits (routing, both products
    # and the combine, on the listed cases).  fp32: 1.5e-7 (tiny preset) and 5.3e-7 (Switch-base width), largest
    # element 3.4e-6.  bf16: 2.3e-3 to 2.4e-3 (the hidden activation and the output are each rounded once), largest
    # element 1.8e-2; `differ`: a token whose best logits agree to the last bits of an fp32 sum may change its expert.
    if c["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 1e-2, "max": 8e-2, "differ": 1e-3}
