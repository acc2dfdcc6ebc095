"""Performance cases of the compressed-MoE decode layer.

Each case is one call (or one short sequence of calls) that a serving program
makes per decode step through ``paper_2609_21137_amd.cardan``, with the buffers
such a program keeps between steps (weights on the device, one workspace,
output tensors) and fresh activations. Together the listed cases cover the
range of the library: batch 1 (a latency chain) to 64 (the largest batch of a
call), the five layer shapes of ``configs``, block lengths d = 8 and 4 (2 in
the draws), ranks 8 to 512, gated and up-only experts, the compressed,
dense-down and dense weight forms, uniform and skewed routing, one call per
layer, the split entry points, and a stack of layers in one call.

Inputs follow the laws of ``synth_device``: x ~ N(0, 1); router, bases ~
N(0, 1/H); code books std 0.02; V and A std 0.01; dense matrices std 0.02;
codes uniform; router bias 1e-3 e (+2 on the first 8 experts of a skewed
layer). Their weights are larger than the last-level cache over the states
that a measurement rotates.
"""

from __future__ import annotations

import functools
import math

import torch

from paper_2609_21137_amd import cardan
from paper_2609_21137_amd.configs import (DSV2_LITE_B1, GEMMA4_B1, NEMOTRON3_B1, OLMOE_B1, QWEN3_B1,
                                          TINY, WIDE_SKEW_B4)

EPS = 1e-6


def _case(w, B, form="layer", **more):
    c = dict(H=w.H, I=w.I, E=w.E, top_k=w.top_k, d=w.d, K=w.K, r=w.r, B=B, form=form,
             relu2=w.act == "relu2_up", skew=bool(w.hot_experts), layers=1, separate=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: launches, hand-offs and host work are all of it
        _case(TINY, 1, name="tiny_b1"),
        # one user's next token on the shape of the headline benchmark
        _case(QWEN3_B1, 1, name="qwen3_b1"),
        # a small server's decode batch on the same shape
        _case(QWEN3_B1, 16, name="qwen3_b16"),
        # the largest batch of one call: nearly every expert is active, several tokens each
        _case(QWEN3_B1, 64, name="qwen3_b64"),
        # a wide layer whose routing is skewed to 8 hot experts
        _case(WIDE_SKEW_B4, 4, name="wide_skew_b4"),
        # an ordinary batch at a large rank (r = 384), few experts
        _case(DSV2_LITE_B1, 8, name="dsv2_lite_b8"),
        # the shorter block length (d = 4) at a large batch: half of the experts get 4+ tokens
        _case(OLMOE_B1, 32, name="olmoe_b32"),
        # up-only squared-ReLU experts at the largest rank (r = 512)
        _case(NEMOTRON3_B1, 16, name="nemotron3_b16"),
        # an odd batch through the split entry points (a program that routes, projects, runs the
        # experts and normalises by separate calls), with a basis of its own for the up projection
        _case(GEMMA4_B1, 7, form="split", separate=True, name="gemma4_split_b7"),
        # compressed gate/up with the down projection left in bf16
        _case(QWEN3_B1, 16, form="dense_down", name="qwen3_dense_down_b16"),
        # the uncompressed layer: the most bytes of one call
        _case(QWEN3_B1, 16, form="dense", name="qwen3_dense_b16"),
        # a stack of layers in one call, normalised between (the decode step of a whole model)
        _case(QWEN3_B1, 16, form="step", layers=4, name="qwen3_step4_b16"),
    ]


def _shape_case(rng, form):
    """A drawn layer: one of the models' shapes, or a generic one with odd sizes."""
    relu2 = form in ("layer", "dense") and rng.random() < 0.25
    if rng.random() < 0.4:
        w = NEMOTRON3_B1 if relu2 else rng.choice((QWEN3_B1, DSV2_LITE_B1, OLMOE_B1, GEMMA4_B1, WIDE_SKEW_B4))
        c = _case(w, 1, form=form)
    else:
        E = int(round(math.exp(rng.uniform(math.log(8), math.log(256)))))
        c = dict(H=64 * int(round(math.exp(rng.uniform(math.log(4), math.log(64))))),
                 I=32 * int(round(math.exp(rng.uniform(math.log(4), math.log(56))))),
                 E=E, top_k=rng.randint(1, min(E, 10)), d=rng.choice((8, 8, 8, 4, 4, 2)),
                 K=rng.choice((256, 256, 256, 128, rng.randint(16, 255))),
                 r=8 * rng.randint(0, 64), B=1, form=form, relu2=relu2, skew=E >= 16 and rng.random() < 0.25,
                 layers=1, separate=False)
        if form == "split":
            c["r"] = max(8, c["r"])
    c["B"] = int(round(math.exp(rng.uniform(0.0, math.log(64)))))
    c["separate"] = c["r"] > 0 and not relu2 and form != "dense" and rng.random() < 0.25
    if form == "step":
        c["layers"] = rng.randint(2, 4)
    if form == "dense":
        c["d"], c["K"], c["r"] = 8, 256, 0
    return c


def draw(rng):
    top = [work(c) for c in listed()]
    most = {m: max(w[m] for w in top) for m in ("bytes", "flops")}
    while True:
        form = rng.choice(("layer",) * 6 + ("split", "dense_down", "dense", "step"))
        c = _shape_case(rng, form)
        stored = c["layers"] * (_expert_bytes(c) * c["E"])
        w = work(c)
        if stored < 1.5e9 and all(w[m] <= most[m] for m in most):
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _shape(c):
    return cardan.make_shape(c["H"], c["I"], c["E"], c["top_k"], c["d"], c["K"], c["r"])


def _tensors(c, gen):
    """One layer's device tensors (compressed and, for the forms that have them, dense)."""
    H, I, E, d, K, r = (c[k] for k in ("H", "I", "E", "d", "K", "r"))

    def normal(shape, std):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(torch.bfloat16)

    def codes(shape):
        return torch.randint(0, K, shape, generator=gen, device="cuda", dtype=torch.uint8)

    T = {"router_w": normal((H, E), H ** -0.5)}
    bias = 1e-3 * torch.arange(E, dtype=torch.float64)
    if c["skew"]:
        bias[:8] += 2.0
    T["router_bias"] = bias.float().cuda()
    gate = not c["relu2"]
    if c["form"] != "dense":
        T["cb_gate"] = normal((K, d), 0.02) if gate else None
        T["cb_up"] = normal((K, d), 0.02)
        T["codes_gate"] = codes((E, H // d, I)) if gate else None
        T["codes_up"] = codes((E, H // d, I))
        if r > 0:
            T["U_gate"] = normal((H, r), H ** -0.5) if gate else None
            T["U_up"] = normal((H, r), H ** -0.5) if c["separate"] or not gate else T["U_gate"]
            T["V_gate"] = normal((E, r, I), 0.01) if gate else None
            T["V_up"] = normal((E, r, I), 0.01)
    if c["form"] not in ("dense", "dense_down"):
        T["cb_down"] = normal((K, d), 0.02)
        T["codes_down"] = codes((E, I // d, H))
        if r > 0:
            T["A_down"] = normal((E, I, r), 0.01)
            T["B_down"] = normal((r, H), H ** -0.5)
    if c["form"] == "dense":
        T["W_gate"] = normal((E, H, I), 0.02) if gate else None
        T["W_up"] = normal((E, H, I), 0.02)
    if c["form"] in ("dense", "dense_down"):
        T["W_down"] = normal((E, I, H), 0.02)
    return T


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    layers = [_tensors(c, gen) for _ in range(c["layers"])]
    x = torch.randn((c["B"], c["H"]), generator=gen, device="cuda").to(torch.bfloat16)
    return layers, x


def prepare(case, seed):
    c = dict(case)
    layers, x = _inputs(c, seed)
    B, H, k, L = c["B"], c["H"], c["top_k"], c["layers"]
    shape = _shape(c)
    s = {"form": c["form"], "relu2": c["relu2"], "shape": shape, "x": x, "ws": cardan.new_workspace(shape, B),
         "out": torch.empty((B, H), dtype=torch.float32, device="cuda")}
    lead = (L,) if c["form"] == "step" else ()
    s["idx"] = torch.empty(lead + (B, k), dtype=torch.int32, device="cuda")
    s["w"] = torch.empty(lead + (B, k), dtype=torch.float32, device="cuda")
    if c["form"] == "dense":
        s["layer"] = cardan.DenseLayer(layers[0])
    else:
        s["layers"] = [cardan.DeviceLayer(t) for t in layers]
        s["layer"] = s["layers"][0]
        s["W_down"] = layers[0].get("W_down")
    if c["form"] == "step":
        s["x_norm"] = torch.empty((L - 1, B, H), dtype=torch.bfloat16, device="cuda")
        s["result"] = {"y": s["out"], "x_norm": s["x_norm"], "topk_idx": list(s["idx"].unbind(0)),
                       "topk_w": list(s["w"].unbind(0))}
    return s


def run(s):
    form, shape, x, ws = s["form"], s["shape"], s["x"], s["ws"]
    if form == "step":
        cardan.moe_decode_step(shape, x, s["layers"], eps=EPS, ws=ws, out=s["out"], x_norm=s["x_norm"],
                               idx=s["idx"], w=s["w"])
        return s["result"]
    if form == "split":
        L = s["layer"]
        T = L.tensors
        idx, w = cardan.route_topk(shape, x, T["router_w"], T["router_bias"], ws=ws)
        z = cardan.shared_proj(shape, x, T["U_gate"], T["U_up"], ws=ws)
        y = cardan.vq_lr_expert_ffn(shape, x, idx, w, z, L, ws=ws, out=s["out"])
        return {"y": y, "topk_idx": idx, "topk_w": w, "z": z, "x_next": cardan.rmsnorm_bf16(y, EPS)}
    kw = dict(ws=ws, out=s["out"], idx=s["idx"], w=s["w"])
    if form == "dense":
        y, idx, w = cardan.dense_moe_layer(shape, x, s["layer"], relu2=s["relu2"], **kw)
    elif form == "dense_down":
        y, idx, w = cardan.moe_layer_dense_down(shape, x, s["layer"], s["W_down"], **kw)
    elif s["relu2"]:
        y, idx, w = cardan.moe_layer_relu2(shape, x, s["layer"], **kw)
    else:
        y, idx, w = cardan.moe_layer(shape, x, s["layer"], **kw)
    return {"y": y, "topk_idx": idx, "topk_w": w}


# ---------------------------------------------------------------------------
# work and tolerance
# ---------------------------------------------------------------------------
def _expert_bytes(c):
    """Weight bytes of one expert."""
    H, I, d, r = c["H"], c["I"], c["d"], c["r"]
    proj = 1 if c["relu2"] else 2
    gu = proj * H * I * 2 if c["form"] == "dense" else proj * (H * I // d + r * I * 2)
    dn = I * H * 2 if c["form"] in ("dense", "dense_down") else I * H // d + I * r * 2
    return gu + dn


@functools.lru_cache(maxsize=None)
def _active(E, k, B, skew):
    """Mean number of distinct experts that B tokens select, over fixed draws of logits N(0, 1) + bias."""
    gen = torch.Generator().manual_seed(0)
    logits = torch.randn((16, B, E), generator=gen) + 1e-3 * torch.arange(E)
    if skew:
        logits[..., :8] += 2.0
    hit = torch.zeros((16, E)).scatter_(1, logits.topk(k, dim=-1).indices.flatten(1), 1.0)
    return float(hit.sum()) / 16


def work(case):
    """Each active expert's weights, the shared tensors and the inputs once, the outputs once."""
    c = case
    H, I, E, k, d, K, r, B = (c[m] for m in ("H", "I", "E", "top_k", "d", "K", "r", "B"))
    if c["form"] == "dense":
        r = 0
    proj = 1 if c["relu2"] else 2
    bases = 2 if c["separate"] else 1
    down = c["form"] not in ("dense", "dense_down")
    nbytes = _active(E, k, B, c["skew"]) * _expert_bytes(c) + H * E * 2 + E * 4 + bases * H * r * 2
    if c["form"] != "dense":
        nbytes += (proj + down) * K * d * 2
    if down:
        nbytes += r * H * 2
    nbytes += B * H * 2 + B * H * 4 + B * k * 8  # x, y, the routing
    S = B * k
    flops = 2 * B * H * E + 2 * B * H * r * bases + S * 2 * H * I * (proj + 1) + S * 2 * r * I * (proj + down)
    if down:
        flops += 2 * B * r * H
    if c["form"] == "split":
        nbytes += 2 * B * r * 4 + B * H * 2
    return {"bytes": c["layers"] * nbytes, "flops": c["layers"] * flops}


def tolerance(case):
    # float32 sums of products of exact bf16 values (and of bf16 hi + lo halves of float32 ones)
    # in another order
    if case["form"] == "step":
        # the bf16 inputs of later layers round another way in a few places, which then can swap
        # two experts of nearly equal logits
        return {"rel": 2e-3, "max": 0.1, "differ": 0.01}
    if case["form"] == "split":
        # x_next is bf16: one place in some thousands rounds the other way
        return {"rel": 2e-4, "max": 0.02, "differ": 0.0}
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _route64(c, T, x):
    logits = x @ T["router_w"].double() + T["router_bias"].double()
    v, idx = torch.topk(logits, c["top_k"], dim=1)
    return idx, torch.softmax(v, dim=1)


def _matrix64(codes, book, d):
    """[n / d, m] codes into [n, m]: element i of block b's code word at row b d + i."""
    n, m = codes.shape
    return book.double()[codes.long()].permute(0, 2, 1).reshape(n * d, m)


def _experts64(c, T, x, idx, w):
    d, r = c["d"], c["r"]
    y = torch.zeros_like(x)

    def product(v, name, e):
        if c["form"] == "dense":
            return v @ T["W_" + name][e].double()
        out = v @ _matrix64(T["codes_" + name][e], T["cb_" + name], d)
        return out + (v @ T["U_" + name].double()) @ T["V_" + name][e].double() if r > 0 else out

    for e in torch.unique(idx).tolist():
        t, j = (idx == e).nonzero(as_tuple=True)
        v = x[t]
        u = product(v, "up", e)
        if c["relu2"]:
            p = u.clamp(min=0).square()
        else:
            p = torch.nn.functional.silu(product(v, "gate", e)) * u
        if c["form"] in ("dense", "dense_down"):
            o = p @ T["W_down"][e].double()
        else:
            o = p @ _matrix64(T["codes_down"][e], T["cb_down"], d)
            if r > 0:
                o = o + (p @ T["A_down"][e].double()) @ T["B_down"].double()
        y.index_add_(0, t, o * w[t, j][:, None])
    return y


def exact(case, seed):
    c = dict(case)
    layers, x = _inputs(c, seed)
    T, x = layers[0], x.double()
    idx, w = _route64(c, T, x)
    if c["form"] == "step":
        # values after the first layer hang on how its output rounds to bf16: no 64-bit value
        none = [None] * (c["layers"] - 1)
        return {"y": None, "x_norm": None, "topk_idx": [idx.int()] + none, "topk_w": [w] + none}
    y = _experts64(c, T, x, idx, w)
    out = {"y": y, "topk_idx": idx.int(), "topk_w": w}
    if c["form"] == "split":
        out["z"] = torch.stack([x @ T["U_gate"].double(), x @ T["U_up"].double()])
        out["x_next"] = y * torch.rsqrt(y.square().mean(dim=1, keepdim=True) + EPS)
    return out
