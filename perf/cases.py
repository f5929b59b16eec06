"""The work a program has this library do, as measurable cases.

A case is one call of the MoE layer (or, for "steps", of its five stand-alone steps in a row) on
one problem statement.  The layer shapes are the ones the benchmark and the tests use: a
DeepSeek-V3-shaped layer (256 experts, top-8, group-limited sigmoid routing) in bf16 and in
block-scaled fp8, whole or as the 32-expert share of one device under expert parallelism, a
Mixtral-shaped layer, a tiny one and generic odd-sized ones; token counts run from one decoded
token to a long prefill.
"""
from __future__ import annotations

import math

import torch

from paper_2602_19128_amd import binding as moe
from paper_2602_19128_amd import synthetic as syn

DEVICE = "cuda"
QBLOCK = 128                 # edge of an fp8 scale block
FP8_MAX = 448.0              # largest finite e4m3 magnitude

# Layer shapes; "softmax" layers route without bias, "sigmoid" ones with bias and expert groups.
DSV3 = dict(H=7168, I=2048, E=256, top_k=8, scoring="sigmoid", n_group=8, topk_group=4, routed_scale=2.5)
MIXTRAL = dict(H=4096, I=14336, E=8, top_k=2, scoring="softmax", n_group=1, topk_group=1, routed_scale=1.0)


def _case(kind, dtype, T, shape, hot=0, local_offset=0, local_experts=0, name=None):
    """dtype: "bf16", "fp8" (hidden states arrive block-quantised) or "fp8_qx" (they arrive as bf16
    and the layer quantises them).  hot: experts whose choice is favoured by +0.5."""
    case = dict(kind=kind, dtype=dtype, T=T, hot=hot, local_offset=local_offset, local_experts=local_experts, **shape)
    if name is not None:
        case["name"] = name
    return case


def _softmax_shape(H, I, E, top_k):
    return dict(H=H, I=I, E=E, top_k=top_k, scoring="softmax", n_group=1, topk_group=1, routed_scale=1.0)


def listed():
    return [
        # the smallest layer the tests run: launches and round trips only
        _case("forward", "bf16", 16, _softmax_shape(256, 128, 8, 2), name="tiny"),
        # a mid-sized layer with sizes that divide nothing evenly (multiples of 64 only)
        _case("forward", "bf16", 333, _softmax_shape(1344, 704, 60, 6), name="odd"),
        # three sequences being decoded with few, large experts
        _case("forward", "bf16", 3, MIXTRAL, name="mixtral_decode"),
        # a prompt of 512 tokens: more weights than arithmetic
        _case("forward", "bf16", 512, MIXTRAL, name="mixtral_prefill"),
        # a long prompt or several: 1024 rows per expert, the matrix cores' regime
        _case("forward", "bf16", 4096, MIXTRAL, name="mixtral_long"),
        # 64 sequences being decoded on a whole DeepSeek-shaped layer: a pure weight stream
        _case("forward", "bf16", 64, DSV3, name="dsv3_decode"),
        # the benchmark's headline: a 4096-token prefill of the same layer
        _case("forward", "bf16", 4096, DSV3, name="dsv3_prefill"),
        # a ragged prefill whose router favours 16 of the 256 experts
        _case("forward", "bf16", 1500, DSV3, hot=16, name="dsv3_skew"),
        # fp8 weights and hidden states, all experts on one device
        _case("forward", "fp8", 1024, DSV3, name="fp8_prefill"),
        # one device's share under 8-way expert parallelism, prefill
        _case("forward", "fp8", 4096, DSV3, local_offset=96, local_experts=32, name="fp8_share"),
        # the same share while decoding, bf16 hidden states quantised by the layer
        _case("forward", "fp8_qx", 200, DSV3, local_offset=32, local_experts=32, name="fp8_share_decode"),
        # the share's steps called one by one (a program that puts its own work in between) on a
        # batch gathered from many sequences: 512 rows per expert
        _case("steps", "fp8", 16384, DSV3, local_offset=160, local_experts=32, name="fp8_share_steps"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(["small", "generic", "mixtral", "dsv3", "fp8_full", "fp8_share", "fp8_share"])
    if family == "small":
        E = rng.randint(4, 16)
        shape = _softmax_shape(64 * rng.randint(2, 16), 64 * rng.randint(1, 12), E, rng.randint(1, min(4, E)))
        return _case("forward", "bf16", _log_int(rng, 1, 64), shape)
    if family == "generic":
        E = rng.randint(17, 96)
        shape = _softmax_shape(64 * rng.randint(8, 40), 64 * rng.randint(4, 24), E, rng.randint(2, 8))
        return _case(rng.choice(["forward", "steps"]), "bf16", _log_int(rng, 8, 4096), shape)
    if family == "mixtral":
        return _case("forward", "bf16", _log_int(rng, 1, 4096), MIXTRAL)
    if family == "dsv3":
        return _case("forward", "bf16", _log_int(rng, 1, 4096), DSV3, hot=rng.choice([0, 0, 16]))
    if family == "fp8_full":
        return _case("forward", rng.choice(["fp8", "fp8_qx"]), _log_int(rng, 1, 4096), DSV3)
    kind = rng.choice(["forward", "forward", "steps"])
    dtype = "fp8" if kind == "steps" else rng.choice(["fp8", "fp8_qx"])
    return _case(kind, dtype, _log_int(rng, 1, 16384), DSV3, local_offset=32 * rng.randint(0, 7), local_experts=32)


def _local_experts(case):
    return case["local_experts"] or case["E"]


def _config(case):
    fp8 = case["dtype"] != "bf16"
    return moe.MoEConfig(case["T"], case["H"], case["I"], case["E"], case["top_k"],
                         {"softmax": 0, "sigmoid": 1}[case["scoring"]], 1, case["n_group"], case["topk_group"], 2,
                         1 if fp8 else 0, case["routed_scale"], case["local_offset"], case["local_experts"],
                         1 if case["dtype"] == "fp8_qx" else 0)


def _bias(case, gen, device):
    if case["scoring"] != "sigmoid":
        return None
    bias = torch.rand((case["E"],), generator=gen, device=device) * 0.2 - 0.1
    if case["hot"]:
        per, size = case["hot"] // case["n_group"], case["E"] // case["n_group"]
        bias.view(case["n_group"], size)[:, :per] += 0.5
    return bias


def _inputs(case, seed):
    """Hidden states ~ N(0,1), router and expert weights ~ N(0, 1/fan_in), the router's bias uniform."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    T, H, I, E, EL = case["T"], case["H"], case["I"], case["E"], _local_experts(case)
    fp8 = case["dtype"] != "bf16"
    x = torch.randn((T, H), generator=gen, device=DEVICE)
    x, x_scale = syn.quantize_rows_1x128(x) if case["dtype"] == "fp8" else (x.to(torch.bfloat16), None)
    router_w = torch.randn((E, H), generator=gen, device=DEVICE) * H ** -0.5
    bias = _bias(case, gen, DEVICE)

    def weights(rows, cols):
        if not fp8:
            w = torch.empty((EL, rows, cols), dtype=torch.bfloat16, device=DEVICE)
            for e in range(EL):
                w[e].normal_(0.0, cols ** -0.5, generator=gen)
            return w, None
        w = torch.empty((EL, rows, cols), dtype=torch.float8_e4m3fn, device=DEVICE)
        scale = torch.empty((EL, rows // QBLOCK, cols // QBLOCK), device=DEVICE)
        for e in range(EL):
            q, s = syn.quantize_blocks_128x128(torch.randn((rows, cols), generator=gen, device=DEVICE) * cols ** -0.5)
            w[e], scale[e] = q, s
        return w, scale

    w1, w1_scale = weights(2 * I, H)
    w2, w2_scale = weights(H, I)
    return dict(x=x, x_scale=x_scale, router_w=router_w, bias=bias, w1=w1, w1_scale=w1_scale, w2=w2, w2_scale=w2_scale)


def prepare(case, seed):
    cfg = _config(case)
    state = dict(kind=case["kind"], cfg=cfg, **_inputs(case, seed))
    if case["kind"] == "forward":
        # a serving loop keeps its output and workspace
        state["out"] = torch.empty((case["T"], case["H"]), dtype=torch.bfloat16, device=DEVICE)
        state["workspace"] = torch.empty((moe.moe_workspace_size(cfg),), dtype=torch.uint8, device=DEVICE)
    return state


def run(state):
    s, cfg = state, state["cfg"]
    if s["kind"] == "forward":
        return moe.moe_forward(cfg, s["x"], s["x_scale"], s["router_w"], s["bias"], s["w1"], s["w1_scale"], s["w2"],
                               s["w2_scale"], out=s["out"], workspace=s["workspace"])
    ids, w = moe.moe_route(cfg, s["x"], s["x_scale"], s["router_w"], s["bias"])
    _, sorted_pair, inv, tiles, sched = moe.moe_permute(cfg, ids)
    act, act_scale = moe.moe_grouped_gemm_swiglu(cfg, s["x"], s["x_scale"], s["w1"], s["w1_scale"], sorted_pair, tiles, sched)
    y = moe.moe_grouped_gemm_down(cfg, act, act_scale, s["w2"], s["w2_scale"], tiles, sched)
    return {"ids": ids, "w": w, "out": moe.moe_combine(cfg, y, w, inv)}


def _route(case, logits, bias):
    """Expert ids [T,k] in descending key order (equal keys: lower index first) and their weights."""
    s = torch.softmax(logits, dim=1) if case["scoring"] == "softmax" else torch.sigmoid(logits)
    key = s if bias is None else s + bias.to(s.dtype)
    if case["n_group"] > 1:
        T, G = key.shape[0], case["n_group"]
        grouped = key.view(T, G, -1)
        score = grouped.topk(2, dim=2).values.sum(dim=2)
        best = torch.sort(score, dim=1, descending=True, stable=True).indices[:, :case["topk_group"]]
        kept = torch.zeros((T, G), dtype=torch.bool, device=key.device).scatter_(1, best, True)
        key = grouped.masked_fill(~kept.unsqueeze(2), -math.inf).view(T, -1)
    ids = torch.sort(key, dim=1, descending=True, stable=True).indices[:, :case["top_k"]]
    w = s.gather(1, ids)
    return ids, w / w.sum(dim=1, keepdim=True) * case["routed_scale"]


def _dequantise(q, scale, rows):
    """fp8 payload [N,K] with one scale per (rows x 128) block, as float64."""
    v = q.double()
    if scale is None:
        return v
    N, K = v.shape
    return (v.view(N // rows, rows, K // QBLOCK, QBLOCK) * scale.double()[:, None, :, None]).view(N, K)


def _quantise_rows(v):
    """Values after a trip through e4m3 with one scale (amax / 448) per 1x128 block."""
    b = v.view(v.shape[0], -1, QBLOCK)
    amax = b.abs().amax(dim=2, keepdim=True)
    scale = torch.where(amax > 0, amax / torch.full_like(amax, FP8_MAX), torch.ones_like(amax))
    q = (b / scale).clamp(-FP8_MAX, FP8_MAX).to(torch.float8_e4m3fn)
    return (q.double() * scale.double()).view(v.shape)


def exact(case, seed):
    """The layer in float64.  The fp8 layers' own quantisation steps (hidden states with "fp8_qx", the
    activations between the projections) are part of what they compute and are applied here too."""
    p = _inputs(case, seed)
    I, lo = case["I"], case["local_offset"]
    fp8 = case["dtype"] != "bf16"
    x = _dequantise(p["x"], p["x_scale"], 1)
    ids, w = _route(case, x @ p["router_w"].double().t(), p["bias"])
    if case["dtype"] == "fp8_qx":
        x = _quantise_rows(p["x"].float())                # binary32 divisions decide the codes
    out = torch.zeros_like(x)
    scale_of = lambda t, e: None if t is None else t[e]
    for e in range(_local_experts(case)):
        token, slot = (ids == lo + e).nonzero(as_tuple=True)
        if token.numel() == 0:
            continue
        gu = x[token] @ _dequantise(p["w1"][e], scale_of(p["w1_scale"], e), QBLOCK).t()
        act = torch.nn.functional.silu(gu[:, :I]) * gu[:, I:]
        if fp8:
            act = _quantise_rows(act)
        y = act @ _dequantise(p["w2"][e], scale_of(p["w2_scale"], e), QBLOCK).t()
        out.index_add_(0, token, y * w[token, slot].unsqueeze(1))
    if case["kind"] == "forward":
        return out
    return {"ids": ids.to(torch.int32), "w": w, "out": out}


def _rows_per_expert(case):
    """Rows each local expert receives from a router of this kind: logits of such inputs are N(0,1)."""
    gen = torch.Generator().manual_seed(1)
    bias = _bias(case, gen, "cpu")
    ids, _ = _route(case, torch.randn((case["T"], case["E"]), generator=gen), bias)
    count = torch.bincount(ids.flatten(), minlength=case["E"])
    return count[case["local_offset"]:case["local_offset"] + _local_experts(case)]


def work(case):
    """Each active expert's weights, the hidden states and the router's weights once, the output once."""
    T, H, I, E = case["T"], case["H"], case["I"], case["E"]
    rows = _rows_per_expert(case)
    active, pairs = int((rows > 0).sum()), int(rows.sum())
    per_weight = 2.0 if case["dtype"] == "bf16" else 1.0 + 4.0 / QBLOCK ** 2
    per_hidden = 1.0 + 4.0 / QBLOCK if case["dtype"] == "fp8" else 2.0
    size = active * 3 * H * I * per_weight + T * H * per_hidden + E * H * 4 + T * H * 2
    if case["kind"] == "steps":
        size += T * case["top_k"] * 8
    return {"bytes": size, "flops": 6 * H * I * pairs + 2 * T * E * H}


def tolerance(case):
    # outputs, activations and expert rows are rounded to bf16 (fp8: also to e4m3): 2.6e-3 to 2.9e-3 from float64
    tol = {"rel": 1e-2}
    if case["kind"] == "steps":
        tol["differ"] = 1e-4                              # experts whose keys tie within fp32 rounding
    return tol
