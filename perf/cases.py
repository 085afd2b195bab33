"""Performance cases of the MoE layer: the calls its users make, through the
entry points of ``paper_2608_17402_amd.binding``.

Kinds of case ("kind"):

  layer     moe_layer_forward of one encoder layer (inference: one image to a
            large batch; GELU or SwiGLU experts; bf16 or fp32)
  backward  moe_grouped_mlp_backward of the routed experts on a routing made
            beforehand (the expensive half of a training step)
  train     one training step of the layer through the stage calls: route,
            permute, routed and shared expert MLPs, combine, expert backward,
            and the load-balancing update of the selection bias

Widths are those of workloads/configs.py; token counts are whole images
(196, 576, 1024 or 1025 tokens each) or a handful of pooled tokens.
"""

from __future__ import annotations

import math

import torch

from paper_2608_17402_amd import binding as mb

# d, E, K, h, h_shared, act of the layer families in workloads/configs.py.
_FAMILIES = {
    "tiny": dict(d=256, E=8, K=2, h=256, hs=0, act="gelu"),
    "vitb": dict(d=768, E=64, K=8, h=384, hs=768, act="gelu"),
    "vitl": dict(d=1024, E=128, K=8, h=512, hs=1024, act="gelu"),
    "vitg": dict(d=1536, E=256, K=8, h=768, hs=1536, act="gelu"),
    "vitg_swiglu": dict(d=1536, E=256, K=8, h=768, hs=1536, act="swiglu"),
    "vith": dict(d=1280, E=31, K=7, h=854, hs=854, act="swiglu"),
}


def _case(name, kind, family, T, dtype="bf16", bias="uniform", **over):
    c = dict(name=name, kind=kind, T=T, dtype=dtype, bias=bias, **_FAMILIES[family])
    c.update(over)
    return c


def listed():
    return [
        # The smallest layer of the configurations: one 224-pixel image, fp32.
        _case("layer_tiny_f32", "layer", "tiny", 196, dtype="f32"),
        # A few pooled tokens (one per clip or crop) through one layer: launch
        # and latency bound, a handful of experts read.
        _case("layer_vitl_5tok", "layer", "vitl", 5),
        # fp32 reference inference of ViT-B widths, four 336-pixel images.
        _case("layer_vitb_f32_4img", "layer", "vitb", 2304, dtype="f32"),
        # Interactive use: one 448-pixel image with its class token, every
        # expert's weights read for some 32 rows each.
        _case("layer_vitg_1img", "layer", "vitg", 1025, bias="zero"),
        _case("layer_vitg_swiglu_1img", "layer", "vitg_swiglu", 1025, bias="zero"),
        # Small serving batches, ragged rows per expert (260 and 448 on average).
        _case("layer_vith_2img", "layer", "vith", 1153),
        _case("layer_vitl_7img", "layer", "vitl", 7175),
        # Offline embedding of large batches: 64 images.
        _case("layer_vith_64img", "layer", "vith", 65536),
        _case("layer_vitg_64img_skew", "layer", "vitg", 65536, bias="skew"),
        # One training step of the layer by its stages, 32 images.
        _case("train_vitb_32img", "train", "vitb", 18432),
        # Expert backward of a training micro-batch and of a large batch.
        _case("backward_vith_4img", "backward", "vith", 4100),
        _case("backward_vitg_64img_skew", "backward", "vitg", 65536, bias="skew", hs=0),
    ]


def _flops(c):
    mats = 3 if c["act"] == "swiglu" else 2
    routed = 2.0 * mats * c["T"] * c["K"] * c["d"] * c["h"]
    shared = 2.0 * mats * c["T"] * c["d"] * c["hs"]
    route = 2.0 * c["T"] * c["d"] * c["E"]
    back = (10.0 if mats == 2 else 16.0) * c["T"] * c["K"] * c["d"] * c["h"]
    return {"layer": routed + shared + route, "backward": back, "train": routed + shared + route + back}[c["kind"]]


def _weight(c):
    """Rough cost of a case: fp32 products run at a fraction of the bf16 rate."""
    return _flops(c) * (16.0 if c["dtype"] == "f32" else 1.0) + 2.0 * c["E"] * c["h"] * c["d"] * 100


_LIMIT = None


def draw(rng):
    global _LIMIT
    if _LIMIT is None:
        _LIMIT = max(_weight(c) for c in listed())
    while True:
        kind = rng.choice(["layer"] * 6 + ["backward", "train"])
        c = dict(_FAMILIES[rng.choice(["vitb", "vitl", "vitg", "vitg_swiglu", "vith", "tiny"])], kind=kind)
        if c["d"] == 256 or (kind == "layer" and rng.random() < 0.3):  # generic widths
            c.update(d=64 * rng.randint(4, 24), E=rng.randint(8, 200), K=rng.randint(1, 8),
                     hs=rng.choice([0, 1, 2]), act=rng.choice(["gelu", "swiglu"]))
            c["h"] = 64 * rng.randint(4, 14) if c["act"] == "gelu" else rng.randint(256, 900)
            c["hs"] *= c["h"]
        c["dtype"] = "f32" if kind == "layer" and c["act"] == "gelu" and rng.random() < 0.25 else "bf16"
        lo, hi = (1, 65536) if kind == "layer" else (512, 65536)
        if c["dtype"] == "f32":
            hi = 4608
        c["T"] = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        c["bias"] = rng.choice(["uniform", "zero", "skew"])
        if kind == "backward":
            c["hs"] = 0
        if _weight(c) <= _LIMIT:
            return c


# ------------------------------------------------------------------- inputs


def _dt(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _ld(c, h):
    return -(-h // 64) * 64 if c["act"] == "swiglu" else h


def _bias_vector(c, gen):
    """Selection biases: balanced ("zero"), as they stand early in training
    ("uniform"), or of a badly balanced layer ("skew": loads from a few tokens
    to several times the mean)."""
    E = c["E"]
    if c["bias"] == "zero":
        return torch.zeros(E, device="cuda")
    if c["bias"] == "uniform":
        return torch.rand(E, generator=gen, device="cuda") * 0.2 - 0.1
    rank = torch.randperm(E, generator=gen, device="cuda").float()
    return 0.3 * (0.5 - torch.log1p(rank) / math.log(1.0 + E))


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt, T, d, E, h, hs = _dt(c), c["T"], c["d"], c["E"], c["h"], c["hs"]
    rows = 2 if c["act"] == "swiglu" else 1

    def normal(*shape, std):
        n = math.prod(shape)
        out = torch.empty(n, dtype=dt, device="cuda")
        for i in range(0, n, 1 << 28):
            m = min(1 << 28, n - i)
            out[i:i + m] = torch.randn(m, generator=gen, device="cuda") * std
        return out.view(*shape)

    def second(*shape):  # second-layer weights, rows padded to a multiple of 64 (SwiGLU)
        w = normal(*shape, std=0.02)
        ld = _ld(c, shape[-1])
        if ld == shape[-1]:
            return w
        p = torch.zeros(*shape[:-1], ld, dtype=dt, device="cuda")
        p[..., :shape[-1]] = w
        return p

    s = dict(x=normal(T, d, std=1.0), w_router=normal(E, d, std=0.02), bias=_bias_vector(c, gen),
             w1=normal(E, rows * h, d, std=0.02), w2=second(E, d, h), w1s=None, w2s=None)
    if hs:
        s["w1s"] = normal(rows * hs, d, std=0.02)
        s["w2s"] = second(d, hs)
    if c["kind"] != "layer":
        s["grad"] = normal(T * c["K"], d, std=0.1)
    return s


def _desc(c, **over):
    kw = dict(T=c["T"], d=c["d"], E=c["E"], K=c["K"], h=c["h"], h_shared=c["hs"], lam=1.0, dtype=c["dtype"],
              flags=mb.MOE_FLAG_SWIGLU if c["act"] == "swiglu" else 0)
    kw.update(over)
    return mb.make_desc(**kw)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = _inputs(c, seed)
    s["case"], s["desc"] = c, _desc(c)
    s["ws"] = mb.alloc_workspace(s["desc"])
    T, d, E, K, dt = c["T"], c["d"], c["E"], c["K"], _dt(c)

    def empty(*shape, dtype=dt):
        return torch.empty(*shape, dtype=dtype, device="cuda")

    s["idx"] = empty(T, K, dtype=torch.int32)
    s["gate"] = empty(T, K, dtype=torch.float32)
    if kind != "backward":
        s["y"] = empty(T, d)
    if kind != "layer":
        s["counts"] = empty(E, dtype=torch.int32)
        s["offsets"] = empty(E + 1, dtype=torch.int32)
        s["slots"] = empty(T * K, dtype=torch.int32)
        s["dx"] = empty(T, d)
        s["dw1"] = torch.empty(s["w1"].shape, dtype=torch.float32, device="cuda")
        s["dw2"] = torch.empty(s["w2"].shape, dtype=torch.float32, device="cuda")
        s["bws"] = mb.alloc_backward_workspace(s["desc"])
    if kind == "backward":  # the forward's routing, kept for the backward
        mb.moe_route(s["desc"], s["x"], s["w_router"], s["bias"], s["idx"], s["gate"], s["ws"])
        mb.moe_permute(s["desc"], s["idx"], s["counts"], s["offsets"], s["slots"], s["ws"])
    if kind == "train":
        s["eout"] = empty(T * K, d)
        s["bias_next"] = torch.empty_like(s["bias"])
        if c["hs"]:  # the shared expert as a group of its own
            s["desc_s"] = _desc(c, E=1, K=1, h=c["hs"], h_shared=0)
            s["ws_s"] = mb.alloc_workspace(s["desc_s"])
            s["slots_s"] = torch.arange(T, dtype=torch.int32, device="cuda")
            s["offsets_s"] = torch.tensor([0, T], dtype=torch.int32, device="cuda")
            s["sout"] = empty(T, d)
    return s


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "layer":
        mb.moe_layer_forward(s["desc"], s["x"], s["w_router"], s["bias"], s["w1"], s["w2"], s["w1s"], s["w2s"],
                             s["y"], s["idx"], s["gate"], s["ws"])
        return [s["y"], s["idx"], s["gate"]]
    if kind == "train":
        mb.moe_route(s["desc"], s["x"], s["w_router"], s["bias"], s["idx"], s["gate"], s["ws"])
        mb.moe_permute(s["desc"], s["idx"], s["counts"], s["offsets"], s["slots"], s["ws"])
        mb.moe_grouped_mlp(s["desc"], s["x"], s["slots"], s["offsets"], s["w1"], s["w2"], s["eout"], s["ws"])
        sout = s.get("sout")
        if sout is not None:
            mb.moe_grouped_mlp(s["desc_s"], s["x"], s["slots_s"], s["offsets_s"], s["w1s"], s["w2s"], sout, s["ws_s"])
        mb.moe_combine(s["desc"], s["eout"], s["gate"], sout, s["y"])
    mb.moe_grouped_mlp_backward(s["desc"], s["x"], s["slots"], s["offsets"], s["w1"], s["w2"], s["grad"], s["dx"],
                                s["dw1"], s["dw2"], s["bws"])
    if kind == "backward":
        return [s["dx"], s["dw1"], s["dw2"]]
    # The new biases go to a second buffer: the step's own stay as they were.
    s["bias_next"].copy_(s["bias"])
    mb.moe_bias_update(s["desc"], s["counts"], s["bias_next"], 1e-3, mb.MOE_BIAS_SIGN)
    return [s["y"], s["idx"], s["gate"], s["dx"], s["dw1"], s["dw2"], s["bias_next"]]


def work(case):
    """Each input read once and each output written once; of the routed
    experts' weights those that some token chooses (expected, balanced load)."""
    c = case
    es = 4 if c["dtype"] == "f32" else 2
    mats = 3 if c["act"] == "swiglu" else 2
    T, d, E, K = c["T"], c["d"], c["E"], c["K"]
    used = E * (1.0 - (1.0 - K / E) ** T)
    wr = used * mats * c["h"] * d
    routed = (wr + mats * c["hs"] * d + E * d) * es + T * d * es
    out = T * d * es + T * K * 8
    back = wr * es + T * d * es + T * K * (d * es + 4) + T * d * es + mats * E * c["h"] * d * 4
    total = {"layer": routed + out, "backward": back,
             "train": routed + out + back - wr * es - T * d * es}[c["kind"]]
    return {"bytes": int(total), "flops": int(_flops(c))}


def tolerance(case):
    # The routing (indices and gates) is defined bit for bit. bf16: outputs
    # are rounded to bf16 twice (expert outputs, y) or at the activation and
    # once more (gradients). fp32: sums in another order.
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4, "differ": 0.0}
    return {"rel": 1e-2, "max": 6e-2, "differ": 0.0}


# ------------------------------------------------------------ 64-bit reference


def _route64(c, s):
    """The routing: logits as fp32 fused multiply-add chains over ascending
    columns (each step rounded to fp32 from 64 bits), then top-K of
    Sigmoid(s) + b in fp32 and the gates in 64 bits."""
    x, w = s["x"], s["w_router"].double().t().contiguous()
    T, E, d = c["T"], c["E"], c["d"]
    logits = torch.empty(T, E, dtype=torch.float64, device="cuda")
    for t0 in range(0, T, 16384):
        xt = x[t0:t0 + 16384].t().double().contiguous()
        acc = torch.zeros(xt.shape[1], E, dtype=torch.float64, device="cuda")
        for k in range(d):
            acc = torch.addcmul(acc, xt[k].unsqueeze(1), w[k].unsqueeze(0)).float().double()
        logits[t0:t0 + 16384] = acc
    sig = torch.sigmoid(logits)
    key = sig.float() + s["bias"]
    order = torch.sort(key, dim=1, descending=True, stable=True).indices[:, :c["K"]]
    g = torch.gather(sig, 1, order)
    return order, g / g.sum(dim=1, keepdim=True)


def _act64(c, w1, x, h):
    if c["act"] == "swiglu":
        return torch.nn.functional.silu(x @ w1[:h].t()) * (x @ w1[h:].t())
    return torch.nn.functional.gelu(x @ w1.t())


def _exact64(c, seed):
    s = _inputs(c, seed)
    T, d, E, K, h, hs = c["T"], c["d"], c["E"], c["K"], c["h"], c["hs"]
    order, gate = _route64(c, s)
    flat = order.reshape(-1)
    slots = torch.sort(flat, stable=True).indices
    counts = torch.bincount(flat, minlength=E)
    ends = torch.cumsum(counts, 0).tolist()
    idx = order.to(torch.int32)
    forward, backward = c["kind"] != "backward", c["kind"] != "layer"
    y = torch.zeros(T, d, dtype=torch.float64, device="cuda") if forward else None
    if backward:
        dxs = torch.zeros(T, d, dtype=torch.float64, device="cuda")
        dw1 = torch.zeros(s["w1"].shape, dtype=torch.float64, device="cuda")
        dw2 = torch.zeros(s["w2"].shape, dtype=torch.float64, device="cuda")
    for e in range(E):
        sl = slots[(ends[e - 1] if e else 0):ends[e]]
        w1, w2 = s["w1"][e].double(), s["w2"][e][:, :h].double()
        for p in range(0, sl.numel(), 16384):
            q = sl[p:p + 16384]
            tok = torch.div(q, K, rounding_mode="floor")
            xe = s["x"][tok].double()
            if forward:
                out = _act64(c, w1, xe, h) @ w2.t()
                y.index_add_(0, tok, out * gate.reshape(-1)[q].unsqueeze(1))
            if backward:
                go = s["grad"][q].double()
                da = go @ w2
                pre = xe @ w1.t()
                if c["act"] == "swiglu":
                    g, u = pre[:, :h], pre[:, h:]
                    sg = torch.sigmoid(g)
                    a = g * sg * u
                    dh = torch.cat([da * u * sg * (1 + g * (1 - sg)), da * g * sg], dim=1)
                else:
                    phi = 0.5 * (1 + torch.erf(pre * math.sqrt(0.5)))
                    a = pre * phi
                    dh = da * (phi + pre * torch.exp(-0.5 * pre * pre) / math.sqrt(2 * math.pi))
                dxs.index_add_(0, tok, dh @ w1)
                dw1[e] += dh.t() @ xe
                dw2[e][:, :h] += go.t() @ a
    if forward and hs:
        for t0 in range(0, T, 16384):
            xe = s["x"][t0:t0 + 16384].double()
            y[t0:t0 + 16384] += _act64(c, s["w1s"].double(), xe, hs) @ s["w2s"][:, :hs].double().t()
    if c["kind"] == "layer":
        return [y, idx, gate]
    if c["kind"] == "backward":
        return [dxs, dw1, dw2]
    sign = torch.sign(counts.double() * E - counts.sum().double())
    return [y, idx, gate, dxs, dw1, dw2, s["bias"].double() - 1e-3 * sign]


def exact(case, seed):
    out = _exact64(case, seed)
    torch.cuda.empty_cache()
    return out
