"""The work a serving program has this library do, as a list of timed cases.

A case is either

* ``call``: one eager ``dmr_qlinear_forward``, the smallest thing a caller can ask for;
* ``step``: the Linear layers of ``layers`` consecutive decoder layers on ``rows`` rows of activations, in the copy
  that ``format`` names (``w4`` group 128, ``w4pc`` per channel, ``w3`` group 128, ``bf16``).  With ``fused`` the
  layers form the dependent chain of a decoder (RMSNorm -> qkv; attention result -> attn_out + residual; RMSNorm ->
  gate_up; SwiGLU -> down + residual) through the fused entry points, attention itself standing as a given
  tensor; without it the plain entry points run on given activations.  Decode and rollout batches replay a HIP graph
  captured once, as a serving loop does; prefill chunks are called eagerly;
* ``convert``: the offline step that makes one low-precision decoder layer from fp32 weights (quantise, re-tile,
  and the bf16 dequantisation that checks it).

Weights are 0.02 N(0,1), activations N(0,1) in bf16; a state holds enough layers that weights come from memory and
not from a cache when states take turns.
"""
import math

import torch

import paper_2602_02711_amd as dmr

GROUP = 128
EPS = 1e-6
# hidden, qkv outputs, SwiGLU width of the 7B-class decoder that the benchmark measures
H7, Q7, I7 = 4096, 6144, 14336
MAX_FLOPS = 3.6e12              # of one pass: 8192 rows through one layer of that decoder
GRAPH_MAX_ROWS = 64             # rollout batches and below are replayed from a graph


def _step(name, format, rows, layers, fused, hidden=H7, qkv=Q7, inter=I7):
    return {"name": name, "kind": "step", "format": format, "rows": rows, "layers": layers, "fused": fused,
            "hidden": hidden, "qkv": qkv, "inter": inter}


def listed():
    return [
        # one small Linear called on its own: launch and host cost
        {"name": "call_w4_1row_1024", "kind": "call", "format": "w4", "rows": 1, "k": 1024, "n": 1024},
        # one token for one rollout on the low-precision copy, and the same step routed to the bf16 copy
        _step("decode_w4_1row", "w4", 1, 4, True),
        _step("decode_bf16_1row", "bf16", 1, 4, True),
        # one token for a group of parallel rollouts
        _step("rollout_w4_8rows", "w4", 8, 4, True),
        _step("rollout_w3_16rows", "w3", 16, 4, True),
        _step("rollout_bf16_32rows", "bf16", 32, 4, True),
        _step("rollout_w4_64rows", "w4", 64, 6, False),
        # a new observation appended to the prompt: short prefill
        _step("chunk_w4_200rows", "w4", 200, 4, True),
        _step("chunk_w4pc_1000rows", "w4pc", 1000, 2, True),
        # a long prompt, in either copy
        _step("prefill_bf16_3000rows", "bf16", 3000, 1, True),
        _step("prefill_w4_8192rows", "w4", 8192, 1, False),
        # making the low-precision copy of one decoder layer
        {"name": "convert_w4_layer", "kind": "convert", "format": "w4", "hidden": H7, "qkv": Q7, "inter": I7},
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(lo * (hi / lo) ** rng.random() + 0.5))


def _decoder(rng):
    """A decoder's widths: hidden 1024..8192, heads of 64..128 with fewer key/value heads, SwiGLU 2..4 times hidden."""
    hidden = 128 * _log_int(rng, 8, 64)
    qkv = hidden + 2 * rng.choice((1, 2, 4, 8)) * rng.choice((64, 80, 96, 128))
    inter = 128 * int(hidden / 128 * rng.uniform(2.0, 4.0) + 0.5)
    return hidden, qkv, inter


def draw(rng):
    kind = rng.choice(("step",) * 10 + ("call", "convert"))
    low = rng.choice(("w4", "w4", "w4", "w4pc", "w3"))
    if kind == "call":
        return {"kind": "call", "format": low, "rows": _log_int(rng, 1, 16), "k": 128 * _log_int(rng, 4, 32),
                "n": 16 * _log_int(rng, 16, 256)}
    hidden, qkv, inter = _decoder(rng)
    if kind == "convert":
        return {"kind": "convert", "format": rng.choice(("w4", "w3")), "hidden": min(hidden, H7),
                "qkv": min(qkv, Q7), "inter": min(inter, I7)}
    fmt = rng.choice((low, low, "bf16"))
    weights = sum(k * n for _, k, n in _linears(hidden, qkv, inter))
    rows = min(_log_int(rng, 1, 8192), int(MAX_FLOPS / (2.0 * weights)))
    fused = rng.random() < 0.7
    # decode: about 0.5 GB of weights to a pass, a chain of at most four decoder layers; prefill: few layers
    layers = max(1, min(4 if fused else 8, int(0.6e9 / (weights * _bytes_per_weight(fmt))))) if rows <= GRAPH_MAX_ROWS else \
        max(1, min(4, int(6e11 / (2.0 * weights * rows))))
    return {"kind": "step", "format": fmt, "rows": rows, "layers": layers, "fused": fused,
            "hidden": hidden, "qkv": qkv, "inter": inter}


def _bytes_per_weight(fmt):
    return {"w4": 0.53125, "w4pc": 0.5, "w3": 0.40625, "bf16": 2.0}[fmt]


def _linears(hidden, qkv, inter):
    return (("qkv", hidden, qkv), ("attn_out", hidden, hidden), ("gate_up", hidden, 2 * inter), ("down", inter, hidden))


def _normal(gen, shape, scale=1.0, dtype=torch.bfloat16):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(scale).to(dtype)


def _layer(fmt, w):
    """What a program keeps of one Linear: the handle of a low-precision layer, or the bf16 weights."""
    if fmt == "bf16":
        return w.to(torch.bfloat16)
    if fmt == "w3":
        return dmr.dmr_qlinear_w3_create(*dmr.dmr_qlinear_quantize_w3(w, GROUP), GROUP)
    qw, s, z = dmr.dmr_qlinear_quantize(w, GROUP)
    if fmt == "w4pc":
        # one scale per row about the row's largest weight; the codes are those of the group-wise quantiser, which
        # cover 0..15 like any checkpoint's
        return dmr.dmr_qlinear_create_per_channel(qw, (w.abs().amax(dim=1) / 7.5).to(torch.bfloat16))
    return dmr.dmr_qlinear_create(qw, s, z, GROUP)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    st = dict(case)
    fmt = case["format"]
    if case["kind"] == "call":
        st["layer"] = _layer(fmt, _normal(gen, (case["n"], case["k"]), 0.02, torch.float32))
        st["x"] = _normal(gen, (case["rows"], case["k"]))
        return st
    H, Q, I = case["hidden"], case["qkv"], case["inter"]
    if case["kind"] == "convert":
        st["w"] = {name: _normal(gen, (n, k), 0.02, torch.float32) for name, k, n in _linears(H, Q, I)}
        return st
    M = case["rows"]
    st["net"] = [{name: _layer(fmt, _normal(gen, (n, k), 0.02, torch.float32)) for name, k, n in _linears(H, Q, I)}
                 for _ in range(case["layers"])]
    if case["fused"]:
        st["gamma"] = [[(1.0 + 0.1 * torch.randn(H, generator=gen, device="cuda")).to(torch.bfloat16) for _ in range(2)]
                       for _ in range(case["layers"])]
        st["h0"] = _normal(gen, (M, H))
        st["attn"] = [_normal(gen, (M, H)) for _ in range(case["layers"])]
        st["buf"] = [{"qkv": torch.empty((M, Q), dtype=torch.bfloat16, device="cuda"),
                      "mid": torch.empty((M, H), dtype=torch.bfloat16, device="cuda"),
                      "gate_up": torch.empty((M, 2 * I), dtype=torch.bfloat16, device="cuda"),
                      "h": torch.empty((M, H), dtype=torch.bfloat16, device="cuda")} for _ in range(case["layers"])]
    else:
        st["x"] = [{name: _normal(gen, (M, k)) for name, k, n in _linears(H, Q, I)} for _ in range(case["layers"])]
        st["y"] = [{name: torch.empty((M, n), dtype=torch.bfloat16, device="cuda") for name, k, n in _linears(H, Q, I)}
                   for _ in range(case["layers"])]
    if M <= GRAPH_MAX_ROWS:
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            _pass(st)
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                _pass(st)
        torch.cuda.synchronize()
        st["graph"] = graph
    return st


def _pass(st):
    """The launches of one step, in order."""
    bf16 = st["format"] == "bf16"
    if not st["fused"]:
        forward = dmr.dmr_qlinear_bf16_forward if bf16 else dmr.dmr_qlinear_forward
        for net, x, y in zip(st["net"], st["x"], st["y"]):
            for name in net:
                forward(net[name], x[name], out=y[name])
        return
    forward = dmr.dmr_qlinear_bf16_forward_fused if bf16 else dmr.dmr_qlinear_forward_fused
    h = st["h0"]
    for net, gamma, attn, buf in zip(st["net"], st["gamma"], st["attn"], st["buf"]):
        forward(net["qkv"], dmr.DMR_PRO_RMSNORM, h, gamma=gamma[0], eps=EPS, out=buf["qkv"])
        forward(net["attn_out"], dmr.DMR_PRO_NONE, attn, residual=h, out=buf["mid"])
        forward(net["gate_up"], dmr.DMR_PRO_RMSNORM, buf["mid"], gamma=gamma[1], eps=EPS, out=buf["gate_up"])
        forward(net["down"], dmr.DMR_PRO_SWIGLU, buf["gate_up"], residual=buf["mid"], out=buf["h"])
        h = buf["h"]


def run(st):
    if st["kind"] == "call":
        return dmr.dmr_qlinear_forward(st["layer"], st["x"])
    if st["kind"] == "convert":
        out = {}
        for name, w in st["w"].items():
            if st["format"] == "w3":
                qw, s, z = dmr.dmr_qlinear_quantize_w3(w, GROUP)
                layer = dmr.dmr_qlinear_w3_create(qw, s, z, GROUP)
            else:
                qw, s, z = dmr.dmr_qlinear_quantize(w, GROUP)
                layer = dmr.dmr_qlinear_create(qw, s, z, GROUP)
            out[name] = [qw, s, z, layer.storage, dmr.dmr_qlinear_dequantize(layer)]
        return out
    if "graph" in st:
        st["graph"].replay()
    else:
        _pass(st)
    return st["buf"] if st["fused"] else st["y"]


def work(case):
    bpw = _bytes_per_weight(case["format"])
    if case["kind"] == "call":
        m, k, n = case["rows"], case["k"], case["n"]
        return {"bytes": k * n * bpw + 2 * m * (k + n), "flops": 2.0 * m * k * n}
    linears = _linears(case["hidden"], case["qkv"], case["inter"])
    weights = sum(k * n for _, k, n in linears)
    if case["kind"] == "convert":
        # fp32 in, canonical arrays out; canonical in, storage out; storage in, bf16 out
        return {"bytes": weights * (4 + 4 * bpw + 2), "flops": 0.0}
    m, L = case["rows"], case["layers"]
    acts = sum(k + n for _, k, n in linears)
    if case["fused"]:
        acts += case["inter"] + 2 * case["hidden"]          # SwiGLU reads twice the layer's input width; residuals
    return {"bytes": L * (weights * bpw + 2.0 * m * acts), "flops": 2.0 * L * m * weights}


def tolerance(case):
    if case["kind"] == "convert":
        return "exact"
    # Against the same pass in fp64 with bf16 roundings at the same places: single Linears 1.1e-4 (bf16 outputs that
    # fall on the other side of a tie) and at most one bf16 ulp, 7.8e-3; chains of four decoder layers, whose bf16
    # residual stream carries such single-ulp differences on, 4e-3 .. 6e-3 and at most 3.6e-2.
    if case["kind"] == "step" and case["fused"]:
        return {"rel": 2e-2, "max": 0.15}
    return {"rel": 5e-4, "max": 2e-2}
