"""The work a user of this framework has it do, as cases that can be timed and checked.

A case is a dict of plain values. `kind` says which public entry points it goes through:

  stack       decode steps through a stack of MoE layers, every layer one `moe_layer_forward`, the step captured
              once into a HIP graph and replayed with each step's hidden states
  layer       one `moe_layer_forward` call (with its routing), launched directly
  routed      one `moe_layer_forward_routed` call: the routing is given by the caller
  expert      one `moe_expert_ffn_q` call
  compress    fp32 weights of an expert -> packed, in the layout a layer is created with
  decompress  packed weights of an expert -> fp32

Weights are N(0, 0.02), hidden states N(0, 1), router weights N(0, 0.02), as in the benchmark's configurations.
"""
import math
import random

import torch

import paper_2308_14352_amd as moeq

DEV = "cuda:0"

# Shapes of the benchmark's configurations: Switch-base, Switch-large and Mixtral-8x7B layers.
SWITCH_BASE = {"d": 768, "f": 3072, "k": 1, "act": "relu", "renorm": False, "group": 32, "x": "f32"}
SWITCH_LARGE = {"d": 1024, "f": 4096, "k": 1, "act": "relu", "renorm": False, "group": 64, "x": "f32"}
MIXTRAL = {"d": 4096, "f": 14336, "k": 2, "act": "swiglu", "renorm": True, "group": 128, "x": "bf16"}


def listed():
    return [
        # the smallest call: one token through one small layer, where launches and latency are everything
        dict(SWITCH_BASE, name="switch_layer_token", kind="layer", experts=8, bits="2:1,4:1,8:1", bias="none",
             layout="columns", tokens=1),
        # single-stream decoding with a Switch-base-64 model: six MoE layers a step, mixed 2/4/8 bits, some experts hot
        dict(SWITCH_BASE, name="switch64_stack_token", kind="stack", experts=64, bits="2:3,4:5,8:2", bias="hot",
             layout="columns", tokens=1, layers=6, steps=8),
        # serving a Switch-large-128 model with eight sequences at a time
        dict(SWITCH_LARGE, name="switch128_stack_batch8", kind="stack", experts=128, bits="2:5,4:13,8:2", bias="none",
             layout="canonical", tokens=8, layers=12, steps=3),
        # single-stream decoding with a Mixtral-8x7B-shaped model (four of its layers), 2- and 4-bit experts
        dict(MIXTRAL, name="mixtral_stack_token", kind="stack", experts=8, bits="2:1,4:1", bias="none",
             layout="stream", tokens=1, layers=4, steps=4),
        # the same layer in a serving loop: a handful of sequences decoded together ...
        dict(MIXTRAL, name="mixtral_layer_batch8", kind="layer", experts=8, bits="2:1,4:1", bias="none",
             layout="stream", tokens=8),
        # ... and an odd two dozen
        dict(MIXTRAL, name="mixtral_layer_batch23", kind="layer", experts=8, bits="2:1,4:1", bias="none",
             layout="stream", tokens=23),
        # a short prompt (or a speculative / chunked prefill) on the layer the decode stack holds
        dict(MIXTRAL, name="mixtral_prompt_117", kind="layer", experts=8, bits="2:1,4:1", bias="normal",
             layout="stream", tokens=117),
        # the largest call: prefill of 2048 tokens, 4- and 8-bit experts unevenly loaded, weights as packed
        dict(MIXTRAL, name="mixtral_prefill_2048", kind="layer", experts=8, bits="4:1,8:1", bias="normal",
             layout="canonical", tokens=2048),
        # a prompt through a Switch-base-64 layer
        dict(SWITCH_BASE, name="switch64_prompt_500", kind="layer", experts=64, bits="2:3,4:5,8:2", bias="hot",
             layout="canonical", tokens=500),
        # one expert on the tokens a caller's own scheduler has collected for it
        dict(SWITCH_LARGE, name="switch_expert_5", kind="expert", experts=2, bits="4:1", bias="none",
             layout="canonical", tokens=5),
        # the offline side: an expert quantized, packed and laid out for the decode kernel
        dict(MIXTRAL, name="compress_mixtral_expert", kind="compress", experts=1, bits="4:1", bias="none",
             layout="stream", tokens=0),
        # ... and a compressed expert brought back to fp32
        dict(MIXTRAL, name="decompress_mixtral_expert", kind="decompress", experts=1, bits="2:1", bias="none",
             layout="canonical", tokens=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges: Switch-like layers of several widths and Mixtral-like ones, every layout and
    entry point, one token up to prompts."""
    big = rng.random() < 0.5
    kind = rng.choice(["stack", "layer", "layer", "layer", "layer", "routed", "expert", "compress", "decompress"])
    if big:
        c = dict(MIXTRAL, f=512 * rng.randint(4, 28), experts=rng.randint(4, 8), bits=rng.choice(["2:1,4:1", "4:1,8:1", "4:1", "2:1,4:1,8:1"]),
                 bias=rng.choice(["none", "normal"]), x=rng.choice(["bf16", "bf16", "f32"]),
                 layout=rng.choice(["stream", "stream", "canonical", "columns"]))
        most = 2048
    else:
        group = rng.choice([32, 32, 64, 128])
        d = 128 * rng.randint(4, 12)
        c = dict(SWITCH_BASE, d=d, f=512 * rng.randint(2, 8), k=rng.choice([1, 1, 2]), group=group,
                 experts=rng.choice([8, 16, 33, 64, 128]), bits=rng.choice(["2:3,4:5,8:2", "2:5,4:13,8:2", "4:1", "8:1"]),
                 bias=rng.choice(["none", "hot"]), x=rng.choice(["f32", "f32", "bf16"]),
                 layout=rng.choice(["canonical", "columns"]))
        most = 1000
    if kind == "stack":
        c.update(tokens=_log_int(rng, 1, 8), layers=2 if big else rng.randint(2, 4), steps=2)
    elif kind == "expert":
        c.update(tokens=_log_int(rng, 1, 24), experts=2, k=1)
    elif kind in ("compress", "decompress"):
        c.update(tokens=0, experts=1, bits=rng.choice(["2:1", "4:1", "8:1"]), k=1)
        if kind == "decompress":
            c.update(layout="canonical")
    else:
        c.update(tokens=_log_int(rng, 1, most))
    c["kind"] = kind
    return c


# ---- inputs ------------------------------------------------------------------------------------------------------

def _gen(seed, *parts):
    z = random.Random(repr((int(seed),) + parts)).getrandbits(62)
    g = torch.Generator(device=DEV)
    g.manual_seed(z)
    return g


def _randn(shape, std, seed, *parts):
    return torch.randn(shape, generator=_gen(seed, *parts), device=DEV, dtype=torch.float32) * std


def _bits_table(case, seed, layer):
    """Bitwidths in the proportions that case["bits"] states, shuffled over the experts."""
    parts = [tuple(int(v) for v in p.split(":")) for p in case["bits"].split(",")]
    total, E = sum(n for _, n in parts), case["experts"]
    table, upto = [], 0
    for b, n in parts:
        upto += n
        table += [b] * (round(E * upto / total) - len(table))
    random.Random(repr((int(seed), layer, "bits"))).shuffle(table)
    return table


def _weights(case, seed, layer, e):
    """fp32 weights of one expert, [out][in]: w_in, w_out and, for SwiGLU, w_gate."""
    d, f = case["d"], case["f"]
    w = {"w_in": _randn((f, d), 0.02, seed, layer, e, "in"), "w_out": _randn((d, f), 0.02, seed, layer, e, "out")}
    if case["act"] == "swiglu":
        w["w_gate"] = _randn((f, d), 0.02, seed, layer, e, "gate")
    return w


def _router(case, seed, layer):
    E = case["experts"]
    Wr = _randn((E, case["d"]), 0.02, seed, layer, "router")
    bias = None
    if case["bias"] == "normal":
        bias = _randn((E,), 0.5, seed, layer, "rbias")
    elif case["bias"] == "hot":                              # a fifth of the experts takes most of the tokens
        bias = torch.zeros(E, device=DEV)
        hot = random.Random(repr((int(seed), layer, "hot"))).sample(range(E), max(1, round(0.2 * E)))
        bias[hot] = 0.445
    return Wr, bias


def _hidden(case, seed, *parts):
    x = _randn((case["tokens"], case["d"]), 1.0, seed, "x", *parts)
    return x.to(torch.bfloat16) if case["x"] == "bf16" else x


def _given_routing(case, seed):
    T, k, E = case["tokens"], case["k"], case["experts"]
    idx = torch.stack([torch.randperm(E, generator=_gen(seed, "ridx", t), device=DEV)[:k] for t in range(T)])
    gate = torch.rand((T, k), generator=_gen(seed, "rgate"), device=DEV) * 0.9 + 0.1
    return idx.to(torch.int32).contiguous(), gate


def _pack(case, w, bits):
    g = case["group"]
    q_in, s_in = moeq.moe_quantize_pack(w["w_in"], bits, g)
    q_out, s_out = moeq.moe_quantize_pack(w["w_out"], bits, g)
    q_g = s_g = None
    if "w_gate" in w:
        q_g, s_g = moeq.moe_quantize_pack(w["w_gate"], bits, g)
    ex = moeq.PackedExpert(bits, q_in, s_in, q_out, s_out, q_g, s_g)
    if case["layout"] == "stream":
        return ex.with_stream_layout(case["d"], case["f"], g)
    return ex.with_out_columns(case["f"], g) if case["layout"] == "columns" else ex


def _layer(case, seed, layer):
    bits = _bits_table(case, seed, layer)
    experts = [_pack(case, _weights(case, seed, layer, e), bits[e]) for e in range(case["experts"])]
    Wr, bias = _router(case, seed, layer)
    return moeq.Layer(case["d"], case["f"], case["k"], case["group"],
                      moeq.MOEQ_ACT_SWIGLU if case["act"] == "swiglu" else moeq.MOEQ_ACT_RELU, case["renorm"],
                      moeq.MOEQ_BF16 if case["x"] == "bf16" else moeq.MOEQ_F32, Wr, bias, experts,
                      moeq.MOEQ_OUT_CANONICAL if case["layout"] == "canonical" else moeq.MOEQ_OUT_COLUMNS,
                      moeq.MOEQ_IN_STREAM if case["layout"] == "stream" else moeq.MOEQ_IN_CANONICAL)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "compress":
        s["w"] = _weights(case, seed, 0, 0)
        s["bits"] = _bits_table(case, seed, 0)[0]
        return s
    if kind == "decompress":
        s["bits"] = _bits_table(case, seed, 0)[0]
        s["ex"] = _pack(case, _weights(case, seed, 0, 0), s["bits"])
        return s
    T, d = case["tokens"], case["d"]
    if kind == "stack":
        L = case["layers"]
        s["layers"] = [_layer(case, seed, l) for l in range(L)]
        s["x"] = [torch.stack([_hidden(case, seed, st, l) for l in range(L)]) for st in range(case["steps"])]
        s["xs"] = torch.zeros_like(s["x"][0])
        s["y"] = torch.zeros((L, T, d), dtype=torch.float32, device=DEV)
        s["out"] = torch.empty((case["steps"], L, T, d), dtype=torch.float32, device=DEV)
        s["ws"] = torch.empty(max(l.workspace_bytes(T) for l in s["layers"]), dtype=torch.uint8, device=DEV)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for l in range(L):
                moeq.moe_layer_forward(s["layers"][l], s["xs"][l], y=s["y"][l], ws=s["ws"])
        return s
    s["layer"] = _layer(case, seed, 0)
    s["x"] = _hidden(case, seed)
    s["ws"] = torch.empty(s["layer"].workspace_bytes(T), dtype=torch.uint8, device=DEV)
    if kind == "routed":
        s["idx"], s["gate"] = _given_routing(case, seed)
    elif kind == "expert":
        s["gate"] = torch.rand((T,), generator=_gen(seed, "egate"), device=DEV) * 0.9 + 0.1
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "stack":
        for st in range(case["steps"]):
            s["xs"].copy_(s["x"][st])
            s["graph"].replay()
            s["out"][st].copy_(s["y"])
        return {"y": s["out"]}
    if kind == "layer":
        y, idx, gate = moeq.moe_layer_forward(s["layer"], s["x"], want_routing=True, ws=s["ws"])
        return {"y": y, "idx": idx, "gate": gate}
    if kind == "routed":
        return {"y": moeq.moe_layer_forward_routed(s["layer"], s["x"], s["idx"], s["gate"], ws=s["ws"])}
    if kind == "expert":
        return {"y": moeq.moe_expert_ffn_q(s["layer"], 1, s["x"], gate=s["gate"], ws=s["ws"])}
    if kind == "compress":
        ex = _pack(case, s["w"], s["bits"])
        named = {"q_in": ex.q_in, "s_in": ex.s_in, "q_gate": ex.q_gate, "s_gate": ex.s_gate, "q_out": ex.q_out,
                 "s_out": ex.s_out}
        return {n: t if t.dtype == torch.uint8 else t.view(torch.int16) for n, t in named.items() if t is not None}
    ex, g = s["ex"], case["group"]
    out = {"w_in": moeq.moe_dequantize(ex.q_in, ex.s_in, case["d"], s["bits"], g),
           "w_out": moeq.moe_dequantize(ex.q_out, ex.s_out, case["f"], s["bits"], g)}
    if ex.q_gate is not None:
        out["w_gate"] = moeq.moe_dequantize(ex.q_gate, ex.s_gate, case["d"], s["bits"], g)
    return out


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def _mean_bits(case):
    parts = [tuple(int(v) for v in p.split(":")) for p in case["bits"].split(",")]
    return sum(b * n for b, n in parts) / sum(n for _, n in parts)


def work(case):
    """Bytes: packed codes and scales of the experts that the tokens are expected to touch, router weights, hidden
    states in, results out. Operations: the multiply-adds of the chosen experts' matrices and of the router."""
    d, f, E, k, T = case["d"], case["f"], case["experts"], case["k"], case["tokens"]
    n_w = (3 if case["act"] == "swiglu" else 2) * d * f
    packed = n_w * (_mean_bits(case) / 8 + 2.0 / case["group"])
    if case["kind"] in ("compress", "decompress"):
        return {"bytes": n_w * 4 + packed, "flops": 0.0}
    xb = 2 if case["x"] == "bf16" else 4
    if case["kind"] == "expert":
        return {"bytes": packed + T * d * (xb + 4), "flops": 2.0 * n_w * T}
    if case["bias"] == "hot":                     # a fifth of the experts takes about six tokens in ten
        hot = max(1, round(0.2 * E))
        p = [0.6 / hot] * hot + [0.4 / max(1, E - hot)] * (E - hot)
    else:
        p = [1.0 / E] * E
    touched = sum(1.0 - (1.0 - min(1.0, k * q)) ** T for q in p)
    routed = case["kind"] == "routed"
    one = {"bytes": touched * packed + (0 if routed else E * d * 4) + T * d * (xb + 4),
           "flops": 2.0 * n_w * T * k + (0 if routed else 2.0 * E * d * T)}
    n = case["layers"] * case["steps"] if case["kind"] == "stack" else 1
    return {"bytes": one["bytes"] * n, "flops": one["flops"] * n}


def tolerance(case):
    """Activations enter the multipliers with 11 significant bits (more on some paths), twice: about 2.5e-4 off the
    64-bit result in the 2-norm, up to 4.5e-4 with 2-bit experts; four times that is stated. Packing and unpacking are
    exact."""
    if case["kind"] in ("compress", "decompress"):
        return "exact"
    return {"rel": 1.8e-3, "max": 1.5e-2, "differ": 0.002}


# ---- the same in 64 bits, plain torch --------------------------------------------------------------------------------

def _dequantized(w, bits, group):
    """The quantization rule (scale = fp16(absmax / qmax), one step up if the largest element would clamp; codes =
    round-half-even of w / scale) and its mirror: the fp64 weights that the packed matrix stands for."""
    rows, cols = w.shape
    qmax = 2 ** (bits - 1) - 1
    g = w.view(rows, cols // group, group)
    a = g.abs().amax(-1)
    s = (a / float(qmax)).to(torch.float16)
    s = torch.where(s.float() * qmax < a, (s.view(torch.int16) + 1).view(torch.float16), s)
    q = (g / s.float()[..., None]).round().clamp(-qmax, qmax)
    q = torch.where((a > 0)[..., None], q, torch.zeros_like(q))
    return (q.double() * s.double()[..., None]).view(rows, cols)


def _ffn64(case, seed, layer, e, bits, x):
    w = _weights(case, seed, layer, e)
    a = x @ _dequantized(w["w_in"], bits, case["group"]).t()
    if case["act"] == "swiglu":
        h = a * torch.sigmoid(a) * (x @ _dequantized(w["w_gate"], bits, case["group"]).t())
    else:
        h = torch.relu(a)
    return h @ _dequantized(w["w_out"], bits, case["group"]).t()


def _route64(case, seed, layer, x):
    Wr, bias = _router(case, seed, layer)
    logits = x @ Wr.double().t() + (0.0 if bias is None else bias.double())
    p = torch.softmax(logits, -1)
    gate, idx = torch.topk(p, case["k"], dim=-1)
    return idx, gate / gate.sum(-1, keepdim=True) if case["renorm"] else gate


def _layer64(case, seed, layer, x, idx, gate):
    bits = _bits_table(case, seed, layer)
    y = torch.zeros((x.shape[0], case["d"]), dtype=torch.float64, device=DEV)
    for e in sorted(set(idx.flatten().tolist())):
        tok, j = torch.nonzero(idx == e, as_tuple=True)
        y.index_add_(0, tok, gate[tok, j].double()[:, None] * _ffn64(case, seed, layer, e, bits[e], x[tok]))
    return y


def exact(case, seed):
    kind = case["kind"]
    if kind == "compress":
        return None
    if kind == "decompress":
        w, bits = _weights(case, seed, 0, 0), _bits_table(case, seed, 0)[0]
        return {n: _dequantized(m, bits, case["group"]) for n, m in w.items()}
    if kind == "stack":
        out = []
        for st in range(case["steps"]):
            ys = []
            for l in range(case["layers"]):
                x = _hidden(case, seed, st, l).double()
                ys.append(_layer64(case, seed, l, x, *_route64(case, seed, l, x)))
            out.append(torch.stack(ys))
        return {"y": torch.stack(out)}
    x = _hidden(case, seed).double()
    if kind == "expert":
        gate = torch.rand((case["tokens"],), generator=_gen(seed, "egate"), device=DEV) * 0.9 + 0.1
        return {"y": gate.double()[:, None] * _ffn64(case, seed, 0, 1, _bits_table(case, seed, 0)[1], x)}
    if kind == "routed":
        return {"y": _layer64(case, seed, 0, x, *_given_routing(case, seed))}
    idx, gate = _route64(case, seed, 0, x)
    return {"y": _layer64(case, seed, 0, x, idx, gate), "idx": idx.to(torch.int32), "gate": gate}
