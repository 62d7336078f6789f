"""GPU parity of prompts: the GEMMs on items of 32 and of 128 pairs at their edges and where the one takes over from the other, and
the kernels that route and group the tokens of such calls, through the C ABI against the oracle."""
import gen
import numpy as np
import oracle
import paper_2308_14352_amd as moeq
import pytest
import torch
from helpers import build_layer_pair, pack_expert_gpu, rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
# Activations enter the multipliers rounded to 11 bits, twice: 2.4e-4 each of the output's scale where the signs are random,
# worst single elements of hundreds of tokens three to four times their root sum.
TOL = 2e-3


@pytest.mark.parametrize("base,d,f,layout", [
    ("c5", 512, 512, "canonical"),      # one chunk, one range of W_out
    ("c5", 1024, 1536, "columns"),      # an odd number of chunks
    ("c1", 512, 1536, "canonical"),     # ReLU: four rows of a matrix where SwiGLU has two of both
    ("c1", 512, 2048, "columns"),       # ranges of W_out
    ("c5", 4096, 1024, "stream"),
    ("c1", 4096, 512, "stream"),
])
@pytest.mark.parametrize("bits", (2, 4, 8))
def test_items_at_their_edges(base, d, f, layout, bits):
    """0, 1, 15..17, 31..33, 63..65 and 129 pairs per expert, and an index outside [0, E)."""
    counts = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 129]
    E = len(counts)
    cfg = gen.tiny_config(base, d, f, n_experts=E, n_layers=1, group=128)
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [bits] * E, columns=layout == "columns", stream=layout == "stream")
    pairs = np.concatenate([np.full(c, e, dtype=np.int32) for e, c in enumerate(counts)])
    rng = np.random.default_rng(7 + bits)
    rng.shuffle(pairs)
    k = cfg.top_k
    pairs = np.concatenate([pairs, np.full(k - len(pairs) % k, E, dtype=np.int32)])
    idx = pairs.reshape(-1, k)
    T = idx.shape[0]
    x = gen.hidden(cfg, 0, 0, T, DEV)
    gate = rng.uniform(0.1, 1.0, size=(T, k)).astype(np.float32)
    args = layer, x, torch.from_numpy(idx).to(DEV), torch.from_numpy(gate).to(DEV)
    y = moeq.moe_layer_forward_routed(*args)
    again = moeq.moe_layer_forward_routed(*args)
    torch.cuda.synchronize()
    assert torch.equal(y, again)
    y_ref = oracle.layer_forward_routed(orc_experts, d, f, 128, int(cfg.swiglu), k, x.float().cpu().numpy(), idx, gate)
    live = np.abs(y_ref).max(axis=1) > 0
    assert rel_err(y.cpu().numpy()[live], y_ref[live]).max() < TOL
    assert not y.cpu().numpy()[~live].any()


@pytest.mark.parametrize("base,E,T", [
    ("c5", 97, 64),        # two kernels: many experts, 32-pair items
    ("c5", 24, 2048),      # 4096 pairs on 24 experts, the most that one workgroup plans, in items of 128
    ("c5", 24, 2049),      # ... and two pairs more
    ("c5", 64, 768),       # its most experts, with as many pairs as it takes for them, in items of 32
    ("c5", 64, 769),       # ... and two pairs more
    ("c5", 65, 40),        # ... and one expert more
    ("c5", 3, 2049),       # many pairs on few experts
    ("c1", 70, 5100),      # more experts, one choice a token
])
def test_planning_of_many_pairs_and_experts(base, E, T):
    """Pairs grouped by one workgroup or by two kernels, for either size of item."""
    d = f = 512
    cfg = gen.tiny_config(base, d, f, n_experts=E, n_layers=1, group=128)
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [(2, 4, 8)[e % 3] for e in range(E)])
    rng = np.random.default_rng(E + T)
    k = cfg.top_k
    idx = rng.integers(0, E, size=(T, k)).astype(np.int32)
    idx[: T // 3, 0] = 1                                     # an expert with a third of the tokens
    idx[5, 0], idx[T - 1, k - 1] = -1, E                     # outside [0, E): weighted 0
    gate = rng.uniform(0.1, 1.0, size=(T, k)).astype(np.float32)
    x = gen.hidden(cfg, 0, 0, T, DEV)
    y = moeq.moe_layer_forward_routed(layer, x, torch.from_numpy(idx).to(DEV), torch.from_numpy(gate).to(DEV))
    torch.cuda.synchronize()
    some = np.unique(np.concatenate([[5, T - 1], rng.integers(0, T, size=300)]))
    y_ref = oracle.layer_forward_routed(orc_experts, d, f, 128, int(cfg.swiglu), k, x[some].float().cpu().numpy(), idx[some], gate[some])
    y = y.cpu().numpy()
    assert np.isfinite(y).all()
    live = np.abs(y_ref).max(axis=1) > 0
    assert rel_err(y[some][live], y_ref[live]).max() < TOL
    assert not y[some][~live].any()


@pytest.mark.parametrize("base,d,f,layout", [
    ("c5", 512, 1024, "canonical"),
    ("c5", 1024, 512, "columns"),
    ("c1", 512, 512, "canonical"),
    ("c1", 512, 1024, "columns"),
    ("c5", 4096, 512, "stream"),
    ("c1", 4096, 512, "stream"),
])
@pytest.mark.parametrize("bits", (2, 4, 8))
def test_items_of_128_pairs_at_their_edges(base, d, f, layout, bits):
    """0, 1, 63..65, 127..129 and 255..257 pairs per expert, well over 72 on average, so that every shape has items of 128; an
    index outside [0, E); tokens between 2^-12 and 2^12 times each other."""
    counts = [0, 1, 63, 64, 65, 127, 128, 129, 255, 256, 257]
    E = len(counts)
    assert sum(counts) > 100 * E
    cfg = gen.tiny_config(base, d, f, n_experts=E, n_layers=1, group=128)
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [bits] * E, columns=layout == "columns", stream=layout == "stream")
    pairs = np.concatenate([np.full(c, e, dtype=np.int32) for e, c in enumerate(counts)])
    rng = np.random.default_rng(17 + bits)
    rng.shuffle(pairs)
    k = cfg.top_k
    pairs = np.concatenate([pairs, np.full(k - len(pairs) % k, E, dtype=np.int32)])
    idx = pairs.reshape(-1, k)
    T = idx.shape[0]
    x = gen.hidden(cfg, 0, 0, T, DEV)
    x = x * torch.from_numpy(2.0 ** rng.integers(-12, 13, (T, 1))).to(DEV).to(x.dtype)
    gate = rng.uniform(0.1, 1.0, size=(T, k)).astype(np.float32)
    y = moeq.moe_layer_forward_routed(layer, x, torch.from_numpy(idx).to(DEV), torch.from_numpy(gate).to(DEV))
    torch.cuda.synchronize()
    some = np.unique(np.concatenate([[T - 1], rng.integers(0, T, size=400)]))
    y_ref = oracle.layer_forward_routed(orc_experts, d, f, 128, int(cfg.swiglu), k, x[some].float().cpu().numpy(), idx[some], gate[some])
    live = np.abs(y_ref).max(axis=1) > 0
    y = y.cpu().numpy()
    assert rel_err(y[some][live], y_ref[live]).max() < TOL
    assert not y[some][~live].any()


def test_one_chunk_of_8_bit_codes():
    """The shortest GEMMs (one chunk of columns, one range of W_out) on 8-bit rows, 0 to 65 pairs per expert."""
    d = f = 512
    counts = [0, 1, 15, 16, 17, 31, 65, 0]
    cfg = gen.tiny_config("c5", d, f, n_experts=len(counts), n_layers=1, group=128)
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [8] * len(counts))
    pairs = np.concatenate([np.full(c, e, dtype=np.int32) for e, c in enumerate(counts)] + [[6]]).astype(np.int32)
    np.random.default_rng(5).shuffle(pairs)
    idx = pairs.reshape(-1, cfg.top_k)
    gate = np.random.default_rng(6).uniform(0.1, 1.0, size=idx.shape).astype(np.float32)
    x = gen.hidden(cfg, 0, 0, idx.shape[0], DEV)
    y = moeq.moe_layer_forward_routed(layer, x, torch.from_numpy(idx).to(DEV), torch.from_numpy(gate).to(DEV))
    torch.cuda.synchronize()
    y_ref = oracle.layer_forward_routed(orc_experts, d, f, 128, int(cfg.swiglu), cfg.top_k, x.float().cpu().numpy(), idx, gate)
    assert rel_err(y.cpu().numpy(), y_ref).max() < TOL


def test_items_of_128_pairs_where_they_are_faster():
    """64 ReLU experts of 1024 x 2048 with 60 pairs each: us with items of 32 / of 128 pairs 158 / 131; with 5 pairs each 74 / 90.
    Every call of more than 72 has items of 128, and the forms differ in the order of their sums (W_out is cut for items of 32)."""
    d, f, E = 1024, 2048, 64
    cfg = gen.tiny_config("c1", d, f, n_experts=E, n_layers=1, group=128)
    layer, _, _, _ = build_layer_pair(cfg, 0, DEV, [4] * E, want_oracle=False)
    n = 74 * E
    x = gen.hidden(cfg, 0, 0, n, DEV)
    idx = torch.randint(0, E, (n, 1), generator=torch.Generator().manual_seed(1), dtype=torch.int32).to(DEV)
    gate = torch.ones((n, 1), device=DEV)
    most, many, few = (moeq.moe_layer_forward_routed(layer, x[:T], idx[:T], gate[:T]) for T in (n, 60 * E, 5 * E))
    torch.cuda.synchronize()
    assert torch.equal(many, most[:60 * E])
    assert not torch.equal(few, most[:5 * E]) and rel_err(few.cpu().numpy(), most[:5 * E].cpu().numpy()).max() < 1e-5


@pytest.mark.parametrize("f", (4096, 8192))
@pytest.mark.parametrize("T", (40, 230))
def test_wide_h(f, T):
    """Activations of h that 512 and 1024 threads stage, for items of 32 and of 128 pairs (230 tokens on three experts)."""
    cfg = gen.tiny_config("c1", 512, f, n_experts=3, n_layers=1, group=128)
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [2, 4, 8])
    x = gen.hidden(cfg, 0, 0, T, DEV)
    idx = (np.arange(T, dtype=np.int32) % 3)[:, None]
    gate = np.linspace(0.3, 1.0, T, dtype=np.float32)[:, None]
    y = moeq.moe_layer_forward_routed(layer, x, torch.from_numpy(idx.copy()).to(DEV), torch.from_numpy(gate).to(DEV))
    torch.cuda.synchronize()
    y_ref = oracle.layer_forward_routed(orc_experts, 512, f, 128, 0, 1, x.float().cpu().numpy(), idx, gate)
    assert rel_err(y.cpu().numpy(), y_ref).max() < TOL


@pytest.mark.parametrize("d,f,E,k,x_dtype,T", [
    (768, 1024, 64, 1, "f32", 300),     # a block of eight experts per wavefront, two tokens a workgroup
    (800, 1024, 9, 3, "bf16", 37),      # two blocks, ranges of columns that do not divide
    (512, 512, 3, 2, "f32", 1030),      # fewer experts than a block; four tokens a workgroup, the last one half empty
    (1024, 512, 130, 2, "f32", 64),     # more experts than lanes
])
def test_routing_of_many_tokens(d, f, E, k, x_dtype, T):
    g = torch.Generator().manual_seed(3)
    Wr, bias = torch.randn((E, d), generator=g).mul_(0.02).to(DEV), torch.randn((E,), generator=g).mul_(0.1).to(DEV)
    x = torch.randn((T, d), generator=g).to(DEV).to(torch.bfloat16 if x_dtype == "bf16" else torch.float32)
    w = {"w_in": torch.randn((f, d), generator=g).to(DEV) * 0.02, "w_out": torch.randn((d, f), generator=g).to(DEV) * 0.02}
    expert = pack_expert_gpu(w, 4, 32).with_out_columns(f, 32)
    layer = moeq.Layer(d, f, k, 32, moeq.MOEQ_ACT_RELU, True, moeq.MOEQ_BF16 if x_dtype == "bf16" else moeq.MOEQ_F32, Wr, bias,
                       [expert] * E, moeq.MOEQ_OUT_COLUMNS, moeq.MOEQ_IN_CANONICAL)
    _, idx, gate = moeq.moe_layer_forward(layer, x, want_routing=True)
    torch.cuda.synchronize()
    idx_ref, gate_ref, _, logits = oracle.router_topk(x.float().cpu().numpy(), Wr.cpu().numpy(), bias.cpu().numpy(), k, True,
                                                      want_logits=True)
    srt = -np.sort(-logits, axis=1)
    keep = (srt[:, :k] - srt[:, 1:k + 1])[:, :E - 1].min(axis=1) >= 1e-5
    assert keep.sum() >= T - 3
    assert np.array_equal(idx.cpu().numpy()[keep], idx_ref[keep])
    assert np.allclose(gate.cpu().numpy()[keep], gate_ref[keep], rtol=2e-5, atol=1e-7)


@pytest.mark.parametrize("d,f,E,k,group,act,x_dtype,T", [
    (512, 512, 3, 2, 128, "relu", "f32", 1030),        # units of four experts, four tokens a workgroup
    (4096, 512, 8, 2, 128, "swiglu", "bf16", 33),
    (1056, 512, 16, 2, 32, "relu", "f32", 300),        # columns that end inside a class
    (768, 1024, 64, 1, 32, "relu", "f32", 257),        # all classes in a unit, the last one empty
    (1024, 512, 130, 2, 128, "relu", "bf16", 64),
    (2048, 512, 600, 8, 128, "swiglu", "f32", 1100),
    (4096, 256, 66, 2, 128, "swiglu", "bf16", 100),    # a grouped decode call
])
def test_layer_calls_route_like_the_router_entry(d, f, E, k, group, act, x_dtype, T):
    """A caller that asks the router first (to fetch experts) and then runs the layer meets the same experts and gates, bit for
    bit, whichever kernels route (decode calls of few experts apart, which route inside their own kernels); and a token's do not
    depend on how many tokens its call has."""
    g = torch.Generator().manual_seed(11)
    Wr, bias = torch.randn((E, d), generator=g).mul_(0.02).to(DEV), torch.randn((E,), generator=g).mul_(0.1).to(DEV)
    x = torch.randn((T, d), generator=g).to(DEV).to(torch.bfloat16 if x_dtype == "bf16" else torch.float32)
    w = {"w_in": torch.randn((f, d), generator=g).to(DEV) * 0.02, "w_out": torch.randn((d, f), generator=g).to(DEV) * 0.02}
    if act == "swiglu":
        w["w_gate"] = w["w_in"].flip(0).contiguous()
    expert = pack_expert_gpu(w, 4, group)
    layer = moeq.Layer(d, f, k, group, moeq.MOEQ_ACT_SWIGLU if act == "swiglu" else moeq.MOEQ_ACT_RELU, True,
                       moeq.MOEQ_BF16 if x_dtype == "bf16" else moeq.MOEQ_F32, Wr, bias, [expert] * E)
    _, idx, gate = moeq.moe_layer_forward(layer, x, want_routing=True)
    idx_r, gate_r, probs = moeq.moe_router_topk(layer, x, want_probs=True)
    few = [moeq.moe_router_topk(layer, x[:n]) for n in (1, 9, 40)]
    if E > 16:
        few += [moeq.moe_layer_forward(layer, x[:n], want_routing=True)[1:] for n in (1, 3)]
    torch.cuda.synchronize()
    assert torch.equal(idx, idx_r) and torch.equal(gate, gate_r)
    assert all(torch.equal(i, idx[:i.shape[0]]) and torch.equal(v, gate[:i.shape[0]]) for i, v in few)
    _, _, probs_ref, _ = oracle.router_topk(x[:20].float().cpu().numpy(), Wr.cpu().numpy(), bias.cpu().numpy(), k, True, want_logits=True)
    assert np.allclose(probs[:20].cpu().numpy(), probs_ref, rtol=1e-4, atol=1e-7)
