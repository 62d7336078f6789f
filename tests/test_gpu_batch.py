"""GPU parity of decode calls of a few tokens on 4096-column layers (pairs grouped by expert, weights streamed once for up
to 16 pairs, 8 in rows and columns), in every layout: the edges of its items, units and chunks, inputs at the ends of their
range and with outliers, and which calls are grouped."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2308_14352_amd as moeq
from paper_2308_14352_amd import binding
from helpers import build_layer_pair, near_tie_tokens, oracle_layer, pack_expert_gpu, pack_expert_oracle, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# On layers in the stream layout x and h enter with 15 bits below the largest of 128 (h: 64) values: an element is off by at
# most 2^-16 of that (about 3.5 standard deviations), 6e-5 / sqrt(3) of a standard deviation, once for x and once for h; the
# largest of 4096 outputs' errors (4 standard deviations) against the largest output (again about 4) stays near that figure. The
# gate product and fp32 sums add less. 4e-4 leaves a factor of five. (On other layers they enter with 30 bits below it.)
TOL = 4e-4


@pytest.mark.parametrize("base,x_dtype,f,k,bits_table,tokens", [
    ("c4", "bf16", 128, 2, [2, 4, 8], (200,)),              # one unit, one chunk; two launches
    ("c4", "f32", 1152, 2, [8, 2, 4, 4], (33, 50, 131)),    # nine scale groups: a last chunk of one
    ("c4", "bf16", 1536, 2, [4, 2], (16, 17, 31)),          # every token on both experts: one and two items of each
    ("c1", "f32", 640, 1, [2, 8, 4], (60, 129)),            # ReLU, top-1
    ("c4", "f32", 384, 5, [2, 2, 4, 8, 8, 4], (60,)),       # five choices: launches of 51 tokens
    ("c1", "bf16", 256, 2, [2 + 2 * (i % 2) for i in range(66)], (100,)),    # more experts than are routed in the kernel
], ids=("one-unit", "nine-groups", "two-items", "relu", "top5", "66-experts"))
@pytest.mark.parametrize("layout", ("stream", "canonical", "columns"))
def test_grouped_decode_calls(base, x_dtype, f, k, bits_table, tokens, layout):
    cfg = replace(gen.tiny_config(base, 4096, f, n_experts=len(bits_table), n_layers=1, group=128), top_k=k, x_dtype=x_dtype)
    layer, orc_experts, Wr, bias = build_layer_pair(cfg, 0, DEV, bits_table, columns=layout == "columns", stream=layout == "stream")
    x = gen.hidden(cfg, 0, 0, max(tokens), DEV)
    y_ref, idx_ref, gate_ref = oracle_layer(cfg, orc_experts, Wr, bias, x)
    skip = set(near_tie_tokens(cfg, Wr, bias, x).tolist())
    first = None
    for T in tokens:
        assert layer.path(T) in {"stream": (moeq.MOEQ_PATH_STREAM,), "canonical": (moeq.MOEQ_PATH_TWO_KERNELS,),
                                 "columns": (moeq.MOEQ_PATH_ONE_KERNEL, moeq.MOEQ_PATH_ONE_KERNEL_MX)}[layout]
        y, idx, gate = moeq.moe_layer_forward(layer, x[:T], want_routing=True)
        y_r = moeq.moe_layer_forward_routed(layer, x[:T], idx, gate)
        torch.cuda.synchronize()
        keep = [t for t in range(T) if t not in skip]
        assert len(keep) >= T - 2
        assert np.array_equal(idx.cpu().numpy()[keep], idx_ref[keep])
        assert np.allclose(gate.cpu().numpy()[keep], gate_ref[keep], rtol=2e-5, atol=1e-7)
        assert rel_err(y.cpu().numpy()[keep], y_ref[keep]).max() < TOL
        assert torch.equal(y, y_r)
        # (the call was grouped: the kernels of a single token round differently)
        assert not torch.equal(y[:1], moeq.moe_layer_forward(layer, x[:1]))
        # a token's result does not depend on the tokens that share its call
        first = y if first is None else first
        n = min(T, first.shape[0])
        assert torch.equal(y[:n], first[:n])
    if layout != "stream" or len(bits_table) > 64:
        return
    # the single-token kernel routes the same way, bit for bit
    _, idx1, gate1 = moeq.moe_layer_forward(layer, x[:1], want_routing=True)
    torch.cuda.synchronize()
    assert torch.equal(idx1, idx[:1]) and torch.equal(gate1, gate[:1])


@pytest.mark.parametrize("bits", (2, 4, 8))
@pytest.mark.parametrize("f,T", [(2304, 20), (1152, 33), (384, 260)])
@pytest.mark.parametrize("layout", ("stream", "canonical", "columns"))
def test_grouped_single_expert_call(bits, f, T, layout):
    cfg = replace(gen.tiny_config("c4", 4096, f, n_experts=2, n_layers=1, group=128), x_dtype="f32")
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [bits, bits], columns=layout == "columns",
                                               stream=layout == "stream")
    x = gen.hidden(cfg, 0, 0, T, DEV)
    gate = torch.linspace(0.2, 1.1, T, device=DEV)
    y0 = gen.normal((T, cfg.d_model), 0.1, 7, DEV)
    y = moeq.moe_expert_ffn_q(layer, 1, x, gate=gate)
    y_acc = moeq.moe_expert_ffn_q(layer, 1, x, gate=gate, y=y0.clone(), accumulate=True)
    torch.cuda.synchronize()
    ref = gate.cpu().numpy()[:, None] * oracle.expert_ffn(orc_experts[1], cfg.d_model, cfg.d_ff, cfg.group, 1, x.cpu().numpy())
    assert rel_err(y.cpu().numpy(), ref).max() < TOL
    assert rel_err((y_acc - y0).cpu().numpy(), ref).max() < TOL + 1e-5


@pytest.mark.parametrize("bits", (2, 4, 8))
@pytest.mark.parametrize("layout,f", [("stream", 5504), ("canonical", 2432), ("columns", 2432)])
def test_output_blocks_taken_in_turn(bits, layout, f):
    """Enough items and chunks that a workgroup of the output kernel takes two blocks of rows (4 and 8 bits; 2 bits: one); a last
    chunk of three groups."""
    cfg = replace(gen.tiny_config("c4", 4096, f, n_experts=2, n_layers=1, group=128), x_dtype="f32")
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [bits, bits], columns=layout == "columns", stream=layout == "stream")
    x = gen.hidden(cfg, 0, 0, 256, DEV)
    gate = torch.linspace(0.2, 1.1, 256, device=DEV)
    y = moeq.moe_expert_ffn_q(layer, 1, x, gate=gate)
    few = moeq.moe_expert_ffn_q(layer, 1, x[:20], gate=gate[:20])
    torch.cuda.synchronize()
    assert torch.equal(y[:20], few)
    y_ref = oracle.expert_ffn(orc_experts[1], 4096, f, cfg.group, int(cfg.swiglu), x[:20].cpu().numpy())
    assert rel_err(few.cpu().numpy(), gate[:20].cpu().numpy()[:, None] * y_ref).max() < TOL


@pytest.mark.parametrize("layout,f", [("stream", 5504), ("columns", 2432)])
def test_output_blocks_taken_in_turn_by_experts_of_every_bitwidth(layout, f):
    """A layer call of 2-, 4- and 8-bit experts, whose output kernel's workgroups take two blocks of rows; a last chunk of three
    groups."""
    cfg = replace(gen.tiny_config("c4", 4096, f, n_experts=3, n_layers=1, group=128), x_dtype="f32")
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [2, 4, 8], columns=layout == "columns", stream=layout == "stream")
    T = 31
    x = gen.hidden(cfg, 0, 0, T, DEV)
    idx = np.stack([np.arange(T) % 3, (np.arange(T) + 1) % 3], 1).astype(np.int32)
    gate = np.linspace(0.2, 1.1, 2 * T, dtype=np.float32).reshape(T, 2)
    args = torch.from_numpy(idx).to(DEV), torch.from_numpy(gate).to(DEV)
    y = moeq.moe_layer_forward_routed(layer, x, *args)
    one = moeq.moe_layer_forward_routed(layer, x[:1], args[0][:1], args[1][:1])
    torch.cuda.synchronize()
    assert not torch.equal(y[:1], one)          # (the call was grouped)
    y_ref = oracle.layer_forward_routed(orc_experts, 4096, f, cfg.group, int(cfg.swiglu), 2, x.cpu().numpy(), idx, gate)
    assert rel_err(y.cpu().numpy(), y_ref).max() < TOL


def test_grouped_call_with_the_ungrouped_workspace():
    """A workspace that only the ungrouped form of a call fits is still taken (a narrow layer with many choices)."""
    cfg = replace(gen.tiny_config("c4", 4096, 128, n_experts=8, n_layers=1, group=128), top_k=8, x_dtype="f32")
    layer, orc_experts, Wr, bias = build_layer_pair(cfg, 0, DEV, [4] * 8, stream=True)
    T = 4
    x = gen.hidden(cfg, 0, 0, T, DEV)
    need = layer.workspace_bytes(T)
    slices = cfg.d_ff // 64
    y = moeq.moe_layer_forward(layer, x, ws=torch.empty(need, dtype=torch.uint8, device=DEV))
    # the ungrouped form: routing, logits and T * slices partial vectors
    part = T * slices * cfg.d_model * 4
    up = lambda v: (v + 255) // 256 * 256
    small = 2 * up(T * 8 * 4) + up(T * 8 * 4) + up(part)
    assert small < need
    y2 = moeq.moe_layer_forward(layer, x, ws=torch.empty(small, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    y_ref, _, _ = oracle_layer(cfg, orc_experts, Wr, bias, x)
    assert rel_err(y.cpu().numpy(), y_ref).max() < TOL and rel_err(y2.cpu().numpy(), y_ref).max() < 2e-3
    with pytest.raises(moeq.MoeqError):
        moeq.moe_layer_forward(layer, x, ws=torch.empty(small - 1, dtype=torch.uint8, device=DEV))


@pytest.mark.parametrize("layout", ("stream", "canonical", "columns"))
def test_grouped_call_at_the_ends_of_the_hidden_states_range(layout):
    """Largest magnitudes next to 2^124 and 2^-96, the range that the entry points state (ReLU: the exact result is then of
    the size of the input)."""
    cfg = replace(gen.tiny_config("c1", 4096, 640, n_experts=3, n_layers=1, group=128), top_k=1, x_dtype="f32")
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [2, 4, 8], columns=layout == "columns", stream=layout == "stream")
    T = 66
    x = gen.hidden(cfg, 0, 0, T, DEV)
    x = x / x.abs().amax(1, keepdim=True)
    idx = (torch.arange(T, device=DEV, dtype=torch.int32) % 3)[:, None].contiguous()
    gate = torch.full((T, 1), 0.125, device=DEV)
    y_ref = oracle.layer_forward_routed(orc_experts, 4096, 640, 128, 0, 1, x.cpu().numpy(), idx.cpu().numpy(), gate.cpu().numpy())
    for e in (123, -95):
        y = moeq.moe_layer_forward_routed(layer, x * 2.0 ** e, idx, gate)
        torch.cuda.synchronize()
        assert rel_err(y.cpu().numpy().astype(np.float64) * 2.0 ** -e, y_ref).max() < TOL


@pytest.mark.parametrize("bits", (2, 4, 8))
@pytest.mark.parametrize("layout", ("canonical", "columns"))
def test_grouped_call_with_outlier_columns_that_meet_zero_weights(bits, layout):
    """An element 2^10 times the others in every scale group, on weights of zero: the results are those of the other
    elements, which keep at least the 11 bits that the single-token kernels give every element. (Layers in the stream layout
    hold 14 bits below the largest of a scale group on every path.)"""
    d, f, g, T = 4096, 1152, 128, 40
    cfg = replace(gen.tiny_config("c4", d, f, n_experts=1, n_layers=1, group=g), top_k=1, x_dtype="f32")
    w = gen.expert_weights(cfg, 0, 0, DEV)
    w["w_in"][:, 5::g] = 0.0
    w["w_gate"][:, 5::g] = 0.0
    ex = pack_expert_gpu(w, bits, g)
    Wr, bias = gen.router_weights(cfg, 0, DEV)
    columns = layout == "columns"
    layer = moeq.Layer(d, f, 1, g, moeq.MOEQ_ACT_SWIGLU, True, moeq.MOEQ_F32, Wr, bias, [ex.with_out_columns(f, g) if columns else ex],
                       moeq.MOEQ_OUT_COLUMNS if columns else moeq.MOEQ_OUT_CANONICAL)
    x = gen.hidden(cfg, 0, 0, T, DEV)
    x[:, 5::g] *= 1024.0
    y = moeq.moe_expert_ffn_q(layer, 0, x)
    torch.cuda.synchronize()
    ref = oracle.expert_ffn(pack_expert_oracle(w, bits, g), d, f, g, 1, x.cpu().numpy())
    assert rel_err(y.cpu().numpy(), ref).max() < TOL


@pytest.mark.parametrize("bits", (2, 4, 8))
@pytest.mark.parametrize("layout", ("stream", "canonical", "columns"))
def test_grouped_call_whose_larger_half_of_h_meets_zero_weights(bits, layout):
    """64 of the 128 columns of h that share a scale are 2^10 times the others and meet weights of zero: the results are
    those of the others."""
    d, f, g, T = 4096, 1152, 128, 60
    cfg = replace(gen.tiny_config("c4", d, f, n_experts=1, n_layers=1, group=g), top_k=1, x_dtype="f32")
    w = gen.expert_weights(cfg, 0, 0, DEV)
    big = torch.arange(f, device=DEV) % 128 < 64
    w["w_gate"][big] *= 1024.0
    w["w_out"][:, big] = 0.0
    ex = pack_expert_gpu(w, bits, g)
    if layout != "canonical":
        ex = ex.with_stream_layout(d, f, g) if layout == "stream" else ex.with_out_columns(f, g)
    Wr, bias = gen.router_weights(cfg, 0, DEV)
    layer = moeq.Layer(d, f, 1, g, moeq.MOEQ_ACT_SWIGLU, True, moeq.MOEQ_F32, Wr, bias, [ex],
                       moeq.MOEQ_OUT_CANONICAL if layout == "canonical" else moeq.MOEQ_OUT_COLUMNS,
                       moeq.MOEQ_IN_STREAM if layout == "stream" else moeq.MOEQ_IN_CANONICAL)
    x = gen.hidden(cfg, 0, 0, T, DEV)
    y = moeq.moe_expert_ffn_q(layer, 0, x)
    torch.cuda.synchronize()
    ref = oracle.expert_ffn(pack_expert_oracle(w, bits, g), d, f, g, 1, x.cpu().numpy())
    assert rel_err(y.cpu().numpy(), ref).max() < TOL


@pytest.mark.parametrize("layout,f,bits,alone,grouped", [
    ("canonical", 4096, 8, (4, 6, 8), (24, 31)),          # us, token by token / grouped: 48 / 77 for 8 tokens, 190 / 69 for 24
    ("canonical", 1024, 8, (8, 16, 24), (100,)),          # 49 / 66 for 24, 152 / 78 for 100
    ("canonical", 1024, 4, (16, 24), (100,)),             # 26 / 46 for 16, 111 / 60 for 100
    ("columns", 1024, 8, (2, 8), (16, 31)),               # 39 / 59 for 8, 73 / 61 for 16
])
def test_one_experts_calls_take_the_faster_form(layout, f, bits, alone, grouped):
    """The forms differ by their error: token by token the activations have 11 bits, grouped (rows, columns) 30."""
    cfg = replace(gen.tiny_config("c4", 4096, f, n_experts=1, n_layers=1, group=128), top_k=1, x_dtype="f32")
    layer, orc_experts, _, _ = build_layer_pair(cfg, 0, DEV, [bits], columns=layout == "columns")
    x = gen.hidden(cfg, 0, 0, max(grouped), DEV)
    ref = oracle.expert_ffn(orc_experts[0], 4096, f, 128, 1, x.cpu().numpy())
    for T in alone + grouped:
        y = moeq.moe_expert_ffn_q(layer, 0, x[:T])
        torch.cuda.synchronize()
        err = rel_err(y.cpu().numpy(), ref[:T]).max()
        assert err < 2e-5 if T in grouped else 5e-5 < err < 2e-3, (T, err)


@pytest.mark.parametrize("base,d,f,group,T", [("c4", 4096, 8192, 128, 12), ("c1", 768, 3072, 32, 500)])
def test_profile_events_of_grouped_calls_bracket_their_phase(base, d, f, group, T):
    """On rows FFN_IN and FFN_OUT time the two phases, not the whole call twice."""
    cfg = gen.tiny_config(base, d, f, n_experts=8, n_layers=1, group=group)
    layer, _, _, _ = build_layer_pair(cfg, 0, DEV, [4] * 8, want_oracle=False)
    x = gen.hidden(cfg, 0, 0, T, DEV)
    ws = torch.empty(layer.workspace_bytes(T), dtype=torch.uint8, device=DEV)
    y = torch.empty((T, d), device=DEV)

    def median_us(which):
        times = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(), b.record()
            if which:
                binding.moe_layer_profile_kernel(layer, which, a.cuda_event, b.cuda_event)
            else:
                a.record()
            moeq.moe_layer_forward(layer, x, y=y, ws=ws)
            if not which:
                b.record()
            binding.moe_layer_profile_kernel(layer, 0)
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        return sorted(times)[7]

    median_us(0)
    whole, t_in, t_out = median_us(0), median_us(binding.MOEQ_KERNEL_FFN_IN), median_us(binding.MOEQ_KERNEL_FFN_OUT)
    assert t_in > 5 and t_out > 5 and t_in + t_out < 1.4 * whole, (whole, t_in, t_out)
