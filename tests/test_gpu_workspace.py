"""What a call computes does not depend on how large a workspace it is given beyond its need, nor on what else its layer
holds: grouped and ungrouped kernels round differently, so the choice shows in the bits."""
from dataclasses import replace

import pytest
import torch

import gen
import paper_2308_14352_amd as moeq
from paper_2308_14352_amd import binding
from helpers import build_layer_pair, pack_expert_gpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("layout", ("stream", "canonical", "columns"))
def test_workspace_made_for_more_tokens_gives_the_same_bits(layout):
    cfg = replace(gen.tiny_config("c4", 4096, 2048, n_experts=8, n_layers=1, group=128), x_dtype="f32")
    layer, _, _, _ = build_layer_pair(cfg, 0, DEV, [2, 4] * 4, want_oracle=False, columns=layout == "columns", stream=layout == "stream")
    x = gen.hidden(cfg, 0, 0, 34, DEV)
    sizes = (2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 16, 17, 23, 31, 32, 33, 34)
    assert all(layer.workspace_bytes(a) <= layer.workspace_bytes(a + 1) for a in range(1, 300))
    for T in sizes:
        fresh = lambda n: torch.empty(layer.workspace_bytes(n), dtype=torch.uint8, device=DEV)
        want = moeq.moe_layer_forward(layer, x[:T], ws=fresh(T))
        want_e = moeq.moe_expert_ffn_q(layer, 3, x[:T], ws=fresh(T))
        for N in [n for n in sizes if n > T]:
            assert torch.equal(moeq.moe_layer_forward(layer, x[:T], ws=fresh(N)), want), (T, N)
            assert torch.equal(moeq.moe_expert_ffn_q(layer, 3, x[:T], ws=fresh(N)), want_e), (T, N)


@pytest.mark.parametrize("base,d,f,E,group,T", [
    ("c4", 4096, 8192, 4, 128, 31),     # grouped decode kernels: 31 tokens in one launch take more than the fixed scratch
    ("c1", 768, 3072, 8, 32, 620),      # grouped GEMMs of narrow layers
])
def test_static_entry_runs_the_grouped_kernels_in_smaller_launches(base, d, f, E, group, T):
    cfg = replace(gen.tiny_config(base, d, f, n_experts=E, n_layers=1, group=group), x_dtype="f32")
    layer, _, _, _ = build_layer_pair(cfg, 0, DEV, [2, 4] * (E // 2), want_oracle=False)
    assert layer.workspace_bytes(T) > binding.moe_static_scratch_bytes()
    x = gen.hidden(cfg, 0, 0, T, DEV)
    want = moeq.moe_layer_forward(layer, x, want_routing=True)
    got = binding.moe_layer_forward_static(layer, x, want_routing=True)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("layout", ("canonical", "columns"))
@pytest.mark.parametrize("f", (1024, 4096))
def test_an_experts_call_does_not_depend_on_the_other_experts(f, layout):
    cfg = replace(gen.tiny_config("c4", 4096, f, n_experts=4, n_layers=1, group=128), x_dtype="f32")
    kw = dict(want_oracle=False, columns=layout == "columns")
    mixed, _, Wr, bias = build_layer_pair(cfg, 0, DEV, [8, 2, 2, 4], **kw)
    alone = moeq.Layer(4096, f, 1, 128, moeq.MOEQ_ACT_SWIGLU, True, moeq.MOEQ_F32, Wr[:1].contiguous(), bias if bias is None else bias[:1].contiguous(),
                       mixed.experts[:1], mixed.out_layout, mixed.in_layout)
    x = gen.hidden(cfg, 0, 0, 40, DEV)
    for T in list(range(2, 18)) + [24, 31, 32, 40]:
        a, b = moeq.moe_expert_ffn_q(mixed, 0, x[:T]), moeq.moe_expert_ffn_q(alone, 0, x[:T])
        assert torch.equal(a, b), T


@pytest.mark.parametrize("act", ("relu", "swiglu"))
def test_workspace_grows_with_the_tokens_over_the_line_to_the_prefill_gemms(act):
    """Layers in columns that group the pairs of 6 to 31 tokens and run other kernels from 32 on: a workspace for more serves those
    calls in as many launches, with the same bits."""
    d, f, g, k = 1024, 24576, 128, 8
    cfg = replace(gen.tiny_config("c1", d, f, n_experts=1, n_layers=1, group=g), x_dtype="f32", act=act)
    ex = pack_expert_gpu(gen.expert_weights(cfg, 0, 0, DEV), 4, g).with_out_columns(f, g)
    layer = moeq.Layer(d, f, k, g, moeq.MOEQ_ACT_SWIGLU if act == "swiglu" else moeq.MOEQ_ACT_RELU, False, moeq.MOEQ_F32,
                       torch.randn((16, d), device=DEV), None, [ex] * 16, moeq.MOEQ_OUT_COLUMNS)
    sizes = [layer.workspace_bytes(T) for T in range(1, 200)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
    x = gen.hidden(cfg, 0, 0, 31, DEV)
    for T in (5, 6, 20, 31):
        want = moeq.moe_layer_forward(layer, x[:T], ws=torch.empty(sizes[T - 1], dtype=torch.uint8, device=DEV))
        assert torch.equal(moeq.moe_layer_forward(layer, x[:T], ws=torch.empty(sizes[31], dtype=torch.uint8, device=DEV)), want), T
