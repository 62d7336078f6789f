"""The routing of calls of few tokens, by the kernels that choose the experts for themselves, against the router entry: ties, logits
of minus infinity, undefined tokens, from few experts to more than any kernel holds in its registers."""
from dataclasses import replace

import pytest
import torch

import gen
import paper_2308_14352_amd as moeq
from helpers import pack_expert_gpu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("columns", (False, True), ids=("canonical", "columns"))
@pytest.mark.parametrize("E,k", [(20, 3), (64, 8), (65, 2), (100, 8), (128, 4), (130, 8), (200, 3), (1024, 8)])
def test_layer_calls_choose_as_the_router_entry_does(E, k, columns):
    d, f, g = 256, 256, 32
    cfg = replace(gen.tiny_config("c1", d, f, n_experts=E, n_layers=1, group=g), top_k=k, x_dtype="f32")
    w = gen.expert_weights(cfg, 0, 0, DEV)
    ex = pack_expert_gpu(w, 4, g)
    ex = ex.with_out_columns(f, g) if columns else ex
    Wr = torch.randn((E, d), generator=torch.Generator(DEV).manual_seed(E), device=DEV)
    # equal rows, in one lane's registers and across lanes and registers: the lowest index comes first
    for a, b in ((1, 17), (3, 64), (0, 66), (2, 129), (64, 128), (5, 999)):
        if b < E:
            Wr[b] = Wr[a]
    x = torch.randn((9, d), generator=torch.Generator(DEV).manual_seed(k), device=DEV)
    x[3] = 0.0                                           # every logit the same
    x[5, 7], x[6, 200], x[7, 0] = float("nan"), float("inf"), float("-inf")
    few = torch.full((E,), float("-inf"), device=DEV)    # fewer finite logits than choices
    few[[0, E // 2, E - 1][:max(1, min(k - 1, 3))]] = 0.25
    for bias in (None, torch.linspace(-1.0, 1.0, E, device=DEV), few):
        layer = moeq.Layer(d, f, k, g, moeq.MOEQ_ACT_RELU, k % 2 == 0, moeq.MOEQ_F32, Wr, bias, [ex] * E,
                           moeq.MOEQ_OUT_COLUMNS if columns else moeq.MOEQ_OUT_CANONICAL)
        want_i, want_g = moeq.moe_router_topk(layer, x)
        for T in (1, 4, 9):
            for t0 in range(0, 9 - T + 1, T):
                y, idx, gate = moeq.moe_layer_forward(layer, x[t0:t0 + T], want_routing=True)
                torch.cuda.synchronize()
                assert torch.equal(idx, want_i[t0:t0 + T]), (T, t0, idx, want_i[t0:t0 + T])
                assert torch.allclose(gate, want_g[t0:t0 + T], rtol=2e-5, atol=1e-7, equal_nan=True), (T, t0)
                undefined = torch.isnan(want_g[t0:t0 + T]).any(1)
                assert torch.equal(~torch.isfinite(y).all(1), undefined), (T, t0)
