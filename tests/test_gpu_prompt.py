"""GPU parity of the kernel that routes calls of many tokens, through the C ABI against the oracle."""
import numpy as np
import oracle
import paper_2308_14352_amd as moeq
import pytest
import torch
from helpers import pack_expert_gpu

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


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
