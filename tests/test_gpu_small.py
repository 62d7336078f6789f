"""GPU parity of the decode kernels for layers whose slices of d_ff, or rows, are a few KB (decode_small.hip), in both layouts of
W_out: widths at the edges of a workgroup's threads, slices of 16 to 128 columns, rows in one pass and in several, every source of
the routing, several choices, scales that are aligned to two bytes only, both ends of the range of x."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2308_14352_amd as moeq
from helpers import near_tie_tokens, pack_expert_gpu, pack_expert_oracle, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# fp32 products and sums throughout: an element of h is a sum of d products, of y one of d_ff, each off by at most a few roundings
# of the largest partial sum and by the square root of their number times 2^-24 in the norm; two such sums in a row, the largest
# of up to 2048 outputs, softmax by the hardware exponential (a few 1e-7): 4 * 2 * sqrt(4096) * 2^-24 = 3e-5
TOL = 3e-5


def odd(t):
    """The same values at an address that is a multiple of two bytes, not of four."""
    b = torch.empty(t.numel() + 3, dtype=t.dtype, device=t.device)
    v = b[1:1 + t.numel()]
    assert v.data_ptr() % 4 == 2
    v.copy_(t.reshape(-1))
    return v.view(t.shape)


@pytest.mark.parametrize("d,f,group,E,k,act,x_dtype,misaligned", [
    (64, 128, 32, 3, 1, "relu", "f32", False),       # fewer columns than a row of lanes folds
    (512, 1024, 32, 64, 2, "relu", "bf16", False),   # logits of 64 experts, one record per lane
    (768, 3072, 32, 65, 1, "relu", "f32", True),     # ... of 65: records from memory
    (768, 768, 96, 5, 3, "relu", "f32", False),     # a group that is no power of two: 4 and 8 bits
    (1024, 3072, 64, 8, 2, "swiglu", "f32", True),   # the widest with two output rows a thread
    (1088, 768, 32, 8, 1, "relu", "f32", True),      # ... and the narrowest with four
    (2048, 512, 128, 140, 2, "relu", "bf16", False), # the widest
    (512, 8192, 32, 4, 1, "relu", "f32", False),     # slices of 32 columns
    (256, 16384, 64, 3, 2, "swiglu", "f32", False),  # of 64: single tokens only
    (256, 32768, 128, 2, 1, "relu", "f32", False),   # of 128 (rows: more columns than they take)
    (2048, 8192, 128, 3, 1, "relu", "f32", False),   # the longest rows of W_out: four of 8 bits a pass (single tokens only)
    (1024, 2048, 32, 130, 5, "relu", "f32", True),   # more experts than two per lane, five choices, workgroups of several passes
])
@pytest.mark.parametrize("columns", (False, True), ids=("canonical", "columns"))
def test_small_slices(d, f, group, E, k, act, x_dtype, misaligned, columns):
    cfg = replace(gen.tiny_config("c1", d, f, n_experts=E, n_layers=1, group=group), top_k=k, x_dtype=x_dtype, act=act)
    distinct = [gen.expert_weights(cfg, 0, e, DEV) for e in range(min(E, 6))]
    widths = (4, 8) if group % 64 and group != 32 else (2, 4) if d == 2048 and columns else (2, 4, 8)     # (8 bits: single tokens)
    packed = [(pack_expert_gpu(w, widths[i % len(widths)], group), pack_expert_oracle(w, widths[i % len(widths)], group))
              for i, w in enumerate(distinct)]
    if columns:
        packed = [(ex.with_out_columns(f, group), o) for ex, o in packed]
    if misaligned:
        for ex, _ in packed:
            ex.s_in, ex.s_out, ex.s_gate = odd(ex.s_in), odd(ex.s_out), None if ex.s_gate is None else odd(ex.s_gate)
    gpu, orc = [[packed[e % len(packed)][i] for e in range(E)] for i in (0, 1)]
    Wr, bias = gen.router_weights(cfg, 0, DEV)
    layer = moeq.Layer(d, f, k, group, moeq.MOEQ_ACT_SWIGLU if act == "swiglu" else moeq.MOEQ_ACT_RELU, cfg.renorm,
                       moeq.MOEQ_BF16 if x_dtype == "bf16" else moeq.MOEQ_F32, Wr, bias, gpu,
                       moeq.MOEQ_OUT_COLUMNS if columns else moeq.MOEQ_OUT_CANONICAL)
    sw, wr, b = int(act == "swiglu"), Wr.cpu().numpy(), None if bias is None else bias.cpu().numpy()
    few = 0 if f > 8192 else (34e6 if d % 512 == 0 else 18e6) / (d * f * (1.5 if sw else 1.0))     # pairs of a call in rows
    if columns:
        few = k if group % 64 == 0 and f // 64 >= 192 or d * f > 1e7 else 1 << 30     # wide slices, or one workgroup a compute unit
    for T in (1, 3):
        x = gen.hidden(cfg, 0, T, T, DEV)
        xh = x.float().cpu().numpy()
        y, idx, gate = moeq.moe_layer_forward(layer, x, want_routing=True)
        y_e = moeq.moe_expert_ffn_q(layer, E - 1, x, gate=gate[:, 0].contiguous())
        torch.cuda.synchronize()
        y_ref, idx_ref, gate_ref = oracle.layer_forward(orc, d, f, group, sw, k, cfg.renorm, wr, b, xh)
        keep = [t for t in range(T) if t not in near_tie_tokens(cfg, Wr, bias, x)]
        tol, tol_e = (TOL if n <= few else 2e-3 for n in (T * k, T))   # (binary16 activations beyond)
        assert np.array_equal(idx.cpu().numpy()[keep], idx_ref[keep])
        assert np.allclose(gate.cpu().numpy()[keep], gate_ref[keep], rtol=2e-5, atol=1e-7)
        assert rel_err(y.cpu().numpy()[keep], y_ref[keep]).max(initial=0) < tol
        e_ref = oracle.expert_ffn(orc[E - 1], d, f, group, sw, xh) * gate.cpu().numpy()[:, :1]
        assert rel_err(y_e.cpu().numpy(), e_ref).max() < tol_e
        # routing given, on tokens of very different scales
        scale = (2.0 ** np.array([-96, 100, 0][:T])[:, None]).astype(np.float32)
        xs = (gen.hidden(replace(cfg, x_dtype="f32"), 0, T + 9, T, DEV) * torch.from_numpy(scale).to(DEV))
        xs = xs.to(torch.bfloat16) if x_dtype == "bf16" else xs
        gi = np.stack([(np.arange(T) * 5 + j) % E for j in range(k)], 1).astype(np.int32)
        gg = np.linspace(0.2, 0.9, T * k, dtype=np.float32).reshape(T, k)
        y_g = moeq.moe_layer_forward_routed(layer, xs, torch.from_numpy(gi).to(DEV), torch.from_numpy(gg).to(DEV))
        torch.cuda.synchronize()
        # (SwiGLU is not homogeneous: the gate's sigmoid is 0 or 1 at these scales, its products leave fp32's range)
        rows = [t for t in range(T) if act == "relu" or scale[t, 0] == 1.0]
        g_ref = oracle.layer_forward_routed(orc, d, f, group, sw, k, xs.float().cpu().numpy(), gi, gg)
        assert rel_err(y_g.cpu().numpy()[rows], g_ref[rows]).max(initial=0) < tol


@pytest.mark.parametrize("d,f,group,E,k,act,T", [
    (1536, 2048, 32, 6, 1, "swiglu", 6),     # 8-bit rows of W_in in passes of half a workgroup's, two matrices
    (1024, 1024, 32, 30, 1, "relu", 23),     # an uneven last block of rows, in both phases
    (512, 2048, 128, 9, 1, "relu", 22),      # long rows of W_out in fewer passes than 32 KB hold
    (512, 512, 64, 4, 1, "relu", 84),        # a token's blocks fewer than the XCDs
    (1024, 4096, 64, 8, 2, "relu", 4),       # the last call under the line (8 pairs) ...
    (1024, 4096, 64, 8, 1, "relu", 9),       # ... and one beyond it
    (768, 3072, 32, 8, 1, "relu", 7),        # the same for widths that are no multiple of 512
    (768, 3072, 32, 8, 1, "relu", 8),
    (2048, 8192, 128, 3, 1, "relu", 2),      # rows of W_out that leave one workgroup a compute unit
])
def test_small_rows_of_several_tokens(d, f, group, E, k, act, T):
    cfg = replace(gen.tiny_config("c1", d, f, n_experts=E, n_layers=1, group=group), top_k=k, x_dtype="f32", act=act)
    distinct = [gen.expert_weights(cfg, 0, e, DEV) for e in range(3)]
    gpu, orc = ([pack(distinct[e % 3], (2, 4, 8)[e % 3], group) for e in range(3)] for pack in (pack_expert_gpu, pack_expert_oracle))
    Wr, bias = gen.router_weights(cfg, 0, DEV)
    layer = moeq.Layer(d, f, k, group, moeq.MOEQ_ACT_SWIGLU if act == "swiglu" else moeq.MOEQ_ACT_RELU, cfg.renorm, moeq.MOEQ_F32, Wr,
                       bias, [gpu[e % 3] for e in range(E)])
    x = gen.hidden(cfg, 0, 0, T, DEV)
    y, idx, gate = moeq.moe_layer_forward(layer, x, want_routing=True)
    y_e = moeq.moe_expert_ffn_q(layer, 2, x)
    torch.cuda.synchronize()
    line = 34e6 if d % 512 == 0 else 18e6
    tol, tol_e = (TOL if n * d * f * (1.5 if act == "swiglu" else 1.0) <= line else 2e-3 for n in (T * k, T))
    sw, xh = int(act == "swiglu"), x.cpu().numpy()
    ref = oracle.layer_forward_routed([orc[e % 3] for e in range(E)], d, f, group, sw, k, xh, idx.cpu().numpy(), gate.cpu().numpy())
    assert rel_err(y.cpu().numpy(), ref).max() < tol
    assert rel_err(y_e.cpu().numpy(), oracle.expert_ffn(orc[2], d, f, group, sw, xh)).max() < tol_e


@pytest.mark.parametrize("d,f,group,E,k,act,bits", [
    (1024, 6144, 32, 8, 1, "relu", 8),       # the launch asks for 78.4 KB of LDS, router inside
    (1024, 6144, 32, 40, 1, "relu", 8),      # ... from the router kernel's logits
    (1024, 6144, 32, 80, 1, "relu", 8),      # ... of more than 64 experts
    (1984, 2048, 32, 70, 1, "relu", 8),      # 80.0 KB: the last of the line
    (1024, 2048, 64, 6, 2, "swiglu", 8),     # two matrices, two choices
    (1056, 6144, 32, 6, 1, "relu", 8),       # just beyond the line: single tokens only
])
def test_small_slices_at_half_a_compute_units_lds(d, f, group, E, k, act, bits):
    cfg = replace(gen.tiny_config("c1", d, f, n_experts=E, n_layers=1, group=group), top_k=k, x_dtype="f32", act=act)
    distinct = [gen.expert_weights(cfg, 0, e, DEV) for e in range(2)]
    gpu = [pack_expert_gpu(w, bits, group).with_out_columns(f, group) for w in distinct]
    orc = [pack_expert_oracle(w, bits, group) for w in distinct]
    Wr, bias = gen.router_weights(cfg, 0, DEV)
    layer = moeq.Layer(d, f, k, group, moeq.MOEQ_ACT_SWIGLU if act == "swiglu" else moeq.MOEQ_ACT_RELU, cfg.renorm, moeq.MOEQ_F32, Wr,
                       bias, [gpu[e % 2] for e in range(E)], moeq.MOEQ_OUT_COLUMNS)
    for T in (1, 2, 5):
        x = gen.hidden(cfg, 0, T, T, DEV)
        y, idx, gate = moeq.moe_layer_forward(layer, x, want_routing=True)
        torch.cuda.synchronize()
        ref = oracle.layer_forward_routed([orc[e % 2] for e in range(E)], d, f, group, int(act == "swiglu"), k, x.cpu().numpy(),
                                          idx.cpu().numpy(), gate.cpu().numpy())
        assert rel_err(y.cpu().numpy(), ref).max() < (2e-3 if d == 1056 and T > 1 else TOL), T


@pytest.mark.parametrize("bits", (2, 4, 8))
@pytest.mark.parametrize("columns", (False, True), ids=("canonical", "columns"))
def test_outlier_columns_that_meet_zero_weights(bits, columns):
    """Columns of x 2^13 times the others, on weights of zero. A zero weight is the code 2^(bits - 1) and its product leaves the sum
    with the offset at the end: d / 128 such products, each in up to 16 roundings of 2^-24 of a partial sum of 2^(bits + 12), are an
    error of 0.3 at 8 bits beside a sum of some 40 sqrt(768) = 1100, 3e-4 of it, less at fewer bits; the largest of 768 outputs."""
    d, f, g, T = 768, 3072, 32, 3
    cfg = gen.tiny_config("c1", d, f, n_experts=1, n_layers=1, group=g)
    w = gen.expert_weights(cfg, 0, 0, DEV)
    w["w_in"][:, 5::128] = 0.0
    ex = pack_expert_gpu(w, bits, g)
    Wr, bias = gen.router_weights(cfg, 0, DEV)
    layer = moeq.Layer(d, f, 1, g, moeq.MOEQ_ACT_RELU, False, moeq.MOEQ_F32, Wr, bias, [ex.with_out_columns(f, g) if columns else ex],
                       moeq.MOEQ_OUT_COLUMNS if columns else moeq.MOEQ_OUT_CANONICAL)
    x = gen.hidden(cfg, 0, 0, T, DEV)
    x[:, 5::128] *= 8192.0
    y = moeq.moe_expert_ffn_q(layer, 0, x)
    torch.cuda.synchronize()
    assert rel_err(y.cpu().numpy(), oracle.expert_ffn(pack_expert_oracle(w, bits, g), d, f, g, 0, x.cpu().numpy())).max() < 1e-3
