"""GPU parity of the compression primitives where their kernels can go wrong: quotients next to a half-integer
(quantizer), group sizes on both sides of its one-pass form, tails and odd groups (decompression)."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2308_14352_amd as moeq

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bits", (2, 4, 8))
@pytest.mark.parametrize("group", (4, 16, 32, 128, 256, 512))
def test_quantize_next_to_half_integers_bit_exact(bits, group):
    """Weights within a few ulp of (k + 1/2) * scale for every k: the code is the rounded IEEE quotient, which the
    quantizer's approximate quotient alone would miss."""
    rows, cols = 67, 1024
    qmax = 2 ** (bits - 1) - 1
    rng = np.random.default_rng(11 * bits + group)
    n_g = rows * cols // group
    absmax = rng.uniform(1e-3, 0.2, n_g).astype(np.float32)
    scale = np.float16(absmax / np.float32(qmax)).astype(np.float32)
    k = rng.integers(-qmax, qmax, (n_g, group))
    w = ((k + 0.5).astype(np.float32) * scale[:, None]).astype(np.float32)
    steps = rng.integers(-3, 4, w.shape)
    w = (w.view(np.int32) + np.where(w != 0, steps, 0).astype(np.int32)).view(np.float32)
    w = np.clip(w, -absmax[:, None], absmax[:, None])
    w[:, 0] = absmax
    w = np.ascontiguousarray(w.reshape(rows, cols))
    q, s = moeq.moe_quantize_pack(torch.from_numpy(w).to(DEV), bits, group)
    torch.cuda.synchronize()
    q_ref, s_ref = oracle.quantize_pack(w, bits, group)
    assert np.array_equal(s.view(torch.int16).cpu().numpy().view(np.uint16), s_ref)
    assert np.array_equal(q.cpu().numpy(), q_ref)


@pytest.mark.parametrize("bits", (2, 4, 8))
@pytest.mark.parametrize("rows,cols,group", [(1, 64, 64), (3, 192, 2), (5, 192, 6), (2, 320, 10), (7, 1056, 96), (129, 2048, 2048)])
def test_dequantize_odd_groups_and_tails(bits, rows, cols, group):
    rng = np.random.default_rng(rows * cols + group)
    q = rng.integers(0, 256, (rows, cols * bits // 8)).astype(np.uint8)
    s = rng.integers(0, 0x7c00, (rows, cols // group)).astype(np.uint16)        # any finite binary16, subnormals too
    w = moeq.moe_dequantize(torch.from_numpy(q).to(DEV), torch.from_numpy(s.view(np.int16)).to(DEV), cols, bits, group)
    torch.cuda.synchronize()
    u = np.stack([(q >> (bits * i)) & (2 ** bits - 1) for i in range(8 // bits)], -1).reshape(rows, cols).astype(np.int32)
    ref = np.repeat(s.view(np.float16).astype(np.float32), group, axis=1) * (u - 2 ** (bits - 1)).astype(np.float32)
    assert np.array_equal(w.cpu().numpy(), ref)
