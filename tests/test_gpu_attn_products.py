"""The causally skipping attention products of a decoder block (P.V, dQ, dK, dV) on each of their kernels: the split
kernel with one and two row groups and the general one, with and without windows, with one contraction per head and with
the heads of a group stacked along K, whole and ragged; blocks bit for bit against the oracle, from a workspace that is
NaN wherever the library did not write."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I
from gemm_rule import attention_configs
from gpu_util import DEV, assert_bits, dev_bf16, dev_f32, host_f32, poisoned_workspace

pytestmark = pytest.mark.gpu
NAMES = ["attn_norm", "w_qkv", "w_o", "ffn_norm", "w_gate_up", "w_down"]
ONE, TWO, GEN = (1, 1), (2, 1), None


@pytest.mark.parametrize("heads,kv,hd,win,seq,batch,pv,dkv", [
    (4, 4, 64, 0, 192, 2, ONE, ONE), (4, 2, 64, 50, 384, 1, ONE, ONE),
    # two row groups: skipped chunks, ranges with unequal counts of real ones, a ragged last chunk
    (4, 4, 64, 0, 512, 4, TWO, TWO), (4, 4, 64, 40, 512, 4, TWO, TWO), (4, 4, 64, 300, 512, 4, TWO, TWO),
    (4, 4, 64, 0, 500, 4, TWO, TWO), (4, 4, 64, 130, 500, 4, TWO, TWO), (2, 2, 128, 70, 1000, 2, TWO, TWO),
    (8, 4, 64, 0, 512, 4, GEN, TWO), (8, 4, 64, 100, 512, 4, GEN, TWO), (8, 2, 64, 33, 384, 8, GEN, TWO),
    # the general kernel: windows in both directions, stacked heads, ragged rows
    (8, 8, 64, 0, 512, 4, GEN, GEN), (8, 8, 64, 90, 512, 4, GEN, GEN), (8, 8, 64, 200, 500, 4, GEN, GEN),
    (16, 8, 32, 0, 512, 4, GEN, GEN), (16, 8, 32, 100, 512, 4, GEN, GEN), (8, 4, 64, 60, 640, 4, GEN, GEN),
    # a short window in a long sequence: dK and dV leave the two row groups
    (2, 2, 64, 100, 4096, 1, TWO, GEN),
])
def test_block(heads, kv, hd, win, seq, batch, pv, dkv):
    print(f"attention products heads={heads}/{kv} hd={hd} win={win} S={seq} B={batch}", flush=True)
    assert attention_configs(batch, heads, kv, seq, hd, win) == (pv, dkv)
    d, F, T = heads * hd, 256, batch * seq
    args = (1, d, heads, hd, F, 100, seq, batch, np.float32(1e-5), kv, 1, 0, win, 0, np.float32(0))
    cfg_o, cfg_c = oracle.ModelCfg(*args), C.ModelCfg(*args)
    x = I.bf16_bits_to_f32(I.normal_bf16((T, d), 4, I.TENSOR_IDS["x_in"]))
    dy = I.bf16_bits_to_f32(I.normal_bf16((T, d), 4, I.TENSOR_IDS["dy_in"]))
    shapes = [(d,), (d + 2 * kv * hd, d), (d, d), (d,), (2 * F, d), (d, F)]
    w = [I.normal_bf16(s, 4, I.TENSOR_IDS[n], std=(0.1 if len(s) == 1 else 0.05), mean=(1.0 if len(s) == 1 else 0.0))
         for s, n in zip(shapes, NAMES)]
    cos, sin = I.rope_tables(seq, hd)
    y_o, dx_o, dw_o = oracle.block_fwd_bwd(cfg_o, batch, x, dy, w, cos, sin)
    ws = poisoned_workspace(C.block_workspace_bytes(cfg_c, batch))
    y = torch.empty((T, d), dtype=torch.float32, device=DEV)
    dx = torch.empty_like(y)
    dw = [torch.empty(s, dtype=torch.float32, device=DEV) for s in shapes]
    C.block_fwd_bwd(cfg_c, batch, dev_f32(x), dev_f32(dy), [dev_bf16(t) for t in w], dev_f32(cos), dev_f32(sin), y,
                    dx, dw, ws)
    torch.cuda.synchronize()
    assert_bits(host_f32(y), y_o, "y")
    assert_bits(host_f32(dx), dx_o, "dx")
    for n, g, go in zip(NAMES, dw, dw_o):
        assert_bits(host_f32(g), go, "d" + n)
