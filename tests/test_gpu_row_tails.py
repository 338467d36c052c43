"""Row kernels at row lengths around their vectors, chunks and launch rules (2048 and 4096 columns), from pointers off
any alignment: norm forward and backward, quantiser steps and causal softmax, bit-identical to the oracle."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I
from gpu_util import DEV, assert_bits, dev_bf16, dev_f32, host_f32, host_u16

pytestmark = pytest.mark.gpu


def off(t):
    """A copy of t that starts one element off the allocation's alignment."""
    u = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)[1:].view(t.shape)
    u.copy_(t)
    return u


@pytest.mark.parametrize("rows,cols", [(5, 1), (33, 3), (40, 2047), (31, 2048), (65, 2049), (9, 2052), (7, 4097), (2, 4100)])
def test_norm_tails(rows, cols):
    print(f"norm {rows}x{cols}", flush=True)
    x = I.normal_f32((rows, cols), 1, 3)
    g = I.normal_bf16((cols,), 1, 200, std=0.1, mean=1.0)
    dy = I.normal_f32((rows, cols), 1, 7)
    eps = np.float32(1e-5)
    y_o, r_o = oracle.rownorm_fwd(x, g, eps)
    dx_o, dg_o = oracle.rownorm_bwd(x, g, r_o, dy)
    xd, gd, dyd = off(dev_f32(x)), off(dev_bf16(g)), off(dev_f32(dy))
    y = off(torch.empty((rows, cols), dtype=torch.bfloat16, device=DEV))
    dx = off(torch.empty((rows, cols), dtype=torch.float32, device=DEV))
    r = torch.empty(rows, dtype=torch.float32, device=DEV)
    dg = torch.empty(cols, dtype=torch.float32, device=DEV)
    C.rownorm(C.FWD, rows, cols, xd, gd, eps, y=y, rstd=r)
    C.rownorm(C.BWD, rows, cols, xd, gd, eps, rstd=r, dy=dyd, dx=dx, dgain=dg)
    torch.cuda.synchronize()
    assert_bits(host_u16(y), y_o, "y")
    assert_bits(host_f32(r), r_o, "rstd")
    assert_bits(host_f32(dx), dx_o, "dx")
    assert_bits(host_f32(dg), dg_o, "dgain")


@pytest.mark.parametrize("window", [0, 1, 100, 600])
@pytest.mark.parametrize("s", [1, 3, 255, 257, 2047, 2048, 2049, 2052, 4095, 4096, 4097])
def test_softmax_tails(s, window):
    print(f"softmax {s} window {window}", flush=True)
    raw = I.normal_f32((1, s, s), 0, I.TENSOR_IDS["scores"]) * np.float32(40)
    c = np.float32(0.125)
    want = oracle.softmax_causal(raw, c, window)
    p = off(torch.empty((1, s, s), dtype=torch.bfloat16, device=DEV))
    C.softmax_xent(C.SOFTMAX_CAUSAL, s, s, off(dev_f32(raw)), p, scale=float(c), window=window)
    torch.cuda.synchronize()
    assert_bits(host_u16(p), want, "probs")


@pytest.mark.parametrize("rows,cols", [(3, 1), (5, 33), (6, 2047), (4, 2048), (3, 2049), (2, 4100)])
def test_quant_scales_tails(rows, cols):
    print(f"quant scales {rows}x{cols}", flush=True)
    w = I.normal_bf16((rows, cols), 0, 11)
    s = torch.empty(rows, dtype=torch.float32, device=DEV)
    C.quant_scales(rows, cols, off(dev_bf16(w)), s)
    torch.cuda.synchronize()
    assert_bits(host_f32(s), oracle.quant_scales(w), "scales")
