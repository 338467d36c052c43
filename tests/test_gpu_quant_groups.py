"""The quantiser's groups of codes with a step per row (values on and one unit beside every rounding boundary, beyond the
clamps, infinite and NaN; steps outside the reciprocal's range) and the step gradient at sizes around its segments and
workgroups from pointers off alignment: bit-identical to the oracle."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I
from gpu_util import DEV, assert_bits, dev_bf16, dev_f32, host_f32

pytestmark = pytest.mark.gpu


def test_rows_near_boundaries():
    print("quantize rows near boundaries", flush=True)
    steps = np.array([0.1416, 1.0, 3e-38, 2.0**-126, 0.33333334, 1e38, 2.0**127, 0.0, -1.0, 1e-40, np.nan], np.float32)
    halves = np.arange(-130, 131, dtype=np.float64) + 0.5
    rows = []
    for s in steps:
        with np.errstate(all="ignore"):
            x = (halves * float(s)).astype(np.float32)
        b = (x.view(np.uint32) >> 16).astype(np.int64)
        row = np.concatenate([b, np.maximum(b - 1, 0), b + 1, [0x7F80, 0xFF80, 0x7FC0, 0, 0x8000, 1, 0x7F7F, 0xFF7F]])
        rows.append(row[: len(row) // 8 * 8])
    x = np.stack(rows).astype(np.uint16)
    q = torch.empty(x.shape, dtype=torch.int8, device=DEV)
    C.quantize(x.shape[0], x.shape[1], dev_bf16(x), dev_f32(steps), 1, q)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(q.cpu().numpy(), oracle.quantize(x, steps, True))


@pytest.mark.parametrize("n", [1, 31, 2047, 2048, 2049, 4095, 4097, 6145, 32767, 32768, 32769, 34817, 100001])
@pytest.mark.parametrize("off", [0, 1])
def test_lsq_sizes(n, off):
    print(f"lsq n={n} offset {off}", flush=True)
    x = I.normal_bf16((1, n), 1, 5, std=4.0)
    dx = I.normal_f32((1, n), 1, 6)
    xd = torch.empty(n + off, dtype=torch.bfloat16, device=DEV)[off:]
    xd.copy_(dev_bf16(x).flatten())
    dd = torch.empty(n + off, dtype=torch.float32, device=DEV)[off:]
    dd.copy_(dev_f32(dx).flatten())
    ws = torch.empty(C.lsq_step_grad_workspace_bytes(1, n), dtype=torch.uint8, device=DEV)
    g = torch.empty(1, dtype=torch.float32, device=DEV)
    C.lsq_step_grad(1, n, xd, dev_f32(np.array([0.05], np.float32)), dd, g, ws)
    torch.cuda.synchronize()
    assert_bits(host_f32(g), np.array([oracle.lsq_step_grad(x, np.float32(0.05), dx)], np.float32), "lsq grad")
