"""Cross-entropy rows at the edges of the launch rule (vocab 10240, 26624 and 57344), of the 8-wide vectors and of the
chunks, and with logits far enough below the row's maximum that their exponential is zero: bit-identical to the oracle.
Infinite logits give the arithmetic's own results (a row of -inf but one target: probability one), and rows that hold a
NaN are NaN."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("z", [0.0, 1e-4])
@pytest.mark.parametrize("vocab", [1, 7, 8, 9, 33, 2049, 10239, 10240, 10241, 26624, 26625, 57344, 57345, 131071, 131072])
def test_xent_rows(vocab, z):
    rows = 5
    print(f"xent rows vocab={vocab} z={z}", flush=True)
    x = I.normal_f32((rows, vocab), 0, I.TENSOR_IDS["logits"]) * np.float32(3)
    x[1, ::3] -= np.float32(300)  # zero exponentials in the row, and a far maximum
    x[2, vocab - 1] += np.float32(90)
    x[3, vocab // 2:] = -np.inf
    x[3, 0] = 1.0
    logits = (x.view(np.uint32) >> 16).astype(np.uint16)
    tgt = np.array([0, vocab - 1, vocab - 1, 0, vocab // 2], np.int32)
    inv = np.float32(1 / rows)
    dl_o, rl_o, ml_o = oracle.xent(logits, tgt, inv, z_loss=z)
    # one element off any alignment
    lg = torch.empty(rows * vocab + 1, dtype=torch.bfloat16, device=DEV)[1:]
    lg.copy_(torch.from_numpy(logits.view(np.int16)).view(torch.bfloat16).flatten())
    dl = torch.zeros(rows * vocab + 2, dtype=torch.bfloat16, device=DEV)
    rl = torch.empty(rows, dtype=torch.float32, device=DEV)
    ml = torch.empty(1, dtype=torch.float32, device=DEV)
    C.softmax_xent(C.XENT, rows, vocab, lg, dl[1:-1], targets=torch.from_numpy(tgt).to(DEV), inv_tokens=float(inv),
                   row_loss=rl, mean_loss=ml, z_loss=z)
    torch.cuda.synchronize()
    out = dl.cpu().view(torch.int16).numpy().view(np.uint16)
    assert out[0] == 0 and out[-1] == 0
    np.testing.assert_array_equal(out[1:-1].reshape(rows, vocab), dl_o)
    np.testing.assert_array_equal(rl.cpu().numpy().view(np.uint32), rl_o.view(np.uint32))
    assert ml.cpu().numpy().view(np.uint32)[0] == np.float32(ml_o).view(np.uint32)


@pytest.mark.parametrize("vocab", [9, 1000, 10241, 57344, 57345])
def test_xent_rows_with_nan(vocab):
    # a NaN logit (either sign, quiet or not), +inf, and a row of -inf make a row of NaN: a NaN must round to a bf16 NaN,
    # never to a number or an infinity (which NaN it is, is not specified).  The rows between stay the oracle's bits.
    rows = 9
    print(f"xent nan rows vocab={vocab}", flush=True)
    logits = I.normal_bf16((rows, vocab), 1, I.TENSOR_IDS["logits"], std=2.0)
    for r, at, bits in ((0, 0, 0x7FC0), (1, vocab - 1, 0xFFC0), (2, vocab // 2, 0x7F81), (3, 1, 0xFFFF), (5, vocab - 2, 0x7F80)):
        logits[r, at] = bits
    logits[6, :] = 0xFF80
    tgt = np.array([0, 1, 2, 1, 0, 0, 0, vocab - 1, 3], np.int32)
    inv = np.float32(1 / rows)
    dl_o, rl_o, _ = oracle.xent(logits, tgt, inv)
    nan_o = (dl_o & 0x7FFF) > 0x7F80
    assert nan_o[[0, 1, 2, 3, 5, 6]].all() and not nan_o[[4, 7, 8]].any()
    dl = torch.zeros((rows, vocab), dtype=torch.bfloat16, device=DEV)
    rl = torch.empty(rows, dtype=torch.float32, device=DEV)
    C.softmax_xent(C.XENT, rows, vocab, torch.from_numpy(logits.view(np.int16)).view(torch.bfloat16).to(DEV), dl,
                   targets=torch.from_numpy(tgt).to(DEV), inv_tokens=float(inv), row_loss=rl)
    torch.cuda.synchronize()
    out, loss = dl.cpu().view(torch.int16).numpy().view(np.uint16), rl.cpu().numpy()
    np.testing.assert_array_equal((out & 0x7FFF) > 0x7F80, nan_o)
    np.testing.assert_array_equal(np.where(nan_o, 0, out), np.where(nan_o, 0, dl_o))
    np.testing.assert_array_equal(np.isnan(loss), np.isnan(rl_o))
    np.testing.assert_array_equal(loss[[4, 7, 8]].view(np.uint32), rl_o[[4, 7, 8]].view(np.uint32))
