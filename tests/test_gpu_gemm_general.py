"""The general canonical GEMM kernel (64 x 64 and 64 x 128 tiles) bit for bit against the oracle.  Outputs that fill the
chip only a little run on the split kernel, so each case here is a batch of one and the same product, large enough that
no split takes it; every matrix of the batch must come out alike."""
import numpy as np
import pytest
import torch

import adversarial as ADV
import oracle
import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I
from gemm_rule import general_batch, split_config
from gpu_util import DEV, assert_bits, dev_bf16, host_f32

pytestmark = pytest.mark.gpu
LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]


def operands(m, n, k, ta, tb, seed):
    a = I.normal_bf16((k, m) if ta else (m, k), seed, I.TENSOR_IDS["gemm_a"])
    b = I.normal_bf16((n, k) if tb else (k, n), seed, I.TENSOR_IDS["gemm_b"])
    return a, b


def check(a, b, ta, tb, m, n, k, what, want=None):
    bt = general_batch(m, n)
    assert split_config(m, n, k, bt) is None
    c = torch.full((bt, m, n), float("nan"), dtype=torch.float32, device=DEV)
    C.gemm_strided_batched(m, n, k, dev_bf16(a), a.shape[1], 0, dev_bf16(b), b.shape[1], 0, c, n, m * n, bt, ta, tb)
    torch.cuda.synchronize()
    assert_bits(host_f32(c[0]), oracle.gemm(a, b, bool(ta), bool(tb)) if want is None else want, what)
    bits = c.view(torch.int32)
    assert torch.equal(bits, bits[:1].expand_as(bits))


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("m,n", [(70, 130), (128, 256)])
@pytest.mark.parametrize("k", [160, 2080, 6144, 16384 + 96, 50304, 128256 + 7])
def test_deep_folds(k, m, n, ta, tb):
    # 5, 65, 192, 515, 1572 and 4009 chunks: every stack depth (3 to 12), odd counts and a ragged last chunk; last tiles
    # that are shifted into the matrix, and whole ones
    print(f"general gemm {m}x{n}x{k} ta={ta} tb={tb}", flush=True)
    a, b = operands(m, n, k, ta, tb, 4)
    check(a, b, ta, tb, m, n, k, f"{m}x{n}x{k}")


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("m,n,k", [(37, 45, 200), (64, 63, 161), (65, 64, 96), (1, 200, 257), (200, 3, 1000), (15, 17, 129)])
def test_edges_of_tiles(m, n, k, ta, tb):
    # matrices smaller than a tile (checked loads) and one row or column beyond one
    print(f"general gemm {m}x{n}x{k} ta={ta} tb={tb}", flush=True)
    a, b = operands(m, n, k, ta, tb, 3)
    check(a, b, ta, tb, m, n, k, f"{m}x{n}x{k}")


@pytest.mark.parametrize("kind", ["wide", "tiny", "ties", "cancel", "huge"])
@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("m,n,k", [(130, 260, 192), (70, 130, 167), (128, 256, 224)])
def test_adversarial_operands(kind, ta, tb, m, n, k):
    print(f"general gemm adversarial {kind} {m}x{n}x{k} ta={ta} tb={tb}", flush=True)
    a, b = ADV.gemm_operands(kind, m, n, k, seed=11)
    a_st = np.ascontiguousarray(a.T) if ta else a
    b_st = np.ascontiguousarray(b.T) if tb else b
    check(a_st, b_st, ta, tb, m, n, k, f"{kind} {m}x{n}x{k}")


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("m,n,k,accum", [(1030, 1060, 200, 3), (1088, 1024, 2048, 2)])
def test_accumulation(m, n, k, accum, ta, tb):
    assert split_config(m, n, k) is None
    print(f"general gemm accum {m}x{n}x{k} accum={accum} ta={ta} tb={tb}", flush=True)
    c = torch.zeros((m, n), dtype=torch.float32, device=DEV)
    grads = []
    for j in range(accum):
        a, b = operands(m, n, k, ta, tb, 20 + j)
        C.gemm(m, n, k, dev_bf16(a), a.shape[1], dev_bf16(b), b.shape[1], c, n, ta, tb,
               accum_scale=float(np.float32(1.0 / accum)))
        grads.append(oracle.gemm(a, b, bool(ta), bool(tb)).reshape(-1))
    torch.cuda.synchronize()
    assert_bits(host_f32(c), oracle.grad_accum(grads, accum, 1, 1).reshape(m, n), f"accum {m}x{n}x{k}")
