"""canon_gemm where the output is too small to fill the chip (K split over wavefronts) and where its last tile is
ragged, against the oracle, bit for bit: every split, at the edges where the next one takes over (256 CUs), every
layout, ragged K, and operands for which rounding, flushes and signed zeros decide."""
import numpy as np
import pytest
import torch

import adversarial as ADV
import oracle
import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I
from gemm_rule import split_config
from gpu_util import DEV, assert_bits, dev_bf16, host_f32

pytestmark = pytest.mark.gpu
LAYOUTS = [(0, 1), (0, 0), (1, 0), (1, 1)]

SHAPES = [
    # 16 x 16 tiles (48 chunks or more): one tile, the last shape that takes them, ragged ends
    (16, 16, 1541), (17, 19, 1536), (256, 256, 1536), (250, 241, 2079),
    # 16 x 32 tiles
    (256, 257, 1536), (16, 32, 64), (100, 300, 97), (40, 33, 1000),
    # 16 x 64 tiles; one chunk and parts of one
    (64, 64, 32), (31, 70, 31), (18, 16, 9), (16, 17, 8), (250, 1000, 300), (256, 1024, 1030),
    # 32 x 64 tiles, over 8 and over more chunks per range
    (272, 1024, 96), (500, 1001, 167), (512, 1024, 33), (400, 700, 1100),
    # past the last split: 64 x 64 tiles whose last rows and columns are ragged and unaligned
    (1100, 1030, 167), (1025, 577, 64), (700, 1333, 100),
]


def operands(m, n, k, ta, tb, seed):
    a = I.normal_bf16((k, m) if ta else (m, k), seed, I.TENSOR_IDS["gemm_a"])
    b = I.normal_bf16((n, k) if tb else (k, n), seed, I.TENSOR_IDS["gemm_b"])
    return a, b


def run(a, b, ta, tb, m, n, k):
    c = torch.full((m, n), float("nan"), dtype=torch.float32, device=DEV)
    C.gemm(m, n, k, dev_bf16(a), a.shape[1], dev_bf16(b), b.shape[1], c, n, ta, tb)
    torch.cuda.synchronize()
    return host_f32(c)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_splits_and_ragged_tiles(m, n, k, ta, tb):
    print(f"gemm split {m}x{n}x{k} ta={ta} tb={tb}", flush=True)
    a, b = operands(m, n, k, ta, tb, 31)
    assert_bits(run(a, b, ta, tb, m, n, k), oracle.gemm(a, b, bool(ta), bool(tb)), f"{m}x{n}x{k}")


@pytest.mark.parametrize("kind", ["wide", "tiny", "ties", "cancel", "huge"])
@pytest.mark.parametrize("m,n,k", [(40, 24, 1575), (120, 200, 167), (90, 1000, 70), (300, 900, 45)])
def test_adversarial_operands(kind, m, n, k):
    # ragged K: the padded terms of the last chunk must leave every partial sum as it is, -0 included
    a, b = ADV.gemm_operands(kind, m, n, k, seed=12)
    want = oracle.gemm(a, b)
    for ta, tb in LAYOUTS:
        print(f"gemm split adversarial {kind} {m}x{n}x{k} ta={ta} tb={tb}", flush=True)
        a_st = np.ascontiguousarray(a.T) if ta else a
        b_st = np.ascontiguousarray(b.T) if tb else b
        assert_bits(run(a_st, b_st, ta, tb, m, n, k), want, f"{kind} {m}x{n}x{k} ta={ta} tb={tb}")


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("m,n,k", [(30, 40, 1600), (100, 130, 200), (200, 900, 100), (400, 1000, 80), (1030, 1100, 70)])
def test_offsets_strides_and_accumulation(m, n, k, ta, tb):
    """Operands and C inside larger arrays (odd leading dimensions and offsets), two accumulating microbatches; the
    elements around C stay as they were."""
    print(f"gemm split strided {m}x{n}x{k} ta={ta} tb={tb}", flush=True)
    cbuf = torch.zeros((m, n + 5), dtype=torch.float32, device=DEV)
    cbuf[:, n:] = 7.0
    grads = []
    for j in range(2):
        a, b = operands(m, n, k, ta, tb, 41 + j)
        big = [torch.full((x.shape[0], x.shape[1] + 3), float("nan"), dtype=torch.bfloat16, device=DEV) for x in (a, b)]
        for t, x in zip(big, (a, b)):
            t[:, 1:1 + x.shape[1]] = dev_bf16(x)
        C.gemm(m, n, k, big[0].data_ptr() + 2, a.shape[1] + 3, big[1].data_ptr() + 2, b.shape[1] + 3, cbuf, n + 5, ta,
               tb, accum_scale=0.5)
        torch.cuda.synchronize()
        grads.append(oracle.gemm(a, b, bool(ta), bool(tb)).reshape(-1))
    got = host_f32(cbuf)
    want = oracle.grad_accum(grads, 2, 1, 1).reshape(m, n)
    assert_bits(got[:, :n], want, f"accum {m}x{n}x{k}")
    assert np.all(got[:, n:] == 7.0)


def test_batched_split():
    bt, m, n, k = 3, 100, 70, 200
    a, b = I.normal_bf16((bt, m, k), 5, 1), I.normal_bf16((bt, n, k), 5, 2)
    c = torch.full((bt, m, n), float("nan"), dtype=torch.float32, device=DEV)
    C.gemm_strided_batched(m, n, k, dev_bf16(a), k, m * k, dev_bf16(b), k, n * k, c, n, m * n, bt, trans_b=1)
    torch.cuda.synchronize()
    for z in range(bt):
        assert_bits(host_f32(c[z]), oracle.gemm(a[z], b[z], False, True), f"batch {z}")


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("bt,m,n,k", [(40, 64, 128, 96), (7, 40, 24, 1575), (9, 16, 33, 70), (13, 50, 70, 40), (256, 16, 64, 33), (61, 40, 100, 9)])
def test_batches_of_few_tiles(bt, m, n, k, ta, tb):
    # tiles of all matrices are dealt to the XCDs in one sequence: counts that are and are not multiples of 8, up to one
    # tile per CU; every matrix its own
    print(f"gemm split batch {bt}x{m}x{n}x{k} ta={ta} tb={tb}", flush=True)
    assert split_config(m, n, k, bt) is not None
    a, b = (I.normal_bf16((bt, *s), 6, i) for i, s in ((1, (k, m) if ta else (m, k)), (2, (n, k) if tb else (k, n))))
    c = torch.full((bt, m, n), float("nan"), dtype=torch.float32, device=DEV)
    C.gemm_strided_batched(m, n, k, dev_bf16(a), a.shape[2], m * k, dev_bf16(b), b.shape[2], n * k, c, n, m * n, bt,
                           trans_a=ta, trans_b=tb)
    torch.cuda.synchronize()
    got = host_f32(c)
    for z in range(bt):
        assert_bits(got[z], oracle.gemm(a[z], b[z], bool(ta), bool(tb)), f"batch {z}")
