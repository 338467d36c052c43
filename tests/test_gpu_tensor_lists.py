"""AdamW and the clip over lists of tensors: counts around the 64 tensors of a launch, sizes around the 512 and 4096
elements of a workgroup and the four-element vectors, empty tensors, buffers off alignment and buffers that are listed twice (each
listing acts, in order), bit-identical to the oracle."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_17380_amd.canon as C
import paper_2609_17380_amd.inputs as I
from gpu_util import DEV, assert_bits, host_f32, host_u16

pytestmark = pytest.mark.gpu
EDGES = [0, 1, 3, 4, 511, 512, 513, 1025, 4095, 4096, 4097, 4099, 8193]


def place(host, dtype, off):
    t = torch.empty(host.size + off, dtype=dtype, device=DEV)[off:]
    t.copy_(torch.from_numpy(host.view(np.int16)).view(torch.bfloat16) if dtype == torch.bfloat16
            else torch.from_numpy(host))
    return t


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("count", [1, 63, 64, 65, 130])
def test_adamw_lists(count, off):
    print(f"adamw {count} tensors offset {off}", flush=True)
    sizes = [EDGES[i % len(EDGES)] for i in range(1, count + 1)]
    p = [I.normal_bf16((n,), i, 40, std=0.1) for i, n in enumerate(sizes)]
    m = [I.normal_f32((n,), i, 41) for i, n in enumerate(sizes)]
    v = [np.square(I.normal_f32((n,), i, 42)) for i, n in enumerate(sizes)]
    g = [I.normal_f32((n,), i, 43) for i, n in enumerate(sizes)]
    decay = [i % 3 == 0 for i in range(count)]
    k = I.adamw_constants()
    dp = [place(x, torch.bfloat16, off) for x in p]
    dm, dv, dg = ([place(x, torch.float32, off) for x in xs] for xs in (m, v, g))
    twice = [0, count - 1]  # listed again at the end
    order = list(range(count)) + twice
    for part in (list(range(count)), twice):
        sub = [[xs[i] for i in part] for xs in (p, m, v, g)]
        oracle.adamw(*sub, [decay[i] for i in part], oracle.AdamWConsts(*k))
    C.adamw(*([xs[i] for i in order] for xs in (dp, dm, dv, dg)), [decay[i] for i in order], C.AdamWConsts(*k))
    torch.cuda.synchronize()
    for i in range(count):
        assert_bits(host_u16(dp[i]), p[i], f"p{i}")
        assert_bits(host_f32(dm[i]), m[i], f"m{i}")
        assert_bits(host_f32(dv[i]), v[i], f"v{i}")


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("count", [2, 63, 64, 65, 130])
def test_clip_lists(count, off):
    print(f"clip {count} tensors offset {off}", flush=True)
    sizes = [EDGES[i % len(EDGES)] for i in range(1, count + 1)]
    if off == 0 and count == 65:
        sizes = [4 * n for n in sizes]  # every boundary on a vector
    g = [I.normal_f32((n,), i, 43) for i, n in enumerate(sizes)]
    dg = [place(x, torch.float32, off) for x in g]
    order = list(range(count)) + [0]  # tensor 0 counts twice and is scaled twice
    norm_o = oracle.global_norm([g[i] for i in order])
    coef = np.float32(1.0) / (norm_o + np.float32(1e-6))
    norm = torch.empty(1, dtype=torch.float32, device=DEV)
    lst = [dg[i] for i in order]
    ws = torch.empty(C.clip_grad_norm_workspace_bytes(lst), dtype=torch.uint8, device=DEV)
    C.clip_grad_norm(lst, C.make_clip(1.0, float("inf"), 0, norm), ws)
    torch.cuda.synchronize()
    assert_bits(host_f32(norm), np.array([norm_o], np.float32), "norm")
    for i in range(count):
        want = g[i] * coef if coef < 1 else g[i]
        if i == 0 and coef < 1:
            want = want * coef
        assert_bits(host_f32(dg[i]), want, f"g{i}")


@pytest.mark.parametrize("sizes", [[255], [257], [1 << 18], [(1 << 18) + 1], [(1 << 25) - 1], [1 << 25], [(1 << 25) + 257],
                                   [1000, (1 << 25) + 769, 513]])
def test_adamw_alone_and_large(sizes):
    # a tensor alone in its launch (one element per thread up to 2^18, two beyond) and those of 2^25 elements, which go
    # by themselves, two blocks of 256 per workgroup
    print(f"adamw alone {sizes}", flush=True)
    p = [I.normal_bf16((n,), i, 40, std=0.1) for i, n in enumerate(sizes)]
    m, g = ([I.normal_f32((n,), i, s) for i, n in enumerate(sizes)] for s in (41, 43))
    v = [np.square(x) for x in m]
    k = I.adamw_constants()
    dp = [place(x, torch.bfloat16, 1) for x in p]
    dm, dv, dg = ([place(x, torch.float32, 1) for x in xs] for xs in (m, v, g))
    oracle.adamw(p, m, v, g, [True] * len(sizes), oracle.AdamWConsts(*k))
    C.adamw(dp, dm, dv, dg, [True] * len(sizes), C.AdamWConsts(*k))
    torch.cuda.synchronize()
    for i in range(len(sizes)):
        assert_bits(host_u16(dp[i]), p[i], f"p{i}")
        assert_bits(host_f32(dm[i]), m[i], f"m{i}")
        assert_bits(host_f32(dv[i]), v[i], f"v{i}")


def test_clip_walks_its_units():
    # more units of 4096 elements than workgroups (65536), in tensors whose borders fall on any stride
    sizes = [3, (1 << 28) + 5, 4097, (1 << 27) + 4096, 0, 9]
    print(f"clip {sizes}", flush=True)
    g = [torch.full((n,), 0.5, dtype=torch.float32, device=DEV) for n in sizes]
    norm = torch.empty(1, dtype=torch.float32, device=DEV)
    ws = torch.empty(C.clip_grad_norm_workspace_bytes(g), dtype=torch.uint8, device=DEV)
    C.clip_grad_norm(g, C.make_clip(1.0, float("inf"), 0, norm), ws)
    torch.cuda.synchronize()
    want = np.float32(0.5) * (np.float32(1.0) / (host_f32(norm)[0] + np.float32(1e-6)))
    for t in g:
        if t.numel():
            assert np.float32(t.min().item()) == want and np.float32(t.max().item()) == want


@pytest.mark.parametrize("sizes", [[(1 << 33) + 5], [1 << 32, (1 << 32) + 777, 1000]])
def test_adamw_more_elements_than_one_grid_takes(sizes):
    # a workgroup of 256 threads per 512 elements: above 8.59e9 elements a launch would have 2^32 threads or more
    print(f"adamw {sizes}", flush=True)
    k = I.adamw_constants()
    one = [np.array([0x3F80], np.uint16)], [np.array([0.5], np.float32)], [np.array([0.25], np.float32)]
    oracle.adamw(*one, [np.array([2.0], np.float32)], [True], oracle.AdamWConsts(*k))
    p = [torch.full((n,), 1.0, dtype=torch.bfloat16, device=DEV) for n in sizes]
    m, v, g = ([torch.full((n,), x, dtype=torch.float32, device=DEV) for n in sizes] for x in (0.5, 0.25, 2.0))
    C.adamw(p, m, v, g, [True] * len(sizes), C.AdamWConsts(*k))
    torch.cuda.synchronize()
    for ts, want in zip((p, m, v), one):
        for t in ts:
            assert_bits((host_u16 if t.dtype == torch.bfloat16 else host_f32)(t[-1:]), want[0], "last element")
            assert int(t.min() == t.max()) == 1
    del p, m, v, g, ts, t
    torch.cuda.empty_cache()
