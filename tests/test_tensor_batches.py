"""Lists of tensors cut into launches (csrc/tensor_batches.h, host code without HIP types): a program built here runs the
cutting on sizes that no memory holds, with the limits of AdamW (a workgroup per 512 elements, at most 2^32 - 1 threads
of 256 per workgroup) and of the clip (units of 4096 walked by a bounded grid)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_17380_amd", "csrc")

# stdin: unit, max_units, large, count, then per tensor its address (four buffers of one element per unit address space)
# and size; stdout: one line per launch, "run units t:start ..." or "alone t"
PROGRAM = r"""
#include <cstdio>
#include <cinttypes>
#include <vector>
#include "tensor_batches.h"
using namespace canon;
int main() {
  int64_t unit, max_units, large, nt;
  if (scanf("%" SCNd64 "%" SCNd64 "%" SCNd64 "%" SCNd64, &unit, &max_units, &large, &nt) != 4) return 1;
  std::vector<int64_t> at(nt), size(nt);
  for (int64_t t = 0; t < nt; ++t)
    if (scanf("%" SCNd64 "%" SCNd64, &at[t], &size[t]) != 2) return 1;
  if (max_units < 0) max_units = kGridMax;
  uint32_t start[kBatchTensors];
  int64_t entry[kBatchTensors];
  return for_tensor_batches(
      nt, size.data(), unit, max_units, large, start, [&](int64_t t, auto f) { f((const void*)at[t], 4 * size[t]); },
      [&](int j, int64_t t) { entry[j] = t; },
      [&](int n, uint32_t units) {
        printf("run %u", units);
        for (int j = 0; j < n; ++j) printf(" %" PRId64 ":%u", entry[j], start[j]);
        for (int j = n; j < kBatchTensors; ++j)
          if (start[j] != 0xFFFFFFFFu) printf(" bad");
        printf("\n");
        return 0;
      },
      [&](int64_t t) { printf("alone %" PRId64 "\n", t); return 0; });
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    d = tmp_path_factory.mktemp("batches")
    (d / "cut.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(d / "cut.cpp"), "-o", str(d / "cut")])

    def run(unit, max_units, large, tensors):
        text = f"{unit} {max_units} {large} {len(tensors)}\n" + "\n".join(f"{a} {n}" for a, n in tensors)
        out = subprocess.run([str(d / "cut")], input=text, capture_output=True, text=True, check=True).stdout
        launches = []
        for line in out.splitlines():
            w = line.split()
            launches.append(("alone", int(w[1])) if w[0] == "alone" else
                            ("run", int(w[1]), [tuple(int(x) for x in e.split(":")) for e in w[2:]]))
        return launches

    return run


def apart(sizes):
    at, out = 1 << 20, []
    for n in sizes:
        out.append((at, n))
        at += 4 * n + 64
    return out


GRID = (2**32 - 1) // 256


@pytest.mark.parametrize("unit,large", [(512, GRID * 512 + 1), (512, 1 << 25)])
@pytest.mark.parametrize("sizes", [
    [1 << 28] * 40,                                  # 1.07e10 elements in all: more workgroups than one launch takes
    [GRID * 512], [GRID * 512 + 1], [(1 << 34) + 5],  # one tensor on either side of the limit
    [1000, (1 << 34) + 5, 7, GRID * 512, 3],
    [33000000] * 300,
])
def test_grids_stay_below_2_to_32_threads(cut, unit, large, sizes):
    seen = []
    for launch in cut(unit, -1, large, apart(sizes)):
        if launch[0] == "alone":
            assert sizes[launch[1]] >= large
            seen.append(launch[1])
            continue
        _, units, entries = launch
        assert 256 * units < 2**32 and len(entries) <= 64
        at = 0
        for t, start in entries:
            assert start == at
            at += -(-sizes[t] // unit)
            seen.append(t)
        assert at == units
    assert sorted(seen) == list(range(len(sizes)))  # each once


def test_overlapping_tensors_keep_their_order(cut):
    a, b, big = (1 << 20, 100), (1 << 21, 100), (1 << 22, 1 << 26)
    inside = (big[0] + 400, 50)  # part of the large one
    got = cut(512, -1, 1 << 25, [a, b, a, big, inside, big, b, (1 << 30, 0)])
    # the second a waits for the first; the large one touches no entry that waits; what overlaps it waits for it
    order = [t for x in got for t in ([x[1]] if x[0] == "alone" else [e[0] for e in x[2]])]
    assert sorted(order) == [0, 1, 2, 3, 4, 5, 6]
    assert order.index(0) < order.index(2) and order.index(3) < order.index(4) < order.index(5)
    assert order.index(1) < order.index(6)
    for x in got:  # no two entries of a launch overlap
        if x[0] == "run":
            assert len({e[0] for e in x[2]} & {0, 2}) < 2 and len({e[0] for e in x[2]} & {1, 6}) < 2


def test_units_of_the_clip_fit_32_bits(cut):
    # 2^40 elements, the most an entry point takes: units of 4096 in 32 bits, with room for a stride past the last
    got = cut(4096, 2**31 - 1, (2**31 - 1) * 4096, apart([1 << 40]))
    assert got == [("run", 1 << 28, [(0, 0)])]
    got = cut(4096, 2**31 - 1, (2**31 - 1) * 4096, apart([1 << 36] * 130))
    assert sum(x[1] for x in got) == 130 * 2**24 and all(x[1] + GRID < 2**32 for x in got)
