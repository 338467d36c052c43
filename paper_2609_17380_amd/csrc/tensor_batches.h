// tensor_batches.h - a list of tensors cut into launches (host side only, no HIP types).
#pragma once
#include <stdint.h>

namespace canon {

// Kernels over a list of tensors take up to kBatchTensors of them per launch, as a table in the kernel arguments
// (4 KiB at most).  Empty tensors are left out; a tensor owns ceil(size / unit) consecutive units of work, start[j]
// being the first of entry j (unused entries 0xFFFFFFFF).
constexpr int kBatchTensors = 64;
// A launch takes fewer than 2^32 threads, so at 256 per workgroup its grid ends here.
constexpr uint32_t kBatchThreads = 256;
constexpr uint32_t kGridMax = 0xFFFFFFFFu / kBatchThreads;

// The buffers of one launch, sorted; a list may name a buffer twice (it is then updated twice, in order), so a tensor
// that touches one of these starts the next launch.
struct BufferSet {
  uintptr_t lo[4 * kBatchTensors], hi[4 * kBatchTensors];
  int n = 0;
  // where [a, b) would stand, or -1 when it overlaps a buffer of the set
  int place(uintptr_t a, uintptr_t b) const {
    int i = n;
    while (i > 0 && lo[i - 1] >= a) --i;
    return (i > 0 && hi[i - 1] > a) || (i < n && lo[i] < b) ? -1 : i;
  }
  bool add(const void* p, int64_t bytes) {  // false: overlaps a buffer of the set (not added)
    const uintptr_t a = (uintptr_t)p, b = a + (uintptr_t)bytes;
    const int i = place(a, b);
    if (i < 0) return false;
    for (int k = n; k > i; --k) {
      lo[k] = lo[k - 1];
      hi[k] = hi[k - 1];
    }
    lo[i] = a;
    hi[i] = b;
    ++n;
    return true;
  }
};

// buffers(t, f): f(pointer, bytes) for each buffer of tensor t (at most 4).  put(j, t) enters t into entry j of the
// table, run(j, units) launches the j entries with so many units in all, at most max_units.  Tensors of at least
// `large` elements, and these must include every one of more than max_units units, are launched by themselves, at
// once, by alone(t): the entries that wait touch none of their buffers.  The first failing status (0 is success)
// ends the list and is returned.
template <class Buffers, class Put, class Run, class Alone>
auto for_tensor_batches(int64_t nt, const int64_t* sizes, int64_t unit, int64_t max_units, int64_t large,
                        uint32_t (&start)[kBatchTensors], Buffers buffers, Put put, Run run, Alone alone)
    -> decltype(alone(0)) {
  typedef decltype(alone(0)) Status;
  BufferSet used;
  int j = 0;
  int64_t units = 0;
  auto flush = [&]() {
    for (int i = j; i < kBatchTensors; ++i) start[i] = 0xFFFFFFFFu;
    const Status e = j > 0 ? run(j, (uint32_t)units) : Status(0);
    j = 0;
    units = 0;
    used.n = 0;
    return e;
  };
  for (int64_t t = 0; t < nt; ++t) {
    if (sizes[t] == 0) continue;
    const bool one = sizes[t] >= large;
    const int64_t b = (sizes[t] + unit - 1) / unit;
    bool apart = true;  // from the buffers of the entries that wait
    buffers(t, [&](const void* p, int64_t bytes) {
      apart = apart && used.place((uintptr_t)p, (uintptr_t)p + (uintptr_t)bytes) >= 0;
    });
    if (!apart || (!one && j > 0 && (j == kBatchTensors || units + b > max_units))) {
      const Status e = flush();
      if (e != Status(0)) return e;
    }
    if (one) {
      const Status e = alone(t);
      if (e != Status(0)) return e;
      continue;
    }
    bool whole = true;  // false: its own buffers overlap, so the set does not hold them all
    buffers(t, [&](const void* p, int64_t bytes) { whole = used.add(p, bytes) && whole; });
    start[j] = (uint32_t)units;
    put(j, t);
    units += b;
    ++j;
    if (!whole) {
      const Status e = flush();
      if (e != Status(0)) return e;
    }
  }
  return flush();
}

}  // namespace canon
