// norm.hip - the global gradient norm of R15 (the optimizer paragraph's clip to a global l2 norm of 1.0),
// the clip coefficient and spike decision (the section on gradient behaviour: a pre-clip norm above 5
// skips five optimizer steps), and the clip itself.
//
// The gradient tensors laid end to end in the declared order are one vector; its sum of squares is R1 over
// that vector's flat index (chunks of 32 may run across a tensor boundary).  Pass 1: one workgroup per
// aligned block of kNormBlockChunks chunks, i.e. one complete (or, for the last, left-filled) subtree of
// the padded tree; each wavefront reads 64 chunks at a time coalesced, squares on the way in, stages them
// in LDS transposed so that lane c runs chunk c's chain, and folds the lanes with the pass-through rule.
// Pass 2: one workgroup folds the block sums (Algorithm 2 over complete subtrees gives the same tree), takes
// the square root and makes the decisions.  HBM bound: 4 bytes read per gradient element.
#include <hip/hip_runtime.h>

#include "canon_dev.h"
#include "canon_internal.h"

namespace canon {

namespace {

constexpr int kWaveSegs = 4;                         // segments of 64 chunks per wavefront
constexpr int kWaveChunks = 64 * kWaveSegs;          // 256 chunks per wavefront
constexpr int kNormBlockChunks = 4 * kWaveChunks;    // 4 wavefronts: 1024 chunks (32768 terms) per workgroup
constexpr int kFinalWaves = 16;                      // wavefronts of the block-sum fold
constexpr int kSegTerms = 64 * kChunk;               // 2048 terms per segment
constexpr float kClipEps = 1e-6f;                    // RN32(1e-6), added to the norm before the division

struct Stage {
  float t[64][36];  // 16-byte stores and reads without bank conflicts
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

// A lane's position in the tensors: flat indexes below `end` lie in tensor `cur`, element j at base[j].  Held in
// registers, so that a load waits for the tables only where it enters another tensor (looked up for every load, the
// two dependent reads left the pass at 156 us for 110 M gradients in 51 tensors; 70 now).
struct TensorPos {
  const float* base;
  int64_t end;
  int cur;
};
__device__ __forceinline__ void enter_tensor(const NormSrc& src, int t, TensorPos& at) {
  at.cur = t;
  at.end = src.start[t + 1];
  at.base = src.ptr[t] - src.start[t];
}

// W consecutive terms starting at flat index j (W = 4: the host guarantees that a W-group never crosses a
// tensor boundary or the end, and that every tensor base is 16-byte aligned).
template <int W, bool MULTI>
__device__ __forceinline__ void load_terms(const NormSrc& src, int64_t n, int64_t j, TensorPos& at, float (&f)[W]) {
  if (j >= n) {
#pragma unroll
    for (int i = 0; i < W; ++i) f[i] = 0.0f;
    return;
  }
  if (MULTI)
    while (j >= at.end) enter_tensor(src, at.cur + 1, at);
  const float* p = at.base + j;
  if (W == 4) {
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  } else {
    f[0] = __builtin_nontemporal_load(p);
  }
}

// first tensor whose range holds flat index j (tensors of size 0 are skipped)
__device__ __forceinline__ int find_tensor(const NormSrc& src, int64_t j) {
  int lo = 0, hi = src.nt - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (src.start[mid] <= j) lo = mid; else hi = mid - 1;
  }
  while (lo < src.nt - 1 && src.start[lo + 1] <= j) ++lo;
  return lo;
}

template <int W, bool MULTI>
__global__ __launch_bounds__(256) void gnorm_block_kernel(int64_t n, NormSrc src, float* __restrict__ part) {
  constexpr int Q = kSegTerms / (64 * W);  // W-groups per lane per segment
  __shared__ __attribute__((aligned(16))) Stage st[4];
  __shared__ float wsum[4];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t nc = (n + kChunk - 1) / kChunk;
  const int64_t cw = (int64_t)blockIdx.x * kNormBlockChunks + (int64_t)w * kWaveChunks;  // wave's first chunk
  TensorPos cur{src.one, 0, 0};
  if (MULTI) enter_tensor(src, find_tensor(src, cw * kChunk + W * lane < n ? cw * kChunk + W * lane : n - 1), cur);
  // the wave's segments are consecutive complete subtrees of 64 chunks: a binary-carry fold over the real
  // ones gives the wave's subtree with the pass-through rule
  LocalFoldN<8> wf;
  float nxt[Q][W];
#pragma unroll
  for (int q = 0; q < Q; ++q) load_terms<W, MULTI>(src, n, cw * kChunk + 64 * W * q + W * lane, cur, nxt[q]);
#pragma unroll
  for (int sg = 0; sg < kWaveSegs; ++sg) {
    const int64_t c0 = cw + 64 * sg;
    if (c0 >= nc) break;
    float f[Q][W];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < W; ++i) f[q][i] = nxt[q][i];
    if (sg + 1 < kWaveSegs) {
#pragma unroll
      for (int q = 0; q < Q; ++q)
        load_terms<W, MULTI>(src, n, (c0 + 64) * kChunk + 64 * W * q + W * lane, cur, nxt[q]);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int local = 64 * W * q + W * lane;
      float* dst = &st[w].t[local >> 5][local & 31];
#pragma unroll
      for (int i = 0; i < W; ++i) f[q][i] = f[q][i] * f[q][i];
      if constexpr (W == 4) *reinterpret_cast<float4*>(dst) = make_float4(f[q][0], f[q][1], f[q][2], f[q][3]);
      else dst[0] = f[q][0];
    }
    __builtin_amdgcn_wave_barrier();  // a wavefront's LDS operations complete in order
    float p = 0.0f;
    const int64_t c = c0 + lane;
    if (c < nc) {
      const int k1 = (int)(n - c * kChunk < kChunk ? n - c * kChunk : kChunk);
      if (k1 == kChunk) {
#pragma unroll
        for (int i = 0; i < kChunk; i += 4) {
          const float4 x = *reinterpret_cast<const float4*>(&st[w].t[lane][i]);
          p = p + x.x; p = p + x.y; p = p + x.z; p = p + x.w;
        }
      } else {
        for (int i = 0; i < k1; ++i) p = p + st[w].t[lane][i];
      }
    }
    const int64_t real = nc - c0;
    const float seg = wave_fold(p, real > 64 ? 64 : (int)real);
    if (lane == 0) wf.push(seg);
    __builtin_amdgcn_wave_barrier();
  }
  if (lane == 0) wsum[w] = wf.result();
  __syncthreads();
  // the workgroup's four waves: pairs of complete subtrees, the right one passed over when it holds no real
  // chunk
  if (threadIdx.x == 0) {
    const int64_t cb = (int64_t)blockIdx.x * kNormBlockChunks;
    float a = wsum[0];
    if (cb + kWaveChunks < nc) a = a + wsum[1];
    if (cb + 2 * kWaveChunks < nc) {
      float b = wsum[2];
      if (cb + 3 * kWaveChunks < nc) b = b + wsum[3];
      a = a + b;
    }
    part[blockIdx.x] = a;
  }
}

// Fold of the block sums, square root, clip coefficient, spike counter.  bad (may be null): a set flag
// means the gradient is not valid (an out-of-range token): the norm is NaN, no update is applied and the
// spike counter is left alone.
__global__ __launch_bounds__(64 * kFinalWaves) void gnorm_final_kernel(
    int64_t nb, const float* __restrict__ part, float max_norm, float spike_norm, int32_t skip_steps,
    const int32_t* __restrict__ bad, float* norm_out, float* coef_out, int32_t* skip_state, int32_t* skip_flag,
    int32_t* skipped_out) {
  // wave w folds the aligned range [w R, (w + 1) R) of block sums, R a power of two >= 64: 64 consecutive
  // sums per read (coalesced) folded across the lanes, those 64-subtrees pushed into a binary-carry fold;
  // then the waves' subtrees are folded level by level with the pass-through rule
  __shared__ float wsum[kFinalWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int64_t R = 64;
  while (kFinalWaves * R < nb) R <<= 1;
  LocalFoldN<24> wf;
  const int64_t r0 = (int64_t)w * R, r1 = (r0 + R < nb) ? r0 + R : nb;
  constexpr int kBatch = 16;
  for (int64_t b = r0; b < r1; b += 64 * kBatch) {
    float v[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int64_t j = b + 64 * i + lane;
      v[i] = j < r1 ? part[j] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int64_t s0 = b + 64 * i;
      if (s0 < r1) {
        const float t = wave_fold(v[i], (int)(r1 - s0 < 64 ? r1 - s0 : 64));
        if (lane == 0) wf.push(t);
      }
    }
  }
  if (lane == 0) wsum[w] = wf.result();
  __syncthreads();
  if (threadIdx.x != 0) return;
  float v[kFinalWaves];
#pragma unroll
  for (int q = 0; q < kFinalWaves; ++q) v[q] = wsum[q];
#pragma unroll
  for (int d = 1; d < kFinalWaves; d <<= 1)
#pragma unroll
    for (int q = 0; q + d < kFinalWaves; q += 2 * d)
      if ((q + d) * R < nb) v[q] = v[q] + v[q + d];
  const float q = v[0];
  float norm = __builtin_sqrtf(q);
  float coef;
  int32_t skip;
  if (bad && *bad) {
    norm = __builtin_nanf("");
    coef = 1.0f;
    skip = 1;
  } else {
    const float den = norm + kClipEps;
    coef = max_norm / den;
    int32_t left = skip_state ? *skip_state : 0;
    if (skip_steps > 0 && !(norm <= spike_norm)) left = skip_steps;
    skip = left > 0;
    if (skip) left -= 1;
    if (skip_state) *skip_state = left;
  }
  if (norm_out) *norm_out = norm;
  *coef_out = coef;
  if (skip_flag) *skip_flag = skip;
  if (skipped_out) *skipped_out = skip;
}

// g <- RN(g * coef) when coef < 1: up to kBatchTensors tensors per launch, kClipBlock elements of one tensor per
// unit of work, any alignment.  110 M elements in 51 tensors, norm and clip: 379 us as a launch per tensor, 200 in one.
// The grid is bounded because every workgroup that finds no clip to do still has to start: 1.28e9 elements in one
// tensor, norm and idle clip 888 us with a workgroup per unit, 828 with kClipGrid; a clip that acts 2650 and 2708
// (16384 workgroups: 818 and 2801).
constexpr int kClipBlock = 4096;
constexpr int64_t kClipUnits = 0x7FFFFFFF;  // per launch: 32-bit counts with room for one stride past the last
constexpr uint32_t kClipGrid = 65536;       // workgroups, which walk the units with the grid as their stride
struct ClipTable {
  float* g[kBatchTensors];
  int64_t n[kBatchTensors];
  uint32_t start[kBatchTensors];
};
struct __attribute__((packed, aligned(4))) ClipF4 {
  float f[4];
};
__global__ __launch_bounds__(kBatchThreads) void clip_scale_kernel(ClipTable tab, uint32_t units,
                                                                   const float* __restrict__ coef) {
  const float c = *coef;
  if (!(c < 1.0f)) return;
  for (uint32_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
    const int t = batch_tensor(tab.start, unit);
    float* __restrict__ g = tab.g[t];
    const int64_t n = tab.n[t], i0 = (int64_t)(unit - tab.start[t]) * kClipBlock + 4 * threadIdx.x;
    if (i0 + kClipBlock - 1024 + 4 <= n) {  // all four vectors: loads in flight before the stores
      ClipF4 x[kClipBlock / 1024];
#pragma unroll
      for (int q = 0; q < kClipBlock / 1024; ++q) x[q] = *reinterpret_cast<const ClipF4*>(g + i0 + 1024 * q);
#pragma unroll
      for (int q = 0; q < kClipBlock / 1024; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[q].f[e] = x[q].f[e] * c;
        *reinterpret_cast<ClipF4*>(g + i0 + 1024 * q) = x[q];
      }
    } else {
      for (int q = 0; q < kClipBlock / 1024; ++q)
        for (int64_t j = i0 + 1024 * q; j < i0 + 1024 * q + 4 && j < n; ++j) g[j] = g[j] * c;
    }
  }
}

struct NormTable {
  const float* ptr[kBatchTensors];
  int64_t start[kBatchTensors];
};
__global__ __launch_bounds__(64) void norm_tables_kernel(NormTable tab, int ptrs, int starts,
                                                         const float** __restrict__ ptr_d,
                                                         int64_t* __restrict__ start_d) {
  const int l = threadIdx.x;
  if (l < ptrs) ptr_d[l] = tab.ptr[l];
  if (l < starts) start_d[l] = tab.start[l];
}

}  // namespace

int64_t gnorm_blocks(int64_t n) {
  const int64_t nc = (n + kChunk - 1) / kChunk;
  return (nc + kNormBlockChunks - 1) / kNormBlockChunks;
}

hipError_t gnorm_launch(const NormSrc& src, int64_t n, int vec4, float* part, const ClipDecision& d, hipStream_t s) {
  const int64_t nb = gnorm_blocks(n);
  if (nb > 0x7fffffff) return hipErrorInvalidValue;
  if (nb > 0) {
    const dim3 grid((unsigned)nb), block(256);
    if (src.nt == 0 || src.one) {
      if (vec4) hipLaunchKernelGGL((gnorm_block_kernel<4, false>), grid, block, 0, s, n, src, part);
      else hipLaunchKernelGGL((gnorm_block_kernel<1, false>), grid, block, 0, s, n, src, part);
    } else {
      if (vec4) hipLaunchKernelGGL((gnorm_block_kernel<4, true>), grid, block, 0, s, n, src, part);
      else hipLaunchKernelGGL((gnorm_block_kernel<1, true>), grid, block, 0, s, n, src, part);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(gnorm_final_kernel, dim3(1), dim3(64 * kFinalWaves), 0, s, nb, part, d.max_norm, d.spike_norm, d.skip_steps,
                     d.bad, d.norm_out, d.coef_out, d.skip_state, d.skip_flag, d.skipped_out);
  return hipGetLastError();
}

hipError_t norm_tables_launch(int64_t nt, const int64_t* sizes, float* const* grads, const float** ptr_d,
                              int64_t* start_d, hipStream_t s) {
  int64_t at = 0;
  for (int64_t t0 = 0; t0 <= nt; t0 += kBatchTensors) {  // entry nt: the end of the last tensor
    NormTable tab{};
    const int starts = (int)(nt + 1 - t0 < kBatchTensors ? nt + 1 - t0 : kBatchTensors);
    const int ptrs = (int)(nt - t0 < starts ? nt - t0 : starts);
    for (int j = 0; j < starts; ++j) {
      tab.start[j] = at;
      if (j < ptrs) {
        tab.ptr[j] = grads[t0 + j];
        at += sizes[t0 + j];
      }
    }
    hipLaunchKernelGGL(norm_tables_kernel, dim3(1), dim3(64), 0, s, tab, ptrs, starts, ptr_d + t0, start_d + t0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t clip_scale_launch(int64_t nt, const int64_t* sizes, float* const* g, const float* coef, hipStream_t s) {
  ClipTable tab;
  return for_tensor_batches(
      nt, sizes, kClipBlock, kClipUnits, kClipUnits * kClipBlock, tab.start,
      [&](int64_t t, auto f) { f(g[t], 4 * sizes[t]); },
      [&](int j, int64_t t) {
        tab.g[j] = g[t];
        tab.n[j] = sizes[t];
      },
      [&](int, uint32_t units) {
        hipLaunchKernelGGL(clip_scale_kernel, dim3(units < kClipGrid ? units : kClipGrid), dim3(kBatchThreads), 0, s,
                           tab, units, coef);
        return hipGetLastError();
      },
      [](int64_t) { return hipErrorInvalidValue; });  // (2^43 elements, beyond the entry points' 2^40)
}

}  // namespace canon
