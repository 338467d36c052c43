// lsq.hip - the gradient of a learned per-tensor activation step of the int8 projections (R19: the paper's
// int8 quantisation-aware training with learned step-size quantisation for activations).
//
// g_s = RN(R1 over the flat index of RN(dx * delta) * gamma), gamma = RN32(1/sqrt(127 K)) (LSQ's gradient
// scale for K features, computed by the caller), where for each element with v = RN(x / s): delta = -128 below
// the integer range, 127 above it, RN(rne(v) - v) inside; 0 when the step is not > 0 once flushed or v is NaN.
// Pass 1: one workgroup per aligned block of 1024 chunks (a complete subtree of the padded tree); each
// wavefront forms 64 chunks of terms at a time from coalesced loads (any alignment), stages them transposed in LDS so that
// lane c runs chunk c's chain, and folds the lanes with the pass-through rule.  Pass 2: one workgroup folds
// the block sums (each thread a complete subtree of consecutive sums, then across threads) and scales.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "canon_dev.h"
#include "canon_internal.h"

namespace canon {

namespace {

constexpr int kWaves = 8;                       // wavefronts of a workgroup
constexpr int kSegs = 2;                        // segments of 64 chunks per wavefront
constexpr int kWaveChunks = 64 * kSegs;         // 128 chunks per wavefront
constexpr int kBlockChunks = kWaves * kWaveChunks;  // 1024 chunks (32768 terms) per workgroup
constexpr int kSegTerms = 64 * kChunk;          // 2048 terms per segment

struct Stage {
  float t[64][36];  // 16-byte stores and reads without bank conflicts
};
struct __attribute__((packed, aligned(4))) Dx4 {
  float f[4];
};
struct __attribute__((packed, aligned(2))) X4 {
  uint32_t w[2];
};

__device__ __forceinline__ float lsq_delta(float x, float s, bool valid) {
  if (!valid) return 0.0f;
  const float v = x / s;  // correctly rounded
  if (!(v == v)) return 0.0f;
  if (v < -128.0f) return -128.0f;
  if (v > 127.0f) return 127.0f;
  return __builtin_rintf(v) - v;  // exact: |rne(v) - v| <= 1/2 (Sterbenz)
}

// Workgroup: 1024 chunks over 8 wavefronts, two segments each, the second one's 24 bytes per term group requested
// before the first one's divisions.  Bound: vector instructions (the correctly rounded quotient) beside 6 bytes per
// term: 8192 x 2048 terms 30 us (4 wavefronts of four segments, loads one group at a time: 49).  The last segment stops
// at its last group: 256 terms 4.7 us (8.5 with every group formed and loaded by element).
__global__ __launch_bounds__(64 * kWaves) void lsq_block_kernel(int64_t n, const uint16_t* __restrict__ x,
                                                                const float* __restrict__ dx,
                                                                const float* __restrict__ sp,
                                                                float* __restrict__ part) {
  constexpr int Q = kSegTerms / (64 * 4);  // 4-term groups per lane per segment
  __shared__ __attribute__((aligned(16))) Stage st[kWaves];
  __shared__ float wsum[kWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float s = step_daz(*sp);
  const bool valid = s > 0.0f;
  const int64_t nc = (n + kChunk - 1) / kChunk;
  const int64_t cw = (int64_t)blockIdx.x * kBlockChunks + (int64_t)w * kWaveChunks;  // wave's first chunk
  Dx4 g[kSegs][Q];
  X4 h[kSegs][Q];
  auto load = [&](int sg) __attribute__((always_inline)) {
    const int64_t j0 = (cw + 64 * sg) * kChunk;
    if (j0 + kSegTerms <= n) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        g[sg][q] = *reinterpret_cast<const Dx4*>(dx + j0 + 256 * q + 4 * lane);
        h[sg][q] = *reinterpret_cast<const X4*>(x + j0 + 256 * q + 4 * lane);
      }
    } else {  // the last segment: groups inside it whole, the last one element by element, +0 beyond the end
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (j0 + 256 * q >= n) break;
        const int64_t j = j0 + 256 * q + 4 * lane;
        g[sg][q] = Dx4{{0.0f, 0.0f, 0.0f, 0.0f}};
        h[sg][q].w[0] = h[sg][q].w[1] = 0;
        if (j + 4 <= n) {
          g[sg][q] = *reinterpret_cast<const Dx4*>(dx + j);
          h[sg][q] = *reinterpret_cast<const X4*>(x + j);
        } else if (j < n) {
#pragma unroll
          for (int i = 0; i < 3; ++i)
            if (j + i < n) {
              g[sg][q].f[i] = dx[j + i];
              h[sg][q].w[i >> 1] |= (uint32_t)x[j + i] << (16 * (i & 1));
            }
        }
      }
    }
  };
  load(0);
  float tot = 0.0f;
#pragma unroll
  for (int sg = 0; sg < kSegs; ++sg) {
    const int64_t c0 = cw + 64 * sg;
    if (c0 >= nc) break;
    if (sg + 1 < kSegs && c0 + 64 < nc) load(sg + 1);
    auto stage = [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int local = 256 * q + 4 * lane;
        if (!whole.value && c0 * kChunk + 256 * q >= n) break;  // no chunk reads these terms
        float t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t b = h[sg][q].w[i >> 1];
          t[i] = g[sg][q].f[i] * lsq_delta(__uint_as_float((i & 1) ? b & 0xFFFF0000u : b << 16), s, valid);
        }
        *reinterpret_cast<float4*>(&st[w].t[local >> 5][local & 31]) = make_float4(t[0], t[1], t[2], t[3]);
      }
    };
    if (c0 * kChunk + kSegTerms <= n) stage(std::true_type{});
    else stage(std::false_type{});
    __builtin_amdgcn_wave_barrier();  // a wavefront's LDS operations complete in order
    float p = 0.0f;
    const int64_t k1 = n - (c0 + lane) * kChunk;
    if (k1 >= kChunk) {
#pragma unroll
      for (int i = 0; i < kChunk; i += 4) {
        const float4 v = *reinterpret_cast<const float4*>(&st[w].t[lane][i]);
        p = p + v.x; p = p + v.y; p = p + v.z; p = p + v.w;
      }
    } else {
      for (int i = 0; i < (int)k1; ++i) p = p + st[w].t[lane][i];
    }
    const int64_t real = nc - c0;
    const float seg = wave_fold(p, real > 64 ? 64 : (int)real);
    tot = sg == 0 ? seg : tot + seg;
    __builtin_amdgcn_wave_barrier();
  }
  if (lane == 0) wsum[w] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {  // the waves' complete subtrees, a right one without real chunks passed over
    const int64_t cb = (int64_t)blockIdx.x * kBlockChunks;
    float v[kWaves];
#pragma unroll
    for (int q = 0; q < kWaves; ++q) v[q] = wsum[q];
#pragma unroll
    for (int d = 1; d < kWaves; d <<= 1)
#pragma unroll
      for (int q = 0; q + d < kWaves; q += 2 * d)
        if (cb + (q + d) * kWaveChunks < nc) v[q] = v[q] + v[q + d];
    part[blockIdx.x] = v[0];
  }
}

// Algorithm 2 over the block sums: thread t folds the aligned run [t G, t G + G) of consecutive sums (a
// complete subtree, G a power of two), then the threads fold with the pass-through rule; times gamma.
__global__ __launch_bounds__(256) void lsq_final_kernel(int64_t nparts, const float* __restrict__ part, float gamma,
                                                        float* __restrict__ out) {
  const int64_t G = block_chunks(nparts, 256);
  const int64_t b0 = (int64_t)threadIdx.x * G;
  LocalFoldN<16> f;
  for (int64_t i = b0; i < b0 + G && i < nparts; ++i) f.push(part[i]);
  const float p = f.result();
  const int64_t nthr = (nparts + G - 1) / G;
  const float total = block_fold(p, nthr);
  if (threadIdx.x == 0) out[0] = total * gamma;
}

}  // namespace

int64_t lsq_grad_parts(int64_t n) { return (n + (int64_t)kBlockChunks * kChunk - 1) / ((int64_t)kBlockChunks * kChunk); }

// ---- the allocation-free variant: the block sums live in a file-scope device array ----
// One copy per GPU, held until the process ends.  Host code never uses the array's name as an address:
// the device address of each GPU's copy comes from hipGetSymbolAddress with that GPU current.
constexpr int64_t kScratchParts = 65536;  // 256 KiB: block sums of up to 2^31 terms
static __device__ __align__(256) float scratch[kScratchParts];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static float* g_scratch_dev[kMaxDevices];  // device address of the current GPU's copy, set on first use

int64_t lsq_noalloc_max_terms() { return kScratchParts * (int64_t)kBlockChunks * kChunk; }

hipError_t lsq_scratch(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) return e != hipSuccess ? e : hipErrorInvalidSymbol;
    g_scratch_dev[dev] = static_cast<float*>(ptr);
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}

hipError_t lsq_grad_launch(int64_t n, const uint16_t* x, const float* s, const float* dx, float gamma, float* part,
                           float* out, hipStream_t st) {
  const int64_t nparts = lsq_grad_parts(n);
  if (nparts == 0) {
    hipLaunchKernelGGL(lsq_final_kernel, dim3(1), dim3(256), 0, st, (int64_t)0, part, gamma, out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(lsq_block_kernel, dim3((unsigned)nparts), dim3(64 * kWaves), 0, st, n, x, dx, s, part);
  hipLaunchKernelGGL(lsq_final_kernel, dim3(1), dim3(256), 0, st, nparts, part, gamma, out);
  return hipGetLastError();
}

}  // namespace canon
