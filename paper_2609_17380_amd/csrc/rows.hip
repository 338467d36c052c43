// rows.hip - row-wise canonical reductions: RMSNorm (R3), causal softmax (R5), cross-entropy (R6) and the
// row pieces of the attention backward.
//
// Layout of every row reduction: the row's chunks of 32 are split into aligned power-of-two blocks of G
// chunks, one block per lane (or thread).  Each lane folds its block with a register binary-carry stack
// (a complete or left-filled subtree of the padded tree), then the lanes are folded across the wavefront or
// workgroup with the pass-through rule, which together give Algorithm 2 over the row's chunks.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "canon_dev.h"
#include "canon_internal.h"

namespace canon {

__device__ __forceinline__ float wave_max(float m) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) m = fmaxf(m, __shfl_xor(m, s, 64));
  return m;
}

// ---- W-wide loads and stores (W = 1 or 4 consecutive elements at any element alignment: gfx950's global accesses
// need none) ----
struct __attribute__((packed, aligned(4))) F4 {
  float x, y, z, w;
};
struct __attribute__((packed, aligned(2))) H4 {
  uint32_t x, y;
};
template <int W>
__device__ __forceinline__ void ldf(const float* p, float (&f)[W]) {
  if constexpr (W == 1) {
    f[0] = p[0];
  } else {
#pragma unroll
    for (int i = 0; i < W; i += 4) {
      const F4 v = *reinterpret_cast<const F4*>(p + i);
      f[i] = v.x; f[i + 1] = v.y; f[i + 2] = v.z; f[i + 3] = v.w;
    }
  }
}

template <int W>
__device__ __forceinline__ void ldb(const uint16_t* p, float (&f)[W]) {
  if constexpr (W == 1) {
    f[0] = bf16_to_f32(p[0]);
  } else {
    const H4 u = *reinterpret_cast<const H4*>(p);
    f[0] = bf16_to_f32((uint16_t)(u.x & 0xFFFFu)); f[1] = bf16_to_f32((uint16_t)(u.x >> 16));
    f[2] = bf16_to_f32((uint16_t)(u.y & 0xFFFFu)); f[3] = bf16_to_f32((uint16_t)(u.y >> 16));
  }
}

template <int W>
__device__ __forceinline__ void stb(uint16_t* p, const uint16_t (&h)[W]) {
  if constexpr (W == 1) {
    p[0] = h[0];
  } else {
    *reinterpret_cast<H4*>(p) = H4{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
  }
}

template <int W>
__device__ __forceinline__ void stf(float* p, const float (&f)[W]) {
  if constexpr (W == 1) {
    p[0] = f[0];
  } else {
#pragma unroll
    for (int i = 0; i < W; i += 4) *reinterpret_cast<F4*>(p + i) = F4{f[i], f[i + 1], f[i + 2], f[i + 3]};
  }
}

// four elements j .. j + 3 of a row of n, those beyond its end as 0 (not read) or not written
// (TAIL: n is not a multiple of 4)
template <bool TAIL>
__device__ __forceinline__ void ldf4(const float* row, int64_t j, int64_t n, float (&f)[4]) {
  if (!TAIL || j + 4 <= n) {
    ldf<4>(row + j, f);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = j + i < n ? row[j + i] : 0.0f;
  }
}
template <bool TAIL>
__device__ __forceinline__ void ldb4(const uint16_t* row, int64_t j, int64_t n, float (&f)[4]) {
  if (!TAIL || j + 4 <= n) {
    ldb<4>(row + j, f);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = j + i < n ? bf16_to_f32(row[j + i]) : 0.0f;
  }
}
template <bool TAIL>
__device__ __forceinline__ void stf4(float* row, int64_t j, int64_t n, const float (&f)[4]) {
  if (!TAIL || j + 4 <= n) {
    stf<4>(row + j, f);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (j + i < n) row[j + i] = f[i];
  }
}
template <bool TAIL>
__device__ __forceinline__ void stb4(uint16_t* row, int64_t j, int64_t n, const uint16_t (&h)[4]) {
  if (!TAIL || j + 4 <= n) {
    stb<4>(row + j, h);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (j + i < n) row[j + i] = h[i];
  }
}

// ------------------------------------------------------------------------------------------------
// Coalesced row reduction for one wavefront.  A segment of 64 chunks (2048 terms) is read coalesced (lane l
// takes terms 64W q + W l .. + W-1), staged in LDS as padded rows [chunk][33], and lane c then runs chunk
// c's chain sequentially from LDS; the chunk partials of all segments collect in `parts` and are folded by
// lane blocks + wave_fold (Algorithm 2).  term(j, f) evaluates terms j .. j+W-1 of the row into f; it is called for
// j < n only, and reads nothing at or past n itself (rows of any length: the last vector may be partial, and the chain
// stops at n whatever f holds there).
struct WaveStage {
  float t[64][33];
};

template <int W, class Term>
__device__ __forceinline__ void wave_segment_chunks(int64_t seg0, int64_t n, WaveStage& st, float* parts, Term term) {
  const int lane = threadIdx.x & 63;
  const int64_t nc = (n + kChunk - 1) / kChunk;
#pragma unroll 2
  for (int q = 0; q < 64 * kChunk / (64 * W); ++q) {
    const int local = 64 * W * q + W * lane;
    const int64_t j = seg0 + local;
    float f[W];
    if (j < n) {
      term(j, f);
    } else {
#pragma unroll
      for (int i = 0; i < W; ++i) f[i] = 0.0f;
    }
    float* dst = &st.t[local >> 5][local & 31];
#pragma unroll
    for (int i = 0; i < W; ++i) dst[i] = f[i];
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
  const int64_t c = seg0 / kChunk + lane;
  if (c < nc) {
    const int64_t k1 = n - c * kChunk < kChunk ? n - c * kChunk : kChunk;
    float s = 0.0f;
    for (int i = 0; i < (int)k1; ++i) s = s + st.t[lane][i];
    parts[c] = s;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
}

// nz: terms at index >= nz are known to be +0 (masked); z0: so are the terms below z0.  Chunks made only of
// such terms have partial +0: those at or after nz, and those of whole staging segments below z0, are not
// staged.
// Algorithm 2 over the nc chunk partials of one row in parts[] (written and made visible by the caller):
// lane l folds the block of G consecutive partials it owns, then the lane results are folded across the
// wavefront.  Returns the row sum in every lane.
__device__ __forceinline__ float fold_parts(const float* parts, int64_t nc) {
  const int lane = threadIdx.x & 63;
  const int64_t G = block_chunks(nc, 64);
  const int64_t c0 = lane * G, c1 = (c0 + G < nc) ? c0 + G : nc;
  LocalFold f;
  for (int64_t c = c0; c < c1; ++c) f.push(parts[c]);
  float tot = wave_fold(f.result(), (int)((nc + G - 1) / G));
  return __shfl(tot, 0, 64);
}

template <int W, class Term>
__device__ __forceinline__ float wave_row_rsum(int64_t n, WaveStage& st, float* parts, Term term, int64_t nz,
                                               int64_t z0 = 0) {
  const int lane = threadIdx.x & 63;
  const int64_t nc = (n + kChunk - 1) / kChunk;
  const int64_t zseg = (z0 / (64 * kChunk)) * (64 * kChunk);
  for (int64_t c = lane; c < zseg / kChunk && c < nc; c += 64) parts[c] = 0.0f;
  for (int64_t seg0 = zseg; seg0 < n && seg0 < nz; seg0 += 64 * kChunk) wave_segment_chunks<W>(seg0, n, st, parts, term);
  for (int64_t c = (nz + kChunk - 1) / kChunk + lane; c < nc; c += 64) parts[c] = 0.0f;
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
  return fold_parts(parts, nc);
}

constexpr int kMaxRowChunks = 64 * 16;  // rows up to 32768 terms in the wave kernels

// The wave kernels take 4 rows per workgroup, with parts[] as dynamic LDS of 4 x (chunks per row) floats.
static inline size_t wave_kernel_lds(int64_t cols) { return sizeof(float) * 4 * (size_t)((cols + kChunk - 1) / kChunk); }

// Register-resident rows (cols <= 2048, or the part H of 2048 terms of a longer one): lane l holds terms
// 4l + 256q .. +3 of its row, read from memory once.  The chunk chains still run one per lane over an LDS transpose
// (rows of 36 floats: 16-byte stores and reads without bank conflicts; a wavefront's LDS operations complete in order).
constexpr int kRegQ = 8;  // 64 x 4 x 8 = 2048 terms
constexpr int64_t kRegCols = 64 * 4 * kRegQ;
struct RegStage {
  float t[64][36];
};

template <int H = 0, int Q>
__device__ __forceinline__ float reg_row_sum(RegStage& st, const float (&e)[Q][4], int64_t n) {
  const int lane = threadIdx.x & 63;
  auto stage = [&](int q) __attribute__((always_inline)) {
    const int local = 256 * q + 4 * lane;
    const float(&v)[4] = e[H * kRegQ + q];
    *reinterpret_cast<float4*>(&st.t[local >> 5][local & 31]) = make_float4(v[0], v[1], v[2], v[3]);
  };
  // short rows leave out the vectors past their end (norm forward of 20000 rows of 16 terms 11.2 -> 9.9 us); with the
  // test in front of every vector the softmax of 2048 keys took 66 us instead of 59
  if (n > 256 * (kRegQ - 1)) {
#pragma unroll
    for (int q = 0; q < kRegQ; ++q) stage(q);
  } else {
#pragma unroll
    for (int q = 0; q < kRegQ - 1; ++q) {
      if (256 * q >= n) break;
      stage(q);
    }
  }
  __builtin_amdgcn_wave_barrier();
  const int nc = (int)((n + kChunk - 1) / kChunk);
  float p = 0.0f;
  const int k1 = (int)n - lane * kChunk;
  if (k1 >= kChunk) {
#pragma unroll
    for (int i = 0; i < kChunk; i += 4) {
      const float4 v = *reinterpret_cast<const float4*>(&st.t[lane][i]);
      p = p + v.x; p = p + v.y; p = p + v.z; p = p + v.w;
    }
  } else {
    for (int i = 0; i < k1; ++i) p = p + st.t[lane][i];
  }
  return __shfl(wave_fold(p, nc), 0, 64);
}

// RMSNorm forward: one wavefront per row, 4 rows per workgroup.
template <bool TAIL, bool F32>
__global__ __launch_bounds__(256) void rownorm_fwd_kernel(int64_t rows, int64_t cols, const float* __restrict__ x,
                                                          const uint16_t* __restrict__ gain, float eps, float inv_d,
                                                          void* __restrict__ y, float* __restrict__ rstd) {
  __shared__ WaveStage st[4];
  extern __shared__ float dyn[];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= rows) return;
  const int64_t nc = (cols + kChunk - 1) / kChunk;
  const float* xr = x + row * cols;
  float ss = wave_row_rsum<4>(cols, st[w], dyn + w * nc, [&](int64_t j, float (&f)[4]) {
    ldf4<TAIL>(xr, j, cols, f);
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = f[i] * f[i];
  }, cols);
  float ms = ss * inv_d;
  float var = ms + eps;
  float r = 1.0f / __builtin_sqrtf(var);
  if (lane == 0) rstd[row] = r;
  for (int64_t k = (int64_t)lane * 4; k < cols; k += 64 * 4) {
    float xv[4], gv[4];
    uint16_t h[4];
    ldf4<TAIL>(xr, k, cols, xv);
    ldb4<TAIL>(gain, k, cols, gv);
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float xn = xv[i] * r;
      o[i] = xn * gv[i];
      h[i] = f32_to_bf16(o[i]);
    }
    if (F32) stf4<TAIL>((float*)y + row * cols, k, cols, o);
    else stb4<TAIL>((uint16_t*)y + row * cols, k, cols, h);
  }
}

// RMSNorm backward (dx): one wavefront per row.
// res (optional): dx = RN(res + the norm's gradient), the residual addition; dxb (optional): bf16 copy of dx.
template <bool TAIL>
__global__ __launch_bounds__(256) void rownorm_bwd_kernel(int64_t rows, int64_t cols, const float* __restrict__ x,
                                                          const uint16_t* __restrict__ gain,
                                                          const float* __restrict__ rstd,
                                                          const float* __restrict__ dy, float inv_d,
                                                          float* __restrict__ dx, const float* __restrict__ res,
                                                          uint16_t* __restrict__ dxb) {
  __shared__ WaveStage st[4];
  extern __shared__ float dyn[];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= rows) return;
  const int64_t nc = (cols + kChunk - 1) / kChunk;
  const float* xr = x + row * cols;
  const float* dyr = dy + row * cols;
  float dot = wave_row_rsum<4>(cols, st[w], dyn + w * nc, [&](int64_t j, float (&f)[4]) {
    float dv[4], gv[4], xv[4];
    ldf4<TAIL>(dyr, j, cols, dv);
    ldb4<TAIL>(gain, j, cols, gv);
    ldf4<TAIL>(xr, j, cols, xv);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float gy = dv[i] * gv[i];
      f[i] = gy * xv[i];
    }
  }, cols);
  const float r = rstd[row];
  float r2 = r * r;
  float r3 = r2 * r;
  float dd = dot * inv_d;
  float q = r3 * dd;
  for (int64_t k = (int64_t)lane * 4; k < cols; k += 64 * 4) {
    float dv[4], gv[4], xv[4], o[4];
    ldf4<TAIL>(dyr, k, cols, dv);
    ldb4<TAIL>(gain, k, cols, gv);
    ldf4<TAIL>(xr, k, cols, xv);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float gy = dv[i] * gv[i];
      float a = r * gy;
      float b = xv[i] * q;
      o[i] = a - b;
    }
    if (res) {
      float rv[4];
      ldf4<TAIL>(res + row * cols, k, cols, rv);
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = rv[i] + o[i];
    }
    stf4<TAIL>(dx + row * cols, k, cols, o);
    if (dxb) {
      uint16_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = f32_to_bf16(o[i]);
      stb4<TAIL>(dxb + row * cols, k, cols, h);
    }
  }
}

// RMSNorm forward and backward with register-resident rows (same arithmetic as the kernels above).
template <bool TAIL, bool F32>
__global__ __launch_bounds__(256) void rownorm_fwd_reg_kernel(int64_t rows, int64_t cols, const float* __restrict__ x,
                                                              const uint16_t* __restrict__ gain, float eps,
                                                              float inv_d, void* __restrict__ y,
                                                              float* __restrict__ rstd) {
  __shared__ __attribute__((aligned(16))) RegStage st[4];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= rows) return;
  const float* xr = x + row * cols;
  float xv[kRegQ][4], sq[kRegQ][4];
#pragma unroll
  for (int q = 0; q < kRegQ; ++q) {
    const int64_t j = 256 * q + 4 * lane;
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (j < cols) ldf4<TAIL>(xr, j, cols, v);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      xv[q][t] = v[t];
      sq[q][t] = v[t] * v[t];
    }
  }
  const float ss = reg_row_sum(st[w], sq, cols);
  float ms = ss * inv_d;
  float var = ms + eps;
  float r = 1.0f / __builtin_sqrtf(var);
  if (lane == 0) rstd[row] = r;
#pragma unroll
  for (int q = 0; q < kRegQ; ++q) {
    const int64_t j = 256 * q + 4 * lane;
    if (j < cols) {
      float gv[4], o[4];
      uint16_t h[4];
      ldb4<TAIL>(gain, j, cols, gv);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float xn = xv[q][t] * r;
        o[t] = xn * gv[t];
        h[t] = f32_to_bf16(o[t]);
      }
      if (F32) stf4<TAIL>((float*)y + row * cols, j, cols, o);
      else stb4<TAIL>((uint16_t*)y + row * cols, j, cols, h);
    }
  }
}

// (bounded to 128 registers, four wavefronts per SIMD: 62.8 -> 58.1 us with the gain's part at 8192 x 2048; with TAIL
// that spills, 69.5 -> 76.5 us at 8192 x 2047)
template <bool TAIL>
__global__ __launch_bounds__(256, TAIL ? 3 : 4) void rownorm_bwd_reg_kernel(int64_t rows, int64_t cols, const float* __restrict__ x,
                                                              const uint16_t* __restrict__ gain,
                                                              const float* __restrict__ rstd,
                                                              const float* __restrict__ dy, float inv_d,
                                                              float* __restrict__ dx, const float* __restrict__ res,
                                                              uint16_t* __restrict__ dxb) {
  __shared__ __attribute__((aligned(16))) RegStage st[4];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= rows) return;
  const float* xr = x + row * cols;
  const float* dyr = dy + row * cols;
  float xv[kRegQ][4], gy[kRegQ][4], tm[kRegQ][4];
#pragma unroll
  for (int q = 0; q < kRegQ; ++q) {
    const int64_t j = 256 * q + 4 * lane;
    float dv[4] = {0.0f, 0.0f, 0.0f, 0.0f}, gv[4] = {0.0f, 0.0f, 0.0f, 0.0f}, xx[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (j < cols) {
      ldf4<TAIL>(dyr, j, cols, dv);
      ldb4<TAIL>(gain, j, cols, gv);
      ldf4<TAIL>(xr, j, cols, xx);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      xv[q][t] = xx[t];
      gy[q][t] = dv[t] * gv[t];
      tm[q][t] = gy[q][t] * xx[t];
    }
  }
  const float dot = reg_row_sum(st[w], tm, cols);
  const float r = rstd[row];
  float r2 = r * r;
  float r3 = r2 * r;
  float dd = dot * inv_d;
  float qq = r3 * dd;
#pragma unroll
  for (int q = 0; q < kRegQ; ++q) {
    const int64_t j = 256 * q + 4 * lane;
    if (j < cols) {
      float o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float a = r * gy[q][t];
        float b = xv[q][t] * qq;
        o[t] = a - b;
      }
      if (res) {
        float rv[4];
        ldf4<TAIL>(res + row * cols, j, cols, rv);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = rv[t] + o[t];
      }
      stf4<TAIL>(dx + row * cols, j, cols, o);
      if (dxb) {
        uint16_t h[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) h[t] = f32_to_bf16(o[t]);
        stb4<TAIL>(dxb + row * cols, j, cols, h);
      }
    }
  }
}

// dgain[k] = R1 over rows t of RN(dy[t,k] * RN(x[t,k] * rstd[t])), in two launches.  First every (chunk of
// 32 rows, column) chain, V per thread (columns along the lanes, so row reads are coalesced), into part[c][k];
// then per column Algorithm 2 over its chunk partials in ascending order: a workgroup of 16 wavefronts
// takes 64 columns, wavefront q folds the aligned power-of-two group of chunks [q*G, q*G + G), and the 16
// group results are folded with the pass-through rule.
// A thread takes V columns and has B rows in flight before their chain steps: V = 4, B = 4 where rows are a multiple of
// 4 long, V = 1, B = 8 otherwise (with the dx kernel, one row in flight -> this: 62.8 -> 57.9 us at 8192 x 2048,
// 24.8 -> 20.3 at 2048 x 2048, 91 -> 70 at 8192 x 2047, where V = 4 with a tail takes 80).
template <int V, int B>
__global__ __launch_bounds__(256 / V) void rownorm_dgain_part_kernel(int64_t rows, int64_t cols,
                                                                     const float* __restrict__ x,
                                                                     const float* __restrict__ rstd,
                                                                     const float* __restrict__ dy,
                                                                     float* __restrict__ part) {
  const int64_t col = (int64_t)blockIdx.x * 256 + threadIdx.x * V;
  const int64_t c = blockIdx.y;
  if (col >= cols) return;
  const int64_t t0 = c * kChunk, t1 = (t0 + kChunk < rows) ? t0 + kChunk : rows;
  float s[V] = {};
  auto steps = [&](int64_t t, auto n) __attribute__((always_inline)) {
    constexpr int N = decltype(n)::value;
    float xv[N][V], dv[N][V];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      ldf<V>(x + (t + i) * cols + col, xv[i]);
      ldf<V>(dy + (t + i) * cols + col, dv[i]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float r = rstd[t + i];
#pragma unroll
      for (int k = 0; k < V; ++k) {
        float xh = xv[i][k] * r;
        float pr = dv[i][k] * xh;
        s[k] = s[k] + pr;
      }
    }
  };
  int64_t t = t0;
  for (; t + B <= t1; t += B) steps(t, std::integral_constant<int, B>{});
  for (; t < t1; ++t) steps(t, std::integral_constant<int, 1>{});
  stf<V>(part + c * cols + col, s);
}

constexpr int kDgainGroups = 16;
__global__ __launch_bounds__(1024) void rownorm_dgain_fold_kernel(int64_t rows, int64_t cols,
                                                                  const float* __restrict__ part,
                                                                  float* __restrict__ dgain) {
  __shared__ float gres[kDgainGroups][64];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t col = (int64_t)blockIdx.x * 64 + lane;
  const int64_t nc = (rows + kChunk - 1) / kChunk;
  const int64_t G = block_chunks(nc, kDgainGroups);
  const int64_t c0 = grp * G, c1 = (c0 + G < nc) ? c0 + G : nc;
  LocalFoldN<22> f;
  if (col < cols) {
    int64_t c = c0;
    for (; c + 4 <= c1; c += 4) {
      const float p0 = part[c * cols + col], p1 = part[(c + 1) * cols + col];
      const float p2 = part[(c + 2) * cols + col], p3 = part[(c + 3) * cols + col];
      f.push(p0); f.push(p1); f.push(p2); f.push(p3);
    }
    for (; c < c1; ++c) f.push(part[c * cols + col]);
  }
  gres[grp][lane] = f.result();
  __syncthreads();
  if (grp == 0 && col < cols) {
    // fold the group results: level by level, a node adds its right neighbour when that subtree is real
    float v[kDgainGroups];
#pragma unroll
    for (int q = 0; q < kDgainGroups; ++q) v[q] = gres[q][lane];
#pragma unroll
    for (int sdist = 1; sdist < kDgainGroups; sdist <<= 1)
#pragma unroll
      for (int q = 0; q + sdist < kDgainGroups; q += 2 * sdist)
        if ((q + sdist) * G < nc) v[q] = v[q] + v[q + sdist];
    dgain[col] = v[0];
  }
}

// Rows of up to 2048 terms stay in registers; longer ones are read again for the output (norm forward / backward at
// 4096 x 4096: 30.5 / 53 us; held in 172 / 296 registers instead, 33 / 58).  TAIL variants take a row length that is
// no multiple of 4 (the last vector by element; without them every row element by element, 8192 x 2047 forward 55 us
// instead of 25).
#define CANON_ROW_KERNEL(LAUNCH, REG, REG_TAIL, GEN, GEN_TAIL)  \
  do {                                                          \
    if (cols <= kRegCols) {                                     \
      if (cols % 4 == 0) LAUNCH(REG, 0);                        \
      else LAUNCH(REG_TAIL, 0);                                 \
    } else {                                                    \
      if (cols % 4 == 0) LAUNCH(GEN, wave_kernel_lds(cols));    \
      else LAUNCH(GEN_TAIL, wave_kernel_lds(cols));             \
    }                                                           \
  } while (0)

template <bool F32>
static hipError_t rownorm_fwd_any(int64_t rows, int64_t cols, const float* x, const uint16_t* gain, float eps,
                                  void* y, float* rstd, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  const float inv_d = (float)(1.0 / (double)cols);  // RN32(1/cols), correctly rounded
  const dim3 grid((unsigned)((rows + 3) / 4));
#define CANON_NORM(K, LDS) \
  hipLaunchKernelGGL(K, grid, dim3(256), LDS, s, rows, cols, x, gain, eps, inv_d, y, rstd)
  CANON_ROW_KERNEL(CANON_NORM, (rownorm_fwd_reg_kernel<false, F32>), (rownorm_fwd_reg_kernel<true, F32>),
                   (rownorm_fwd_kernel<false, F32>), (rownorm_fwd_kernel<true, F32>));
#undef CANON_NORM
  return hipGetLastError();
}

hipError_t rownorm_fwd_launch(int64_t rows, int64_t cols, const float* x, const uint16_t* gain, float eps, uint16_t* y,
                              float* rstd, hipStream_t s) {
  return rownorm_fwd_any<false>(rows, cols, x, gain, eps, y, rstd, s);
}

hipError_t rownorm_fwd_f32_launch(int64_t rows, int64_t cols, const float* x, const uint16_t* gain, float eps,
                                  float* y, float* rstd, hipStream_t s) {
  return rownorm_fwd_any<true>(rows, cols, x, gain, eps, y, rstd, s);
}

// dx doubles as the scratch of the dgain chunk partials (ceil(rows/32) x cols floats <= rows x cols), so
// the dgain launches run before the dx kernel overwrites it.
hipError_t rownorm_bwd_launch(int64_t rows, int64_t cols, const float* x, const uint16_t* gain, const float* rstd,
                              const float* dy, float* dx, float* dgain, hipStream_t s, const float* res,
                              uint16_t* dxb) {
  if (dgain && res && res == dx) return hipErrorInvalidValue;  // dx holds the dgain partials before res is read
  if (rows == 0) {
    if (dgain) return hipMemsetAsync(dgain, 0, sizeof(float) * cols, s);
    return hipSuccess;
  }
  const float inv_d = (float)(1.0 / (double)cols);
  if (dgain) {
    const int64_t nc = (rows + kChunk - 1) / kChunk;
    const dim3 pgrid((unsigned)((cols + 255) / 256), (unsigned)nc);
    if (cols % 4 == 0)
      hipLaunchKernelGGL((rownorm_dgain_part_kernel<4, 4>), pgrid, dim3(64), 0, s, rows, cols, x, rstd, dy, dx);
    else
      hipLaunchKernelGGL((rownorm_dgain_part_kernel<1, 8>), pgrid, dim3(256), 0, s, rows, cols, x, rstd, dy, dx);
    hipLaunchKernelGGL(rownorm_dgain_fold_kernel, dim3((unsigned)((cols + 63) / 64)), dim3(1024), 0, s, rows, cols,
                       dx, dgain);
  }
  const dim3 grid((unsigned)((rows + 3) / 4));
#define CANON_NORM(K, LDS) \
  hipLaunchKernelGGL(K, grid, dim3(256), LDS, s, rows, cols, x, gain, rstd, dy, inv_d, dx, res, dxb)
  CANON_ROW_KERNEL(CANON_NORM, rownorm_bwd_reg_kernel<false>, rownorm_bwd_reg_kernel<true>, rownorm_bwd_kernel<false>,
                   rownorm_bwd_kernel<true>);
#undef CANON_NORM
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// LSQ step re-pin of the int8 quantised linear: per row r of a bf16 matrix,
// s[r] = RN(RN(2 * RN(R1(|w[r,:]|) * RN(1/cols))) * RN32(1/sqrt(127))).  One wavefront per row.
constexpr uint32_t kInvSqrtQmaxBits = 0x3DB5BB09u;  // RN32(1/sqrt(127))

template <bool TAIL>
__global__ __launch_bounds__(256) void quant_scales_kernel(int64_t rows, int64_t cols, const uint16_t* __restrict__ w,
                                                           float inv_k, float* __restrict__ scale) {
  __shared__ WaveStage st[4];
  extern __shared__ float dyn[];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wv;
  if (row >= rows) return;
  const int64_t nc = (cols + kChunk - 1) / kChunk;
  const uint16_t* wr = w + row * cols;
  const float a = wave_row_rsum<4>(cols, st[wv], dyn + wv * nc, [&](int64_t j, float (&f)[4]) {
    ldb4<TAIL>(wr, j, cols, f);
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __builtin_fabsf(f[i]);
  }, cols);
  const float mean = a * inv_k;
  const float two = 2.0f * mean;
  if (lane == 0) scale[row] = two * __uint_as_float(kInvSqrtQmaxBits);
}

// The same for rows held in registers: one read of the row
template <bool TAIL>
__global__ __launch_bounds__(256) void quant_scales_reg_kernel(int64_t rows, int64_t cols,
                                                               const uint16_t* __restrict__ w, float inv_k,
                                                               float* __restrict__ scale) {
  __shared__ __attribute__((aligned(16))) RegStage st[4];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wv;
  if (row >= rows) return;
  const uint16_t* wr = w + row * cols;
  float e[kRegQ][4];
#pragma unroll
  for (int q = 0; q < kRegQ; ++q) {
    const int64_t j = 256 * q + 4 * lane;
    if (j < cols) {
      float f[4];
      ldb4<TAIL>(wr, j, cols, f);
#pragma unroll
      for (int t = 0; t < 4; ++t) e[q][t] = __builtin_fabsf(f[t]);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) e[q][t] = 0.0f;
    }
  }
  const float a = reg_row_sum(st[wv], e, cols);
  const float mean = a * inv_k;
  const float two = 2.0f * mean;
  if (lane == 0) scale[row] = two * __uint_as_float(kInvSqrtQmaxBits);
}

hipError_t quant_scales_launch(int64_t rows, int64_t cols, const uint16_t* w, float* scale, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  const float inv_k = (float)(1.0 / (double)cols);  // RN32(1/cols)
  const dim3 grid((unsigned)((rows + 3) / 4));
#define CANON_SCALES(K, LDS) hipLaunchKernelGGL(K, grid, dim3(256), LDS, s, rows, cols, w, inv_k, scale)
  CANON_ROW_KERNEL(CANON_SCALES, quant_scales_reg_kernel<false>, quant_scales_reg_kernel<true>,
                   quant_scales_kernel<false>, quant_scales_kernel<true>);
#undef CANON_SCALES
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Causal softmax of raw scores: row r is query i = r mod cols; one wavefront per row, coalesced.  With
// window > 0 query i sees keys j0 = max(0, i - window + 1) .. i (the hybrid attention's windowed layers).
// band = 1 writes only the columns [wlo, whi) that the causally skipping products read (kAttnLead).
__device__ __forceinline__ void band_cols(int band, int64_t i, int64_t window, int64_t cols, int64_t& wlo,
                                          int64_t& whi) {
  if (!band) return;
  const int64_t lo = i - window - kAttnLead, hi = (i / 128) * 128 + 128;
  wlo = (window > 0 && lo > 0) ? lo : 0;
  whi = hi < cols ? hi : cols;
}
template <bool TAIL>
__global__ __launch_bounds__(256) void softmax_causal_kernel(int64_t rows, int64_t cols, const float* __restrict__ raw,
                                                             float scale, int64_t window,
                                                             uint16_t* __restrict__ probs, int band) {
  __shared__ WaveStage st[4];
  extern __shared__ float dyn[];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= rows) return;
  const int64_t nc = (cols + kChunk - 1) / kChunk;
  const int64_t i = row % cols;
  const int64_t j0 = (window > 0 && i - window + 1 > 0) ? i - window + 1 : 0;
  const float* rr = raw + row * cols;
  float m = -__builtin_inff();
  // keys before the window are not read: whole wavefront strides below j0 are skipped, and the loads of
  // vectors wholly below j0 are left out (their terms are +0 either way)
  for (int64_t j = (j0 / (64 * 4)) * (64 * 4) + (int64_t)lane * 4; j <= i; j += 64 * 4) {
    float v[4];
    ldf4<TAIL>(rr, j, cols, v);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if ((j + t <= i && j + t >= j0)) m = fmaxf(m, v[t] * scale);
  }
  m = wave_max(m);
  // masked keys enter the chain as +0 terms
  const float S = wave_row_rsum<4>(cols, st[w], dyn + w * nc, [&](int64_t j, float (&f)[4]) {
    float v[4];
    if (j + 4 - 1 >= j0) ldf4<TAIL>(rr, j, cols, v);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float e = 0.0f;
      if ((j + t <= i && j + t >= j0)) {
        float sc = v[t] * scale;
        e = cexp_neg(sc - m);
      }
      f[t] = e;
    }
  }, i + 1, j0);
  const float rcp = 1.0f / S;
  int64_t wlo = 0, whi = cols;  // columns written
  band_cols(band, i, window, cols, wlo, whi);
  for (int64_t j = (wlo / (64 * 4)) * (64 * 4) + (int64_t)lane * 4; j < whi; j += 64 * 4) {
    uint16_t o[4];
    if (j <= i && j + 4 - 1 >= j0) {
      float v[4];
      ldf4<TAIL>(rr, j, cols, v);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        o[t] = 0;
        if ((j + t <= i && j + t >= j0)) {
          float sc = v[t] * scale;
          float e = cexp_neg(sc - m);
          o[t] = f32_to_bf16(e * rcp);
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) o[t] = 0;
    }
    stb4<TAIL>(probs + row * cols, j, cols, o);
  }
}

// Rows held in registers, read from memory once (cols <= 256 Q, Q = 8 or 16).  A wavefront's vectors q are each wholly
// outside the visible keys j0 .. i (+0 terms, no work), wholly inside (no masks) or on an edge.  Bound: the reads of
// the visible scores and the writes of every probability, 268 MB at 16 heads x 2048: 59 us (masks on every term 84);
// 4 heads x 4096: 58 us (98).
template <int Q, bool TAIL>
__global__ __launch_bounds__(256) void softmax_causal_reg_kernel(int64_t rows, int64_t cols,
                                                                 const float* __restrict__ raw, float scale,
                                                                 int64_t window, uint16_t* __restrict__ probs,
                                                                 int band) {
  __shared__ __attribute__((aligned(16))) RegStage st[4];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= rows) return;
  const int i = __builtin_amdgcn_readfirstlane((int)(row % cols));  // column indices fit in int
  const int j0 = (window > 0 && i - window + 1 > 0) ? (int)(i - window + 1) : 0;
  const float* rr = raw + row * cols;
  auto any = [&](int q) { return 256 * q <= i && 256 * q + 255 >= j0; };   // some visible key in vectors q
  auto all = [&](int q) { return 256 * q + 255 <= i && 256 * q >= j0; };   // nothing but visible keys
  float e[Q][4];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
#pragma unroll
    for (int t = 0; t < 4; ++t) e[q][t] = 0.0f;
    const int j = 256 * q + 4 * lane;
    if (any(q) && j <= i && j + 3 >= j0) ldf4<TAIL>(rr, j, cols, e[q]);
  }
  float m = -__builtin_inff();
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (!any(q)) continue;
    const int j = 256 * q + 4 * lane;
#pragma unroll
    for (int t = 0; t < 4; ++t) e[q][t] = e[q][t] * scale;
    if (all(q)) {
#pragma unroll
      for (int t = 0; t < 4; ++t) m = fmaxf(m, e[q][t]);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (j + t <= i && j + t >= j0) m = fmaxf(m, e[q][t]);
    }
  }
  m = wave_max(m);
  // masked keys enter the chain as +0 terms
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (!any(q)) continue;
    const int j = 256 * q + 4 * lane;
#pragma unroll
    for (int t = 0; t < 4; ++t) e[q][t] = cexp_neg(e[q][t] - m);
    if (!all(q)) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (!(j + t <= i && j + t >= j0)) e[q][t] = 0.0f;
    }
  }
  float S = reg_row_sum<0>(st[w], e, cols < kRegCols ? cols : kRegCols);
  if constexpr (Q > kRegQ) {  // 64 chunks are a complete subtree: the other half adds last
    if (i >= kRegCols) S = S + reg_row_sum<1>(st[w], e, cols - kRegCols);
    else S = S + 0.0f;
  }
  const float rcp = 1.0f / S;
  int64_t wlo = 0, whi = cols;  // columns written
  band_cols(band, i, window, cols, wlo, whi);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = 256 * q + 4 * lane;
    if (j < whi && j + 3 >= wlo) {
      uint16_t o[4] = {0, 0, 0, 0};
      if (any(q)) {  // a masked key's probability is +0 * rcp, a NaN if S is: keep its zero
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = f32_to_bf16(e[q][t] * rcp);
        if (!all(q)) {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (!(j + t <= i && j + t >= j0)) o[t] = 0;
        }
      }
      stb4<TAIL>(probs + row * cols, j, cols, o);
    }
  }
}

// Windowed rows (0 < window <= kBandWin): the visible keys j0 .. i lie in the 768 columns [base, base + 768),
// base = j0 rounded down to 256, which lane l holds as float4 vectors at base + 256 q + 4 l (q < 3): the row
// is read from memory once.  The band's 24 chunks are staged in LDS and chained by lanes 0 .. 23 (every
// other chunk of the row is a +0 partial), and the nc partials are folded as in wave_row_rsum.
constexpr int64_t kBandWin = 512;
struct BandStage {
  float t[24][33];
};
template <bool TAIL>
__global__ __launch_bounds__(256) void softmax_band_kernel(int64_t rows, int64_t cols, const float* __restrict__ raw,
                                                           float scale, int64_t window, uint16_t* __restrict__ probs,
                                                           int band) {
  __shared__ BandStage st[4];
  extern __shared__ float dyn[];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= rows) return;
  const int64_t nc = (cols + kChunk - 1) / kChunk;
  float* parts = dyn + w * nc;
  const int64_t i = row % cols;
  const int64_t j0 = (i - window + 1 > 0) ? i - window + 1 : 0;
  const int64_t base = (j0 / 256) * 256;
  const float* rr = raw + row * cols;
  auto seen = [&](int64_t j) { return j <= i && j >= j0; };
  float e[3][4];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int64_t j = base + 256 * q + 4 * lane;
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (j <= i && j + 3 >= j0) ldf4<TAIL>(rr, j, cols, v);
#pragma unroll
    for (int t = 0; t < 4; ++t) e[q][t] = v[t];
  }
  float m = -__builtin_inff();
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (seen(base + 256 * q + 4 * lane + t)) m = fmaxf(m, e[q][t] * scale);
  m = wave_max(m);
  // masked keys enter the chain as +0 terms
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float x = 0.0f;
      if (seen(base + 256 * q + 4 * lane + t)) {
        float sc = e[q][t] * scale;
        x = cexp_neg(sc - m);
      }
      e[q][t] = x;
    }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int local = 256 * q + 4 * lane;
    float* dst = &st[w].t[local >> 5][local & 31];
#pragma unroll
    for (int t = 0; t < 4; ++t) dst[t] = e[q][t];
  }
  for (int64_t c = lane; c < nc; c += 64) parts[c] = 0.0f;
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
  const int64_t cb = base / kChunk + lane;  // this lane's band chunk
  if (lane < 24 && cb < nc) {
    const int64_t k1 = cols - cb * kChunk < kChunk ? cols - cb * kChunk : kChunk;
    float p = 0.0f;
    for (int k = 0; k < (int)k1; ++k) p = p + st[w].t[lane][k];
    parts[cb] = p;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
  const float S = fold_parts(parts, nc);
  const float rcp = 1.0f / S;
  int64_t wlo = 0, whi = cols;  // columns written
  band_cols(band, i, window, cols, wlo, whi);
  for (int64_t j = (wlo / 256) * 256 + 4 * lane; j < whi; j += 256) {
    uint16_t o[4] = {0, 0, 0, 0};
    const int64_t d = j - base;
    if (d >= 0 && d < 768) {
      const int q = (int)(d >> 8);
      float x[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = q == 0 ? e[0][t] : (q == 1 ? e[1][t] : e[2][t]);
#pragma unroll
      for (int t = 0; t < 4; ++t) o[t] = seen(j + t) ? f32_to_bf16(x[t] * rcp) : (uint16_t)0;
    }
    stb4<TAIL>(probs + row * cols, j, cols, o);
  }
}

hipError_t softmax_causal_launch(int64_t rows, int64_t cols, const float* raw, float scale, int64_t window,
                                 uint16_t* probs, hipStream_t s, int band) {
  if (rows == 0) return hipSuccess;
  const dim3 grid((unsigned)((rows + 3) / 4));
#define CANON_SOFTMAX(K, LDS) \
  hipLaunchKernelGGL(K, grid, dim3(256), LDS, s, rows, cols, raw, scale, window, probs, band)
  if (window > 0 && window <= kBandWin) {
    if (cols % 4 == 0) CANON_SOFTMAX(softmax_band_kernel<false>, wave_kernel_lds(cols));
    else CANON_SOFTMAX(softmax_band_kernel<true>, wave_kernel_lds(cols));
  } else {
    if (cols > kRegCols && cols <= 2 * kRegCols) {
      if (cols % 4 == 0) CANON_SOFTMAX((softmax_causal_reg_kernel<2 * kRegQ, false>), 0);
      else CANON_SOFTMAX((softmax_causal_reg_kernel<2 * kRegQ, true>), 0);
    } else {
      CANON_ROW_KERNEL(CANON_SOFTMAX, (softmax_causal_reg_kernel<kRegQ, false>),
                       (softmax_causal_reg_kernel<kRegQ, true>), softmax_causal_kernel<false>,
                       softmax_causal_kernel<true>);
    }
  }
#undef CANON_SOFTMAX
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Cross-entropy, one workgroup of NT threads per row, the row read from memory once: thread t holds the 8 logits
// 8 (t + NT q) .. + 7 for q < Q.  EXPS keeps the exponentials in registers (one cexp per logit, rows up to 26624);
// longer rows keep the bf16 logits in 64 or 108 registers, so that two (one) workgroups of 16 wavefronts share a CU,
// and evaluate cexp again for the output (50304 logits, one run under a lower clock than the figures below: with the
// exponentials kept, 512 threads 584 us, 1024 threads, one workgroup per CU, 543; logits kept 531).  The exponentials are staged SEG vectors at a time as chunk rows of 36
// floats (16-byte stores, and 16-byte reads without bank conflicts), thread c running chunk c's chain.  Rows start at
// any element (16-byte accesses need no alignment).
// Bound: vector instructions, about 56 per logit with two cexp of 22 (no range selects where no logit is far enough
// below the maximum).  8192 x 50304: 742 -> 516 us (3.2 TB/s); 8192 x 50257: 1999 -> 555; 8192 x 20000: 323 -> 203.
struct __attribute__((packed, aligned(2))) Row8 {
  uint32_t w[4];
};
__device__ __forceinline__ void widen_row8(const Row8& u, float (&f)[8]) {  // a subnormal is flushed by its first use
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(u.w[i] << 16);
    f[2 * i + 1] = __uint_as_float(u.w[i] & 0xFFFF0000u);
  }
}

template <int NT, int Q, bool EXPS>
__global__ __launch_bounds__(NT) void xent_row_kernel(int vocab, const uint16_t* __restrict__ logits,
                                                      const int32_t* __restrict__ targets, float inv_tokens,
                                                      float z_loss, float z2, uint16_t* __restrict__ dlogits,
                                                      float* __restrict__ row_loss) {
  constexpr int SEG = NT == 1024 ? 2 : 4, CPS = NT / 4;  // vectors staged at a time; chunks per vector index
  __shared__ __attribute__((aligned(16))) float st[SEG][CPS][36];
  extern __shared__ float parts[];
  __shared__ float red[2][NT / 64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, t = threadIdx.x;
  const int64_t row = blockIdx.x;
  const uint16_t* lr = logits + row * vocab;
  const int n8 = vocab >> 3, tail = vocab & 7, nv = n8 + (tail ? 1 : 0);
  Row8 raw[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j8 = t + NT * q;
    if (j8 < n8) {
      raw[q] = *reinterpret_cast<const Row8*>(lr + 8 * (int64_t)j8);
    } else if (j8 < nv) {  // the partial last vector, filled up with its first logit
#pragma unroll
      for (int i = 0; i < 4; ++i)
        raw[q].w[i] = (uint32_t)lr[8 * j8 + (2 * i < tail ? 2 * i : 0)] |
                      ((uint32_t)lr[8 * j8 + (2 * i + 1 < tail ? 2 * i + 1 : 0)] << 16);
    }
  }
  float m = -__builtin_inff(), lo = __builtin_inff();
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (t + NT * q < nv) {
      float f[8];
      widen_row8(raw[q], f);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        m = fmaxf(m, f[i]);
        lo = fminf(lo, f[i]);
      }
    }
  }
  m = wave_max(m);
  lo = -wave_max(-lo);
  if (lane == 0) {
    red[0][w] = m;
    red[1][w] = lo;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    m = fmaxf(m, red[0][i]);
    lo = fminf(lo, red[1][i]);
  }
  const bool mid = cexp_is_mid(lo - m);  // no logit of the row is far enough below m for a zero
  float e[EXPS ? Q : 1][8];
  auto exps = [&](auto all_mid, const Row8& r, float (&x)[8]) __attribute__((always_inline)) {
    float f[8];
    widen_row8(r, f);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = all_mid.value ? cexp_mid(f[i] - m) : cexp_neg(f[i] - m);
  };
  const int nc = (vocab + kChunk - 1) / kChunk;
  auto sums = [&](auto all_mid) __attribute__((always_inline)) {
#pragma unroll
    for (int s0 = 0; s0 < Q; s0 += SEG) {
      if (NT * s0 < nv) {
#pragma unroll
        for (int b = 0; b < SEG; ++b) {
          const int q = s0 + b;
          if (q < Q && t + NT * q < nv) {
            float x[8];
            exps(all_mid, raw[q], x);
            float4* dst = reinterpret_cast<float4*>(&st[b][t >> 2][8 * (t & 3)]);
            dst[0] = make_float4(x[0], x[1], x[2], x[3]);
            dst[1] = make_float4(x[4], x[5], x[6], x[7]);
            if (EXPS) {
#pragma unroll
              for (int i = 0; i < 8; ++i) e[q % (EXPS ? Q : 1)][i] = x[i];
            }
          }
        }
        __syncthreads();
        const int c = CPS * s0 + t;  // this thread's chunk of the staged vectors
        if (t < SEG * CPS && c < nc) {
          const float* src = &st[0][0][0] + 36 * t;
          float sacc = 0.0f;
          const int k1 = vocab - c * kChunk;
          if (k1 >= kChunk) {
#pragma unroll
            for (int i = 0; i < kChunk; i += 4) {
              const float4 v = *reinterpret_cast<const float4*>(src + i);
              sacc = sacc + v.x; sacc = sacc + v.y; sacc = sacc + v.z; sacc = sacc + v.w;
            }
          } else {
            for (int i = 0; i < k1; ++i) sacc = sacc + src[i];
          }
          parts[c] = sacc;
        }
        __syncthreads();
      }
    }
  };
  if (mid) sums(std::true_type{});
  else sums(std::false_type{});
  // Algorithm 2 over the chunk partials: 256 threads, each an aligned block of G of them
  const int G = (int)block_chunks(nc, 256), np = (nc + G - 1) / G;
  if (w < 4) {
    const int c0 = t * G, c1 = c0 + G < nc ? c0 + G : nc;
    LocalFoldN<5> f;  // G <= 16
    for (int c = c0; c < c1; ++c) f.push(parts[c]);
    const int nl = np - 64 * w;
    const float r = wave_fold(f.result(), nl < 0 ? 0 : (nl > 64 ? 64 : nl));
    if (lane == 0) red[0][w] = r;
  }
  __syncthreads();
  float S = red[0][0];
  if (64 < np) S = S + red[0][1];
  if (128 < np) {
    float b = red[0][2];
    if (192 < np) b = b + red[0][3];
    S = S + b;
  }
  const int32_t y = targets[row];
  const bool valid = y >= 0 && y < vocab;
  // z-loss (weight z_loss, z2 = RN(2 z_loss)): the row loss gains RN(z_loss * RN(lse^2)) and every
  // probability is scaled by RN(1 + RN(z2 * lse)) before the target is subtracted
  const float lse = m + clog(S);
  const bool zl = z_loss != 0.0f;
  const float zt = z2 * lse;
  const float pscale = 1.0f + zt;
  if (t == 0) {
    float ce = lse - bf16_to_f32(lr[valid ? y : 0]);
    if (zl) {
      const float l2 = lse * lse;
      const float zterm = z_loss * l2;
      ce = ce + zterm;
    }
    row_loss[row] = valid ? ce : __builtin_nanf("");
  }
  const float rcp = 1.0f / S;
  uint16_t* dr = dlogits + row * vocab;
  auto out = [&](auto all_mid) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int j8 = t + NT * q;
      if (j8 < nv) {
        float x[8];
        if (EXPS) {
#pragma unroll
          for (int i = 0; i < 8; ++i) x[i] = e[q % (EXPS ? Q : 1)][i];
        } else {
          exps(all_mid, raw[q], x);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = x[i] * rcp;
        if (zl) {
#pragma unroll
          for (int i = 0; i < 8; ++i) x[i] = x[i] * pscale;
        }
        if ((y >> 3) == j8) {  // the target's one; elsewhere p - 0 = p
#pragma unroll
          for (int i = 0; i < 8; ++i) x[i] = x[i] - (8 * j8 + i == y ? 1.0f : 0.0f);
        }
        Row8 h;
#pragma unroll
        for (int i = 0; i < 4; ++i) h.w[i] = pack_bf16(x[2 * i] * inv_tokens, x[2 * i + 1] * inv_tokens);
        if (j8 < n8) {
          *reinterpret_cast<Row8*>(dr + 8 * (int64_t)j8) = h;
        } else {
#pragma unroll
          for (int i = 0; i < 7; ++i)
            if (i < tail) dr[8 * j8 + i] = (uint16_t)(h.w[i >> 1] >> (16 * (i & 1)));
        }
      }
    }
  };
  if (EXPS || mid) out(std::true_type{});
  else out(std::false_type{});
}

// mean_loss = RN(R1(row_loss) * inv_tokens): one workgroup.
__global__ __launch_bounds__(256) void mean_loss_kernel(int64_t rows, const float* __restrict__ row_loss,
                                                        float inv_tokens, float* __restrict__ out) {
  const int64_t nc = (rows + kChunk - 1) / kChunk;
  const int64_t G = block_chunks(nc, 256);
  const int64_t c0 = threadIdx.x * G, c1 = (c0 + G < nc) ? c0 + G : nc;
  LocalFold f;
  for (int64_t c = c0; c < c1; ++c) {
    float s = 0.0f;
    const int64_t k1 = (c + 1) * kChunk < rows ? (c + 1) * kChunk : rows;
    if (k1 - c * kChunk == kChunk) {  // all loads in flight before the chain
      float v[kChunk];
#pragma unroll
      for (int i = 0; i < kChunk; ++i) v[i] = row_loss[c * kChunk + i];
#pragma unroll
      for (int i = 0; i < kChunk; ++i) s = s + v[i];
    } else {
      for (int64_t t = c * kChunk; t < k1; ++t) s = s + row_loss[t];
    }
    f.push(s);
  }
  const float S = block_fold(f.result(), (nc + G - 1) / G);
  if (threadIdx.x == 0) out[0] = S * inv_tokens;
}

hipError_t xent_launch(int64_t rows, int64_t vocab, const uint16_t* logits, const int32_t* targets, float inv_tokens,
                       float z_loss, uint16_t* dlogits, float* row_loss, float* mean_loss, hipStream_t s) {
  if (rows > 0) {
    const size_t lds = sizeof(float) * (size_t)((vocab + kChunk - 1) / kChunk);
    const float z2 = 2.0f * z_loss;  // exact
    const dim3 grid((unsigned)rows);
    const int v = (int)vocab;  // at most 131072: 16 vectors of 8 for each of 1024 threads
#define CANON_XENT(NT, Q, EXPS)                                                                                  \
  hipLaunchKernelGGL((xent_row_kernel<NT, Q, EXPS>), grid, dim3(NT), lds, s, v, logits, targets, inv_tokens, z_loss, z2, \
                     dlogits, row_loss)
    if (vocab <= 256 * 8 * 5) CANON_XENT(256, 5, true);
    else if (vocab <= 256 * 8 * 13) CANON_XENT(256, 13, true);
    else if (vocab <= 1024 * 8 * 7) CANON_XENT(1024, 7, false);
    else CANON_XENT(1024, 16, false);
#undef CANON_XENT
  }
  if (mean_loss)
    hipLaunchKernelGGL(mean_loss_kernel, dim3(1), dim3(256), 0, s, rows, row_loss, inv_tokens, mean_loss);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// D[bh][i] = R1 over d of fma(dO[i,d], O[i,d]) (bf16 operands, [T, ld] layout, head h at column h*hd).
// A row takes a group of G lanes (G = the chunk count rounded up to a power of two): lane r of the group
// runs the chain of chunk r over its 32 columns (16-byte loads when aligned, so the lanes of a group read the
// row's consecutive 64-byte pieces), and the group's first lane folds the chunk partials with Algorithm 2.
template <int G>
__global__ __launch_bounds__(256) void attn_rowdot_kernel(int64_t B, int64_t H, int64_t S, int64_t hd,
                                                          const uint16_t* __restrict__ dO,
                                                          const uint16_t* __restrict__ O, int64_t ld, int vec,
                                                          float* __restrict__ D) {
  const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = tid / G;
  const int r = (int)(tid % G);
  const int lane = threadIdx.x & 63;
  const bool live = row < B * H * S;
  const int nch = (int)((hd + kChunk - 1) / kChunk);
  float p = 0.0f;
  if (live && r < nch) {
    const int64_t i = row % S, bh = row / S, b = bh / H, h = bh % H;
    const int64_t off = (b * S + i) * ld + h * hd + (int64_t)r * kChunk;
    const uint16_t* a = dO + off;
    const uint16_t* o = O + off;
    const int64_t n = hd - (int64_t)r * kChunk < kChunk ? hd - (int64_t)r * kChunk : kChunk;
    if (vec && n == kChunk) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint4 av = reinterpret_cast<const uint4*>(a)[q];
        const uint4 ov = reinterpret_cast<const uint4*>(o)[q];
        const uint32_t aw[4] = {av.x, av.y, av.z, av.w}, ow[4] = {ov.x, ov.y, ov.z, ov.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p = __builtin_fmaf(__uint_as_float(aw[e] << 16), __uint_as_float(ow[e] << 16), p);
          p = __builtin_fmaf(__uint_as_float(aw[e] & 0xFFFF0000u), __uint_as_float(ow[e] & 0xFFFF0000u), p);
        }
      }
    } else {
      for (int64_t k = 0; k < n; ++k) p = __builtin_fmaf(bf16_to_f32(a[k]), bf16_to_f32(o[k]), p);
    }
  }
  float parts[G];
#pragma unroll
  for (int q = 0; q < G; ++q) parts[q] = __shfl(p, (lane & ~(G - 1)) + q, 64);
  if (live && r == 0) {
    LocalFold f;
    for (int q = 0; q < nch; ++q) f.push(parts[q]);
    D[row] = f.result();
  }
}

// head dims above 16 chunks: one thread per row, chunks in order
__global__ __launch_bounds__(256) void attn_rowdot_wide_kernel(int64_t B, int64_t H, int64_t S, int64_t hd,
                                                               const uint16_t* __restrict__ dO,
                                                               const uint16_t* __restrict__ O, int64_t ld,
                                                               float* __restrict__ D) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= B * H * S) return;
  const int64_t i = idx % S, bh = idx / S, b = bh / H, h = bh % H;
  const uint16_t* a = dO + (b * S + i) * ld + h * hd;
  const uint16_t* o = O + (b * S + i) * ld + h * hd;
  LocalFold f;
  for (int64_t c0 = 0; c0 < hd; c0 += kChunk) {
    float p = 0.0f;
    const int64_t c1 = c0 + kChunk < hd ? c0 + kChunk : hd;
    for (int64_t k = c0; k < c1; ++k) p = __builtin_fmaf(bf16_to_f32(a[k]), bf16_to_f32(o[k]), p);
    f.push(p);
  }
  D[idx] = f.result();
}

hipError_t attn_rowdot_launch(int64_t B, int64_t H, int64_t S, int64_t hd, const uint16_t* dO, const uint16_t* O,
                              int64_t ld, float* D, hipStream_t s) {
  const int64_t n = B * H * S;
  if (n == 0) return hipSuccess;
  const int64_t nch = (hd + kChunk - 1) / kChunk;
  if (nch > 16) {
    hipLaunchKernelGGL(attn_rowdot_wide_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, B, H, S, hd, dO,
                       O, ld, D);
    return hipGetLastError();
  }
  const int vec = ((uintptr_t)dO & 15) == 0 && ((uintptr_t)O & 15) == 0 && ld % 8 == 0 && hd % 8 == 0;
  auto go = [&](auto gc) {
    constexpr int G = decltype(gc)::value;
    const int64_t threads = n * G;
    hipLaunchKernelGGL(attn_rowdot_kernel<G>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, B, H, S, hd,
                       dO, O, ld, vec, D);
  };
  if (nch <= 1) go(std::integral_constant<int, 1>{});
  else if (nch <= 2) go(std::integral_constant<int, 2>{});
  else if (nch <= 4) go(std::integral_constant<int, 4>{});
  else if (nch <= 8) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 16>{});
  return hipGetLastError();
}

}  // namespace canon
