// gemm_split.hip - the canonical GEMM (R1, R2) for outputs too small to fill the chip: K split over wavefronts.
//
// The general kernel (gemm.hip) gives a 64 x 64 or 64 x 128 output tile to one workgroup, which runs the tile's
// chunks one after the other.  With fewer tiles than CUs that leaves the other CUs idle, and a workgroup alone on its
// CU also waits at every chunk's boundary (about 0.8 us per chunk of 0.43 us of matrix work).  Here a workgroup of 8
// wavefronts owns 16 RG x (64 / KB) outputs and the K chunks are dealt to (8 / RG) KB ranges: the wavefronts, and
// inside a wavefront the KB blocks of v_mfma_f32_16x16x1_4b_f32 that do not differ in their columns.  A range is
// G consecutive chunks, G a power of two and the range's start a multiple of it, so a range's fold is a complete
// (the last one: left-filled) subtree of Algorithm 2's tree, and the ranges' results are folded pairwise, a
// right neighbour without chunks passed over: the same additions in the same order as one binary-carry stack.
// What bounds it: the chain of the longest range, its chunk boundaries (fold, staging: vector instructions that take
// issue cycles from the matrix core) and, below about 8 us, the launch.
//
// A ragged last chunk is padded with products -0 * 1 = -0, and s + (-0) = s for every s, so its chain is the chain
// of its real terms.  Rows and columns beyond the matrix are loaded as its last row or column and not stored.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "canon_dev.h"
#include "canon_internal.h"

namespace canon {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int SW = 8;   // wavefronts of a workgroup (K ranges per block)
constexpr int KC = 32;  // chunk length
// Fold stack of a range: register levels, then private memory.  With two register levels the scratch accesses, one
// dependent round trip per four chunks, doubled a chunk's time.  Of at most 4095 chunks (the library's 12 levels) a
// range of RG row groups and KB K blocks holds up to 4096 / (SW / RG * KB), a power of two.
template <int KB>
constexpr int kRegLevels = KB == 1 ? 5 : 3;
constexpr int kMaxChunks = 4096;
template <int RG, int KB>
constexpr int mem_levels() {
  int levels = 1;
  while ((SW / RG * KB << (levels - 1)) < kMaxChunks) ++levels;
  return levels - kRegLevels<KB>;
}
constexpr uint32_t kPadA = 0x8000u, kPadB = 0x3F80u;  // bf16 -0 and 1

// K block of accumulator register v (KB > 1: the instruction's block v / 4 is column block * KB + K block)
template <int KB>
__device__ __forceinline__ constexpr int kblock(int v) { return (v >> 2) % KB; }

// Binary-carry stack over one wavefront's ranges, n[kb] chunks each; a push of local chunk q beyond a block's own
// chunks leaves that block's entries alone.
template <int KB, int LEVELS>
struct SplitMem {
  float s[LEVELS][16];
  __device__ __forceinline__ void push(v16f p, uint32_t c, const bool (&live)[KB]) {
    int L = 0;
    for (; c & 1; c >>= 1, ++L) {
#pragma unroll
      for (int v = 0; v < 16; ++v) p[v] = s[L][v] + p[v];
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (live[kblock<KB>(v)]) s[L][v] = p[v];
  }
  __device__ __forceinline__ void result(v16f& r, bool (&have)[KB], const uint32_t (&n)[KB], int lev) const {
#pragma unroll 1
    for (int L = 0; L < LEVELS; ++L, ++lev)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        if ((n[kb] >> lev) & 1) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (kblock<KB>(v) == kb) r[v] = have[kb] ? s[L][v] + r[v] : s[L][v];
          have[kb] = true;
        }
  }
};
template <int KB, int R>
struct SplitFold {
  v16f s;
  SplitFold<KB, R - 1> up;
  template <class Mem>
  __device__ __forceinline__ void push(const v16f& p, uint32_t c, const bool (&live)[KB], Mem& mem) {
    if (c & 1) {
      up.push(s + p, c >> 1, live, mem);
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (live[kblock<KB>(v)]) s[v] = p[v];
    }
  }
  // lowest occupied level first, then the others in ascending level order
  template <class Mem>
  __device__ __forceinline__ void result(v16f& r, bool (&have)[KB], const uint32_t (&n)[KB], int lev,
                                         const Mem& mem) const {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
      if ((n[kb] >> lev) & 1) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kblock<KB>(v) == kb) r[v] = have[kb] ? s[v] + r[v] : s[v];
        have[kb] = true;
      }
    up.result(r, have, n, lev + 1, mem);
  }
};
template <int KB>
struct SplitFold<KB, 0> {
  template <class Mem>
  __device__ __forceinline__ void push(const v16f& p, uint32_t c, const bool (&live)[KB], Mem& mem) {
    mem.push(p, c, live);
  }
  template <class Mem>
  __device__ __forceinline__ void result(v16f& r, bool (&have)[KB], const uint32_t (&n)[KB], int lev,
                                         const Mem& mem) const {
    mem.result(r, have, n, lev);
  }
};

typedef float v4f __attribute__((ext_vector_type(4)));

struct __attribute__((packed, aligned(2))) Vec8 {  // 8 elements at any element alignment
  uint32_t w[4];
};

// Operand blocks of 16 rows (columns) x 32 k: loaded by one wavefront, one 16-byte load per lane, and staged in LDS
// as widened fp32 rows of LDK floats (16-byte reads of 16 rows, and the k-major stores below, touch distinct banks).
// KCONT: k contiguous in memory, lane l loads k segment l % 4 of row l / 4.  Else k-major: lane l loads rows
// 8 (l % 2) .. + 7 of k = l / 2 and scatters them.
constexpr int LDK = KC + 4, BLOCK = 16 * LDK;  // floats
template <bool KCONT>
struct Stage {
  // idx0: the block's first row (all 16 inside the matrix when k-major); last: the matrix's last row.  WHOLE: the
  // chunk has 32 terms; else k >= K is pad (K >= 8; the load is moved back inside the row and shifted).  Byte offsets
  // stay below 2^32 (the launcher's bound).
  template <bool WHOLE>
  static __device__ __forceinline__ Vec8 load(const uint16_t* base, uint32_t ld, uint32_t idx0, uint32_t last,
                                              uint32_t k0, uint32_t K, uint32_t pad, int lane) {
    const char* p = reinterpret_cast<const char*>(base);
    if (KCONT) {
      const uint32_t row = idx0 + (lane >> 2), k = k0 + 8 * (lane & 3), kk = WHOLE || k + 8 <= K ? k : K - 8;
      Vec8 v = *reinterpret_cast<const Vec8*>(p + 2u * ((row < last ? row : last) * ld + kk));
      if (!WHOLE) {
        const uint32_t sh = k - kk, pp = pad | (pad << 16);
        auto down = [&](bool c, int words) {  // c: drop the lowest 2 words elements
          const uint32_t u[8] = {v.w[0], v.w[1], v.w[2], v.w[3], pp, pp, pp, pp};
#pragma unroll
          for (int x = 0; x < 4; ++x) v.w[x] = c ? u[x + words] : u[x];
        };
        const uint32_t u[5] = {v.w[0], v.w[1], v.w[2], v.w[3], pp};
#pragma unroll
        for (int x = 0; x < 4; ++x) v.w[x] = (sh & 1) ? (u[x] >> 16) | (u[x + 1] << 16) : u[x];
        down(sh & 2, 1);
        down(sh & 4, 2);
        down(sh >= 8, 4);
      }
      return v;
    }
    const uint32_t k = k0 + (lane >> 1), kk = WHOLE || k < K ? k : K - 1;
    Vec8 v = *reinterpret_cast<const Vec8*>(p + 2u * (kk * ld + idx0 + 8 * (lane & 1)));
    if (!WHOLE) {
#pragma unroll
      for (int x = 0; x < 4; ++x) v.w[x] = k < K ? v.w[x] : (pad | (pad << 16));
    }
    return v;
  }
  static __device__ __forceinline__ void store(float* blk, const Vec8& v, int lane) {
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = __uint_as_float((e & 1) ? (v.w[e >> 1] & 0xFFFF0000u) : (v.w[e >> 1] << 16));
    if (KCONT) {
      v4f* d = reinterpret_cast<v4f*>(blk + (lane >> 2) * LDK + 8 * (lane & 3));
      d[0] = v4f{f[0], f[1], f[2], f[3]};
      d[1] = v4f{f[4], f[5], f[6], f[7]};
    } else {
      float* d = blk + 8 * (lane & 1) * LDK + (lane >> 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e * LDK] = f[e];
    }
  }
};

// RG row groups of 16 rows x S = 8 / RG K ranges per instruction block: wavefront w = s RG + rg.  The RG wavefronts
// of a range share its staged operands (two buffers, a barrier per chunk); with RG = 1 a wavefront stages for itself
// (one buffer: its LDS operations complete in order) and no barrier is needed before the fold.
// CZ: the causal chunk ranges (KMODE_TRAIL, KMODE_LEAD, windows, K segments) as in gemm.hip, for this tile's
// rows; a chunk outside them is a +0 partial.  KB = 1 only.
template <bool TA, bool TB, int RG, int KB, bool CZ>
__global__ __launch_bounds__(64 * SW, 2) void gemm_split_kernel(GemmArgs g, uint32_t tiles_m, uint32_t tiles,
                                                                uint32_t G) {
  static_assert(RG == 1 || KB == 1, "row groups or K blocks");
  constexpr int S = SW / RG, R = S * KB, TM = 16 * RG, TN = 64 / KB;
  typedef Stage<!TA> SA;
  typedef Stage<TB> SB;
  constexpr int NA = RG > 1 ? RG : KB;                         // staged blocks of A (and 4 of B) per range
  constexpr int NBUF = RG > 1 ? 2 : 1, RBUF = (NA + 4) * BLOCK;  // floats per buffer
  constexpr int LOADA = RG > 1 ? 1 : KB, LOADB = 4 / RG;       // blocks each wavefront loads
  constexpr int PFLOATS = SW * 16 * 64;                        // the ranges' results
  __shared__ __attribute__((aligned(16))) float lds[RBUF * NBUF * S > PFLOATS ? RBUF * NBUF * S : PFLOATS];
  // each XCD (every 8th workgroup) takes a contiguous run of the batch's tiles, row tiles fastest, so that its L2 holds
  // a few column panels or matrices (40 x 64 x 128 x 512, four tiles each: 10.1 us; numbered within each matrix, half
  // of the XCDs had no work, 19.2)
  const uint32_t at = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const uint32_t z = at / tiles, tile = at - z * tiles;
  if (z >= (uint32_t)g.batch) return;
  const uint32_t tn = tile / tiles_m, tm = tile - tn * tiles_m;
  const uint32_t nb2 = (uint32_t)g.nb2, z1 = z / nb2, z2 = z - z1 * nb2;
  const uint16_t* A = g.a + z1 * g.sa1 + z2 * g.sa2;
  const uint16_t* B = g.b + z1 * g.sb1 + (g.b_group > 1 ? z2 / (uint32_t)g.b_group : z2) * g.sb2;
  const uint32_t m = (uint32_t)g.m, n = (uint32_t)g.n, K = (uint32_t)g.k, nc = (K + KC - 1) / KC;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rg = w % RG, ws = w / RG;
  // this wavefront's rows; a block past the matrix's end is loaded as its last 16 rows (or columns)
  const uint32_t row0 = tm * TM + 16 * rg, col0 = tn * TN;
  const uint32_t lrow0 = row0 + 16 > m ? m - 16 : row0;
  auto lcol0 = [&](int cb) {
    const uint32_t c = col0 + 16 * cb;
    return c + 16 > n ? n - 16 : c;
  };

  // causal range of real chunks within each K segment of spc chunks
  uint32_t spc = nc, lb = 0, le = nc;
  if (CZ) {
    if (g.kseg > 0) spc = (uint32_t)g.kseg / KC;
    le = spc;
    const int64_t r0 = tm * TM, last = r0 + TM < m ? r0 + TM : m, win = g.kwin;
    if (g.kmode == KMODE_TRAIL) {
      const uint32_t ce = (uint32_t)((last + KC - 1) / KC);
      le = ce < spc ? ce : spc;
      if (win > 0 && r0 - win + 1 > 0) {
        const uint32_t cb = (uint32_t)((r0 - win + 1) / KC);
        lb = cb < le ? cb : le;
      }
    } else if (g.kmode == KMODE_LEAD) {
      lb = (uint32_t)(r0 / KC) < spc ? (uint32_t)(r0 / KC) : spc;
      if (win > 0) {
        const int64_t ce = (last - 2 + win) / KC + 1;
        le = ce < (int64_t)spc ? (uint32_t)ce : spc;
        if (le < lb) le = lb;
      }
    }
  }
  // real chunks among the first c
  auto reals = [&](uint32_t c) {
    const uint32_t sg = g.kseg > 0 ? c / spc : 0u, cl = c - sg * spc;
    return sg * (le - lb) + (cl < lb ? 0u : (cl < le ? cl : le) - lb);
  };

  uint32_t cnt[KB], first[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    first[kb] = (ws * KB + kb) * G;
    cnt[kb] = first[kb] >= nc ? 0u : (nc - first[kb] < G ? nc - first[kb] : G);
  }
  v16f r;
#pragma unroll
  for (int v = 0; v < 16; ++v) r[v] = 0.0f;
  const uint32_t n0 = cnt[0];  // the longest of this wavefront's ranges
  float* la = lds + ws * NBUF * RBUF;
  struct Raw {
    Vec8 a[LOADA], b[LOADB];
  };
  auto load_as = [&](auto whole, uint32_t q, Raw& x) {
    int l = lane;
    if (!whole.value) asm volatile("" : "+v"(l));  // the rare path's masks are not kept live across the loop
#pragma unroll
    for (int i = 0; i < LOADA; ++i) {  // K block i; a range without this chunk: loaded, never folded
      const uint32_t c = first[i] + q < nc ? first[i] + q : nc - 1;
      x.a[i] = SA::template load<whole.value>(A, (uint32_t)g.lda, lrow0, m - 1, c * KC, K, kPadA, l);
    }
#pragma unroll
    for (int i = 0; i < LOADB; ++i) {
      const int b = RG > 1 ? rg + RG * i : i;  // block b: column block b / KB, K block b % KB
      const uint32_t c = first[b % KB] + q < nc ? first[b % KB] + q : nc - 1;
      x.b[i] = SB::template load<whole.value>(B, (uint32_t)g.ldb, lcol0(b / KB), n - 1, c * KC, K, kPadB, l);
    }
  };
  const uint32_t cfull = K / KC;  // chunks with 32 terms
  auto load = [&](uint32_t q, Raw& x) {
    if (first[KB - 1] + q < cfull) load_as(std::true_type{}, q, x);
    else load_as(std::false_type{}, q, x);
  };
  auto stage = [&](const Raw& x, int buf) {
    float* d = la + buf * RBUF;
#pragma unroll
    for (int i = 0; i < LOADA; ++i) SA::store(d + (RG > 1 ? rg : i) * BLOCK, x.a[i], lane);
#pragma unroll
    for (int i = 0; i < LOADB; ++i) SB::store(d + (NA + (RG > 1 ? rg + RG * i : i)) * BLOCK, x.b[i], lane);
    __builtin_amdgcn_wave_barrier();
  };
  const int blk = lane >> 4;
  const float* fa0 = la + (RG > 1 ? rg : blk % KB) * BLOCK + (lane & 15) * LDK;
  const float* fb0 = la + (NA + blk) * BLOCK + (lane & 15) * LDK;
  auto frag = [&](int buf, int g4, v4f& ya, v4f& yb) {
    ya = *reinterpret_cast<const v4f*>(fa0 + buf * RBUF + 4 * g4);
    yb = *reinterpret_cast<const v4f*>(fb0 + buf * RBUF + 4 * g4);
  };
  SplitFold<KB, kRegLevels<KB>> fold;
  SplitMem<KB, mem_levels<RG, KB>()> mem;
  uint32_t pos = 0;  // local chunks pushed
  auto push = [&](const v16f& p) {
    bool live[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) live[kb] = pos < cnt[kb];
    fold.push(p, pos, live, mem);
    ++pos;
  };
  auto next = [&](uint32_t q) {  // the next real local chunk after q, or n0
    ++q;
    if (CZ && q < n0) {
      const uint32_t c = first[0] + q, cl = g.kseg > 0 ? c % spc : c;
      if (lb >= le) q = n0;
      else if (cl < lb) q += lb - cl;
      else if (cl >= le) q += spc - cl + lb;  // the next segment's first
    }
    return q < n0 ? q : n0;
  };
  // One chunk: local chunk qa, staged in buffer buf.  x holds the operands of qb, the next one: they are staged
  // under this chunk's last products, and then x receives those of qd, three chunks ahead.
  v4f fa, fb;
  auto chunk = [&](uint32_t qa, uint32_t qb, uint32_t qd, int buf, Raw& x) {
    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    if (CZ)
      while (pos < qa) push(acc);  // skipped chunks: +0
    if (RG > 1) frag(buf, 0, fa, fb);
#pragma unroll
    for (int g4 = 0; g4 < KC / 4; ++g4) {
      v4f na = fa, nb = fb;
      if (g4 + 1 < KC / 4) frag(buf, g4 + 1, na, nb);
      if (g4 + 1 == KC / 4 && qb < n0) {
        stage(x, RG > 1 ? buf ^ 1 : 0);
        if (qd < n0) load(qd, x);
        if (RG == 1) frag(0, 0, na, nb);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(fa[e], fb[e], acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      fa = na;
      fb = nb;
    }
    push(acc);
  };
  // chunks every range's wavefronts step through together (RG > 1): the largest count of real chunks
  uint32_t steps = n0;
  if (RG > 1) {
    steps = nc < G ? nc : G;
    if (CZ) {
      steps = 0;
      for (uint32_t c0 = 0; c0 < nc; c0 += G) {
        const uint32_t k = reals(c0 + G < nc ? c0 + G : nc) - reals(c0);
        steps = k > steps ? k : steps;
      }
    }
  }
  Raw x0, x1;
  uint32_t qa = next(~0u), qb = next(qa), qc = next(qb);
  if (qa < n0) {
    load(qa, x0);
    if (qb < n0) load(qb, x1);
    stage(x0, 0);
    if (qc < n0) load(qc, x0);
    if (RG == 1) frag(0, 0, fa, fb);
  }
  if (RG > 1) __syncthreads();
  for (uint32_t j = 0; j < steps; j += 2) {
    if (RG == 1 && qa >= n0) break;
    const uint32_t qd = next(qc), qe = next(qd);
    if (qa < n0) chunk(qa, qb, qd, 0, x1);
    if (RG > 1) __syncthreads();
    if (RG > 1 ? j + 1 < steps : qb < n0) {
      if (qb < n0) chunk(qb, qc, qe, NBUF - 1, x0);
      if (RG > 1) __syncthreads();
    }
    qa = qc;
    qb = qd;
    qc = qe;
  }
  if (CZ) {
    v16f z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.0f;
    while (pos < n0) push(z);
  }
  {
    bool have[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) have[kb] = false;
    fold.result(r, have, cnt, 0, mem);
  }
  __syncthreads();
  float(*part)[16][64] = reinterpret_cast<float(*)[16][64]>(lds);
  if (n0 > 0) {
#pragma unroll
    for (int v = 0; v < 16; ++v) part[w][v][lane] = r[v];
  }
  __syncthreads();

  // Outputs of row group rg: register u = (column block cb, rr) of lane l is row rr + 4 (l / 16), column l % 16 of
  // the block; its range kb of K range s is accumulator (cb * KB + kb) * 4 + rr of wavefront s RG + rg.
  const uint32_t nr = (nc + G - 1) / G;  // ranges with chunks
  if (row0 >= m) return;
#pragma unroll
  for (int u = ws; u < 16 / KB; u += S) {
    const int cb = u >> 2, rr = u & 3;
    float x[R];
#pragma unroll
    for (int q = 0; q < R; ++q)
      x[q] = (uint32_t)q < nr ? part[(q / KB) * RG + rg][((cb * KB + q % KB) << 2) + rr][lane] : 0.0f;
#pragma unroll
    for (int s = 1; s < R; s <<= 1)
#pragma unroll
      for (int q = 0; q + s < R; q += 2 * s)
        if ((uint32_t)(q + s) < nr) x[q] = x[q] + x[q + s];
    const float d = x[0];
    const uint32_t i = lrow0 + rr + 4 * (lane >> 4), j = lcol0(cb) + (lane & 15);
    if (i >= row0 && j >= col0 + 16 * cb) {
      const int64_t o = z1 * g.sc1 + z2 * g.sc2 + (int64_t)i * g.ldc + j;
      float* C = (float*)g.c;
      if (g.epi == EPI_RES) {
        C[o] = (g.res + z1 * g.sc1 + z2 * g.sc2)[(int64_t)i * g.ldres + j] + d;
      } else if (g.epi == EPI_ACCUM) {
        const float t = d * g.epi_scale;
        C[o] = C[o] + t;
      } else if (g.out_bf16) {
        ((uint16_t*)g.c)[o] = f32_to_bf16(d);
      } else {
        C[o] = d;
      }
    }
  }
}

template <bool TA, bool TB>
hipError_t launch(const GemmArgs& g, int cfg, bool cz, hipStream_t s) {
  const int rg = cfg >> 4, kb = cfg & 15;
  const uint32_t tm = (uint32_t)((g.m + 16 * rg - 1) / (16 * rg)), tn = (uint32_t)((g.n + 64 / kb - 1) / (64 / kb));
  const uint32_t tiles = tm * tn, nc = (uint32_t)((g.k + KC - 1) / KC);
  uint32_t G = 1;
  while (G * (SW / rg) * kb < nc) G <<= 1;
  const dim3 grid((unsigned)((tiles * g.batch + 7) / 8 * 8)), block(64 * SW);  // (at most a workgroup per CU)
#define CANON_SPLIT(RG, KB, CZ) \
  hipLaunchKernelGGL((gemm_split_kernel<TA, TB, RG, KB, CZ>), grid, block, 0, s, g, tm, tiles, G)
  if (cz) {
    if (rg == 1) CANON_SPLIT(1, 1, true);
    else CANON_SPLIT(2, 1, true);
  } else if (rg == 2) CANON_SPLIT(2, 1, false);
  else if (kb == 1) CANON_SPLIT(1, 1, false);
  else if (kb == 2) CANON_SPLIT(1, 2, false);
  else CANON_SPLIT(1, 4, false);
#undef CANON_SPLIT
  return hipGetLastError();
}

}  // namespace

// The configuration (16 * row groups + K blocks) to run g with, or 0 when the general kernel is the better one: the
// smallest split whose workgroups still find a CU each.  Measured at K = 4096, row/row, against the general kernel
// (us): 256 x 256 (1, 4) 15 against 99; 100 x 1000 (1, 2) 21 against 100; 256 x 768 (1, 1) 32 against 100;
// 512 x 1024 (2, 1) 57 against 101.  One step further, 1024 x 1024 in 256 tiles of 64 rows, it ties (97-110
// against 101), and with two workgroups on a CU it loses (333 x 1555 (2, 1) 108 against 101).
// Causal products of S queries (split against general, us; h heads of 64): P.V, S = 512, 8 heads (1, 1) 9.0 against 39;
// S = 2048, 4 heads (2, 1) 35 against 138, with a window of 100 15 against 27; dK / dV, S = 2048, 4 heads (2, 1) 33
// against 65, window 512 25 against 26, window 100 14 against 15; 4 query heads per key head, 16 heads (2, 1) 113 against
// 254, window 20 29 against 49.  Only dK / dV of one head with a window that is short in a long sequence loses, where
// the real chunks lie in one or two of the four ranges and the others push their +0: S = 4096, 2 heads 18.0 against
// 15.0 (window 20), 30 against 29 (512), 45 against 43 (1024); S = 8192, 1 head 56 against 48 (1024).  With one row group
// the split is the faster one there too (S = 4096, 1 head, window 20 9.9 against 14.5).
int gemm_split_config(const GemmArgs& g, int64_t cus) {
  const int64_t lim = int64_t(1) << 30;  // operand elements: byte offsets below 2^32
  if (g.epi == EPI_DS || g.tri_lower || g.m < 16 || g.n < 16 || g.m > lim || g.n > lim || g.k < 8) return 0;
  if ((g.trans_a ? g.k : g.m) * g.lda > lim || (g.trans_b ? g.n : g.k) * g.ldb > lim) return 0;
  if (g.nb2 < 1 || g.batch > 65535) return 0;
  auto fits = [&](int64_t rows, int64_t cols) {
    return ((g.m + rows - 1) / rows) * ((g.n + cols - 1) / cols) * g.batch <= cus;
  };
  const int64_t nc = (g.k + KC - 1) / KC;
  if (g.kmode == KMODE_FULL && g.kseg == 0) {
    if (nc >= 48 && fits(16, 16)) return 16 + 4;  // below 48 chunks 32 ranges leave wavefronts idle (K = 256: 6.0 against 5.1)
    if (nc >= 2 && fits(16, 32)) return 16 + 2;
  }
  if (fits(16, 64)) return 16 + 1;
  const bool short_window = g.kmode == KMODE_LEAD && g.kseg == 0 && g.kwin > 0 && 4 * g.kwin <= g.k && nc >= 128;
  if (fits(32, 64) && !short_window) return 32 + 1;
  return 0;
}

hipError_t gemm_split_launch(const GemmArgs& g, int cfg, hipStream_t s) {
  const bool cz = g.kmode != KMODE_FULL || g.kseg > 0;
  if (!g.trans_a && g.trans_b) return launch<false, true>(g, cfg, cz, s);
  if (!g.trans_a) return launch<false, false>(g, cfg, cz, s);
  if (!g.trans_b) return launch<true, false>(g, cfg, cz, s);
  return launch<true, true>(g, cfg, cz, s);
}

}  // namespace canon
