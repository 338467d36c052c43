// hash.hip - the canonical state hash H1 on the device.
//
// H1 (this library's definition; the paper hashes every step's state on the host and leaves the function
// open): SHA-256 (FIPS 180-4) over a fixed tree.
//   * a tensor of n bytes is cut into nb = ceil(n/64) blocks of 64 bytes (the last may be shorter) and
//     W = max(1, ceil(nb/1024)) leaves; leaf l holds blocks l, l+W, l+2W, ... in order (interleaved, so the
//     lanes of a wavefront, one leaf each, read neighbouring blocks);
//   * leaf digest = SHA-256(leaf bytes); the leaf digests fold pairwise level by level,
//     SHA-256(left || right), an odd last node passing up unchanged;
//   * tensor digest = SHA-256(0x02 || index as 8 bytes LE || n as 8 bytes LE || root);
//   * state digest = SHA-256(0x03 || tensor digests in order).
// Integer arithmetic only: the result is the same on every device.
#include <hip/hip_runtime.h>

#include "canon_internal.h"

namespace canon {

// SHA-256 round constants and initial state (FIPS 180-4, sections 4.2.2 and 5.3.3)
constexpr uint32_t kSha256K[64] = {
    0x428a2f98u, 0x71374491u, 0xb5c0fbcfu, 0xe9b5dba5u, 0x3956c25bu, 0x59f111f1u, 0x923f82a4u, 0xab1c5ed5u,
    0xd807aa98u, 0x12835b01u, 0x243185beu, 0x550c7dc3u, 0x72be5d74u, 0x80deb1feu, 0x9bdc06a7u, 0xc19bf174u,
    0xe49b69c1u, 0xefbe4786u, 0x0fc19dc6u, 0x240ca1ccu, 0x2de92c6fu, 0x4a7484aau, 0x5cb0a9dcu, 0x76f988dau,
    0x983e5152u, 0xa831c66du, 0xb00327c8u, 0xbf597fc7u, 0xc6e00bf3u, 0xd5a79147u, 0x06ca6351u, 0x14292967u,
    0x27b70a85u, 0x2e1b2138u, 0x4d2c6dfcu, 0x53380d13u, 0x650a7354u, 0x766a0abbu, 0x81c2c92eu, 0x92722c85u,
    0xa2bfe8a1u, 0xa81a664bu, 0xc24b8b70u, 0xc76c51a3u, 0xd192e819u, 0xd6990624u, 0xf40e3585u, 0x106aa070u,
    0x19a4c116u, 0x1e376c08u, 0x2748774cu, 0x34b0bcb5u, 0x391c0cb3u, 0x4ed8aa4au, 0x5b9cca4fu, 0x682e6ff3u,
    0x748f82eeu, 0x78a5636fu, 0x84c87814u, 0x8cc70208u, 0x90befffau, 0xa4506cebu, 0xbef9a3f7u, 0xc67178f2u};
constexpr uint32_t kSha256H0[8] = {0x6a09e667u, 0xbb67ae85u, 0x3c6ef372u, 0xa54ff53au,
                                   0x510e527fu, 0x9b05688cu, 0x1f83d9abu, 0x5be0cd19u};


constexpr uint32_t rotr_c(uint32_t x, int n) { return (x >> n) | (x << (32 - n)); }
// round constant + schedule word of the padding block that follows a 64-byte message (a node of the tree): constants
struct PadKw {
  uint32_t v[64];
  constexpr PadKw() : v{} {
    uint32_t w[64] = {};
    w[0] = 0x80000000u;
    w[15] = 512u;
    for (int t = 16; t < 64; ++t) {
      const uint32_t s0 = rotr_c(w[t - 15], 7) ^ rotr_c(w[t - 15], 18) ^ (w[t - 15] >> 3);
      const uint32_t s1 = rotr_c(w[t - 2], 17) ^ rotr_c(w[t - 2], 19) ^ (w[t - 2] >> 10);
      w[t] = w[t - 16] + s0 + w[t - 7] + s1;
    }
    for (int t = 0; t < 64; ++t) v[t] = kSha256K[t] + w[t];
  }
};
constexpr PadKw kPadKw{};

__device__ __forceinline__ uint32_t rotr(uint32_t x, int n) { return (x >> n) | (x << (32 - n)); }
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);  // one instruction for two XORs
}

// the working variables of one compression
struct ShaVars {
  uint32_t a, b, c, d, e, f, g, h;
  __device__ __forceinline__ void from(const uint32_t (&s)[8]) {
    a = s[0]; b = s[1]; c = s[2]; d = s[3]; e = s[4]; f = s[5]; g = s[6]; h = s[7];
  }
  __device__ __forceinline__ void add_to(uint32_t (&s)[8]) const {
    s[0] += a; s[1] += b; s[2] += c; s[3] += d; s[4] += e; s[5] += f; s[6] += g; s[7] += h;
  }
  // one round, kw = round constant + schedule word: 14 vector instructions
  __device__ __forceinline__ void round(uint32_t kw) {
    const uint32_t S1 = xor3(rotr(e, 6), rotr(e, 11), rotr(e, 25));
    const uint32_t ch = __builtin_amdgcn_bitop3_b32(e, f, g, 0xCA);  // e ? f : g
    const uint32_t x = h + kw + ch;
    const uint32_t S0 = xor3(rotr(a, 2), rotr(a, 13), rotr(a, 22));
    const uint32_t mj = __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);  // majority
    const uint32_t y = S0 + mj + x;
    h = g; g = f; f = e; e = x + S1 + d;
    d = c; c = b; b = a; a = y + S1;
  }
  // the rounds so far are done here: the compiler would otherwise move them past the barriers that follow
  __device__ __forceinline__ void pin() {
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(e), "+v"(f), "+v"(g), "+v"(h));
  }
  __device__ __forceinline__ void rounds16(const uint32_t (&kw)[16]) {
#pragma unroll
    for (int t = 0; t < 16; ++t) round(kw[t]);
  }
};

__device__ __forceinline__ void sha_init(uint32_t (&s)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) s[i] = kSha256H0[i];
}

// the next 16 words of the message schedule
__device__ __forceinline__ void expand16(uint32_t (&w)[16]) {
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const uint32_t w15 = w[(t + 1) & 15], w2 = w[(t + 14) & 15];
    const uint32_t s0 = xor3(rotr(w15, 7), rotr(w15, 18), w15 >> 3);
    const uint32_t s1 = xor3(rotr(w2, 17), rotr(w2, 19), w2 >> 10);
    w[t] = w[t] + s0 + (w[(t + 9) & 15] + s1);
  }
}

// a whole compression of one block (big-endian words; w is used up)
__device__ __forceinline__ void compress(uint32_t (&s)[8], uint32_t (&w)[16]) {
  ShaVars v;
  v.from(s);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q) expand16(w);
    uint32_t kw[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) kw[t] = w[t] + kSha256K[16 * q + t];
    v.rounds16(kw);
  }
  v.add_to(s);
}

// SHA-256(left || right), the two digests as 16 words
__device__ __forceinline__ void hash_node(uint32_t (&s)[8], uint32_t (&w)[16]) {
  sha_init(s);
  compress(s, w);
  ShaVars v;
  v.from(s);
#pragma unroll
  for (int t = 0; t < 64; ++t) v.round(kPadKw.v[t]);
  v.add_to(s);
}

// Level by level fold of m digests in a (8 words each), b the other buffer of the ping-pong: pairs are hashed, an odd
// last one passes up unchanged.  All threads of the workgroup call it; returns the buffer with the result in front.
template <int THREADS>
__device__ __forceinline__ uint32_t* fold_digests(uint32_t* a, uint32_t* b, int64_t m) {
  while (m > 1) {
    const int64_t pairs = m / 2;
    for (int64_t i = threadIdx.x; i < (m + 1) / 2; i += THREADS) {
      uint32_t out[8];
      if (i < pairs) {
        uint32_t w[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) w[k] = a[16 * i + k];
        hash_node(out, w);
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) out[k] = a[16 * i + k];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) b[8 * i + k] = out[k];
    }
    __syncthreads();
    uint32_t* t = a;
    a = b;
    b = t;
    m = (m + 1) / 2;
  }
  return a;
}

__device__ __forceinline__ uint32_t bswap(uint32_t x) { return __builtin_bswap32(x); }

struct __attribute__((packed)) Bytes16 {  // 16 bytes at any alignment (global loads need none on gfx950)
  uint32_t w[4];
};

// Leaves of one tensor and the first levels of its tree: a workgroup takes 64 PAIRS leaves, one per lane of PAIRS
// wavefronts, and folds their digests to one node.  A leaf is a serial chain of up to 1024 compressions, and a state
// of a few GB has little more than one wavefront of leaves per SIMD, so what counts is how long a lane takes for one
// block.  A wavefront that runs the rounds (14 instructions each) has a partner that loads the blocks one ahead and
// expands the message schedule (10 instructions per word), 16 words at a time through two LDS buffers and a barrier;
// the rounds use a group of 16 one barrier after they read it.  A wavefront alone on its SIMD issues a vector
// instruction every 5.5 to 9 cycles, so the 903 instructions of a block's rounds take 2.3 us.  Rounds and schedule in
// one lane, 1698 instructions with the loads exposed, took 3.6-4.4 us: a tensor of 1 MB 3.7 ms, now 2.4; 60 tensors of
// 1 MB 5.0 ms, now 2.4; 4.8 GB 6.9 ms, now 5.4.  PAIRS = 1 spreads few leaves over the SIMDs; PAIRS = 4 gives the four
// SIMDs of a CU equal shares, which is what counts once every SIMD has several wavefronts and the 1448 instructions
// of a block are the bound (12 GB: 8.1 ms against 10.6 with PAIRS = 1, and 10.1 before).
template <int PAIRS>
__global__ __launch_bounds__(128 * PAIRS) void hash_leaves_kernel(const HashTensor* __restrict__ tens,
                                                                  const int32_t* __restrict__ wg_tensor,
                                                                  const int64_t* __restrict__ wg_first,
                                                                  uint32_t* __restrict__ node_out) {
  constexpr int LEAVES = 64 * PAIRS;
  __shared__ uint32_t kw[PAIRS][2][16][64];
  const HashTensor T = tens[wg_tensor[blockIdx.x]];
  const int64_t first = wg_first[blockIdx.x], W = T.leaves, n = T.nbytes, nfull = n / 64;
  const int tail = (int)(n - nfull * 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, pair = wv % PAIRS;
  const int64_t l = first + 64 * pair + lane;
  // blocks of leaf l: its whole blocks l, l + W, ..., the partial last block of the tensor if it is the next one,
  // and the padding
  const int64_t mine = l < W ? (nfull > l ? (nfull - 1 - l) / W + 1 : 0) : 0;
  const bool owns = l < W && tail > 0 && nfull % W == l;
  const int fill = owns ? tail : 0;
  const int64_t count = l < W ? mine + (fill >= 56 ? 2 : 1) : 0;
  const int64_t most = (nfull > first ? (nfull - 1 - first) / W + 1 : 0) + (tail >= 56 ? 2 : 1);  // of the workgroup
  if (wv >= PAIRS) {
    const uint8_t* base = static_cast<const uint8_t*>(T.ptr);
    Bytes16 nx[4];
    auto fetch = [&](int64_t i) {
      if (i < mine) {
        const Bytes16* p = reinterpret_cast<const Bytes16*>(base + (l + i * W) * 64);
#pragma unroll
        for (int q = 0; q < 4; ++q) nx[q] = p[q];
      }
    };
    fetch(0);
    for (int64_t i = 0; i < most; ++i) {
      uint32_t w[16] = {};
      if (i < mine) {
#pragma unroll
        for (int t = 0; t < 16; ++t) w[t] = bswap(nx[t >> 2].w[t & 3]);
      } else if (i < count) {  // the partial block and the padding
        const int64_t j = i - mine;
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          uint32_t x = 0;
          for (int e = 0; e < 4; ++e) {
            const int at = 64 * (int)(j < 2 ? j : 2) + 4 * t + e;
            const uint32_t v = at < fill ? base[nfull * 64 + at] : (at == fill ? 0x80u : 0u);
            x = (x << 8) | v;
          }
          w[t] = x;
        }
        if (i + 1 == count) {
          const uint64_t bits = 8 * (uint64_t)(mine * 64 + fill);
          w[14] = (uint32_t)(bits >> 32);
          w[15] = (uint32_t)bits;
        }
      }
      fetch(i + 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q) expand16(w);
#pragma unroll
        for (int t = 0; t < 16; ++t) kw[pair][q & 1][t][lane] = w[t] + kSha256K[16 * q + t];
        __syncthreads();
      }
    }
    __syncthreads();
  } else {
    uint32_t s[8];
    sha_init(s);
    ShaVars v;
    uint32_t ka[16], kb[16];
    auto take = [&](int q, uint32_t (&k)[16]) {
      __syncthreads();
#pragma unroll
      for (int t = 0; t < 16; ++t) k[t] = kw[pair][q & 1][t][lane];
    };
    take(0, ka);
    for (int64_t i = 0; i < most; ++i) {
      v.from(s);
      take(1, kb);
      v.rounds16(ka);
      v.pin();
      take(2, ka);
      v.rounds16(kb);
      v.pin();
      take(3, kb);
      v.rounds16(ka);
      v.pin();
      if (i + 1 < most) take(0, ka);
      v.rounds16(kb);
      if (i < count) v.add_to(s);
    }
    __syncthreads();
    uint32_t* d = &kw[0][0][0][0] + 8 * (64 * pair + lane);
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = s[k];
  }
  __syncthreads();
  uint32_t* buf = &kw[0][0][0][0];
  const uint32_t* r = fold_digests<128 * PAIRS>(buf, buf + 8 * LEAVES, W - first < LEAVES ? W - first : LEAVES);
  if (threadIdx.x < 8) node_out[8 * (T.node_offset + first / LEAVES) + threadIdx.x] = r[threadIdx.x];
}

// The upper levels of each tensor's tree (one workgroup per tensor, ping-pong between two buffers), then the tensor
// digest: SHA-256 of 49 bytes, one block.
__global__ __launch_bounds__(256) void hash_tree_kernel(const HashTensor* __restrict__ tens, int64_t group,
                                                        uint32_t* bufA, uint32_t* bufB,
                                                        uint32_t* __restrict__ tensor_out) {
  const HashTensor T = tens[blockIdx.x];
  const uint32_t* r = fold_digests<256>(bufA + 8 * T.node_offset, bufB + 8 * T.node_offset,
                                        (T.leaves + group - 1) / group);
  if (threadIdx.x != 0) return;
  // 0x02, index and byte count (8 bytes each, little-endian), root, 0x80, length 392 bits
  const uint32_t i0 = bswap(blockIdx.x), n0 = bswap((uint32_t)T.nbytes), n1 = bswap((uint32_t)(T.nbytes >> 32));
  uint32_t w[16] = {0x02000000u | (i0 >> 8), i0 << 24, n0 >> 8, (n0 << 24) | (n1 >> 8), (n1 << 24) | (r[0] >> 8)};
#pragma unroll
  for (int k = 0; k < 7; ++k) w[5 + k] = (r[k] << 24) | (r[k + 1] >> 8);
  w[12] = (r[7] << 24) | 0x00800000u;
  w[13] = 0;
  w[14] = 0;
  w[15] = 392;
  uint32_t s[8];
  sha_init(s);
  compress(s, w);
#pragma unroll
  for (int k = 0; k < 8; ++k) tensor_out[8 * blockIdx.x + k] = s[k];
}

// state digest = SHA-256(0x03 || tensor digests); written as 32 bytes.  One wavefront: the schedules of 64 blocks at
// a time are expanded one per lane, then every lane runs the serial rounds.
__global__ __launch_bounds__(64) void hash_state_kernel(int64_t n_tensors, const uint32_t* __restrict__ td,
                                                        uint8_t* __restrict__ out) {
  __shared__ uint32_t kw[64][64];  // [word][block]
  const int64_t words = 8 * n_tensors, blocks = (32 * n_tensors + 1 + 9 + 63) / 64;
  uint32_t s[8];
  sha_init(s);
  for (int64_t b0 = 0; b0 < blocks; b0 += 64) {
    const int64_t b = b0 + threadIdx.x;
    if (b < blocks) {
      uint32_t w[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) {  // the message is the digests' words one byte later
        const int64_t j = 16 * b + t;
        const uint32_t hi = j == 0 ? 0x03u : (j - 1 < words ? td[j - 1] & 0xFFu : 0u);
        const uint32_t lo = j < words ? td[j] >> 8 : (j == words ? 0x800000u : 0u);
        w[t] = (hi << 24) | lo;
      }
      if (b + 1 == blocks) {
        const uint64_t bits = 8 * (uint64_t)(32 * n_tensors + 1);
        w[14] = (uint32_t)(bits >> 32);
        w[15] = (uint32_t)bits;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q) expand16(w);
#pragma unroll
        for (int t = 0; t < 16; ++t) kw[16 * q + t][threadIdx.x] = w[t] + kSha256K[16 * q + t];
      }
    }
    __syncthreads();
    const int64_t here = blocks - b0 < 64 ? blocks - b0 : 64;
    for (int64_t i = 0; i < here; ++i) {
      ShaVars v;
      v.from(s);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t k[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) k[t] = kw[16 * q + t][i];
        v.rounds16(k);
      }
      v.add_to(s);
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int k = 0; k < 8; ++k)
    for (int i = 0; i < 4; ++i) out[4 * k + i] = (uint8_t)(s[k] >> (24 - 8 * i));
}

// Leaves per workgroup for a state of so many leaves in all (a fixed line, the same on every
// device): from one and a half groups of 256 per CU on, the four-pair workgroups are the faster ones.
int64_t hash_leaf_group(int64_t total_leaves) { return total_leaves >= 256 * 384 ? 256 : kHashLeafGroupMin; }

int64_t hash_leaf_count(int64_t nbytes) {
  const int64_t nb = (nbytes + 63) / 64;
  const int64_t w = (nb + 1023) / 1024;
  return w < 1 ? 1 : w;
}

hipError_t hash_launch(int64_t n_tensors, const HashTensor* tens_dev, int64_t group, int64_t n_wg,
                       const int32_t* wg_tensor, const int64_t* wg_first, uint32_t* node_a, uint32_t* node_b,
                       uint32_t* tensor_digests, uint8_t* out, hipStream_t s) {
  if (n_wg > 0 && group == kHashLeafGroupMin)
    hipLaunchKernelGGL(hash_leaves_kernel<1>, dim3((unsigned)n_wg), dim3(128), 0, s, tens_dev, wg_tensor, wg_first,
                       node_a);
  else if (n_wg > 0)
    hipLaunchKernelGGL(hash_leaves_kernel<4>, dim3((unsigned)n_wg), dim3(512), 0, s, tens_dev, wg_tensor, wg_first,
                       node_a);
  if (n_tensors > 0)
    hipLaunchKernelGGL(hash_tree_kernel, dim3((unsigned)n_tensors), dim3(256), 0, s, tens_dev, group, node_a, node_b,
                       tensor_digests);
  hipLaunchKernelGGL(hash_state_kernel, dim3(1), dim3(64), 0, s, n_tensors, tensor_digests, out);
  return hipGetLastError();
}

}  // namespace canon
