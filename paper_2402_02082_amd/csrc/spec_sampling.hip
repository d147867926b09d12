// Chain verification with speculative sampling (arXiv 2402.02082, Sec. 3:
// the accepted draft tokens plus one target token extend the prefix, and the
// emitted tokens follow the target's sampling distribution; Sec. 5.1: the
// GliDe-only experiments verify gamma = 5 chains this way).
//
// One 1024-thread workgroup per sequence.  Proposal token x_i is accepted when
// r_i * p_D(x_i) < p_T(x_i) (float32), tested for every position at once; the
// first rejection j picks the residual row max(0, p_T_j - p_D_j), no
// rejection picks the target row after the last token.  The token is drawn by
// inverse CDF over fixed-point weights floor(p * 2^32): integer sums do not
// depend on the order of summation, so the draw is a function of the inputs
// alone.  Each wave owns a contiguous region of the row and reads it in tiles
// of 256 tokens, four consecutive tokens a lane; the waves' sums tell which
// region holds floor(u * W), and that wave scans its tiles for the token.
//
// Bound: latency -- the dependent reads of the tokens, their probabilities
// and the row, then the sums.  With a contiguous run of tokens per thread a
// row load touched 64 cache lines for 1 KB, and every weight went through
// float64: 13.0 us for 16 sequences of V = 32000.  A tile load is 1 KB
// contiguous, and a probability below 1 converts exactly in float32: 8.3 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace glide {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ uint64_t fixed_weight(float p) {
  // p >= 0 (negatives count as 0); p * 2^32 is exact in float64
  return p > 0.f ? (uint64_t)((double)p * 4294967296.0) : 0;
}

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int d) {
  const uint32_t lo = __shfl_up((uint32_t)v, d), hi = __shfl_up((uint32_t)(v >> 32), d);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = __shfl_xor((uint32_t)v, m), hi = __shfl_xor((uint32_t)(v >> 32), m);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane), hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

constexpr int kTile = 256;  // tokens a wave reads at once
constexpr int kTiles = 8;   // tiles held in registers (V <= 32768: a wave's whole region)
constexpr int kGroup = kTile * kTiles;

// Values of tokens v0 + 256 u + 4 lane .. + 3 of the chosen row (0 at and
// past v1): the target's (mode 1) or the residual max(0, target - draft).
__device__ __forceinline__ void load_group(float (&p)[kTiles][4], const float* pt, const float* pd, int v0, int v1,
                                           int mode, bool vec, int lane) {
  float d[kTiles][4];
#pragma unroll
  for (int u = 0; u < kTiles; ++u) {
    const int v = v0 + kTile * u + 4 * lane;
    if (vec) {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
      if (v < v1) {
        a = *(const float4*)(pt + v);
        if (mode == 0) b = *(const float4*)(pd + v);
      }
      p[u][0] = a.x, p[u][1] = a.y, p[u][2] = a.z, p[u][3] = a.w;
      d[u][0] = b.x, d[u][1] = b.y, d[u][2] = b.z, d[u][3] = b.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[u][e] = v + e < v1 ? pt[v + e] : 0.f;
        d[u][e] = mode == 0 && v + e < v1 ? pd[v + e] : 0.f;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kTiles; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) p[u][e] = fmaxf(p[u][e] - d[u][e], 0.f);
}

// s[u]: sum of the lane's four weights of tile u.  p * 2^32 is exact in
// float32, and below 2^32 its integer part fits 32 bits; only values of 1 and
// more take the float64 conversion.
__device__ __forceinline__ void group_weights(const float (&p)[kTiles][4], uint64_t (&s)[kTiles]) {
  float top = 0.f;
#pragma unroll
  for (int u = 0; u < kTiles; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) top = fmaxf(top, p[u][e]);
  if (__any(top >= 1.f)) {
#pragma unroll
    for (int u = 0; u < kTiles; ++u)
      s[u] = (fixed_weight(p[u][0]) + fixed_weight(p[u][1])) + (fixed_weight(p[u][2]) + fixed_weight(p[u][3]));
  } else {
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
      s[u] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) s[u] += (uint32_t)(p[u][e] * 4294967296.f);
    }
  }
}

// Called by a whole wave: the token of the group starting at v0 whose running
// weight first exceeds `left` (written by its lane), or `left` less the
// group's weight.  Returns whether the token was in the group.
__device__ bool find_in_group(const float (&p)[kTiles][4], int v0, uint64_t& left, int lane, int32_t* token) {
  uint64_t s[kTiles], own[kTiles];
  group_weights(p, own);
#pragma unroll
  for (int u = 0; u < kTiles; ++u) s[u] = own[u];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
      const uint64_t y = shfl_up_u64(s[u], d);
      if (lane >= d) s[u] += y;
    }
  }
  bool found = false;
#pragma unroll
  for (int u = 0; u < kTiles; ++u) {
    if (!found) {
      const uint64_t tile = readlane_u64(s[u], 63);
      if (left < tile) {
        found = true;
        uint64_t run = s[u] - own[u];
        if (run <= left && left < s[u]) {
          int at = 3;
#pragma unroll
          for (int e = 0; e < 3; ++e) {
            run += fixed_weight(p[u][e]);
            if (run > left) {
              at = e;
              break;
            }
          }
          *token = v0 + kTile * u + 4 * lane + at;
        }
      } else {
        left -= tile;
      }
    }
  }
  return found;
}

__global__ __launch_bounds__(kThreads) void spec_sample_kernel(const int32_t* __restrict__ draft_tokens,
                                                               const float* __restrict__ p_draft,
                                                               const float* __restrict__ p_target,
                                                               const float* __restrict__ uniforms,
                                                               int gamma, int V,
                                                               int32_t* __restrict__ accept_len,
                                                               int32_t* __restrict__ next_token) {
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* u = uniforms + (size_t)b * (gamma + 1);
  const float draw = u[gamma];
  __shared__ int first_reject;
  __shared__ uint64_t wave_sum[kWaves];

  // Acceptance tests of every position (gamma <= 64: wave 0).
  if (tid < 64) {
    bool rejected = false;
    if (lane < gamma) {
      int x = draft_tokens[(size_t)b * gamma + lane];
      x = x < 0 ? 0 : (x >= V ? V - 1 : x);
      const float pd = p_draft[((size_t)b * gamma + lane) * V + x];
      const float pt = p_target[((size_t)b * (gamma + 1) + lane) * V + x];
      rejected = !(u[lane] * pd < pt);
    }
    const uint64_t rej = __ballot(rejected);
    if (lane == 0) first_reject = rej ? __ffsll((long long)rej) - 1 : gamma;
  }
  __syncthreads();
  const int j = __builtin_amdgcn_readfirstlane(first_reject);
  const float* pt = p_target + ((size_t)b * (gamma + 1) + j) * V;
  const float* pd = p_draft + ((size_t)b * gamma + (j < gamma ? j : 0)) * V;
  const bool vec = (V & 3) == 0 && ((((uintptr_t)p_target) | ((uintptr_t)p_draft)) & 15) == 0;

  const int region = (V + kWaves * kTile - 1) / (kWaves * kTile) * kTile;  // tokens per wave
  const int v0 = min(V, wave * region), v1 = min(V, v0 + region);
  int mode = j < gamma ? 0 : 1;
  float p[kTiles][4];
  uint64_t total = 0, before = 0, mine = 0, first = 0;  // first: the lane's share of the region's first group
  for (int pass = 0; pass < 2; ++pass) {
    mine = 0;
    for (int g = v0; g < v1; g += kGroup) {
      uint64_t s[kTiles];
      load_group(p, pt, pd, g, v1, mode, vec, lane);
      group_weights(p, s);
#pragma unroll
      for (int t = 0; t < kTiles; ++t) mine += s[t];
      if (g == v0) first = mine;
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) mine += shfl_xor_u64(mine, m);
    if (lane == 0) wave_sum[wave] = mine;
    __syncthreads();
    total = before = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint64_t s = wave_sum[w];
      if (w < wave) before += s;
      total += s;
    }
    __syncthreads();  // wave_sum is reused by the next pass
    if (total > 0 || mode == 1) break;
    mode = 1;  // a residual of zero weight: draw from the target row itself
  }
  if (total == 0) {
    if (tid == 0) {
      accept_len[b] = j;
      next_token[b] = 0;
    }
    return;
  }
  uint64_t t = (uint64_t)((double)draw * (double)total);
  if (t >= total) t = total - 1;
  if (t < before || t >= before + mine) return;
  if (lane == 0) accept_len[b] = j;
  uint64_t left = t - before;
  int g = v0;
  if (region > kGroup) {
    // a first group without the token is passed over unread: rows of 32772
    // tokens, all accepted, 12.1 us with it searched
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) first += shfl_xor_u64(first, m);
    if (left >= first) {
      left -= first;
      g += kGroup;
    }
  }
  bool held = true;  // the region's last group is still in registers
  for (; g < v1; g += kGroup) {
    if (!held || g + kGroup < v1) {
      load_group(p, pt, pd, g, v1, mode, vec, lane);
      held = false;
    }
    if (find_in_group(p, g, left, lane, next_token + b)) return;
  }
}

}  // namespace

hipError_t launch_spec_sample(const int32_t* draft_tokens, const float* p_draft, const float* p_target,
                              const float* uniforms, int B, int gamma, int V, int32_t* accept_len,
                              int32_t* next_token, hipStream_t stream) {
  hipLaunchKernelGGL(spec_sample_kernel, dim3(B), dim3(kThreads), 0, stream, draft_tokens, p_draft, p_target,
                     uniforms, gamma, V, accept_len, next_token);
  return hipGetLastError();
}

}  // namespace glide
