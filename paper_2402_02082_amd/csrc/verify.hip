// Greedy verification of a candidate tree (arXiv 2402.02082, Sec. 3: with
// greedy "speculative decoding" acceptance a proposed token is kept exactly
// when it equals the target's greedy token; Sec. 4.2 verifies the whole
// expanded proposal in one pass; Sec. 5.1 uses greedy acceptance for CaPE).
//
//   argmax_rows   one workgroup per logits row: the first index of the row
//                 maximum; 1024 threads while every row's workgroup fits on
//                 the chip at once (a 32000-entry row is one round of
//                 loads), 256 beyond that, so that no rows wait for a
//                 second round of workgroups.
//   tree_verify   one wave per sequence, one lane per node: a node is
//                 accepted iff every node on its root path matches, i.e. its
//                 ancestor-or-self bitmask has no non-matching bit; the
//                 deepest accepted node (lowest index on ties) wins.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace glide {
namespace {

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = __shfl_xor((uint32_t)v, m), hi = __shfl_xor((uint32_t)(v >> 32), m);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src) {
  const uint32_t lo = __shfl((uint32_t)v, src), hi = __shfl((uint32_t)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    const uint64_t o = shfl_xor_u64(v, m);
    v = o > v ? o : v;
  }
  return v;
}

// One step of the wave maximum below: the value of another lane of the
// 16-lane DPP row.
template <int CTRL>
__device__ __forceinline__ float row_swap(float v) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), CTRL, 0xF, 0xF, true));
}

// Max over a wave, in every lane: within the DPP rows (neighbours, pairs,
// half mirror, mirror), then across the rows with gfx950's row swaps.
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, row_swap<0xB1>(v));
  v = fmaxf(v, row_swap<0x4E>(v));
  v = fmaxf(v, row_swap<0x141>(v));
  v = fmaxf(v, row_swap<0x140>(v));
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Min over a wave, in every lane, by the same steps.
__device__ __forceinline__ int wave_min(int v) {
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = min((int)a[0], (int)a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return min((int)b[0], (int)b[1]);
}

// One workgroup of kThreads per row; each thread requests 8 float4 (32
// values) at once, so with 1024 threads a 32000-entry row is a single round
// of loads.  A thread keeps its largest value and that value's first index
// (a strictly larger value moves both: three instructions a value); the
// row's maximum is reduced first, then the lowest index among the threads
// that hold it.  Ordered 64-bit (value, ~index) keys through every step took
// about ten instructions a value: 132 rows of 32000 6.6 us, now 4.5.
constexpr int kArgmaxVec = 8;

template <int kArgmaxThreads>
__global__ __launch_bounds__(kArgmaxThreads) void argmax_rows_kernel(const float* __restrict__ logits,
                                                                     int V, int32_t* __restrict__ idx) {
  const int row = blockIdx.x, tid = threadIdx.x;
  const float* p = logits + (size_t)row * V;
  float best = -INFINITY;
  int at = INT32_MAX;  // of a value above -inf
  auto take = [&](float x, int i) {
    const bool more = x > best;
    best = more ? x : best;
    at = more ? i : at;
  };
  if ((V & 3) == 0 && (((uintptr_t)p) & 15) == 0) {
    const float4* p4 = (const float4*)p;
    const int n4 = V / 4;
    for (int i0 = 0; i0 < n4; i0 += kArgmaxThreads * kArgmaxVec) {
      float4 x[kArgmaxVec];
#pragma unroll
      for (int u = 0; u < kArgmaxVec; ++u) {
        const int i = i0 + tid + kArgmaxThreads * u;
        x[u] = i < n4 ? p4[i] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      }
#pragma unroll
      for (int u = 0; u < kArgmaxVec; ++u) {
        const int i = 4 * (i0 + tid + kArgmaxThreads * u);
        take(x[u].x, i);
        take(x[u].y, i + 1);
        take(x[u].z, i + 2);
        take(x[u].w, i + 3);
      }
    }
  } else {
    for (int i = tid; i < V; i += kArgmaxThreads) take(p[i], i);
  }
  __shared__ float wave_best[kArgmaxThreads / 64];
  __shared__ int first;
  const float w = wave_max(best);
  if ((tid & 63) == 0) wave_best[tid >> 6] = w;
  if (tid == 0) first = INT32_MAX;
  __syncthreads();
  float m = wave_best[0];
#pragma unroll
  for (int i = 1; i < kArgmaxThreads / 64; ++i) m = fmaxf(m, wave_best[i]);
  bool holds = best == m && at != INT32_MAX;
  if (__builtin_expect(__popcll(__ballot(holds)) > 4, 0)) {
    // equal values: one LDS atomic for the wave (17 rows of 32000 equal
    // values: 6.7 us with an atomic each)
    at = wave_min(holds ? at : INT32_MAX);
    holds = (tid & 63) == 0;
  }
  if (holds) atomicMin(&first, at);
  __syncthreads();
  if (tid == 0) idx[row] = first == INT32_MAX ? 0 : first;  // a row of nothing above -inf: its first entry
}

__global__ __launch_bounds__(64) void tree_verify_kernel(const int32_t* __restrict__ target_argmax,
                                                         const int32_t* __restrict__ cand,
                                                         const int32_t* __restrict__ parents, int N,
                                                         int32_t* __restrict__ accept_len,
                                                         int32_t* __restrict__ last_node,
                                                         int32_t* __restrict__ bonus) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int32_t* ta = target_argmax + (size_t)b * (N + 1);
  int p = -1;
  bool match = false;
  uint64_t anc = 0;
  if (lane < N) {
    p = parents[(size_t)b * N + lane];
    if (p < -1 || p >= lane) p = -1;
    match = cand[(size_t)b * N + lane] == ta[p + 1];
    anc = 1ull << lane;
  }
  const uint64_t matched = __ballot(match);
  // Ancestor-or-self masks by pointer doubling (six rounds cover depth 64).
#pragma unroll
  for (int round = 0; round < 6; ++round) {
    const int src = p < 0 ? lane : p;
    const uint64_t a_up = shfl_u64(anc, src);
    const int p_up = __shfl(p, src);
    if (p >= 0) {
      anc |= a_up;
      p = p_up;
    }
  }
  const bool accepted = lane < N && (anc & ~matched) == 0;
  const int depth = __popcll(anc);
  // Deepest accepted node, then the lowest index.
  uint64_t key = accepted ? (((uint64_t)depth << 8) | (uint64_t)(255 - lane)) : 0;
  key = wave_max_u64(key);
  if (lane == 0) {
    const int len = (int)(key >> 8);
    const int last = key ? 255 - (int)(key & 255) : -1;
    accept_len[b] = len;
    if (last_node) last_node[b] = last;
    if (bonus) bonus[b] = ta[last + 1];
  }
}

}  // namespace

hipError_t launch_argmax_rows(const float* logits, int rows, int V, int32_t* idx,
                              hipStream_t stream) {
  // two 1024-thread workgroups fit on a CU
  if (rows <= 2 * kNumCU)
    hipLaunchKernelGGL(argmax_rows_kernel<1024>, dim3(rows), dim3(1024), 0, stream, logits, V, idx);
  else
    hipLaunchKernelGGL(argmax_rows_kernel<256>, dim3(rows), dim3(256), 0, stream, logits, V, idx);
  return hipGetLastError();
}

hipError_t launch_tree_verify(const int32_t* target_argmax, const int32_t* cand,
                              const int32_t* parents, int B, int N, int32_t* accept_len,
                              int32_t* last_node, int32_t* bonus, hipStream_t stream) {
  hipLaunchKernelGGL(tree_verify_kernel, dim3(B), dim3(64), 0, stream, target_argmax, cand, parents,
                     N, accept_len, last_node, bonus);
  return hipGetLastError();
}

}  // namespace glide
