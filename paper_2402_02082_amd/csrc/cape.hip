// CaPE proposal expansion on the GPU (arXiv 2402.02082, Sec. 4.2,
// "Proposal Expansion"; linearisation from "Verification of Expanded
// Proposals"; verification budget from Sec. 5.3; fixed-size variant from
// Sec. 5.4).
//
// Two kernels:
//   cape_top8_part  one workgroup per 4096-token part of a draft row: the 8
//                   best (prob desc, id asc) tokens of the part, ranked among
//                   the few that pass a threshold;
//   cape_assemble   one workgroup per sequence: merges the parts into the
//                   row's top 8 -- the proposal token and the largest possible
//                   expansion set (S(p) <= 7) -- then applies S(p), the budget
//                   cut and the linearisation into a parent-indexed tree.
// Every decision is an exact comparison of the float32 inputs (keys are the
// order-preserving integer image of the float, ties broken by token id), so
// the result is bit-exact by construction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace glide {
namespace {

constexpr int kTopK = 8;
constexpr int kThreads = 256;

// Order-preserving map float32 -> uint32 (+0 and -0 map to the same value).
__device__ __forceinline__ uint32_t ordered_bits(float x) {
  uint32_t u = __float_as_uint(x);
  if (u == 0x80000000u) u = 0;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_ordered_bits(uint32_t o) {
  const uint32_t u = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
  return __uint_as_float(u);
}

// Larger key = more probable token; equal probabilities: lower id is larger.
__device__ __forceinline__ uint64_t rank_key(float p, int id) {
  return ((uint64_t)ordered_bits(p) << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)id);
}

__device__ __forceinline__ int key_id(uint64_t key) {
  return (int)(0xFFFFFFFFu - (uint32_t)key);
}

// Top 8 of two descending lists of 8, descending (bitonic merge: the
// element-wise max of a and reversed b holds the 8 largest keys as a bitonic
// sequence, which three compare-exchange stages sort).
__device__ __forceinline__ void merge_top8(uint64_t (&a)[kTopK], const uint64_t (&b)[kTopK]) {
#pragma unroll
  for (int i = 0; i < kTopK; ++i) a[i] = a[i] > b[kTopK - 1 - i] ? a[i] : b[kTopK - 1 - i];
#pragma unroll
  for (int dist = kTopK / 2; dist > 0; dist >>= 1)
#pragma unroll
    for (int i = 0; i < kTopK; ++i)
      if ((i & dist) == 0) {
        const uint64_t x = a[i], y = a[i + dist];
        a[i] = x > y ? x : y;
        a[i + dist] = x > y ? y : x;
      }
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = __shfl_xor((uint32_t)v, m), hi = __shfl_xor((uint32_t)(v >> 32), m);
  return ((uint64_t)hi << 32) | lo;
}

// Butterfly merge of the lists held by the lanes [0, width) of a wave; every
// lane ends with the top 8 of its aligned group of `width` lanes.
__device__ __forceinline__ void wave_merge_top8(uint64_t (&top)[kTopK], int width) {
  for (int m = 1; m < width; m <<= 1) {
    uint64_t other[kTopK];
#pragma unroll
    for (int j = 0; j < kTopK; ++j) other[j] = shfl_xor_u64(top[j], m);
    merge_top8(top, other);
  }
}

// Elements of a draft row handled by one workgroup: 256 threads x 16.
constexpr int kPart = kThreads * 16;

__device__ __forceinline__ int parts_per_row(int V) { return (V + kPart - 1) / kPart; }

// Max over the 16 lanes of a DPP row, in every lane of the row: swaps of
// neighbours, pairs, quads (half mirror) and halves (mirror).
__device__ __forceinline__ float row16_max(float v) {
  auto step = [&](float o) { v = fmaxf(v, o); };
  step(__uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0xB1, 0xF, 0xF, true)));
  step(__uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x4E, 0xF, 0xF, true)));
  step(__uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x141, 0xF, 0xF, true)));
  step(__uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x140, 0xF, 0xF, true)));
  return v;
}

constexpr int kWaves = kThreads / 64;
constexpr int kPerWave = 128;  // candidates a wave can hold

// Top-8 keys of one 4096-element part of one draft row.
//
// Every thread requests its 16 values at once.  The maxima of 16 thread
// groups are paired, and the smallest of the eight pair maxima is passed by
// at least eight values and, on values in random order, by about 22.  Those
// are ranked by counting.
//
// Where more values pass it than a wave can hold (many equal ones, as the
// zeros of filtered rows, or sorted rows), the threshold is the largest of the
// waves' eighth largest thread maxima: a wave's values above it are in at most
// seven threads, and of those equal to it the first eight are enough.
//
// Bound: latency (one round of loads, then short dependent steps).  A sorted
// top 8 per thread, merged across lanes and waves, took 9.8 us for 64 rows of
// 32000 (5 rows: 7.5); this takes 5.8 (4.6).
__global__ __launch_bounds__(kThreads) void cape_top8_part(const float* __restrict__ probs, int V,
                                                           uint64_t* __restrict__ top_out) {
  const int part = blockIdx.x, row = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = gridDim.x;
  const float* p = probs + (size_t)row * V;
  const int base = part * kPart, left = min(kPart, V - base);
  uint64_t* out = top_out + ((size_t)row * P + part) * kTopK;
  __shared__ __attribute__((aligned(16))) float group_max[16];
  __shared__ uint64_t cand[kWaves][kPerWave];
  __shared__ int cand_n[kWaves];
  __shared__ uint32_t wave_eighth[kWaves];

  // x[j]: the part's element index_of(j); elements past the row are -inf here
  // and never candidates.  Float4 loads leave whole threads of a part below
  // 4 * kThreads elements without any, and groups without a maximum.
  const bool vec = (V & 3) == 0 && (((uintptr_t)p) & 15) == 0 && left >= 4 * kThreads;
  float x[16];
  if (vec) {
    const float4* p4 = (const float4*)(p + base);
    float4 x4[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = tid + kThreads * u;
      x4[u] = 4 * i < left ? p4[i] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[4 * u] = x4[u].x;
      x[4 * u + 1] = x4[u].y;
      x[4 * u + 2] = x4[u].z;
      x[4 * u + 3] = x4[u].w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int i = tid + kThreads * j;
      x[j] = i < left ? p[base + i] : -INFINITY;
    }
  }
  auto index_of = [&](int j) { return vec ? 4 * (tid + kThreads * (j >> 2)) + (j & 3) : tid + kThreads * j; };

  float mx = x[0];
#pragma unroll
  for (int j = 1; j < 16; ++j) mx = fmaxf(mx, x[j]);
  mx = row16_max(mx);
  if ((lane & 15) == 0) group_max[tid >> 4] = mx;
  __syncthreads();
  float t = INFINITY;
#pragma unroll
  for (int i = 0; i < 8; ++i) t = fminf(t, fmaxf(group_max[i], group_max[i + 8]));

  const uint64_t below = (1ull << lane) - 1ull;
  int n = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const bool hit = !(x[j] < t) && index_of(j) < left;  // NaN: its key is the largest
    const uint64_t hits = __ballot(hit);
    if (hits) {
      const int slot = n + __popcll(hits & below);
      if (hit && slot < kPerWave) cand[wave][slot] = rank_key(x[j], base + index_of(j));
      n += __popcll(hits);
    }
  }
  int cn[kWaves], total;
  auto meet = [&]() {  // every wave's candidates are in place; the largest count
    if (lane == 0) cand_n[wave] = n;
    __syncthreads();
    int most = total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      cn[w] = __builtin_amdgcn_readfirstlane(cand_n[w]);
      total += cn[w];
      most = max(most, cn[w]);
    }
    return most;
  };
  if (meet() > kPerWave) {
    uint32_t o[16], top = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      o[j] = index_of(j) < left ? ordered_bits(x[j]) : 0;
      top = max(top, o[j]);
    }
    // the wave's eighth largest thread maximum: of the thread maxima that fewer
    // than eight exceed, the one that most exceed
    int above = 0;
#pragma unroll
    for (int i = 0; i < 64; ++i) above += (uint32_t)__builtin_amdgcn_readlane(top, i) > top;
    uint64_t eighth = 0;
#pragma unroll
    for (int k = 0; k < kTopK; ++k) {
      const uint64_t at = __ballot(above == k);
      eighth = at ? at : eighth;
    }
    uint32_t e8 = __builtin_amdgcn_readlane(top, __ffsll((long long)eighth) - 1);
    if (lane == 0) wave_eighth[wave] = e8;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) e8 = max(e8, wave_eighth[w]);
    n = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const bool hit = o[j] > e8;
      const uint64_t hits = __ballot(hit);
      if (hit) cand[wave][n + __popcll(hits & below)] = rank_key(x[j], base + index_of(j));
      n += __popcll(hits);
    }
    // equal values in the order of their ids: element by element of a thread
    // where it holds four in a row, otherwise thread by thread
    int ties = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (ties < kTopK) {
        bool tie[4];
        int first[4], upto = ties;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          tie[e] = o[4 * u + e] == e8 && index_of(4 * u + e) < left;
          const uint64_t hits = __ballot(tie[e]);
          first[e] = __popcll(hits & below) + (vec ? 0 : upto);
          upto += __popcll(hits);
        }
        int at = ties + first[0] + first[1] + first[2] + first[3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int slot = vec ? at : first[e];
          if (tie[e] && slot < kTopK) cand[wave][n + slot] = rank_key(x[4 * u + e], base + index_of(4 * u + e));
          at += tie[e];
        }
        ties = upto;
      }
    }
    n += min(ties, kTopK);
    meet();
  }

  // each wave ranks its own candidates against all (keys are distinct)
#pragma unroll
  for (int own = lane; own < kPerWave; own += 64) {
    if (own - lane < n) {
      const uint64_t mine = own < n ? cand[wave][own] : 0;
      int rank = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
#pragma unroll 4
        for (int i = 0; i < cn[w]; ++i) rank += cand[w][i] > mine;
      }
      if (own < n && rank < kTopK) out[rank] = mine;
    }
  }
  if (tid >= total && tid < kTopK) out[tid] = 0;  // a part of fewer than eight elements
}

// S(p): 7, 5, 3, 1 on (0, 0.3], (0.3, 0.6], (0.6, 0.8], (0.8, 1].
__device__ __forceinline__ int expansion_size(float p) {
  if (p <= 0.3f) return 7;
  if (p <= 0.6f) return 5;
  if (p <= 0.8f) return 3;
  return 1;
}

// One workgroup per sequence.  First each wave merges the per-part top-8
// lists of its positions into one top-8 list per position (bitonic merges
// across lanes); eight waves, so that proposals of up to eight tokens load
// every list in one round.  Then wave 0 assembles the tree: candidate c
// enumerates (position i, rank r) in linearisation order, and its confidence
// key is the top-8 key itself.  Sizes, offsets and (up to 64 candidates) the
// budget ranks pass between lanes in registers: reading them from LDS inside
// the counting loops cost a dependent LDS round trip per candidate (16-node
// tree of 5 tokens 6.1 -> 5.1 us, eight trees of 8 tokens 6.6 -> 5.9 us).
constexpr int kAsmThreads = 512;

__global__ __launch_bounds__(kAsmThreads) void cape_assemble(const uint64_t* __restrict__ part_top,
                                                             int gamma, int V, int k, int fixed,
                                                             int n_max, int32_t* __restrict__ tokens,
                                                             int32_t* __restrict__ parents,
                                                             int32_t* __restrict__ n_nodes) {
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int P = parts_per_row(V);
  const int C = P * kTopK;  // merge candidates per position

  __shared__ uint64_t top[kMaxNodes][kTopK];
  for (int i = wave; i < gamma; i += kAsmThreads / 64) {
    const uint64_t* src = part_top + ((size_t)b * gamma + i) * C;
    // Lane l holds the lists of parts l, l + 64, ...; fold them, then merge
    // across lanes.
    uint64_t best[kTopK];
#pragma unroll
    for (int j = 0; j < kTopK; ++j) best[j] = 0;
    for (int part = lane; part < P; part += 64) {
      uint64_t l[kTopK];
#pragma unroll
      for (int j = 0; j < kTopK; ++j) l[j] = src[part * kTopK + j];
      merge_top8(best, l);
    }
    int width = 1;
    while (width < min(P, 64)) width <<= 1;
    wave_merge_top8(best, width);
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < kTopK; ++j) top[i][j] = best[j];
    }
  }
  __syncthreads();
  if (wave != 0) return;

  __shared__ uint64_t cand_key[kMaxNodes * 7];
  __shared__ int cand_pos[kMaxNodes * 7];

  int size = 0;
  if (lane < gamma) {
    const uint64_t k0 = top[lane][0];
    if (fixed) {
      size = k;
    } else {
      size = expansion_size(from_ordered_bits((uint32_t)(k0 >> 32)));
      if (k > 0) size = min(size, k);
    }
    size = min(size, V - 1);
    tokens[(size_t)b * n_max + lane] = key_id(k0);
    parents[(size_t)b * n_max + lane] = lane - 1;
  }
  int Ctot = 0;
  for (int i = 0; i < gamma; ++i) Ctot += __builtin_amdgcn_readlane(size, i);
  uint64_t my_key = 0;  // the lane's candidate of the first 64
  int my_pos = 0;
  for (int cb = 0; cb < Ctot; cb += 64) {
    // position of candidate cb + lane: the number of positions that end at
    // or before it
    const int cidx = cb + lane;
    int pos = 0, start = 0, end = 0;
    for (int i = 0; i < gamma; ++i) {
      end += __builtin_amdgcn_readlane(size, i);
      if (cidx >= end) {
        pos = i + 1;
        start = end;
      }
    }
    const uint64_t key = cidx < Ctot ? top[pos][cidx - start + 1] : 0;
    if (cb == 0) {
      my_key = key;
      my_pos = pos;
    }
    if (cidx < Ctot) {
      cand_key[cidx] = key;
      cand_pos[cidx] = pos;
    }
  }
  __builtin_amdgcn_wave_barrier();

  const int budget = n_max - gamma;
  int written = 0;  // kept candidates in earlier chunks
  // Rank in (prob desc, position asc, rank asc): probability is the high half
  // of the key; cidx order is (position, rank) order.
  int ahead64 = 0;
  if (Ctot > budget && Ctot <= 64) {
    const uint32_t pc = (uint32_t)(my_key >> 32);
    for (int o = 0; o < Ctot; ++o) {
      const uint32_t po = __builtin_amdgcn_readlane(pc, o);
      ahead64 += (po > pc) || (po == pc && o < lane);
    }
  }
  for (int cb = 0; cb < Ctot; cb += 64) {
    const int cidx = cb + lane;
    bool kept = false;
    uint64_t key = my_key;
    int pos = my_pos;
    if (cidx < Ctot) {
      if (Ctot > 64) {
        key = cand_key[cidx];
        pos = cand_pos[cidx];
      }
      if (Ctot <= budget) {
        kept = true;
      } else if (Ctot <= 64) {
        kept = ahead64 < budget;
      } else {
        const uint32_t pc = (uint32_t)(key >> 32);
        int ahead = 0;
        for (int o = 0; o < Ctot; ++o) {
          const uint32_t po = (uint32_t)(cand_key[o] >> 32);
          ahead += (po > pc) || (po == pc && o < cidx);
        }
        kept = ahead < budget;
      }
    }
    const uint64_t mask = __ballot(kept);
    if (kept) {
      const int slot = gamma + written + __popcll(mask & ((1ull << lane) - 1ull));
      tokens[(size_t)b * n_max + slot] = key_id(key);
      parents[(size_t)b * n_max + slot] = pos - 1;
    }
    written += __popcll(mask);
  }
  const int n = gamma + written;
  for (int j = n + lane; j < n_max; j += 64) {
    tokens[(size_t)b * n_max + j] = -1;
    parents[(size_t)b * n_max + j] = -1;
  }
  if (lane == 0) n_nodes[b] = n;
}

}  // namespace

size_t cape_workspace_bytes(int B, int gamma, int V) {
  return (size_t)B * gamma * ((V + kPart - 1) / kPart) * kTopK * sizeof(uint64_t);
}

hipError_t launch_cape_expand(const float* probs, int B, int gamma, int V, int k, int fixed,
                              int n_max, int32_t* tokens, int32_t* parents, int32_t* n_nodes,
                              void* ws, hipStream_t stream) {
  uint64_t* top = (uint64_t*)ws;
  const int P = (V + kPart - 1) / kPart;
  hipLaunchKernelGGL(cape_top8_part, dim3(P, B * gamma), dim3(kThreads), 0, stream, probs, V, top);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cape_assemble, dim3(B), dim3(kAsmThreads), 0, stream, top, gamma, V, k, fixed,
                     n_max, tokens, parents, n_nodes);
  return hipGetLastError();
}

}  // namespace glide
