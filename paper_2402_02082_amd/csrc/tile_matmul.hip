// Projections of many activation rows (a prompt's positions when the draft
// prefills, or a large batch of draft steps; arXiv 2402.02082, Sec. 4.1:
// Q^{m,j} = H^m W_j and Concat(hd_1..hd_h) W^O):
//
//   out[m, n] = sum_k a[m, k] * w_t[n, k]      a [M, K], w_t [N, K] (bf16)
//
// The few-row kernels (rows_matmul.hip) stream the weights once per 128 rows
// and read every activation row once per 16 output features; past 128 rows
// that is matrix work held up by operand traffic.  Here each workgroup owns
// a 2-D tile of the output and stages 64-wide K chunks of both operands
// through LDS with memory-to-LDS loads, two to four chunks deep.
//
// What bounds it: at 256 x 128 each CU takes one tile (two waves per SIMD)
// and the matrix cores run at about half their rate, the rest going to the
// chunk barrier and the LDS reads; a CU's loads (64 bytes a cycle into LDS)
// would need 75 % of the product's time, where 128 x 128 tiles need all of
// it.  The chunk loop must stay free of address arithmetic: with offsets
// recomputed per load it issued four vector instructions per product and
// took 75-82 us, without 62.  K = N = 4096, row-major weights: 2048 rows
// 335 -> 62 us (1100 TFLOP/s), 512 rows 87 -> 24 us, 130 rows 30 -> 16 us
// against the few-row kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace glide {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr uint32_t kDesc3 = 0x00020000u;
constexpr int kBK = 64;               // K values per staged chunk (128 bytes a row)

// Buffer descriptor of bytes [skip, bytes) behind `base` (empty past the end).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_from(const char* base, int skip, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base) + skip, (short)0, max(bytes - skip, 0), kDesc3);
}

// 16 bytes per lane from byte offset `off` to dst + 16 * lane (LDS).
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, char* dst, int off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)dst, 16, off, 0, 0, 0);
}

// This wave's loads of the next chunk have landed (at most PENDING later ones
// are in flight) and its LDS reads of the chunk before are done; after the
// barrier everyone's, so that chunk's stage is free.  (A __syncthreads()
// would wait for every outstanding memory-to-LDS load.)
template <int PENDING>
__device__ __forceinline__ void wait_and_meet() {
  static_assert(PENDING >= 0 && PENDING < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(PENDING) : "memory");
  asm volatile("s_barrier" ::: "memory");
}

template <int WM, int WN, int MT, int NT, int S, bool PACKED>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2)))
void tile_matmul_kernel(const uint16_t* __restrict__ a, const uint16_t* __restrict__ w_t,
                        uint16_t* __restrict__ out, int M, int K, int N, int m_tiles, int n_tiles, bool vec_out) {
  constexpr int kWaves = WM * WN;
  constexpr int kTM = 16 * MT * WM, kTN = 16 * NT * WN;
  constexpr int kABytes = kTM * kBK * 2, kWBytes = kTN * kBK * 2;
  constexpr int kAInstr = kABytes / 1024 / kWaves, kWInstr = kWBytes / 1024 / kWaves;
  constexpr int kStage = kABytes + kWBytes;
  static_assert(kAInstr * kWaves * 1024 == kABytes && kWInstr * kWaves * 1024 == kWBytes, "whole loads");
  __shared__ __attribute__((aligned(1024))) char lds[S * kStage];

  // Tile order: workgroups are dealt to the eight XCDs round-robin by linear
  // id; XCD x takes a contiguous run of the tile order, in which eight
  // m-tiles share each n-tile, so its L2 serves both operands' reuse.
  const int T = m_tiles * n_tiles, lin = blockIdx.x;
  const int x = lin % 8, q = T / 8, rem = T % 8;
  const int idx = x * q + min(x, rem) + lin / 8;
  const int group = idx / (8 * n_tiles), in_group = idx % (8 * n_tiles);
  const int gm = min(8, m_tiles - 8 * group);
  const int m0 = (8 * group + in_group % gm) * kTM, n0 = (in_group / gm) * kTN;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int c = lane & 15, g = lane >> 4;
  const int wm = wave % WM, wn = wave / WM;
  const int k_steps = (K + 31) / 32, chunks = (K + kBK - 1) / kBK;

  // Both operands are read through descriptors that start at the chunk's
  // first column and end with the tile's last row (row-major) or block
  // (packed), so rows past M and N read nothing.
  const char* a_base = (const char*)(a + (size_t)m0 * K);
  const int a_bytes = min(kTM, M - m0) * K * 2;
  const char* w_base = (const char*)(PACKED ? w_t + (size_t)(n0 / 16) * k_steps * 512 : w_t + (size_t)n0 * K);
  const int w_bytes = PACKED ? min(kTN / 16, (N + 15) / 16 - n0 / 16) * k_steps * 1024 : min(kTN, N - n0) * K * 2;
  constexpr int kWChunk = PACKED ? 2048 : kBK * 2;  // a chunk's step in w

  // This lane's part of instruction i, which fills an operand's units
  // [64 i, 64 i + 64): row-major, eight rows' 128 contiguous bytes; packed,
  // the 1 KB block of 16-row tile i / 2, step i % 2 of the chunk.
  int a_off[kAInstr], w_off[kWInstr];
  const int sub = lane >> 3;
#pragma unroll
  for (int j = 0; j < kAInstr; ++j) {
    const int row = 8 * (wave + kWaves * j) + sub;
    a_off[j] = row * K * 2 + 16 * ((lane & 7) ^ ((row >> 1) & 7));
  }
#pragma unroll
  for (int j = 0; j < kWInstr; ++j) {
    const int i = wave + kWaves * j, row = 8 * i + sub;
    w_off[j] = PACKED ? ((i >> 1) * k_steps + (i & 1)) * 1024 + 16 * lane
                      : row * K * 2 + 16 * ((lane & 7) ^ ((row >> 1) & 7));
  }
  auto stage = [&](int ch, char* base) {
    const bool live = ch < chunks;
    const __amdgpu_buffer_rsrc_t ra = rsrc_from(a_base, ch * (kBK * 2), live ? a_bytes : 0);
    const __amdgpu_buffer_rsrc_t rw = rsrc_from(w_base, ch * kWChunk, live ? w_bytes : 0);
#pragma unroll
    for (int j = 0; j < kAInstr; ++j)
      load_to_lds(ra, base + (wave + kWaves * j) * 1024, a_off[j]);
#pragma unroll
    for (int j = 0; j < kWInstr; ++j)
      load_to_lds(rw, base + kABytes + (wave + kWaves * j) * 1024, w_off[j]);
  };

  f32x4_t acc[NT][MT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Operand units of this lane: row 16 t + c of the wave's tile t, unit
  // 4 st + g of the chunk (the row's swizzle depends on c alone).
  const int sw = (c >> 1) & 7;
  const int lane_unit[2] = {c * 8 + (g ^ sw), c * 8 + ((4 + g) ^ sw)};
  auto compute = [&](const char* base, int k_left) {
    const char* abase = base + MT * wm * 2048;
    const char* wbase = base + kABytes + NT * wn * 2048;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      u32x4_t av[MT], wv[NT];
#pragma unroll
      for (int j = 0; j < MT; ++j) av[j] = *(const u32x4_t*)(abase + 2048 * j + 16 * lane_unit[st]);
#pragma unroll
      for (int i = 0; i < NT; ++i)
        wv[i] = *(const u32x4_t*)(wbase + (PACKED ? 2048 * i + 1024 * st + 16 * lane : 2048 * i + 16 * lane_unit[st]));
      if (k_left < kBK && 32 * st + 8 * g >= k_left) {
        // columns past K hold the next row's values, or nothing
#pragma unroll
        for (int j = 0; j < MT; ++j) av[j] = u32x4_t{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < NT; ++i) wv[i] = u32x4_t{0, 0, 0, 0};
      }
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wv[i]),
                                                             __builtin_bit_cast(bf16x8_t, av[j]), acc[i][j], 0, 0, 0);
    }
  };
  constexpr int kPending = (S - 2) * (kAInstr + kWInstr);

#pragma unroll
  for (int ch = 0; ch < S - 1; ++ch) stage(ch, lds + ch * kStage);
  const int whole = K / kBK;  // chunks without columns past K
  for (int ch0 = 0; ch0 < whole; ch0 += S) {
#pragma unroll
    for (int u = 0; u < S; ++u) {
      if (ch0 + u < whole) {
        wait_and_meet<kPending>();
        stage(ch0 + u + S - 1, lds + ((u + S - 1) % S) * kStage);
        compute(lds + u * kStage, kBK);
      }
    }
  }
  if (whole < chunks) {
    wait_and_meet<kPending>();
    compute(lds + (whole % S) * kStage, K - whole * kBK);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // Lane (c, g) holds output row 16 j + c, features 16 i + 4 g .. + 3.
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    const int m = m0 + 16 * (MT * wm + j) + c;
    if (m < M) {
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const int n = n0 + 16 * (NT * wn + i) + 4 * g;
        const u32x2_t v = {
            __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{acc[i][j][0], acc[i][j][1]}), bf16x2_t)),
            __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{acc[i][j][2], acc[i][j][3]}), bf16x2_t))};
        uint16_t* dst = out + (size_t)m * N + n;
        if (vec_out) {
          if (n < N) *(u32x2_t*)dst = v;  // N % 4 == 0: all four or none
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n + r < N) dst[r] = (uint16_t)(v[r >> 1] >> (16 * (r & 1)));
        }
      }
    }
  }
}

// Output tiles of the three launch shapes (rows x features).
struct Big { static constexpr int kWM = 4, kWN = 2, kMT = 4, kNT = 4, kS = 2; };    // 256 x 128, eight waves
struct Mid { static constexpr int kWM = 2, kWN = 2, kMT = 4, kNT = 2, kS = 3; };    // 128 x 64
struct Small { static constexpr int kWM = 2, kWN = 2, kMT = 2, kNT = 2, kS = 4; };  // 64 x 64

template <class C>
long tiles_of(int M, int N) {
  constexpr int tm = 16 * C::kMT * C::kWM, tn = 16 * C::kNT * C::kWN;
  return (long)((M + tm - 1) / tm) * ((N + tn - 1) / tn);
}

template <class C, bool PACKED>
hipError_t launch(const uint16_t* a, const uint16_t* w, uint16_t* out, int M, int K, int N, hipStream_t stream) {
  constexpr int tm = 16 * C::kMT * C::kWM, tn = 16 * C::kNT * C::kWN, threads = 64 * C::kWM * C::kWN;
  const int nt = (N + tn - 1) / tn;
  const bool vec = N % 4 == 0 && ((uintptr_t)out & 7) == 0;
  // a launch holds fewer than 2^31 threads: more m-tiles take further launches
  const long most = ((1L << 31) - 1) / ((long)nt * threads);
  const int step = (int)(most < 1 ? 1 : (most > (1 << 22) ? (1 << 22) : most)) * tm;
  for (int m0 = 0; m0 < M; m0 += step) {
    const int rows = min(step, M - m0), mt = (rows + tm - 1) / tm;
    hipLaunchKernelGGL((tile_matmul_kernel<C::kWM, C::kWN, C::kMT, C::kNT, C::kS, PACKED>), dim3(mt * nt),
                       dim3(threads), 0, stream, a + (size_t)m0 * K, w, out + (size_t)m0 * N, rows, K, N, mt, nt, vec);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || M - m0 <= step) return e;
  }
  return hipSuccess;
}

template <bool PACKED>
hipError_t launch_shape(const uint16_t* a, const uint16_t* w, uint16_t* out, int M, int K, int N,
                        hipStream_t stream) {
  // Time per 64-wide K chunk with n tiles on a CU, from K = N = 4096: 256 x
  // 128 one tile 1.0 us; 128 x 64 one 0.38, two 0.65, four 1.26; 64 x 64 one
  // 0.25, two 0.42, four 0.78.  The larger tile wins once it gives every CU
  // one: 2048 rows 66 against 81 and 100 us, 1024 rows 55 against 41 and 50,
  // 512 rows 54 against 24 and 28, 256 rows 53 against 23 and 17.
  auto per_cu = [](long tiles) { return (double)((tiles + kNumCU - 1) / kNumCU); };
  const double big = 1.0 * per_cu(tiles_of<Big>(M, N));
  const double mid = 0.05 + 0.33 * per_cu(tiles_of<Mid>(M, N));
  const double small = 0.06 + 0.19 * per_cu(tiles_of<Small>(M, N));
  if (big <= mid && big <= small) return launch<Big, PACKED>(a, w, out, M, K, N, stream);
  if (mid <= small) return launch<Mid, PACKED>(a, w, out, M, K, N, stream);
  return launch<Small, PACKED>(a, w, out, M, K, N, stream);
}

}  // namespace

hipError_t launch_tile_matmul(const void* a, const void* w, void* out, int M, int K, int N, bool packed,
                              hipStream_t stream) {
  return packed ? launch_shape<true>((const uint16_t*)a, (const uint16_t*)w, (uint16_t*)out, M, K, N, stream)
                : launch_shape<false>((const uint16_t*)a, (const uint16_t*)w, (uint16_t*)out, M, K, N, stream);
}

}  // namespace glide
