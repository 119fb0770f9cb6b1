// Sign products on the matrix cores as 4-bit floats (e2m1: +-1 against +-1/2,
// which give the half-codes (dot - K % 2) / 2 exactly; a 32 x 32 x 64 product
// takes 32 cycles, twice the int8 rate):
//   k_bgemm_q8_e2m1  binary GEMM into 8-bit half-codes
// Matrix and vector instructions of a SIMD do not overlap here (32 fp32 FMAs
// and two of these products take 128 cycles, as they would one after the
// other), so the cost of a tile is the sum of both; FMA, add and move issue
// every 2.2 cycles with two waves, most other vector instructions every 4.3.

#include "bigcn_device.h"

#include <algorithm>

namespace bigcn {
namespace {

typedef int int8v_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

// 32 sign bits as 32 e2m1 values (4 bits: sign, then the magnitude MAG): bit
// 4 m + i goes to nibble m of register i, set bits negative.
template <uint32_t MAG>
__device__ inline int4_t sign_nibbles(uint32_t w) {
  constexpr uint32_t S = 0x88888888u, T = 0x11111111u * MAG;
  int4_t r;
  r[0] = (int)(((w << 3) & S) | T);
  r[1] = (int)(((w << 2) & S) | T);
  r[2] = (int)(((w << 1) & S) | T);
  r[3] = (int)((w & S) | T);
  return r;
}

// Nibbles of the bits set in m: 0xF, else 0 (the order of sign_nibbles).
__device__ inline int4_t mask_nibbles(uint32_t m) {
  int4_t r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t x = (m << (3 - i)) & 0x88888888u;
    x |= x >> 1;
    x |= x >> 2;
    r[i] = (int)x;
  }
  return r;
}

// D = A B + C over 64 e2m1 inputs: lane l gives row (A) / column (B) l & 31,
// inputs 32 (l >> 5) .. + 31, and holds D[8 b + 4 (l >> 5) + i][l & 31] at
// index 4 b + i.
__device__ inline float16_t mfma_e2m1(const int4_t& a, const int4_t& b, const float16_t& c) {
  const int8v_t av = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
  const int8v_t bv = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4 /* A: e2m1 */,
                                                         4 /* B: e2m1 */, 0, 0, 0, 0);
}

// ------------------------------------------ binary GEMM, e2m1 operands ----
//
// k_bgemm_pop_q8's results (8-bit half-codes, exact rows and flags) for 65-256
// output columns, on the matrix cores: 32-row tiles, the signs as e2m1 +-1
// against +-1/2 weights (zero past K) that the block keeps in LDS, so a
// 32 x 32 x 64 product takes 32 cycles and the kernel is bound by the codes it
// writes (2.45 M x 256 x 256: 479 us with bit counts, 226 us here for 627 MB
// written; 233 K x 256 x 602: 110 -> 42 us; 169 K x 256 x 256: 42 -> 19 us; at
// 2-10 K rows the two are level).  Lane l holds column l & 31 of every 32-column tile, whose bytes
// fill the interleaved row layout in pieces of 32 lanes: whole 128-byte lines
// for 129-256 columns.
template <int NT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void k_bgemm_q8_e2m1(
    const uint64_t* __restrict__ F, int64_t M, int64_t ldf, const uint64_t* __restrict__ B,
    int32_t N, int64_t ldb, int32_t K, int8_t* __restrict__ C8, int64_t ldc8,
    _Float16* __restrict__ C16, int64_t ldc16, float* __restrict__ g) {
  constexpr int NB = NT / 2;
  extern __shared__ __attribute__((aligned(16))) int4_t s_b[];  // [kw][NT][64]
  const int lane = threadIdx.x & 63;
  const int half = lane >> 5, m = lane & 31;
  const int kw = (K + 63) >> 6;
  for (int i = wave_index_in_block(); i < kw * NT; i += kWavesPerBlock) {
    const int ks = i / NT, col = 32 * (i % NT) + m;
    const int left = K - 64 * ks - 32 * half;
    const uint32_t mask = left >= 32 ? ~0u : left <= 0 ? 0u : (1u << left) - 1;
    const int4_t mk = mask_nibbles(mask);
    const uint64_t w = col < N ? B[col * ldb + ks] : 0ull;
    int4_t v = sign_nibbles<1>(half != 0 ? (uint32_t)(w >> 32) : (uint32_t)w);
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] &= col < N ? mk[u] : 0;
    s_b[i * 64 + lane] = v;
  }
  __syncthreads();
  const int par = K & 1;
  float16_t c0;
#pragma unroll
  for (int i = 0; i < 16; ++i) c0[i] = par != 0 ? -0.5f : 0.f;
  const __amdgpu_buffer_rsrc_t rsc = raw_rsrc(C8, (uint32_t)(M * ldc8));
  const int64_t tiles = (M + 31) / 32;
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  for (int64_t tile = (int64_t)blockIdx.x * kWavesPerBlock + wave_index_in_block(); tile < tiles;
       tile += nwaves) {
    const int64_t r0 = 32 * tile;
    const uint64_t* frow = F + (r0 + m < M ? r0 + m : M - 1) * ldf;
    float16_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = c0;
    uint64_t w = frow[0];
    for (int ks = 0; ks < kw; ++ks) {
      const uint64_t wn = ks + 1 < kw ? frow[ks + 1] : 0ull;
      const int4_t a = sign_nibbles<2>(half != 0 ? (uint32_t)(w >> 32) : (uint32_t)w);
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = mfma_e2m1(a, s_b[(ks * NT + t) * 64 + lane], acc[t]);
      w = wn;
    }
    // acc[t][i]: half-code of row r0 + 8 (i / 4) + 4 half + i % 4, column
    // 32 t + m.  1.5 2^23 + code has the code's two's complement low byte.
    // (Rows past M fall outside the buffer's range.)
    const uint32_t off = (uint32_t)((r0 + 4 * half) * ldc8) + NB * m;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t ro = off + (uint32_t)(8 * (i / 4) + (i & 3)) * (uint32_t)ldc8;
#pragma unroll
      for (int p = 0; p < 2; ++p) {  // columns m + 32 p + 64 c
        int x[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c)
          x[c] = __builtin_bit_cast(int, acc[2 * c + p][i] + 12582912.f);
        const uint32_t v = pack_low_bytes<NB>(x);
        if constexpr (NB == 4)
          __builtin_amdgcn_raw_buffer_store_b32(v, rsc, (int)(ro + 128 * p), 0, 0);
        else
          __builtin_amdgcn_raw_buffer_store_b16((uint16_t)v, rsc, (int)(ro + 64 * p), 0, 0);
      }
    }
    if (K <= 255) continue;  // every code fits
    float hi = 0.f, lo = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        hi = fmaxf(hi, acc[t][i]);
        lo = fminf(lo, acc[t][i]);
      }
    if (__builtin_amdgcn_ballot_w64(hi > 127.f || lo < -128.f) == 0) continue;
    // Some row of the tile has a product that leaves its byte (rare): the
    // tile's rows one by one, lane l on columns l + 64 c, by bit counts.
    for (int64_t r = r0; r < r0 + 32 && r < M; ++r) {
      int dot[NB];
      bool big = false;
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const int col = lane + 64 * c;
        int pc = 0;
        if (col < N)
          for (int ks = 0; ks < kw; ++ks) pc += __builtin_popcountll(F[r * ldf + ks] ^ B[col * ldb + ks]);
        dot[c] = K - 2 * pc;
        const int code = (dot[c] - par) >> 1;
        big |= col < N && (code < -128 || code > 127);
      }
      if (__builtin_amdgcn_ballot_w64(big) == 0) continue;
      store_exact<NB>(C16 + r * ldc16 + NB * lane, dot);
      if (lane == 0) g[r] = -fabsf(g[r]);
    }
  }
}

}  // namespace

// The weights of a block take 1 KB of LDS per 64 inputs and 32 columns; up to
// 80 KB (640 inputs for 256 columns, 1280 for 128) leave room for two blocks
// on a CU.
static size_t e2m1_lds(int32_t N, int32_t K) {
  return (size_t)((K + 63) >> 6) * (N <= 128 ? 4 : 8) * 1024;
}

bool bgemm_q8_e2m1_supported(int64_t M, int32_t N, int32_t K) {
  return M > 0 && N > 64 && N <= 256 && e2m1_lds(N, K) <= 80 * 1024;
}

hipError_t launch_bgemm_q8_e2m1(const uint64_t* F, int64_t M, int64_t ldf, const uint64_t* B,
                                int32_t N, int64_t ldb, int32_t K, int8_t* C8, int64_t ldc8,
                                void* C16, int64_t ldc16, float* g, hipStream_t stream) {
  if (!bgemm_q8_e2m1_supported(M, N, K)) return hipErrorInvalidValue;
  const size_t lds = e2m1_lds(N, K);
  const int64_t tiles = (M + 31) / 32;
  const dim3 grid((unsigned)std::min<int64_t>((tiles + kWavesPerBlock - 1) / kWavesPerBlock, 1024));
#define BIGCN_E2M1(NT)                                                                   \
  do {                                                                                   \
    if (lds > 65536) {                                                                   \
      const hipError_t e = hipFuncSetAttribute(                                          \
          (const void*)k_bgemm_q8_e2m1<NT>, hipFuncAttributeMaxDynamicSharedMemorySize,  \
          80 * 1024);                                                                    \
      if (e != hipSuccess) return e;                                                     \
    }                                                                                    \
    hipLaunchKernelGGL(k_bgemm_q8_e2m1<NT>, grid, dim3(kBlock), lds, stream, F, M, ldf, B, \
                       N, ldb, K, C8, ldc8, (_Float16*)C16, ldc16, g);                   \
  } while (0)
  if (N <= 128)
    BIGCN_E2M1(4);
  else
    BIGCN_E2M1(8);
#undef BIGCN_E2M1
  return hipGetLastError();
}

}  // namespace bigcn
