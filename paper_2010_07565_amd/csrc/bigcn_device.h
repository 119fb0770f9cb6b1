// Device code shared by the aggregations: wave primitives, the 8-bit row
// stores, and what happens to a finished output row (epilogue, fused next
// layer, rows cut by a chunk boundary).
#pragma once

#include "bigcn_internal.h"

#include <hip/hip_fp16.h>

namespace bigcn {
namespace {

constexpr int kBlock = 256;  // 4 waves
constexpr int kWavesPerBlock = kBlock / 64;

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef int int4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// Buffer resource for raw (unformatted) loads: base, stride 0, byte range,
// and the gfx9 default of the fourth descriptor word.  Loads past the range
// return zero.
template <typename T>
__device__ inline __amdgpu_buffer_rsrc_t raw_rsrc(const T* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0, (int)bytes,
                                           0x00020000);
}

constexpr uint32_t kPastEnd = 0x80000000u;  // buffer offset past every range: loads give 0

__device__ inline int wave_index_in_block() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// DPP lane exchange within rows of 16 lanes (quad_perm, row_mirror and
// row_half_mirror controls of gfx9 DPP).
template <int CTRL>
__device__ inline float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                       0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

__device__ inline float wave_sum(float v) {
  // Order-fixed sum, the same in every lane: pairs (xor 1, xor 2), then the
  // mirrored half rows and rows of 16 lanes, then the four rows' sums read
  // out and added as (r0 + r1) + (r2 + r3).
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  const float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
  const float b = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
  const float c = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
  const float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
  return (a + b) + (c + d);
}

// Between a wave's LDS stores and its lanes' loads of each other's values (and
// the other way round): a wave's LDS operations complete in order, so it takes
// no instruction, but neither the compiler's moves nor lanes run apart may
// cross it.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

typedef float float2_t __attribute__((ext_vector_type(2)));

// Lane swaps between two registers: swap32 exchanges lanes 32..63 of a with
// lanes 0..31 of b; swap16 exchanges the odd 16-lane rows of a with the even
// rows of b.  (The results are read into scalars before the bit casts.)
__device__ inline void swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  const uint32_t x = r[0], y = r[1];
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}
__device__ inline void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  const uint32_t x = r[0], y = r[1];
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}

// 8-bit half-codes of one row, NB per lane (lane l: columns l + 64 c), and a
// flagged row's exact products in the same order.
template <int NB>
__device__ inline void store_codes(int8_t* p, uint32_t packed) {
  if constexpr (NB == 4)
    *reinterpret_cast<uint32_t*>(p) = packed;
  else if constexpr (NB == 2)
    *reinterpret_cast<uint16_t*>(p) = (uint16_t)packed;
  else
    *reinterpret_cast<uint8_t*>(p) = (uint8_t)packed;
}

// The low bytes of NB ints as one word (byte c from v[c]), by byte permutes.
template <int NB>
__device__ inline uint32_t pack_low_bytes(const int* v) {
  if constexpr (NB == 4) {
    // v_perm: selector bytes 0-3 take the second operand's bytes, 4-7 the
    // first's, 0x0C gives zero
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x0C0C0400u);
    return __builtin_amdgcn_perm((uint32_t)v[3], (uint32_t)v[2], 0x04000C0Cu) | lo;
  } else if constexpr (NB == 2) {
    return __builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x0C0C0400u);
  } else {
    return (uint32_t)v[0] & 0xFFu;
  }
}

// store_codes for a row address the whole wave shares: a buffer resource
// built on the scalar unit and a lane offset, no per-lane address math.
template <int NB>
__device__ inline void store_codes_row(int8_t* row, int lane, uint32_t packed) {
  const __amdgpu_buffer_rsrc_t rs = raw_rsrc(row, 64u * NB);
  if constexpr (NB == 4)
    __builtin_amdgcn_raw_buffer_store_b32(packed, rs, lane * 4, 0, 0);
  else if constexpr (NB == 2)
    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)packed, rs, lane * 2, 0, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)packed, rs, lane, 0, 0);
}

template <int NB>
__device__ inline void store_exact(_Float16* p, const int* v) {
  if constexpr (NB == 4) {
    half4_t h;
#pragma unroll
    for (int c = 0; c < 4; ++c) h[c] = (_Float16)v[c];
    *reinterpret_cast<half4_t*>(p) = h;
  } else if constexpr (NB == 2) {
    half2_t h;
    h[0] = (_Float16)v[0];
    h[1] = (_Float16)v[1];
    *reinterpret_cast<half2_t*>(p) = h;
  } else {
    *p = (_Float16)v[0];
  }
}

// Stages packed weight rows into LDS as [kw][CN][64]: entry (w*CN + c)*64 + l
// holds word w of the column lane l owns in slot c, so that for a fixed
// (w, c) the 64 lanes read 64 consecutive words.  Lane l owns columns
// j0 + CN*l + c (consecutive) or, with IL, l + 64*c (lane-interleaved).
template <int CN, bool IL = false>
__device__ inline void stage_weights(uint64_t* sB, const uint64_t* __restrict__ B,
                                     int32_t N, int64_t ldb, int kw, int j0) {
  for (int idx = threadIdx.x; idx < kw * CN * 64; idx += kBlock) {
    const int l = idx & 63;
    const int c = (idx >> 6) % CN;
    const int w = idx / (64 * CN);
    const int j = IL ? l + 64 * c : j0 + l * CN + c;
    sB[idx] = j < N ? B[(int64_t)j * ldb + w] : 0ull;
  }
  __syncthreads();
}

// a + b where b may be a product: b is rounded first (no fused multiply-add),
// so that the self term of a two-weight layer of 65-256 outputs is the same
// whichever kernel adds it (up to 64 outputs one kernel does, finish_slot, which
// may contract it).  (A select between the product and the sum did not keep the
// compiler from contracting them in every kernel.)
__device__ inline float add_rounded(float a, float b) {
#pragma clang fp contract(off)
  return a + b;
}

__device__ inline float act(float v, int relu) { return relu ? fmaxf(v, 0.f) : v; }

// Destination-side factor of Ã for a row with deg entries: D̂^-1/2 (mean 0,
// symmetric), D̂^-1 (mean 1), or none (mean 2: the transpose of the mean
// normalisation, whose factor sits on the source side).
__device__ inline float row_factor_deg(int64_t deg, int mean) {
  const float dg = (float)deg;
  return mean == 2 ? 1.0f : mean ? 1.0f / dg : 1.0f / sqrtf(dg);
}

// Partial rows of the 8-bit path: NB floats per lane at p = base + NB*lane.
template <int NB>
__device__ inline void store_partial(float* p, const float4_t v) {
  if constexpr (NB == 4)
    *reinterpret_cast<float4_t*>(p) = v;
  else if constexpr (NB == 2)
    *reinterpret_cast<float2_t*>(p) = float2_t{v[0], v[1]};
  else
    *p = v[0];
}

template <int NB>
__device__ inline float4_t load_partial(const float* p) {
  float4_t v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (NB == 4) {
    v = *reinterpret_cast<const float4_t*>(p);
  } else if constexpr (NB == 2) {
    const float2_t x = *reinterpret_cast<const float2_t*>(p);
    v[0] = x[0];
    v[1] = x[1];
  } else {
    v[0] = *p;
  }
  return v;
}

// What the aggregation does with a finished output row in the 8-bit path.
// Lane l holds columns l + 64c of the row (c < NB, interleaved).
//   NX == 0: write act(rowfac*alpha*acc + b) to out (columns l + 64c).
//   NX == 2: as 0, plus the self term of a two-weight GraphSAGE layer:
//            |g_r| * alpha_self[k] * Cself[r][k] (exact half products of the
//            node's own features with the self weights) before bias / act.
//   NX == 1: the next layer (K' = d inputs, d' <= 256 outputs, NBN bytes per
//            lane) is fused: its sign bits are the ballots of the output
//            values (word c = ballot of slot c, because lane l holds element
//            l + 64c), its scale is their mean magnitude (summed per lane
//            over c, then a butterfly: the order of the pack kernel), and its
//            products against the next weights (in LDS) are written as 8-bit
//            half-codes with the exact fallback, as k_bgemm_pop_q8 does.
//   NX == 4: the next layer reads packed signs: the row's words (the ballots
//            of NX == 1) and scale are written, no products are formed.
// With NX == 1 or 4 the output row is also written to out if out != nullptr.
struct NextLayer {
  int32_t dn;          // next layer's output width d'
  int8_t* C8;          // codes [n][ldc8]
  int64_t ldc8;
  _Float16* C16;       // exact fallback rows [n][ldc16]
  int64_t ldc16;
  float* g;            // next layer's per-node scale
  int sym;             // fold D̂^-1/2 into the next scale
  const _Float16* Cself;  // NX == 2: self products [n][ldself], natural order
  int64_t ldself;
  const float* gself;     // NX == 2: per-node scale (its magnitude is β_i)
  const int32_t* slot;    // nullable: row r's next products / self products
                          // sit at row slot[r] (the source order), else at r
  const uint64_t* F;      // NX == 3: the layer's packed signs, row r at F + r ldF
  int64_t ldF;            // (r = slot[r] when slot is given)
  int32_t kin;            // NX == 3: the layer's input width
  uint64_t* Fn;           // NX == 4: the next layer's packed signs [n][ldFn],
  int64_t ldFn;           // ldFn words (NB, or 2 where NB is 1: the pad word is zero)
};

// The next layer's weights as finish_row reads them.
struct NextRegs {
  const uint64_t* sB;  // LDS: next weights, [kw'][NBN][64] interleaved columns
  uint64_t wr[4];      // or, when NB * NBN <= 4, this lane's words in registers:
                       // wr[w * NBN + c] = word w of column lane + 64c
};

// Everything finish_row reads besides a row's sums and the next weights:
// the first argument of the kernels that finish rows, so that it starts the
// kernel-argument segment.  finish_row reads it afresh at each call (scalar
// loads from that segment behind an opaque pointer, which the compiler
// cannot hoist) instead of the kernel holding its fields in scalar
// registers through the edge loop, where they would crowd out the loop's
// own values.  The per-column alpha, bias and alpha_self sit in LDS
// (stage_epi).
struct FinishArgs {
  NextLayer nx;
  float* out;            // [n][ldo]; nullable when a next layer is formed
  int64_t ldo;
  const float* alpha;    // this layer's alpha [d]
  const float* bias;     // [d] or null
  const float* alpha_s;  // two-weight layer: the self weights' alpha [d]
  int mean;              // destination factor, see row_factor_deg
  int relu;
  int32_t d;             // output width, at most 256
};

// The kernels' FinishArgs from a launcher's arguments.
inline FinishArgs finish_args(int mean, const float* g, int32_t d, const float* alpha,
                              const float* bias, int relu, float* out, int64_t ldo,
                              const FusedNext& fn) {
  FinishArgs fa;
  NextLayer& nx = fa.nx;
  nx.dn = fn.d_out;
  nx.C8 = fn.C8;
  nx.ldc8 = fn.ldc8;
  nx.C16 = (_Float16*)fn.C16;
  nx.ldc16 = fn.ldc16;
  nx.g = fn.g;
  nx.sym = !mean;
  nx.slot = fn.slot;
  nx.Cself = (const _Float16*)fn.Cself;
  nx.ldself = fn.ldself;
  nx.gself = g;
  nx.F = fn.F;
  nx.ldF = fn.ldF;
  nx.kin = fn.kin;
  nx.Fn = fn.Fn;
  nx.ldFn = fn.ldFn;
  fa.out = out;
  fa.ldo = ldo;
  fa.alpha = alpha;
  fa.bias = bias;
  fa.alpha_s = fn.alpha_self;
  fa.mean = mean;
  fa.relu = relu;
  fa.d = d;
  return fa;
}

typedef const __attribute__((address_space(4))) FinishArgs* KernargFinish;
__device__ inline FinishArgs fresh_finish() {
#if defined(__HIP_DEVICE_COMPILE__)
  KernargFinish p = (KernargFinish)__builtin_amdgcn_kernarg_segment_ptr();
  __asm__ volatile("" : "+s"(p));
  return *p;
#else
  return FinishArgs{};  // (the host pass only parses device functions)
#endif
}

// LDS copy of alpha, bias and alpha_self (zero past d) for finish_row, one
// column per thread of the block; ends in a barrier.
__device__ inline void stage_epi(float (*s_epi)[256], const FinishArgs& fa) {
  static_assert(kBlock == 256, "one column per thread");
  const int t = threadIdx.x;
  const bool ok = t < fa.d;
  s_epi[0][t] = ok ? fa.alpha[t] : 0.f;
  s_epi[1][t] = ok && fa.bias != nullptr ? fa.bias[t] : 0.f;
  s_epi[2][t] = ok && fa.alpha_s != nullptr ? fa.alpha_s[t] : 0.f;
  __syncthreads();
}

// Without a fused next layer and with groups of 8 edges (short epilogues,
// frequent on graphs of short rows) the epilogue's arguments stay in the
// kernel's scalar registers and alpha, bias and alpha_self of a lane's
// columns in its registers: a kernel-argument read and LDS reads at every
// finished row measured slower there (arxiv-shaped, 123 -> 139-144 us), and
// these variants have the registers to spare.  finish_row's EPI_LDS says
// which form it takes.
template <int NB>
struct EpiRegs {
  float alpha[NB], bias[NB], alpha_s[NB];
};
template <int NB>
__device__ inline void make_epi_regs(EpiRegs<NB>& er, const FinishArgs& fa, int lane) {
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    const int k = lane + 64 * c;
    const bool ok = k < fa.d;
    er.alpha[c] = ok ? fa.alpha[k] : 0.f;
    er.bias[c] = ok && fa.bias != nullptr ? fa.bias[k] : 0.f;
    er.alpha_s[c] = ok && fa.alpha_s != nullptr ? fa.alpha_s[k] : 0.f;
  }
}

// The first kw of a row's NW packed words (zero past kw), the row address
// the same in every lane: read-only, so they come through scalar loads.
template <int NW>
__device__ inline void load_row_words(uint64_t (&fw)[NW], const uint64_t* __restrict__ row,
                                      int kw) {
#pragma unroll
  for (int w = 0; w < NW; ++w) fw[w] = w < kw ? row[w] : 0ull;
}

// Lane 0's v to *p, and lanes 0 .. n - 1's words to p[0 .. n), through
// buffers of that size (no branch on the lane, see finish_row).
template <typename T>
__device__ inline void store_first(T* p, int lane, T v) {
  static_assert(sizeof(T) == 4, "one dword");
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), raw_rsrc(p, 4u),
                                        lane * 4, 0, 0);
}
__device__ inline void store_words(uint64_t* p, uint32_t n, int lane, uint64_t v) {
  typedef uint32_t uint2_b __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2_b, v), raw_rsrc(p, n * 8u),
                                        lane * 8, 0, 0);
}

template <int NX, int NB, int NBN, bool EPI_LDS>
__device__ inline void finish_row(int64_t r, int64_t deg, const float4_t acc,
                                  const float (*s_epi)[256], const EpiRegs<NB>& er,
                                  const NextRegs& nr, const FinishArgs& fa_arg, int lane) {
  // EPI_LDS: the arguments are read afresh (see FinishArgs) and alpha /
  // bias come from LDS; else from the kernel argument's scalar registers
  // and the lane's registers (EpiRegs).
  const FinishArgs fa = EPI_LDS ? fresh_finish() : fa_arg;
  const NextLayer& nx = fa.nx;
  bool valid[NB];  // column lane + 64c < d
#pragma unroll
  for (int c = 0; c < NB; ++c) valid[c] = lane + 64 * c < fa.d;
  const float rowfac = deg > 0 ? row_factor_deg(deg, fa.mean) : 0.f;
  int64_t dst = r;  // row of the next products / self products
  if (NX != 0 && nx.slot != nullptr) dst = nx.slot[r];
  float self[NB];
  if constexpr (NX == 3) {
    // The two-weight layer's self products, formed here: the row's own
    // packed signs (wave-uniform, scalar loads) against the self weights
    // staged in LDS (NBN words per lane and column) -- the products Cself
    // holds for NX == 2, exactly.
    const int kws = (nx.kin + 63) >> 6;  // <= NBN
    uint64_t fw[NBN];
    load_row_words<NBN>(fw, nx.F + dst * nx.ldF, kws);
    const float gi = fabsf(nx.gself[dst]);
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      uint32_t pc = 0;
#pragma unroll
      for (int w = 0; w < NBN; ++w) {
        if (w >= kws) continue;  // wave-uniform
        const uint64_t z = fw[w] ^ nr.sB[(w * NB + c) * 64 + lane];
        pc += __builtin_popcount((uint32_t)z);
        pc += __builtin_popcount((uint32_t)(z >> 32));
      }
      const int dot = nx.kin - 2 * (int)pc;
      self[c] = valid[c] ? gi * (EPI_LDS ? s_epi[2][lane + 64 * c] : er.alpha_s[c]) * (float)dot
                         : 0.f;
    }
  }
  if (NX == 2) {
    const float gi = fabsf(nx.gself[dst]);
    // (columns past d fall outside the buffer: zero)
    const __amdgpu_buffer_rsrc_t rsc = raw_rsrc(nx.Cself + dst * nx.ldself, (uint32_t)fa.d * 2u);
    float cs[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c)
      cs[c] = (float)__builtin_bit_cast(
          _Float16, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsc, (lane + 64 * c) * 2, 0, 0));
#pragma unroll
    for (int c = 0; c < NB; ++c)
      self[c] = valid[c] ? gi * (EPI_LDS ? s_epi[2][lane + 64 * c] : er.alpha_s[c]) * cs[c] : 0.f;
  }
  float v[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    const float al = EPI_LDS ? s_epi[0][lane + 64 * c] : er.alpha[c];
    const float bi = EPI_LDS ? s_epi[1][lane + 64 * c] : er.bias[c];
    float t = deg > 0 ? fmaf(acc[c], rowfac * al, bi) : bi;
    if (NX == 2 || NX == 3) t = add_rounded(t, self[c]);
    v[c] = act(t, fa.relu);
  }
  // Loads and stores go through buffers that end with the row, so lanes past
  // it need no branch: with one in the callers' row loops the compiler ran
  // those loops apart for the lanes on either side of it, and cross-lane
  // reads of the row window found lanes that had not moved on yet (after rows
  // without entries some rows were then never written).
  if ((NX != 1 && NX != 4) || fa.out != nullptr) {
    const __amdgpu_buffer_rsrc_t rso = raw_rsrc(fa.out + r * fa.ldo, (uint32_t)fa.d * 4u);
#pragma unroll
    for (int c = 0; c < NB; ++c)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v[c]), rso,
                                            (lane + 64 * c) * 4, 0, 0);
  }
  if (NX != 1 && NX != 4) return;
  // Next layer: signs (one ballot per 64 elements = one packed word) and
  // mean magnitude, exactly as the pack kernel forms them.
  uint64_t word[NB];
  float l1 = 0.f;
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    word[c] = __builtin_amdgcn_ballot_w64(valid[c] && v[c] >= 0.f);
    l1 += valid[c] ? fabsf(v[c]) : 0.f;
  }
  l1 = wave_sum(l1);
  float sc = l1 / (float)fa.d;
  if (nx.sym) sc = sc * (deg > 0 ? 1.0f / sqrtf((float)deg) : 0.f);
  if constexpr (NX == 4) {
    uint64_t mine = 0;  // lane w: word w (the pad word of a narrow row stays zero)
#pragma unroll
    for (int c = 0; c < NB; ++c) mine = lane == c ? word[c] : mine;
    store_words(nx.Fn + dst * nx.ldFn, (uint32_t)nx.ldFn, lane, mine);
    store_first(nx.g + dst, lane, sc);
    return;
  }
  const int kwn = (fa.d + 63) >> 6;  // <= NB
  const int Kn = fa.d;
  const int par = Kn & 1;
  bool big = false;
  uint32_t packed = 0;
  int dot[NBN];
#pragma unroll
  for (int c = 0; c < NBN; ++c) {
    uint32_t pc = 0;
#pragma unroll
    for (int w = 0; w < NB; ++w) {
      if (w >= kwn) break;
      const uint64_t bw = NB * NBN <= 4 ? nr.wr[(w * NBN + c) & 3]
                                        : nr.sB[(w * NBN + c) * 64 + lane];
      const uint64_t z = word[w] ^ bw;
      pc += __builtin_popcount((uint32_t)z);
      pc += __builtin_popcount((uint32_t)(z >> 32));
    }
    dot[c] = Kn - 2 * (int)pc;
    const int code = (dot[c] - par) >> 1;
    big |= (lane + 64 * c < nx.dn) && (code < -128 || code > 127);
    packed |= (uint32_t)(uint8_t)(int8_t)code << (8 * c);
  }
  store_codes_row<NBN>(nx.C8 + dst * nx.ldc8, lane, packed);
  const bool flag = __builtin_amdgcn_ballot_w64(big) != 0;
  if (flag) store_exact<NBN>(nx.C16 + dst * nx.ldc16 + NBN * lane, dot);
  store_first(nx.g + dst, lane, flag ? -sc : sc);
}

// The next layer's weights for finish_row: in registers when a lane needs
// at most four words (NB * NBN <= 4; no LDS, no block barrier), else staged
// in LDS by the whole block (stage_weights, which ends in a barrier).
template <int NB, int NBN>
__device__ inline void load_next_weights(NextRegs& nx, int32_t dn, uint64_t* sBn,
                                         const uint64_t* __restrict__ Bn, int64_t ldbn,
                                         int32_t d, int lane) {
  const int kwn = (d + 63) >> 6;
  if constexpr (NB * NBN <= 4) {
#pragma unroll
    for (int w = 0; w < NB; ++w)
#pragma unroll
      for (int c = 0; c < NBN; ++c) {
        const int col = lane + 64 * c;
        nx.wr[(w * NBN + c) & 3] =
            (w < kwn && col < dn) ? Bn[(int64_t)col * ldbn + w] : 0ull;
      }
    nx.sB = nullptr;
  } else {
    stage_weights<NBN, true>(sBn, Bn, dn, ldbn, kwn, 0);
    nx.sB = sBn;
  }
}

// The row holding edge s, rowptr[r] <= s < rowptr[r+1] (rows without
// entries are skipped), by a wave-wide search: each step the 64 lanes probe
// 64 evenly spaced row starts of the current range [lo, hi), which shrinks
// 65-fold; once it is at most 64 rows wide, lane l loads the start and end
// of row lo + l.  Returns r; lo, and this lane's start / end, are the window
// the aggregation walks from.  Requires rowptr[0] <= s < rowptr[n].
__device__ inline int64_t find_row(const int64_t* __restrict__ rowptr, int64_t n, int64_t s,
                                   int lane, int64_t& lo_out, int64_t& start_l,
                                   int64_t& end_l) {
  int64_t lo = 0, hi = n;
  while (hi - lo > 64) {
    const int64_t step = (hi - lo + 64) / 65;
    const int64_t p = lo + (int64_t)(lane + 1) * step;
    const bool le = p < hi && rowptr[p] <= s;
    const int c = (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(le));
    const int64_t nhi = lo + (int64_t)(c + 1) * step;
    lo += (int64_t)c * step;
    if (nhi < hi) hi = nhi;
  }
  start_l = rowptr[lo + lane < n ? lo + lane : n];
  end_l = rowptr[lo + 1 + lane < n ? lo + 1 + lane : n];
  lo_out = lo;
  const uint64_t done = __builtin_amdgcn_ballot_w64(lo + 1 + lane <= n && end_l <= s);
  return lo + (int64_t)__builtin_popcountll(done);
}

__device__ inline int64_t readlane64(int64_t v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Fix-up of the 8-bit path: rows cut by chunk boundaries, partial rows in
// interleaved order, finished with the same finish_row.  One wave serves
// four workers: their cut rows, row bounds and first two partial rows are
// loaded together (lanes 0..3 fetch the per-worker scalars), then the rows
// are finished in worker order.
template <int NX, int NB, int NBN>
__global__ __launch_bounds__(kBlock) void k_spmm_fix_q8(
    FinishArgs fa, const int64_t* __restrict__ rowptr, int64_t chunk, int64_t workers,
    int32_t dpad, const int32_t* __restrict__ tail_row,
    const float* __restrict__ head, const float* __restrict__ tail,
    const uint64_t* __restrict__ Bn, int64_t ldbn) {
  extern __shared__ uint64_t sBn[];
  __shared__ float s_epi[3][256];
  const int lane = threadIdx.x & 63;
  NextRegs nr = {};
  if (NX == 1) load_next_weights<NB, NBN>(nr, fa.nx.dn, sBn, Bn, ldbn, fa.d, lane);
  // NX == 3: the self weights, NBN words by NB columns per lane, in LDS
  if (NX == 3) load_next_weights<NBN, NB>(nr, fa.d, sBn, Bn, ldbn, fa.nx.kin, lane);
  constexpr bool kEpiLds = NX == 1 || NX == 3 || NX == 4;  // where finish_row reads alpha / bias
  if constexpr (kEpiLds) stage_epi(s_epi, fa);
  EpiRegs<NB> er = {};
  if constexpr (!kEpiLds) make_epi_regs<NB>(er, fa, lane);
  const int64_t w0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave_index_in_block()) * 4;
  if (w0 >= workers) return;
  // lane q < 4: worker w0 + q's cut row and that row's bounds
  const int64_t wq = w0 + (lane & 3);
  const int32_t rq = wq < workers ? tail_row[wq] : -1;
  const int64_t bq = rq >= 0 ? rowptr[rq] : 0;
  const int64_t eq = rq >= 0 ? rowptr[rq + 1] : 0;
  float4_t acc[4], nxt[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {  // tail of the worker and the next head
    const int32_t r = __builtin_amdgcn_readlane(rq, q);
    if (r >= 0) {
      const int64_t w = w0 + q;
      acc[q] = load_partial<NB>(tail + w * dpad + NB * lane);
      nxt[q] = load_partial<NB>(head + (w + 1) * dpad + NB * lane);
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int32_t r = __builtin_amdgcn_readlane(rq, q);
    if (r < 0) continue;
    const int64_t w = w0 + q;
    const int64_t e = readlane64(eq, q);
    const int64_t wend = (e - 1) / chunk;  // > w: a cut row continues past w
    float4_t a = acc[q] + nxt[q];
    int64_t v = w + 2;
    for (; v + 8 <= wend + 1; v += 8) {  // eight loads in flight, added in order
      float4_t h[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) h[u] = load_partial<NB>(head + (v + u) * dpad + NB * lane);
#pragma unroll
      for (int u = 0; u < 8; ++u) a += h[u];
    }
    for (; v <= wend; ++v) a += load_partial<NB>(head + v * dpad + NB * lane);
    finish_row<NX, NB, NBN, kEpiLds>(r, e - readlane64(bq, q), a, s_epi, er, nr, fa, lane);
  }
}

}  // namespace
}  // namespace bigcn
