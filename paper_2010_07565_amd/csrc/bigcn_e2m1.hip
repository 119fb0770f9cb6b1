// Sign products on the matrix cores as 4-bit floats (e2m1: +-1 against +-1/2,
// which give the half-codes (dot - K % 2) / 2 exactly; a 32 x 32 x 64 product
// takes 32 cycles, twice the int8 rate):
//   k_spmm_sign      aggregation that gathers packed signs and forms the
//                    products itself
//   k_bgemm_q8_e2m1  binary GEMM into 8-bit half-codes
// The 100 -> 256 aggregation of the products-shaped graph keeps the matrix core
// busy for 40 % of the SIMD cycles; in 62 % of those a vector instruction issues as
// well.  Vector instructions, at four cycles each, take 78 %, either kind 93 %: it
// is bound by vector issue, with most of the products beside it.

#include "bigcn_device.h"

#include <algorithm>
#include <type_traits>

namespace bigcn {
namespace {

typedef int int8v_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t uint4_v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2_v __attribute__((ext_vector_type(2)));

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

// old with lane i's (wave-uniform i) value replaced by v (wave-uniform); the
// intrinsic has no builtin of its own.
extern "C" __device__ int amdgcn_writelane(int v, int i, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ inline int write_lane(int v, int i, int old) { return amdgcn_writelane(v, i, old); }

// v summed over lanes 0 .. lane.
__device__ inline int wave_prefix(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

__device__ inline int from_lane(int v, int src) {  // src per lane
  return __builtin_amdgcn_ds_bpermute(src * 4, v);
}
__device__ inline float lane_float(float v, int i) {  // i wave-uniform
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), i));
}

// The sums of k_spmm_wave_q8 (the same chunks of edges, rows cut by a chunk
// boundary left to k_spmm_fix_q8) with a gather of packed signs: 16 or 32
// bytes an edge instead of the 128 or 256 of ready products, whose lines past
// L2 bound k_spmm_wave_q8.  Here a tile of 32 edges is bound by its vector
// instructions: for 128 inputs and 256 outputs 128 FMAs and ~110 others, beside
// 16 products of 32 cycles.  Products-shaped graph (2.45 M nodes, 126 M entries),
// 100 -> 256: 4.31 -> 2.90 ms, 0.45 lines an edge past L2 instead of 1.9; 100 -> 128
// layer with its pack 3.08 -> 2.14 ms.  A wave takes `run` consecutive chunks.
//
// A wave works through a chunk in tiles of four blocks of eight edges.  A
// block holds edges of one row only (the first block of a row starts at the
// row's first edge rounded down to an even position; places before the row,
// past it or past the chunk count with scale zero), so a tile may hold up to
// four short rows.  Edge 2 i + h of block b is row 8 b + 4 h + i of the
// matrix tile: lanes 0-31 then hold the products of the even edges and
// lanes 32-63 those of the odd ones, in order, which are the two chains
// (a0, a1) k_spmm_wave_q8 keeps, so the sums are the same additions.
//
// Per tile: 32 x K signs as e2m1 +-1 against the weights' +-1/2 (zero past
// K), accumulated from 0 or, for odd K, -1/2, give the half-codes
// (dot - K % 2) / 2 exactly.  KS: inputs in steps of 64 (a lane's sign words
// of a row: KS dwords), NT: output columns in tiles of 32.
//
// Rows are taken 64 at a time (the window, a row per lane): their degrees,
// factors and places are formed for all lanes at once, a prefix sum numbers
// their blocks, and for 64 blocks at a time (a batch) every lane looks up
// the row, first edge and length of one block.  What a finished row of a
// fused layer leaves (signs, scale) waits in the row's lane and is stored
// once per window.
//
// The layer's weights are read from LDS at every product (in registers they
// left two waves per SIMD and 0.3 ms more there), at three waves per SIMD
// half of the LDS rate.
//
// ID: the products are the signs themselves (the weights are the identity,
// K columns): out = rowfac sum_e g_j sign(h_j), as the backward pass needs it.
// Tile t's columns are then one dword of the signs, so it takes one product
// (whatever KS), and the two operands it needs stay in registers.  The rows of
// F are ldw words apart there (W is not used).
template <int KS, int NT, int NX, int NBN, int P, bool ID = false>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3))) void k_spmm_sign(
    FinishArgs fa, int64_t n, int64_t nnz, const int64_t* __restrict__ rowptr,
    const int32_t* __restrict__ colidx, const float* __restrict__ g,
    const uint64_t* __restrict__ F, const uint64_t* __restrict__ W, int64_t ldw, int32_t K,
    int32_t chunk, int32_t run, int64_t workers, int32_t dpad, int32_t* __restrict__ tail_row,
    float* __restrict__ head, float* __restrict__ tails, const uint64_t* __restrict__ Bn,
    int64_t ldbn) {
  constexpr int NB = NT / 2;  // finished columns per lane
  extern __shared__ uint64_t sBn[];
  __shared__ __attribute__((aligned(16))) int4_t s_w[ID ? 1 : NT * KS * 64];  // this layer's weights
  __shared__ float s_epi[3][256];
  __shared__ __attribute__((aligned(16))) float4_t s_ab[2][64];  // alpha, bias of a lane's columns
  __shared__ __attribute__((aligned(16))) float s_gw[kWavesPerBlock][64];
  const int lane = threadIdx.x & 63;
  const int wave = wave_index_in_block();
  const int half = lane >> 5;
  NextRegs nr = {};
  if (NX == 1) load_next_weights<NB, NBN>(nr, fa.nx.dn, sBn, Bn, ldbn, fa.d, lane);
  if (NX == 3) load_next_weights<NBN, NB>(nr, fa.d, sBn, Bn, ldbn, fa.nx.kin, lane);
  // This layer's weights: column 32 t + (lane & 31), dwords half KS + ks.
  auto weights = [&](int t, int ks) -> int4_t {
    const int dw = half * KS + ks;
    const int left = K - 32 * dw;
    const uint32_t m = left >= 32 ? ~0u : left <= 0 ? 0u : (1u << left) - 1;
    const int4_t mk = mask_nibbles(m);
    const int col = 32 * t + (lane & 31);
    uint32_t w = 0;
    if (m != 0 && col < fa.d) w = reinterpret_cast<const uint32_t*>(W + col * ldw)[dw];
    int4_t v = sign_nibbles<1>(w);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] &= mk[i];
    return v;
  };
  // ID: -1/2 (set bits expand to -1) at the lane's column, for tiles of either
  // half of the signs
  int4_t one[2] = {};
  if constexpr (ID) {
    static_assert(NX == 0 && P == 0 && NT <= 2 * KS, "a sign dword per tile");
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = (lane & 3) == i ? (int)(9u << (4 * ((lane & 31) >> 2))) : 0;
      one[0][i] = half == 0 ? v : 0;
      one[1][i] = half == 0 ? 0 : v;
    }
  } else {
    for (int t = wave; t < NT; t += kWavesPerBlock)
#pragma unroll
      for (int k = 0; k < KS; ++k) s_w[(t * KS + k) * 64 + lane] = weights(t, k);
  }
  if (threadIdx.x < 128) {  // (zero past d)
    const bool al = threadIdx.x < 64;
    const float* src = al ? fa.alpha : fa.bias;
    float4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NB; ++c)
      if (lane + 64 * c < fa.d && src != nullptr) v[c] = src[lane + 64 * c];
    s_ab[al ? 0 : 1][lane] = v;
  }
  stage_epi(s_epi, fa);  // ends in a barrier
  const int64_t w0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * run;  // first chunk
  if (w0 >= workers) return;
  const int64_t w1 = w0 + run < workers ? w0 + run : workers;
  const int64_t s = w0 * chunk;  // positions below count from this edge
  const int len = (int)((w1 * chunk < nnz ? w1 * chunk : nnz) - s);
  const bool at_end = s + len == nnz;

  auto rel = [&](int64_t v) -> int {
    const int64_t x = v - s;
    return (int)(x < -1 ? -1 : (x > len + 1 ? len + 1 : x));
  };
  int64_t base, start_l, end_l;  // the window: lane l holds row base + l
  find_row(rowptr, n, s, lane, base, start_l, end_l);

  float16_t c0;
#pragma unroll
  for (int i = 0; i < 16; ++i) c0[i] = P != 0 ? -0.5f : 0.f;

  const __amdgpu_buffer_rsrc_t rsf = raw_rsrc(
      F, ID ? (uint32_t)((n - 1) * ldw * 8 + KS * 8) : (uint32_t)(n * (KS * 8)));
  const uint32_t f_row = ID ? (uint32_t)ldw * 8u : KS * 8u;
  const __amdgpu_buffer_rsrc_t rsg = raw_rsrc(g, (uint32_t)(n * 4));
  const __amdgpu_buffer_rsrc_t rsi = raw_rsrc(colidx + s, (uint32_t)len * 4u);
  // this lane's matrix row: block mb of the tile, edge me of the block
  const int mb = (lane >> 3) & 3;
  const int me = 2 * (lane & 3) + ((lane >> 2) & 1);
  float* gw = &s_gw[wave][0];
  const float4_t zero4 = {0.f, 0.f, 0.f, 0.f};

  // Window state per lane: bounds (relative), destination factor, the row's
  // place in the next layer's (or its own, NX 3) buffers, its own scale (NX 3).
  int st, en, dst_l = 0;
  float rf_l, gi_l = 0.f;
  uint64_t done = 0;  // rows finished in this window
  // NX 4, per lane: the finished row's packed words and sum of magnitudes
  int wlo[NB], whi[NB];
  float l1_l = 0.f;
#pragma unroll
  for (int c = 0; c < NB; ++c) wlo[c] = whi[c] = 0;
  auto open_window = [&]() {
    const int64_t rr = base + lane;
    const bool in = rr < n;
    st = rel(start_l);
    en = rel(end_l);
    const int64_t deg = end_l - start_l;
    rf_l = deg > 0 ? row_factor_deg(deg, fa.mean) : 0.f;
    if (NX != 0) {
      dst_l = (int)rr;
      if (fa.nx.slot != nullptr && in) dst_l = fa.nx.slot[rr];
      if (NX == 3) gi_l = in ? fabsf(fa.nx.gself[dst_l]) : 0.f;
    }
    done = 0;
  };
  auto close_window = [&]() {
    if constexpr (NX == 4) {
      const NextLayer nx = fresh_finish().nx;
      float sc = l1_l / (float)fa.d;
      if (nx.sym) sc = sc * rf_l;  // D̂^-1/2: the symmetric destination factor
      // (rows of NB words; lanes without a finished row store past the end,
      // without a branch in the window loop: see finish_row)
      const uint32_t off = ((done >> lane) & 1) != 0 ? 0u : kPastEnd;
      const __amdgpu_buffer_rsrc_t rsn = raw_rsrc(nx.Fn, (uint32_t)(n * (NB * 8)));
#pragma unroll
      for (int c = 0; c < NB; c += 2) {
        const uint4_v two = {(uint32_t)wlo[c], (uint32_t)whi[c], (uint32_t)wlo[c + 1],
                             (uint32_t)whi[c + 1]};
        __builtin_amdgcn_raw_buffer_store_b128(
            two, rsn, (int)(((uint32_t)dst_l * (NB * 8u) + 8u * c) | off), 0, 0);
      }
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, sc),
                                            raw_rsrc(nx.g, (uint32_t)(n * 4)),
                                            (int)((uint32_t)dst_l * 4u | off), 0, 0);
    }
  };
  // The epilogue of finish_row for row i of the window: the same operations,
  // with what every row needs formed per window.
  // (rows without entries, empty, get the bias: not 0 * alpha, which may overflow)
  auto finish = [&](int i, const float4_t acc, bool empty) {
    const FinishArgs f = NX == 0 || NX == 4 ? fa : fresh_finish();
    const float rf = lane_float(rf_l, i);
    const int64_t r = base + i;
    const int64_t dst = NX == 1 || NX == 3 ? (int64_t)__builtin_amdgcn_readlane(dst_l, i) : 0;
    float self[NB];
    if constexpr (NX == 3) {
      const int kws = (f.nx.kin + 63) >> 6;
      uint64_t fw[NBN];
      load_row_words<NBN>(fw, f.nx.F + dst * f.nx.ldF, kws);
      const float gi = lane_float(gi_l, i);
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
        const int dot = f.nx.kin - 2 * (int)pc;
        self[c] = lane + 64 * c < f.d ? gi * s_epi[2][lane + 64 * c] * (float)dot : 0.f;
      }
    }
    float v[NB];
    const float4_t al = s_ab[0][lane], bi = s_ab[1][lane];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      float t = empty ? bi[c] : fmaf(acc[c], rf * al[c], bi[c]);
      if (NX == 3) t = add_rounded(t, self[c]);
      v[c] = act(t, f.relu);
    }
    if ((NX != 1 && NX != 4) || f.out != nullptr) {  // (see finish_row)
      const FinishArgs o = fresh_finish();
      const __amdgpu_buffer_rsrc_t rso = raw_rsrc(o.out + r * o.ldo, (uint32_t)o.d * 4u);
#pragma unroll
      for (int c = 0; c < NB; ++c)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v[c]), rso,
                                              (lane + 64 * c) * 4, 0, 0);
    }
    if constexpr (NX == 1 || NX == 4) {
      uint64_t word[NB];
      float l1 = 0.f;
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        word[c] = __builtin_amdgcn_ballot_w64(lane + 64 * c < f.d && v[c] >= 0.f);
        // (past d, which is more than half the columns, the sums are of zeros only
        // while every scale is finite)
        l1 += c < NB / 2 || lane + 64 * c < f.d ? fabsf(v[c]) : 0.f;
      }
      l1 = wave_sum(l1);
      if constexpr (NX == 4) {
        l1_l = lane == i ? l1 : l1_l;
#pragma unroll
        for (int c = 0; c < NB; ++c) {
          wlo[c] = write_lane((int)(uint32_t)word[c], i, wlo[c]);
          whi[c] = write_lane((int)(uint32_t)(word[c] >> 32), i, whi[c]);
        }
        done |= 1ull << i;
      } else {
        static_assert(NX != 1 || NBN == 1, "next products of at most 64 columns");
        float sc = l1 / (float)f.d;
        if (f.nx.sym) sc = sc * rf;
        const int kwn = (f.d + 63) >> 6;
        uint32_t pc = 0;
#pragma unroll
        for (int w = 0; w < NB; ++w) {
          if (w >= kwn) break;
          const uint64_t z = word[w] ^ nr.wr[w];
          pc += __builtin_popcount((uint32_t)z);
          pc += __builtin_popcount((uint32_t)(z >> 32));
        }
        const int dot[1] = {f.d - 2 * (int)pc};
        const int code = (dot[0] - (f.d & 1)) >> 1;
        const bool big = lane < f.nx.dn && (code < -128 || code > 127);
        store_codes_row<1>(f.nx.C8 + dst * f.nx.ldc8, lane, (uint32_t)(uint8_t)(int8_t)code);
        const bool flag = __builtin_amdgcn_ballot_w64(big) != 0;
        if (flag) store_exact<1>(f.nx.C16 + dst * f.nx.ldc16 + lane, dot);
        store_first(f.nx.g + dst, lane, flag ? -sc : sc);
      }
    }
  };

  open_window();
  // rows without entries at the run's first position, before the window
  for (int64_t q = base - 1; q >= 0 && rowptr[q] == s; --q) {
    const EpiRegs<NB> er = {};
    finish_row<NX, NB, NBN, true>(q, 0, zero4, s_epi, er, nr, fa, lane);
  }

  for (int64_t w = w0; w < w1; ++w) {
    const int cs = (int)(w - w0) * chunk;  // this chunk
    const int ce = cs + chunk < len ? cs + chunk : len;
    float acc[NT];
    float gsum = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = 0.f;
    // columns lane + 64 c from the two chains of 32-column tiles 2 c, 2 c + 1
    auto both_chains = [&](float a, float b) -> float {
      swap32(a, b);
      return a + b;
    };
    int open_row = -1;  // lane of the row that reaches past the chunk
    for (;;) {  // windows
      const int lo = st > cs ? st : cs;
      const int hi = en < ce ? en : ce;
      const int nb = hi > lo ? (hi - (lo & ~1) + 7) >> 3 : 0;
      const int pre = wave_prefix(nb);  // blocks of rows 0 .. lane
      const int total = __builtin_amdgcn_readlane(pre, 63);
      const uint64_t ahead = __builtin_amdgcn_ballot_w64(st < cs);  // began before the chunk
      // rows with edges here, in order; rows without any entry
      uint64_t rows = __builtin_amdgcn_ballot_w64(nb > 0);
      uint64_t empty = __builtin_amdgcn_ballot_w64(
          st == en && st >= cs && base + lane < n &&
          (st < ce || (at_end && ce == len && st == len)));
      while (empty != 0) {
        const int i = __builtin_ctzll(empty);
        empty &= empty - 1;
        finish(i, zero4, true);
      }
      struct Tile {  // gathered
        uint32_t f[KS];  // lane: sign dwords half KS .. of matrix row lane & 31
        float g;         // lane < 32: scale of matrix row lane
        int ended;       // bit b: block b ends its row; bit 4: the tile exists
      };
      struct Next {  // looked up
        uint32_t j;    // lane: source of matrix row lane & 31
        uint32_t bad;  // kPastEnd on lanes without an edge, else 0
        int ended;
      };
      uint32_t desc = 0;     // lane l: block l of the batch, first place << 8 | empty places
      uint64_t ends = 0;     // blocks of the batch that end their row
      int next_block = 0;    // of the window
      auto look_up = [&]() -> Next {
        Next x;
        if (next_block >= total) {
          x.j = 0;
          x.bad = kPastEnd;
          x.ended = 0;
          return x;
        }
        if ((next_block & 63) == 0) {  // a new batch: lane l takes block next_block + l
          const int blk = next_block + lane;
          int i = 0;  // its row: the first with pre > blk
#pragma unroll
          for (int step = 32; step > 0; step >>= 1)
            if (from_lane(pre, i + step - 1) <= blk) i += step;
          const int lo_i = from_lane(lo, i), hi_i = from_lane(hi, i), en_i = from_lane(en, i);
          const int first = from_lane(pre - nb, i);
          const int e0 = (lo_i & ~1) + 8 * (blk - first);
          const bool in = blk < total;
          const int cnt = hi_i - e0 < 8 ? hi_i - e0 : 8;
          const uint32_t empty = in ? ((0xFFu << cnt) & 0xFFu) | (e0 < lo_i ? 1u : 0u) : 0xFFu;
          desc = ((uint32_t)e0 << 8) | empty;
          ends = __builtin_amdgcn_ballot_w64(in && e0 + 8 >= hi_i && en_i <= ce);
        }
        const int k = next_block & 63;
        const uint32_t d = (uint32_t)from_lane((int)desc, k + mb);
        x.bad = (d << (31 - me)) & kPastEnd;
        const uint32_t eo = ((d >> 6) & ~3u) + 4u * me;
        x.j = __builtin_amdgcn_raw_buffer_load_b32(rsi, (int)(eo | x.bad), 0, 0);
        x.ended = (int)((ends >> k) & 15) | 16;
        next_block += 4;
        return x;
      };
      auto gather = [&](const Next& x) -> Tile {
        Tile tl;
        const uint32_t fo = (x.j * f_row + half * (KS * 4u)) | x.bad;
        const uint32_t go = (x.j * 4u) | (half != 0 ? kPastEnd : 0u) | x.bad;
        if constexpr (KS == 4) {
          const uint4_v v = __builtin_bit_cast(
              uint4_v, __builtin_amdgcn_raw_buffer_load_b128(rsf, (int)fo, 0, 0));
#pragma unroll
          for (int k = 0; k < 4; ++k) tl.f[k] = v[k];
        } else {
          static_assert(KS == 2, "16- or 32-byte sign rows");
          const uint2_v v = __builtin_bit_cast(
              uint2_v, __builtin_amdgcn_raw_buffer_load_b64(rsf, (int)fo, 0, 0));
          tl.f[0] = v[0];
          tl.f[1] = v[1];
        }
        tl.g = __builtin_bit_cast(float,
                                  __builtin_amdgcn_raw_buffer_load_b32(rsg, (int)go, 0, 0));
        tl.ended = x.ended;
        return tl;
      };

      // indices three tiles ahead of the sums, signs and scales two ahead
      Next x = look_up();
      Next y = look_up();
      Next xx = look_up();
      Tile cur = gather(x);
      Tile nxt = gather(y);
      while (cur.ended != 0) {
        const Next xn = look_up();
        const Tile nn = gather(xx);
        xx = xn;
        wave_lds_sync();
        gw[lane] = cur.g;  // (lanes 32-63: zero, not read)
        wave_lds_sync();
        int4_t av[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) av[k] = sign_nibbles<2>(cur.f[k]);
        float gv[16];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const float4_t q = *reinterpret_cast<const float4_t*>(gw + 8 * b + 4 * half);
#pragma unroll
          for (int i = 0; i < 4; ++i) gv[4 * b + i] = q[i];
        }
        float gs[4] = {0.f, 0.f, 0.f, 0.f};  // P: sum of g of the row up to block b, in edge order
        if constexpr (P != 0) {
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const float4_t q0 = *reinterpret_cast<const float4_t*>(gw + 8 * b);
            const float4_t q1 = *reinterpret_cast<const float4_t*>(gw + 8 * b + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              gsum += q0[i];
              gsum += q1[i];
            }
            gs[b] = gsum;
            if ((cur.ended >> b) & 1) gsum = 0.f;
          }
        }
        auto products = [&](int t) -> float16_t {
          if constexpr (ID) return mfma_e2m1(av[t % KS], one[t / KS], c0);
          float16_t d = c0;
#pragma unroll
          for (int k = 0; k < KS; ++k) d = mfma_e2m1(av[k], s_w[(t * KS + k) * 64 + lane], d);
          return d;
        };
        if (cur.ended == 16) {  // no row ends in this tile
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float16_t d = products(t);
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t] = fmaf(d[i], gv[i], acc[t]);
          }
        } else {
          float4_t z[4] = {zero4, zero4, zero4, zero4};
          float e[2][4];
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float16_t d = products(t);
            float a = acc[t];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
#pragma unroll
              for (int i = 0; i < 4; ++i) a = fmaf(d[4 * b + i], gv[4 * b + i], a);
              e[t & 1][b] = a;
              a = ((cur.ended >> b) & 1) ? 0.f : a;
            }
            acc[t] = a;
            if ((t & 1) != 0) {
#pragma unroll
              for (int b = 0; b < 4; ++b) z[b][t / 2] = both_chains(e[0][b], e[1][b]);
            }
          }
          uint32_t todo = (uint32_t)cur.ended & 15u;
          do {
            const int b = __builtin_ctz(todo);
            todo &= todo - 1;
            float4_t sum = b == 0 ? z[0] : b == 1 ? z[1] : b == 2 ? z[2] : z[3];
            if constexpr (P != 0) {
              const float q = b == 0 ? gs[0] : b == 1 ? gs[1] : b == 2 ? gs[2] : gs[3];
              sum = 2.f * sum + q;
            } else {
              sum = 2.f * sum;
            }
            const int i = __builtin_ctzll(rows);
            rows &= rows - 1;
            if ((ahead >> i) & 1)
              store_partial<NB>(head + w * dpad + NB * lane, sum);
            else
              finish(i, sum, false);
          } while (todo != 0);
        }
        cur = nxt;
        nxt = nn;
      }
      if (rows != 0) open_row = __builtin_ctzll(rows);  // goes on past the chunk
      // On to the next window while rows there start in this chunk (rows
      // without entries at the very end included).
      const int last_end = __builtin_amdgcn_readlane(en, 63);
      if (base + 64 >= n || last_end > ce || (last_end == ce && !(at_end && ce == len))) break;
      close_window();
      base += 64;
      start_l = rowptr[base + lane < n ? base + lane : n];
      end_l = rowptr[base + lane < n ? base + lane + 1 : n];
      open_window();
    }
    int tail = -1;  // the row that goes on from this chunk
    if (open_row >= 0) {
      const bool before = __builtin_amdgcn_readlane(st, open_row) < cs;
      float4_t sum = zero4;
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        sum[c] = 2.f * both_chains(acc[2 * c], acc[2 * c + 1]);
        if constexpr (P != 0) sum[c] += gsum;
      }
      store_partial<NB>((before ? head : tails) + w * dpad + NB * lane, sum);
      if (!before) tail = (int)(base + open_row);
    }
    store_first(tail_row + w, lane, tail);
  }
  close_window();
}

// ------------------------------------------ binary GEMM, e2m1 operands ----
//
// k_bgemm_pop_q8's results (8-bit half-codes, exact rows and flags) for 65-256
// output columns, on the matrix cores: 32-row tiles, the signs as e2m1 +-1
// against +-1/2 weights (zero past K) that the block keeps in LDS, so a
// 32 x 32 x 64 product takes 32 cycles and the kernel is bound by the codes it
// writes (2.45 M x 256 x 256: 479 us with bit counts, 226 us here for 627 MB
// written; 233 K x 256 x 602: 110 -> 42 us; 169 K x 256 x 256: 42 -> 19 us; with
// few rows the weights' expansion bounds it, see bgemm_q8_on_matrix_cores).  Lane l holds column l & 31 of every 32-column tile, whose bytes
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

template <int KS, int NT, int NX, int NBN, bool ID = false>
hipError_t sign_launch(int64_t n, int64_t nnz, const int64_t* rowptr, const int32_t* colidx,
                       const float* g, const uint64_t* F, const uint64_t* wbits, int64_t ldw,
                       int32_t K, const FinishArgs& fa, const SpmmPlan& p, void* ws,
                       const FusedNext& fn, hipStream_t stream) {
  constexpr int NB = NT / 2;
  char* base = (char*)ws;
  int32_t* tail_row = (int32_t*)(base + p.off_tailrow);
  float* head = (float*)(base + p.off_head);
  float* tail = (float*)(base + p.off_tail);
  const size_t lds =
      NX == 3 ? (size_t)((fn.kin + 63) >> 6) * NB * 64 * sizeof(uint64_t) : 0;
  const uint64_t* wB = NX == 3 ? fn.wself : fn.wbits;
  const int64_t ldB = NX == 3 ? fn.ldw_self : fn.ldw;
  // About 16 K waves (each starts by looking up its first row and staging
  // weights: 4 K measured 20 % slower on the largest graphs for their uneven
  // ends, 32 K and 64 K within 2 % either way).
  const int32_t run = (int32_t)((p.workers + 16383) / 16384);
  const int64_t waves = (p.workers + run - 1) / run;
  const dim3 grid((unsigned)((waves + kWavesPerBlock - 1) / kWavesPerBlock));
#define BIGCN_SIGN(PV)                                                                       \
  hipLaunchKernelGGL((k_spmm_sign<KS, NT, NX, NBN, PV, ID>), grid, dim3(kBlock), lds, stream, fa, \
                     n, nnz, rowptr, colidx, g, F, wbits, ldw, K, (int32_t)p.chunk, run, p.workers, p.dpad, \
                     tail_row, head, tail, wB, ldB)
  if constexpr (ID) {
    BIGCN_SIGN(0);
  } else {
    if (K & 1)
      BIGCN_SIGN(1);
    else
      BIGCN_SIGN(0);
  }
#undef BIGCN_SIGN
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t fix_waves = (p.workers + 3) / 4;
  hipLaunchKernelGGL((k_spmm_fix_q8<NX, NB, NBN>),
                     dim3((unsigned)((fix_waves + kWavesPerBlock - 1) / kWavesPerBlock)),
                     dim3(kBlock), lds, stream, fa, rowptr, p.chunk, p.workers, p.dpad,
                     tail_row, head, tail, wB, ldB);
  return hipGetLastError();
}

template <int KS, int NT>
hipError_t sign_kind(int64_t n, int64_t nnz, const int64_t* rowptr, const int32_t* colidx,
                     const float* g, const uint64_t* F, const uint64_t* wbits, int64_t ldw,
                     int32_t K, const FinishArgs& fa, const SpmmPlan& p, void* ws,
                     const FusedNext& fn, hipStream_t stream) {
#define BIGCN_KIND(NX, NBN)                                                                 \
  return sign_launch<KS, NT, NX, NBN>(n, nnz, rowptr, colidx, g, F, wbits, ldw, K, fa, p, \
                                      ws, fn, stream)
  switch (fn.kind) {
    case 0: BIGCN_KIND(0, 1);
    case 1: BIGCN_KIND(1, 1);
    case 3: BIGCN_KIND(3, 16 / (NT / 2));  // NBN: the self weights' words per lane
    case 4: BIGCN_KIND(4, 1);
  }
#undef BIGCN_KIND
  return hipErrorInvalidValue;
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

// Where gathering signs is faster than gathering codes (whole passes, codes
// against signs, with the GEMM that only codes need; nodes, entries):
//   up to 128 inputs, up to 128 outputs: from 2 M entries (100 -> 128: 169 K, 2.5 M 113 ->
//     102 us; 60 K, 2.3 M 82 -> 70; 700 K, 2.1 M, three a row, 273 -> 262).  Below that a
//     launch's few tiles per wave do not pay for its start (30 K, 0.8 M: 65 -> 75).
//   129-256 outputs: from 4 M where 256 fp32 columns are written (169 K, 2.5 M 150 -> 157;
//     1.2 M, 5.2 M 711 -> 699; 233 K, 115 M 2330 -> 1990); from 2 M where they leave signs
//     (128 -> 256 -> 256 -> 40: 169 K, 2.5 M 416 -> 405; 60 K, 2.5 M 298 -> 292; but 65 -> 192
//     -> 65: 700 K, 2.9 M, four a row, 569 -> 581, 2.4 M, 12 M 2003 -> 1866).  Where they leave
//     a narrow layer's products, which a tile's long epilogue forms row by row, rows
//     have to be longer (100 -> 256 -> 47: 700 K, 2.1 M, three a row, 556 -> 622;
//     1.2 M, 5.2 M 981 -> 1075; 2.4 M, 12 M 2047 -> 2125; 300 K, 3.5 M (12) 371 -> 388, 300 K,
//     5.3 M (18) 445 -> 440, 1.2 M, 15 M (13) 1413 -> 1383, 60 K, 2.5 M (41) 201 -> 201,
//     20 K, 2.4 M (120) 130 -> 120)
//   a two-weight layer's epilogue is longer yet (169 K nodes: pass 665 -> 702; 2.4 M, 9.6 M
//     (four a row) 100 -> 128 1528 -> 1618; 2.4 M, 28 M (12) 1813 -> 1751; 250 K, 8.6 M
//     339 -> 303; 2.4 M, 120 M 3111 -> 2567)
//   129-256 inputs double the matrix work: up to 128 outputs on large graphs (200 -> 128:
//     250 K, 8.9 M 271 -> 263; 2.4 M, 30 M 1500 -> 1380; 256 -> 70: 2.4 M, 12 M (five a row)
//     1177 -> 1200; but 169 K, 2.5 M 142 -> 155); two-weight layers are at best level
//     (1.2 M, 14 M 1097 -> 1179; 2.4 M, 120 M 3446 -> 3445); with 256 outputs codes stay
//     ahead where they fit the last-level cache (233 K nodes: 2.4 against 2.9 ms) and
//     are level elsewhere.
bool sign_supported(int64_t n, int64_t nnz, int32_t d, int32_t K, bool two_weight, int leaves) {
  constexpr int64_t M = 1 << 20;
  if (d <= 64 || K > 256 || !q8_supported(n, d, K)) return false;
  if (K > 128) return !two_weight && d <= 128 && nnz >= 8 * M && nnz >= 8 * n;
  if (two_weight) return nnz >= 8 * M && nnz >= 8 * n;
  if (d <= 128) return nnz >= 2 * M;
  if (leaves == 4) return nnz >= (nnz >= 8 * n ? 2 : 8) * M;
  if (leaves == 1) return (nnz >= 2 * M && nnz >= 32 * n) || (nnz >= 4 * M && nnz >= 12 * n);
  return nnz >= 4 * M;
}

hipError_t launch_spmm_sign(int64_t n, int64_t nnz, const int64_t* rowptr,
                            const int32_t* colidx, int mean, const float* g,
                            const uint64_t* F, const uint64_t* wbits, int64_t ldw, int32_t K,
                            int32_t d, const float* alpha, const float* bias, int relu,
                            float* out, int64_t ldo, const SpmmPlan& p, void* ws,
                            const FusedNext* next, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  FusedNext none = {};
  const FusedNext& fn = next != nullptr ? *next : none;
  // a fused next layer of products (kind 1) has at most 64 columns here
  if (!sign_supported(n, nnz, d, K, fn.kind == 3, fn.kind == 3 ? 0 : fn.kind) ||
      (fn.kind == 1 && q8_lane_bytes(fn.d_out) != 1) ||
      (fn.kind == 4 && fn.ldFn != q8_lane_bytes(d)) ||
      (fn.kind == 3 && !self_in_epilogue_supported(nnz, d, fn.kin)))
    return hipErrorInvalidValue;
  const FinishArgs fa = finish_args(mean, g, d, alpha, bias, relu, out, ldo, fn);
#define BIGCN_KSNT(KS, NT)                                                               \
  return sign_kind<KS, NT>(n, nnz, rowptr, colidx, g, F, wbits, ldw, K, fa, p, ws, fn, \
                           stream)
  if (K > 128) BIGCN_KSNT(4, 4);
  if (d <= 128) BIGCN_KSNT(2, 4);
  BIGCN_KSNT(2, 8);
#undef BIGCN_KSNT
}

hipError_t launch_spmm_scaled_signs(int64_t n, int64_t nnz, const int64_t* rowptr,
                                    const int32_t* colidx, int mean, const float* g,
                                    const uint64_t* F, int64_t ldf, int32_t K,
                                    const float* ones, float* out, int64_t ldo,
                                    const SpmmPlan& p, void* ws, hipStream_t stream) {
  // (the kernel's buffers address the signs and scales by 31-bit offsets)
  if (n < 1 || nnz < 1 || K < 1 || K > 256 || ldf < sign_row_words(K) ||
      n * ldf * 8 >= (1ll << 31) || p.dpad < 64 * q8_lane_bytes(K))
    return hipErrorInvalidValue;
  const FusedNext none = {};
  const FinishArgs fa = finish_args(mean, g, K, ones, nullptr, 0, out, ldo, none);
#define BIGCN_ID(KS, NT)                                                                    \
  return sign_launch<KS, NT, 0, 1, true>(n, nnz, rowptr, colidx, g, F, nullptr, ldf, K, fa, p, \
                                         ws, none, stream)
  if (K <= 64) BIGCN_ID(2, 2);
  if (K <= 128) BIGCN_ID(2, 4);
  BIGCN_ID(4, 8);
#undef BIGCN_ID
}

}  // namespace bigcn
