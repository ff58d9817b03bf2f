// Per-tile pieces of the gfx950 decode-attention kernels (Sec. 2, Eq. gqa_attention): loading a
// 16-row K/V tile of one KV head, and folding it into one wave's online softmax for the G query
// heads of that KV head.  Both contractions run on the matrix cores, and the probabilities go
// from one to the other without leaving their lane:
//
//   * K rows come in whole (1 KB of consecutive rows per wave-wide load) and pass through a
//     wave-private LDS slice into the matrix-core layout, 16 bytes of another row per lane.
//     Loading that layout straight from memory touches 64 cache lines per load where 8 would do,
//     which held a CU at 35 GB/s (one 32K sequence, G = 7, 64 workgroups: 36 us against 27 us).
//   * QK^T: v_mfma_f32_16x16x32_bf16 with A = the 16 K rows (M = rows, K = head dim) and B = the
//     query vectors (N = 16 columns).  Lane (quad, n) of the score tile holds rows 4*quad ..
//     4*quad+3 of column n.  Column n carries query head n % S, S = 4 (G <= 4) or 8: every head
//     stands in 16 / S columns, so 16 / S lanes hold the same scores.
//   * online softmax in the log2 domain (exp2, scale folded with log2 e).  The cross-lane maximum
//     and the rescaling of the outputs sit in a wave-uniform branch, taken when a score of the
//     tile exceeds the running maximum: for most tiles at a walk's beginning, few later on.  (No
//     probability exceeds 1 then, so sums of large values stay in range.  Letting scores exceed
//     the maximum by 2^8 before raising it saves 1.5 % of a full layer of one 32K sequence and 3 %
//     of a sparse layer of 2-4 tiles per wave (11.1 us), and nothing from 0.1 GB on.)  Each lane
//     sums the probabilities of its own rows.  A weight below 2^-126 of the largest counts as zero
//     (v_exp_f32).
//   * P.V: v_mfma_f32_16x16x16_bf16 with A = P (M = columns n of the score tile, K = the 16 rows)
//     and B = V (N = 16 head-dim columns).  The A operand's lane (quad, m) holds rows 4*quad ..
//     4*quad+3 of m, which is the score tile's own layout.  An fp32 probability is the exact sum
//     of three bf16 terms (its upper 8 significant bits, the next 8, the last 8), and the copies
//     of a head's column carry one term each: with S = 4 three of the four copies make one MFMA,
//     with S = 8 two terms make one and the third a second one, the first copies carrying half of
//     the first term in each: a lower term is often zero, zero times an infinite V is NaN, and so
//     the rows of the first term, which is zero only where the probability is, say alone what an
//     infinite V gives (sum_keep_inf).  V is bf16 as it is, the products
//     are exact and the sums fp32, so no probability is rounded.  Lane (quad, n) loads 8 (d = 128)
//     or 4 (d = 64) consecutive columns of rows 4*quad .. 4*quad+3, and MFMA c takes column
//     (D/16)*n + c from lane n: the operand is two byte permutes of the lane's own registers.
//
// Bound: HBM, as soon as the per-tile chain of a wave is shorter than its share of the memory
// rate.  With P.V on the vector ALUs (32*G fma per tile, P through LDS, a cross-lane maximum and
// sum per tile) and uncoalesced K loads the chain took 1.1 us per 8 KB tile, i.e. 29 GB/s per CU
// with one wave per SIMD however many loads were in flight, while a CU alone reads 57 GB/s: grids
// below 256 workgroups and the few tiles per wave of small launches were bound by it.  Measured
// on MI355X, before and after the tile alone, the work cut the same (us per layer): one 32K
// sequence, 28/4 heads, 64 workgroups 43.5 and 26.6; 64 sequences of 600-1500 tokens, 12/2 heads
// 26.5 and 20.0; 20 sequences of 12289 tokens, 40/8 heads 219 and 183; 32 ragged sequences of
// 16K-32K, 32/8 heads (3.2 GB, at the memory rate either way) 494 and 493.
//
// The split of an fp32 operand into bf16 terms is that of Henry, Tang and Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations" (2019), the online
// softmax that of Milakov and Gimelshein, "Online normalizer calculation for softmax" (2018).
#pragma once

#include "internal.h"
#include "wave.h"

namespace delta {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

constexpr float kNegInfF = -__builtin_huge_valf();

template <int D>
struct Geo {
  static constexpr int NK = D / 32;     // MFMA k-steps = 16-byte K loads per lane per tile
  static constexpr int CPR = D / 8;     // 16-byte pieces of a K row
  static constexpr int RPL = 64 / CPR;  // K rows per wave-wide load
  static constexpr int NC = D / 16;     // V columns per lane = P.V MFMAs per tile and term group
  static constexpr int NW = D / 32;     // 32-bit words of a lane's V columns of one row
  // register tiles per wave: loads of R - 1 tiles stay in flight while one is consumed
  static constexpr int R = D == 128 ? 3 : 4;
};

template <int W>
struct VWords;
template <>
struct VWords<4> { typedef u32x4 type; };
template <>
struct VWords<2> { typedef u32x2 type; };

template <int D>
struct Tile {
  u32x4 k[Geo<D>::NK];   // load i: row k_row<D>(i, lane), piece lane % CPR
  typename VWords<Geo<D>::NW>::type v[4];   // rows 4*quad .. 4*quad+3
  uint32_t kmask;   // bit r: row r valid (wave-uniform)
};

// Columns of the score tile per copy of the query heads (column n carries head n % kCopy<G>).
template <int G>
constexpr int kCopy = G <= 4 ? 4 : 8;

// One wave's running softmax state for the G query heads of one KV head: the maximum of head
// n % S in use (the same in every lane of that head), the sum over the lane's own rows, and the
// unnormalised outputs as P.V leaves them: o[c][r] = row 4*quad + r (a term of head
// (4*quad + r) % S) of head-dim column NC*n + c.
template <int D, int G>
struct WaveSoftmax {
  float m_run, l_run;
  f32x4 o[Geo<D>::NC];
  __device__ __forceinline__ void init() {
    m_run = kNegInfF;
    l_run = 0.f;
#pragma unroll
    for (int c = 0; c < Geo<D>::NC; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
};

__device__ __forceinline__ u32x4 load16(const uint16_t* p) {
  return *reinterpret_cast<const u32x4*>(p);
}
// K/V rows are read once per launch: non-temporal loads.  Measured on MI355X they raise the
// streaming rate of the full and sparse layers by 5-20 % over ordinary loads.
__device__ __forceinline__ u32x4 load16_stream(const uint16_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}

__device__ __forceinline__ u32x2 load8_stream(const uint16_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
}
// A lane's V columns of one row: D/16 bf16.
template <int D>
__device__ __forceinline__ auto load_v_stream(const uint16_t* p) {
  if constexpr (D == 128) return load16_stream(p);
  else return load8_stream(p);
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// Compiler-level ordering for LDS traffic that stays inside one wave (the LDS unit executes
// one wave's requests in order; this only stops the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The query operand of the MFMA: the G query vectors of KV head g (row `qrow` = b*Hq + g*G of
// q), lane (quad, hcol) holding 8 head-dim values of head hcol % S; columns of no head are zero.
template <int D, int G>
__device__ __forceinline__ void load_query(bf16x8 (&qb)[Geo<D>::NK], const uint16_t* q,
                                           size_t qrow, int lane) {
  const int quad = lane >> 4, head = (lane & 15) % kCopy<G>;
  const uint16_t* qp = q + (qrow + min(head, G - 1)) * D + 8 * quad;
#pragma unroll
  for (int ks = 0; ks < Geo<D>::NK; ++ks) {
    u32x4 w = load16(qp + 32 * ks);
    if (head >= G) w = u32x4{0u, 0u, 0u, 0u};
    qb[ks] = __builtin_bit_cast(bf16x8, w);
  }
}

template <int D>
__device__ __forceinline__ int k_row(int i, int lane) { return Geo<D>::RPL * i + lane / Geo<D>::CPR; }

// Buffer-resource word 3 for raw (unformatted, stride 0) buffer access on gfx950, and the
// cache-policy operand of the buffer builtins for non-temporal loads.
constexpr int kRawBufferFlags = 0x00020000;
constexpr int kNonTemporal = 2;

// Loads the [16, D] K and V tile that starts at kt / vt (one page of one KV head; both
// wave-uniform).  With real == false the loads are still issued, so that a loop's memory waits
// stay uniform, but from an empty buffer: they return zeros and read nothing.  (Buffer loads: the
// address is a scalar descriptor and a lane offset that no tile changes.  With global loads the
// compiler sometimes formed 64-bit lane addresses in registers of tiles still in flight, whose
// loads it then waited for.)
template <int D>
__device__ __forceinline__ void load_page_tile(Tile<D>& t, const uint16_t* kt, const uint16_t* vt,
                                               bool real, int lane) {
  using Gm = Geo<D>;
  const int quad = lane >> 4, hcol = lane & 15;
  const int bytes = real ? 16 * D * 2 : 0;
  const __amdgpu_buffer_rsrc_t rk =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(kt), 0, bytes, kRawBufferFlags);
  const __amdgpu_buffer_rsrc_t rv =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(vt), 0, bytes, kRawBufferFlags);
  const int ko = 16 * lane, vo = 2 * (quad * 4 * D + Gm::NC * hcol);
#pragma unroll
  for (int i = 0; i < Gm::NK; ++i)
    t.k[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, ko + 1024 * i, 0, kNonTemporal));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (D == 128)
      t.v[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, vo + 2 * D * i, 0, kNonTemporal));
    else
      t.v[i] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rv, vo + 2 * D * i, 0, kNonTemporal));
  }
}

// 16-byte piece c of row r of a K tile in the wave's LDS slice (16 * D bf16): the pieces of a row
// are permuted by the row, so that 16 lanes reading the same piece of 16 rows touch all 64 banks
// (d = 128: 256-byte rows; d = 64: two rows per 256 bytes).
template <int D>
__device__ __forceinline__ int k_slot(int r, int c) {
  return r * D + 8 * (c ^ (D == 128 ? r : (r >> 1) & 7));
}

// The A operand of QK^T: lane (quad, m) gets pieces 4*ks + quad of row m.
template <int D>
__device__ __forceinline__ void k_operand(const Tile<D>& t, uint16_t* lk, u32x4 (&ka)[Geo<D>::NK],
                                          int lane) {
  using Gm = Geo<D>;
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < Gm::NK; ++i)
    *reinterpret_cast<u32x4*>(lk + k_slot<D>(k_row<D>(i, lane), lane % Gm::CPR)) = t.k[i];
  wave_lds_sync();
#pragma unroll
  for (int ks = 0; ks < Gm::NK; ++ks)
    ka[ks] = *reinterpret_cast<const u32x4*>(lk + k_slot<D>(lane & 15, 4 * ks + (lane >> 4)));
}

// Folds one tile's score tile (acc: lane (quad, hcol) holds q_(hcol % S) . k_r for rows
// r = 4*quad .. 4*quad+3, unscaled) into the wave's softmax state.  With LOGITS, the tile's
// scaled log2-domain logits go to logit_slot[head][16] (LDS).
template <int D, int G, bool LOGITS>
__device__ __forceinline__ void fold_tile(f32x4 acc, Tile<D>& t, float scale_log2,
                                          WaveSoftmax<D, G>& st, float* logit_slot, int lane) {
// Every scaled score is rounded before anything else sees it, the maximum and the stored logit
// too: with the scaling contracted into the difference's fma, the maximum's own rounding error
// would be left in the exponent, which for scores of 2^32 and more is a weight of 0 or infinity.
#pragma clang fp contract(off)
  using Gm = Geo<D>;
  constexpr int S = kCopy<G>;
  const int quad = lane >> 4, hcol = lane & 15;
  const uint32_t kmask = __builtin_amdgcn_readfirstlane(t.kmask);
  acc *= scale_log2;
  if (kmask != 0xffffu) {   // rows past the end (their K and V may hold NaN)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = (kmask >> (4 * quad + r)) & 1u;
      acc[r] = ok ? acc[r] : kNegInfF;
#pragma unroll
      for (int w = 0; w < Gm::NW; ++w) t.v[r][w] = ok ? t.v[r][w] : 0u;
    }
  }
  if (LOGITS && hcol < G)
    *reinterpret_cast<f32x4*>(logit_slot + hcol * 16 + 4 * quad) = acc;

  float m_use = st.m_run;
  const float mx = fmaxf(fmaxf(acc[0], acc[1]), fmaxf(acc[2], acc[3]));
  // a difference, negated, so that a maximum of -inf (nothing folded in yet: inf, or NaN where the
  // tile's scores are -inf too) and NaN scores take the branch
  if (__any(!(mx - m_use <= 0.f))) {
    const float m_new = fmaxf(st.m_run, max_xor32(max_xor16(mx)));
    m_use = (m_new == kNegInfF) ? 0.f : m_new;
    const float alpha = exp2f(st.m_run - m_use);
    st.m_run = m_new;
    st.l_run *= alpha;
    // the factor of output row 4*quad + r, from a lane of its head
    float row[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float lo = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(alpha), r));
      const float hi = S == 8 ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(alpha), 4 + r)) : lo;
      row[r] = (quad & 1) ? hi : lo;
    }
#pragma unroll
    for (int c = 0; c < Gm::NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) st.o[c][r] *= row[r];
  }
  float p[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(acc[r] - m_use);
  st.l_run += (p[0] + p[1]) + (p[2] + p[3]);

  // The term of the probabilities that this lane's copy of the head carries: p less the upper
  // parts that the lower copies carry.  (With S = 4 the fourth copy carries a third term again;
  // its output rows are dropped in the end.)
  constexpr uint32_t kHigh = 0xffff0000u;
  const uint32_t m1 = hcol >= S ? kHigh : 0u, m2 = hcol >= 2 * S ? kHigh : 0u;
  auto high = [](float x, uint32_t m) { return __uint_as_float(__float_as_uint(x) & m); };
  auto pack = [](float lo, float hi) {   // the upper halves of two floats
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
  };
  const float part = S == 8 && hcol < S ? 0.5f : 1.f;   // (exact, the fma too)
  float a1[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    a1[r] = fmaf(p[r], part, -high(p[r], m1));
    if (S == 4) a1[r] -= high(a1[r], m2);
  }
  const u32x2 pa = {pack(a1[0], a1[1]), pack(a1[2], a1[3])};
  u32x2 pb = {0u, 0u};
  if (S == 8) {   // the third term, from the second copies; the other half of the first copies' term
    float a2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) a2[r] = a1[r] - high(a1[r], kHigh);
    pb = u32x2{pack(a2[0], a2[1]), pack(a2[2], a2[3])};
    pb[0] = hcol >= S ? pb[0] : pa[0];
    pb[1] = hcol >= S ? pb[1] : pa[1];
  }
#pragma unroll
  for (int c = 0; c < Gm::NC; ++c) {
    const uint32_t pick = (c & 1) ? 0x07060302u : 0x05040100u;
    const int w = c / 2;
    const u32x2 vb = {__builtin_amdgcn_perm(t.v[1][w], t.v[0][w], pick),
                      __builtin_amdgcn_perm(t.v[3][w], t.v[2][w], pick)};
    st.o[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(i16x4, pa),
                                                        __builtin_bit_cast(i16x4, vb), st.o[c], 0, 0, 0);
    if (S == 8)
      st.o[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(i16x4, pb),
                                                          __builtin_bit_cast(i16x4, vb), st.o[c], 0, 0, 0);
  }
}

// Folds one tile into the wave's softmax state, QK^T on the matrix cores (see the file header).
template <int D, int G, bool LOGITS>
__device__ __forceinline__ void process_tile(Tile<D>& t, const bf16x8 (&qb)[Geo<D>::NK],
                                             float scale_log2, WaveSoftmax<D, G>& st,
                                             uint16_t* lk, float* logit_slot, int lane) {
  u32x4 ka[Geo<D>::NK];
  k_operand<D>(t, lk, ka, lane);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < Geo<D>::NK; ++ks)
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[ks]), qb[ks],
                                                  acc, 0, 0, 0);
  fold_tile<D, G, LOGITS>(acc, t, scale_log2, st, logit_slot, lane);
}

// The same score tile with QK^T on the vector ALUs, a build option (DELTA_QK_VALU) kept for
// comparing the two engines.  Lane (quad, r) holds 32 head-dim values of K row r (the registers
// of the matrix-core operand) and forms their dot products with the same 32 values of every
// query head (sq: the wave's LDS copy of the G query vectors, bf16 [G][D]) with
// v_dot2_f32_bf16; the four quads' partial sums are added across lanes, and the tile goes
// through the wave's LDS slice into the matrix-core layout that fold_tile reads.
template <int D, int G>
__device__ __forceinline__ void stage_query_lds(const bf16x8 (&qb)[Geo<D>::NK], uint16_t* sq,
                                                int lane) {
  const int quad = lane >> 4, hcol = lane & 15;
  if (hcol < G) {
#pragma unroll
    for (int ks = 0; ks < Geo<D>::NK; ++ks)
      *reinterpret_cast<bf16x8*>(sq + hcol * D + 32 * ks + 8 * quad) = qb[ks];
  }
}

template <int D, int G, bool LOGITS>
__device__ __forceinline__ void process_tile_valu(Tile<D>& t, const uint16_t* sq,
                                                  float scale_log2, WaveSoftmax<D, G>& st, float* lp,
                                                  uint16_t* lk, float* logit_slot, int lane) {
  const int quad = lane >> 4, r = lane & 15;
  u32x4 ka[Geo<D>::NK];
  k_operand<D>(t, lk, ka, lane);
  float part[G];
#pragma unroll
  for (int h = 0; h < G; ++h) part[h] = 0.f;
#pragma unroll
  for (int ks = 0; ks < Geo<D>::NK; ++ks) {
    const u32x4 kw = ka[ks];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const u32x4 qw = *reinterpret_cast<const u32x4*>(sq + h * D + 32 * ks + 8 * quad);
      // v_dot2_f32_bf16 written out: with hipcc of ROCm 7.2 at -O3 the builtin
      // (__builtin_amdgcn_fdot2_f32_bf16) compiled to the same operand pair repeated for the
      // four pairs of a 16-byte chunk (wrong sums; found with a one-tile check against the
      // matrix-core tile), the instruction itself gives the right ones
#pragma unroll
      for (int c = 0; c < 4; ++c)
        asm volatile("v_dot2_f32_bf16 %0, %1, %2, %0" : "+v"(part[h]) : "v"(kw[c]), "v"(qw[c]));
    }
  }
#pragma unroll
  for (int h = 0; h < G; ++h) part[h] = sum_xor32(sum_xor16(part[h]));
  wave_lds_sync();
  if (quad == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) lp[r * 8 + h] = part[h];
  }
  wave_lds_sync();
  f32x4 acc;
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = r % kCopy<G> < G ? lp[(4 * quad + i) * 8 + r % kCopy<G>] : 0.f;
  fold_tile<D, G, LOGITS>(acc, t, scale_log2, st, logit_slot, lane);
}

template <int W>
struct FloatVec { typedef float type __attribute__((ext_vector_type(W))); };
template <>
struct FloatVec<1> { typedef float type; };

// upper + lower of the rows of a first and of lower terms (float2: upper, lower).  Where the upper
// sum is infinite it is the result: the lower one may be NaN then (see the file header).
__device__ __forceinline__ float sum_keep_inf(float2 v) {
  return __builtin_isinf(v.x) ? v.x : v.x + v.y;
}

// The wave's complete sums and outputs: afterwards every lane holds the sum of head hcol % S in
// l_run, and emit(head, column, w consecutive outputs) has been called for every output of the G
// heads, each by one lane.  The rows that belong to one head (its terms) stand in different
// 16-lane rows of the wave; a swap of two registers' halves brings two sums' addends together
// at once, so adding and spreading them over the lanes takes NC*4 swaps and adds in all.
template <int D, int G, class F>
__device__ __forceinline__ void reduce_outputs(WaveSoftmax<D, G>& st, int lane, F&& emit) {
  constexpr int NC = Geo<D>::NC, S = kCopy<G>;
  const int quad = lane >> 4, hcol = lane & 15;
  st.l_run = sum_xor32(sum_xor16(st.l_run));
  float h[NC / 2][4];   // lanes 0-31: columns c < NC/2, lanes 32-63: columns c + NC/2
#pragma unroll
  for (int c = 0; c < NC / 2; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = st.o[c][r], y = st.o[c + NC / 2][r];
      if (S == 4) {   // the fourth copy repeats the third term
        x = lane < 48 ? x : 0.f;
        y = lane < 48 ? y : 0.f;
      }
      h[c][r] = sum_keep_inf(swap32(x, y));
    }
  constexpr int W = S == 4 ? NC / 4 : NC / 2;
  const int col = NC * hcol + (quad >> 1) * (NC / 2) + (S == 4 ? (quad & 1) * (NC / 4) : 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int head = S == 4 ? r : 4 * (quad & 1) + r;
    typename FloatVec<W>::type v;
    float e[W];
#pragma unroll
    for (int j = 0; j < W; ++j) e[j] = S == 4 ? sum_keep_inf(swap16(h[j][r], h[j + NC / 4][r])) : h[j][r];
    __builtin_memcpy(&v, e, sizeof(v));
    if (head < G) emit(head, col, v);
  }
}

}  // namespace delta
