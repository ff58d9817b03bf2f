// Split-K paged decode attention for gfx950, in three row modes (full / Delta / sparse).
//
// What it computes (Sec. 2, Eq. gqa_attention; App. A, Alg. 1): for sequence b and query
// head j, out = sum_t softmax_t(scale * q_j . k_t) v_t over the rows of the sequence that the
// mode selects, with k_t, v_t read from KV head j / G.  With logits on (Delta layers) the
// scaled logits of every token (group-major: [b][kv group][page][head in group][row]) and the
// per-head log-sum-exp are also written, for the page scoring of Sec. 4 ("Selection
// mechanism", "Page-based DELTA").
//
// Work decomposition.  A group is one 16-token page tile [16, D] of K and of V (4 KB each at
// D = 128, contiguous in HBM), or 16 gathered token rows in token-level sparse mode.  The grid
// is (split, kv head g, sequence b), 4 waves per workgroup.  Statically, workgroup (split, g,
// b) takes the run of `gps` groups starting at split * gps of pair (b, g).  The balanced
// decomposition instead cuts the batch's actual groups, in (b, g, page) order, into equal runs,
// one for each CU, each run possibly spanning pairs: for ragged batches, lengths far below the
// host's bound, and pair counts that would leave CUs with one static piece more than others
// (20 sequences of 12289 tokens with 8 KV heads are 320 static workgroups on 256 CUs: 183 us
// against 159).  Full and Delta launches only: sparse ones are cut by the shape.  Waves take a
// piece's groups in turn and keep their own online-softmax state; all G query heads of the KV
// group share every K/V byte read.
//
// Per group and wave:
//   * QK^T on the matrix cores: v_mfma_f32_16x16x32_bf16 with A = the 16 K rows (M = rows,
//     K = head dim) and B = the G query vectors, each in two or four of the 16 columns; D/32
//     MFMAs give the 16 x 16 score tile, lane l holding rows 4*(l/16)..+3 of column l%16.
//   * online softmax in the log2 domain (exp2, scale folded with log2 e), the wave's maximum
//     formed only for tiles that raise it;
//   * P.V on the matrix cores too, the probabilities split exactly into three bf16 terms that
//     never leave their lane (attn_tile.h has the layouts and the reasons).
//   Each wave keeps a ring of R register tiles: while one group is consumed, the K/V loads of
//   the next R - 1 groups are in flight.  With logits on, the logits of a chunk of groups are
//   staged in LDS and written by the whole workgroup between chunks.
//
// Combine.  The 4 waves merge through LDS into one (max, sum, o) partial per piece, written to
// the workspace with device-coherent stores.  The last workgroup of each (b, g) to arrive
// (device-scope atomic counter) folds the pair's partials in a fixed order, so results do not
// depend on arrival order, writes bf16 outputs (and the log-sum-exp), and re-arms the counter to
// zero for the next launch.  A pair that is one piece skips all of this and has its outputs
// written directly.  Small launches are bound by this chain: per-workgroup timestamps of a sparse
// layer of 8 sequences, 128 pages, 28/4 heads (256 workgroups, 33.7 MB, 11.3 us; before, 12.0) show
// the page list in LDS at 1.5 us, the stream's end at 7.1, the waves merged 0.7 us later (1.2
// with every lane adding every term), the partial acknowledged and counted after 0.4 us each,
// and the last arriver's fold taking 1.7 us.
//
// Eight waves per workgroup instead of four: a three-layer step at 1K tokens 30.9 against 23.2 us,
// sparse layers 14.5 against 11; the large layers within 2 %.  A shared pool of tail runs taken
// by ticket: 3-20 % slower on every layer of 0.3 GB and more.
#include <type_traits>

#include "attn_tile.h"
#include "debug_check.h"
#include "internal.h"
#include "wave.h"

namespace delta {
namespace {

constexpr float kNegInf = kNegInfF;
constexpr int kCoherent = 16;   // cache-policy operand of the buffer builtins: device-coherent (sc1)
constexpr int kPastEnd = 0x7ffffff0;   // a byte offset past every buffer
// LDS floats for staging Delta-layer logits (128 KB: one Delta workgroup per CU; measured on
// MI355X, fewer and larger chunk flushes beat two resident workgroups with half the staging).
constexpr int kStageFloats = 32768;

// Page list entries of the selected-page mode: the page, and whether only the sequence's tail
// rows (kPartialPage) or none of its rows (kEmptyPage, the sign bit) exist.
constexpr int kPageMask = 0x3fffffff;
constexpr int kPartialPage = 0x40000000;
constexpr int kEmptyPage = (int)0x80000000;

template <int D, int G, int MODE, bool LOGITS, bool BAL>
__global__ __launch_bounds__(kAttnThreads, LOGITS ? 1 : 2) void attn_kernel(const AttnArgs a) {
  static_assert(!BAL || MODE == ROWS_DENSE, "the balanced decomposition is for dense launches");
  using Gm = Geo<D>;
  constexpr int R = Gm::R;
  constexpr int T = kAttnThreads, NW = T / 64;
  constexpr int kSeg = kMaxRowSlots / (MODE == ROWS_SEL_TOKEN ? 16 : 1);   // groups listed at once
  static_assert(kSeg % (4 * NW) == 0, "a wave's share of a piece does not depend on the listing");
  // (not const: the piece loop below makes them opaque once per piece)
  int tid = threadIdx.x;
  int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform (scalar)
  int quad = lane >> 4;   // score-tile rows 4*quad .. 4*quad+3
  int hcol = lane & 15;   // score-tile column: query head hcol % kCopy<G> of the group
  const int Hq = a.n_q_heads;

  // ---- staging: the page (or row) list of groups [g0, g0 + cand) of sequence b, to LDS, and
  // the query operand of (b, KV head g).
  // (Debug builds check every physical page and selected unit here and flag bad ones; see
  // checked_page.)
  bf16x8 qb[Gm::NK];
  __shared__ int s_rows[kMaxRowSlots];
  auto stage_list = [&](int b, int g0, int cand) {
    const int32_t* pt = a.page_table + (size_t)b * a.max_pages;
    // selected pages: the length says which of them is the partial last one; debug builds also
    // check the selected units against it
    const int s_len = MODE == ROWS_SEL_PAGE || (DELTA_DEBUG && MODE != ROWS_DENSE) ? a.seq_lens[b] : 0;
    if (MODE == ROWS_DENSE) {
      for (int i = tid; i < cand; i += T)
        s_rows[i] = checked_page(pt[g0 + i], a.n_pages, a.status);
    } else if (MODE == ROWS_SEL_PAGE) {
      // with precomputed physical pages the index and the page arrive together
      const int32_t* sel = a.sel_idx + (size_t)b * a.sel_stride;
      const int32_t* phys = a.sel_phys ? a.sel_phys + (size_t)b * a.sel_stride : nullptr;
      for (int i = tid; i < cand; i += T) {
        const int u = sel[g0 + i];
        const int ph = phys ? phys[g0 + i] : 0;
        const bool ok = u >= 0 && u < a.max_pages;
        if (DELTA_DEBUG && u >= 0 && 16 * u >= s_len) debug_flag(a.status, DELTA_DEBUG_SELECTION);
        const int page = ok ? checked_page(phys ? ph : pt[u], a.n_pages, a.status) : 0;
        // (a page index needs 30 bits at most: a page is at least 2 KB)
        const int rows = s_len - 16 * (ok ? u : 0);
        s_rows[i] = page | (rows >= 16 ? 0 : rows > 0 ? kPartialPage : kEmptyPage);
      }
    } else {
      const int32_t* sel = a.sel_idx + (size_t)b * a.sel_stride;
      const int32_t* phys = a.sel_phys ? a.sel_phys + (size_t)b * a.sel_stride : nullptr;
      const int n_rows = min(16 * cand, a.sel_stride - 16 * g0);
      for (int i = tid; i < 16 * cand; i += T) {
        int packed = -1;
        if (i < n_rows) {
          const int t = sel[16 * g0 + i];
          const int ph = phys ? phys[16 * g0 + i] : 0;
          if (DELTA_DEBUG && t >= s_len) debug_flag(a.status, DELTA_DEBUG_SELECTION);
          if (t >= 0 && t < 16 * a.max_pages) {
            const int page = checked_page(phys ? ph >> 4 : pt[t >> 4], a.n_pages, a.status);
            packed = page * 16 + (phys ? ph & 15 : t & 15);
          }
        }
        s_rows[i] = packed;
      }
    }
  };
  auto stage = [&](int b, int g, int g0, int cand) {
    load_query<D, G>(qb, a.q, (size_t)b * Hq + g * G, lane);
    stage_list(b, g0, min(cand, kSeg));
  };
  // nothing to attend to (an empty sequence, or no selected unit): defined output (zeros),
  // log-sum-exp = -inf
  auto write_empty = [&](int b, int g) {
    for (int i = tid; i < G * D; i += T) a.out[((size_t)b * Hq + g * G) * D + i] = 0;
    if (LOGITS && tid < G) a.lse[(size_t)b * Hq + g * G + tid] = kNegInf;
  };

  // shared state of the attention of one piece
  constexpr int kChunk = (kStageFloats / (G * 16)) / 16 * 16;
  __shared__ __attribute__((aligned(16))) float s_stage[LOGITS ? kChunk * G * 16 : 1];
  __shared__ float s_m[NW][kMaxGroup], s_l[NW][kMaxGroup];
  // each wave's K tile on its way to the matrix cores, later its outputs; then the outputs of
  // the thread groups that merge partials
  union WaveSpace {
    uint16_t k[16 * D];
    float o[G][D];
  };
  __shared__ __attribute__((aligned(16))) WaveSpace s_w[NW];
  __shared__ int s_last;
#if DELTA_QK_VALU
  __shared__ __attribute__((aligned(16))) uint16_t s_qv[NW][G * D];
  __shared__ float s_p[NW][16 * 8];   // wave-private: the score tile
#endif
  constexpr int E = G * D / 4;             // threads that cover a group's outputs, four each
  constexpr int NP = T / E;                // such thread groups in the workgroup
  static_assert(E <= T && D % 4 == 0 && NP <= 4 * NW, "outputs and thread groups fit");

  // ---- attention of groups [g0, g0 + ng) of (sequence b, KV head g), staged by stage(); the
  // piece is partial `slot` of the n_valid partials of its pair (n_valid == 1: the whole pair)
  auto run = [&](int b, int g, int g0, int ng, int slot, int n_valid, int s_b, int sel_n) {
    const int bg = b * a.n_kv_heads + g;
    const size_t head_off = (size_t)g * 16 * D;
    // Loads tile `li` of the listed groups (the first is group l0 of the pair).  `row` is its
    // page list entry (page modes), read from LDS one tile ahead.  A prefetch past the wave's
    // last group (real == false) is still issued, so that the loop's memory waits stay uniform,
    // but reads nothing (a page tile) or one cache line per load instruction (gathered rows).
    const int s_last_page = (s_b - 1) >> 4;
    const uint32_t tail_mask = 0xffffu >> (15 - ((s_b - 1) & 15));   // rows of the last page
    auto load_tile = [&](Tile<D>& t, int row, int li, int l0, bool real) {
      if (MODE == ROWS_SEL_TOKEN) {
        // every row is its own (page, row); rows past the selection re-read the group's first
        const int* rows = s_rows + 16 * li;
        const int first = rows[0];
        t.kmask = (uint32_t)__ballot(rows[hcol] >= 0 && 16 * (l0 + li) + hcol < sel_n) & 0xffffu;
#pragma unroll
        for (int i = 0; i < Gm::NK; ++i) {
          const int r = k_row<D>(i, lane);
          const int kr = ((t.kmask >> r) & 1u) && real ? rows[r] : first;
          t.k[i] = load16_stream(a.k_cache + (size_t)(kr >> 4) * a.page_stride + head_off +
                                 (size_t)(kr & 15) * D + (real ? 8 * (lane % Gm::CPR) : 0));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * quad + i;
          const int vr = ((t.kmask >> r) & 1u) && real ? rows[r] : first;
          t.v[i] = load_v_stream<D>(a.v_cache + (size_t)(vr >> 4) * a.page_stride + head_off +
                                    (size_t)(vr & 15) * D + (real ? Gm::NC * hcol : 0));
        }
      } else {
        row = __builtin_amdgcn_readfirstlane(row);
        const size_t page = (size_t)(row & kPageMask) * a.page_stride + head_off;
        if (MODE == ROWS_DENSE) t.kmask = l0 + li == s_last_page ? tail_mask : 0xffffu;
        else t.kmask = row < 0 ? 0u : (row & kPartialPage) ? tail_mask : 0xffffu;
        load_page_tile<D>(t, a.k_cache + page, a.v_cache + page, real, lane);
      }
    };

    WaveSoftmax<D, G> st;
    st.init();
    const int Hq_row = b * Hq + g * G;
    // Logits on: the workgroup keeps the logits of a chunk of kChunk groups in LDS ([group]
    // [head][16], the global layout) and writes the chunk out cooperatively between chunks.
    // Bound: the writes, which HBM takes at about 2.5 TB/s while it serves the other workgroups'
    // reads (64 sequences of 18432 tokens with 12/2 heads: 57 MB, 23 us of 205; pausing the walk
    // itself costs nothing measurable).  Stores of single tiles cost several times that.  Stores
    // written through (sc1) against non-temporal and ordinary ones, us per Delta layer: 222.5,
    // 228.5, 231; 16 x 32K with 32/8 heads 373, 378, 387; 32 ragged 16K-32K 616, 623, 644.
#if DELTA_QK_VALU
    // build option: QK^T on the vector ALUs, the query vectors read from the wave's LDS copy
    stage_query_lds<D, G>(qb, s_qv[wave], lane);
    wave_lds_sync();
    auto process = [&](Tile<D>& t, int slot_in_chunk) {
      process_tile_valu<D, G, LOGITS>(t, s_qv[wave], a.scale_log2, st, s_p[wave], s_w[wave].k,
                                      s_stage + slot_in_chunk * G * 16, lane);
    };
#else
    auto process = [&](Tile<D>& t, int slot_in_chunk) {
      process_tile<D, G, LOGITS>(t, qb, a.scale_log2, st, s_w[wave].k,
                                 s_stage + slot_in_chunk * G * 16, lane);
    };
#endif

    // The waves take a piece's groups in turn: one at a time in short pieces, so that every wave
    // has its share, and blocks of four in pieces of 128 groups or more, where pages in order
    // stream better that way (64 sequences of 18432 tokens, 12/2 heads, blocks of 1, 2, 4, 8 and
    // 16: Delta layer 225, 220, 218, 222, 223 us, full layer 190, 187, 186, 187, 186; 16 x 32K,
    // 32/8 heads 336, 338, 339, 374, 367; blocks of four cost 64 sequences of 600-1500 tokens
    // 20.6 us instead of 19.7).  A wave walks
    // its groups [kb, ke) of the listed ones with a ring of R register tiles: tile k lives in
    // slot k % R, and while it is consumed the loads of tiles k + 1 .. k + R - 1 are in flight.
    // Every load is issued unconditionally and the loop has no other exits, so the compiler's
    // wait for tile k never drains the younger loads.  With logits on, the groups are walked in
    // chunks with the ring drained at each chunk end; the chunk loop is uniform over the
    // workgroup (its barriers are reached by every wave).
    const int sh = ng >= 128 ? 2 : 0, in_block = (1 << sh) - 1;
    auto group_of = [&](int k) { return NW * (k & ~in_block) + (wave << sh) + (k & in_block); };
    auto count_of = [&](int n) {   // this wave's groups among the first n
      const int blocks = n / (NW << sh) << sh;
      return blocks + min(1 << sh, max(0, n - NW * blocks - (wave << sh)));
    };
    auto walk = [&](int kb, int ke, int l0, int c0) {
      if (kb >= ke) return;
      // (the scheduler must not reorder the loads of different tiles: the compiler's wait for
      // the oldest tile would then drain the younger ones)
      int row = s_rows[MODE == ROWS_SEL_TOKEN ? 0 : group_of(kb)];
      auto fetch = [&](Tile<D>& t, int k) {
        __builtin_amdgcn_sched_barrier(0);
        load_tile(t, row, group_of(min(k, ke - 1)), l0, k < ke);
        if (MODE != ROWS_SEL_TOKEN) row = s_rows[group_of(min(k + 1, ke - 1))];
        __builtin_amdgcn_sched_barrier(0);
      };
      Tile<D> t[R];
#pragma unroll
      for (int i = 0; i < R - 1; ++i) fetch(t[i], kb + i);
      for (int k = kb; k < ke; k += R) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          fetch(t[(r + R - 1) % R], k + r + R - 1);
          if (k + r < ke) process(t[r], group_of(k + r) - c0);
        }
      }
    };
    for (int l0 = 0; l0 < ng; l0 += kSeg) {
      if (l0 > 0) {   // the next part of a long piece's list, once every wave is done with this one
        lds_barrier();
        stage_list(b, g0 + l0, min(kSeg, ng - l0));
      }
      lds_barrier();   // the list is in LDS; the query loads may still be in flight
      const int nl = min(kSeg, ng - l0);
      if (!LOGITS) {
        walk(0, count_of(nl), g0 + l0, 0);
      } else {
        for (int c0 = 0; c0 < nl; c0 += kChunk) {
          const int n = min(kChunk, nl - c0);
          walk(c0 / NW, count_of(c0 + n), g0 + l0, c0);
          // chunk [c0, c0 + n) goes to [b][kv group][page ...][head][16], contiguous
          lds_barrier();
          const int nf = n * G * 16;
          float* dst = a.logits + (((size_t)b * a.n_kv_heads + g) * a.logit_pages + g0 + l0 + c0) * G * 16;
          const __amdgpu_buffer_rsrc_t out =
              __builtin_amdgcn_make_buffer_rsrc(dst, 0, nf * 4, kRawBufferFlags);
          for (int i = 4 * tid; i < nf; i += 4 * T)
            __builtin_amdgcn_raw_buffer_store_b128(
                *reinterpret_cast<const u32x4*>(s_stage + i), out, 4 * i, 0, kCoherent);
          if (c0 + n < nl) lds_barrier();
        }
      }
    }

    // ---- the wave's sums and outputs to LDS ------------------------------------------------
    reduce_outputs<D, G>(st, lane, [&](int head, int col, auto v) {
      *reinterpret_cast<decltype(v)*>(&s_w[wave].o[head][col]) = v;
    });
    if (quad == 0 && hcol < G) {
      s_m[wave][hcol] = st.m_run;
      s_l[wave][hcol] = st.l_run;
    }
    lds_barrier();

    // ---- merge the waves into one partial of the piece -------------------------------------
    // From here on thread t of the first E owns the four consecutive outputs 4t .. 4t+3 of head
    // h (D is a multiple of 4), so every partial, output and merge access is one 16- or 8-byte
    // access and each thread needs the running max and sum of one head.
    const int e = tid % E, part = tid / E;   // (part: thread group of the merge of partials)
    const bool owner = tid < E;
    const int h = 4 * e / D;
    const int dc = 4 * e % D;
    // weights of partial sums relative to their common maximum; 0 while there is none
    auto weight = [](float m, float mu) { return __builtin_amdgcn_exp2f(m - mu); };
    auto finite_or_0 = [](float m) { return m == kNegInf ? 0.f : m; };
    float M = kNegInf, L = 0.f;
    f32x4 O = {0.f, 0.f, 0.f, 0.f};
    if (owner) {
#pragma unroll
      for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w][h]);
      const float Mu = finite_or_0(M);
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = weight(s_m[w][h], Mu);
        O += f * *reinterpret_cast<const f32x4*>(&s_w[w].o[h][dc]);
        L += f * s_l[w][h];
      }
    }
    auto store_out = [&](const f32x4& v, float lsum, float mx) {
      // (divided, not multiplied by 1 / lsum: that product's extra rounding moves quotients half
      // way between two bf16 values, as equal weights give)
      uint2 packed;
      packed.x = (uint32_t)f32_to_bf16_rne(v[0] / lsum) | ((uint32_t)f32_to_bf16_rne(v[1] / lsum) << 16);
      packed.y = (uint32_t)f32_to_bf16_rne(v[2] / lsum) | ((uint32_t)f32_to_bf16_rne(v[3] / lsum) << 16);
      *reinterpret_cast<uint2*>(a.out + (size_t)(Hq_row + h) * D + dc) = packed;
      if (LOGITS && dc == 0) a.lse[(size_t)Hq_row + h] = mx + log2f(lsum);
    };

    // A pair that is one piece needs no combine: the workgroup writes the output itself.
    if (n_valid == 1) {
      if (owner) store_out(O, L, M);
      return;
    }

    // ---- combine ----------------------------------------------------------------------
    // Partials are written and read only with device-coherent accesses (the sc1 cache policy:
    // written through to memory, and read past any stale copy in another XCD's L2), so no L2
    // write-back or invalidation is needed to publish them.  Each thread waits until its
    // partial stores are complete, the barrier makes that true for the whole workgroup, and
    // only then does one thread count the workgroup in with a device-scope atomic; the
    // workgroup that brings the count to n_valid reads every partial after the atomic has
    // returned.  (A release/acquire fence pair would instead write back and invalidate the
    // whole L2 of the XCD once per workgroup; measured on MI355X that serialises launches of
    // many workgroups.)
    const int pair_floats = a.slots * G * D;
    const __amdgpu_buffer_rsrc_t po = __builtin_amdgcn_make_buffer_rsrc(
        a.part_o + (size_t)bg * pair_floats, 0, pair_floats * 4, kRawBufferFlags);
    const __amdgpu_buffer_rsrc_t pml = __builtin_amdgcn_make_buffer_rsrc(
        a.part_ml + (size_t)bg * a.slots * G * 2, 0, a.slots * G * 8, kRawBufferFlags);
    const int o_off = (h * D + dc) * 4;   // this thread's bytes inside one slot's G x D block
    if (owner) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, O), po, o_off,
                                             slot * G * D * 4, kCoherent);
      if (dc == 0)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, make_float2(M, L)), pml,
                                              h * 8, slot * G * 8, kCoherent);
    }
    __builtin_amdgcn_s_waitcnt(0);   // this thread's partial stores are complete
    __syncthreads();
    if (tid == 0) {
      const int prev = __hip_atomic_fetch_add(&a.counters[(size_t)bg * kCounterStride], 1, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
      s_last = prev == n_valid - 1;
    }
    __syncthreads();
    if (!s_last) return;

    // The workgroup's NP thread groups fold the pair's partials, group p the slots p, p + NP, ...
    // in that order, up to 16 at a time, and the groups' results are folded in group order: the
    // result does not depend on the order in which workgroups finished.  A batch's loads are all
    // in flight at once; issuing them is what takes the time (32 loads 0.9 us, their return
    // another 0.3 us), so a batch is no larger than the slots left.
    M = kNegInf;
    L = 0.f;
    O = f32x4{0.f, 0.f, 0.f, 0.f};
    auto fold = [&](int c0, auto size) {   // slots c0 + part, c0 + part + NP, ...
      constexpr int N = decltype(size)::value;
      float2 ml[N];
      f32x4 pv[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        // (an offset past the buffer reads zeros without touching memory)
        const int c = c0 + part + i * NP;
        const bool ok = c < n_valid;
        ml[i] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(
            pml, ok ? h * 8 + c * G * 8 : kPastEnd, 0, kCoherent));
        pv[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
            po, ok ? o_off + c * G * D * 4 : kPastEnd, 0, kCoherent));
      }
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (c0 + part + i * NP >= n_valid) ml[i].x = kNegInf;
      float bm = M;
#pragma unroll
      for (int i = 0; i < N; ++i) bm = fmaxf(bm, ml[i].x);
      const float Mu = finite_or_0(bm);
      const float rs = weight(M, Mu);
      L *= rs;
      O *= rs;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float f = weight(ml[i].x, Mu);
        L += f * ml[i].y;
        O += f * pv[i];
      }
      M = bm;
    };
    if (part < NP) {
      for (int c0 = 0; c0 < n_valid;) {
        const int left = n_valid - c0;   // (uniform)
        if (left <= 4 * NP) {
          fold(c0, std::integral_constant<int, 4>{});
          c0 += 4 * NP;
        } else if (left <= 8 * NP) {
          fold(c0, std::integral_constant<int, 8>{});
          c0 += 8 * NP;
        } else {
          fold(c0, std::integral_constant<int, 16>{});
          c0 += 16 * NP;
        }
      }
    }
    if (NP > 1) {
      float* so = reinterpret_cast<float*>(s_w);      // [NP][G][D]
      float* sml = reinterpret_cast<float*>(s_rows);  // [NP][G][2]
      static_assert(NP * G * D * 4 <= sizeof(s_w) && NP * G * 2 <= kMaxRowSlots, "merge space");
      if (part > 0 && part < NP) {
        *reinterpret_cast<f32x4*>(so + (part * E + e) * 4) = O;
        if (dc == 0) {
          sml[(part * G + h) * 2] = M;
          sml[(part * G + h) * 2 + 1] = L;
        }
      }
      __syncthreads();
      if (owner) {
        float m[NP], Mn = M;
#pragma unroll
        for (int q = 1; q < NP; ++q) {
          m[q] = sml[(q * G + h) * 2];
          Mn = fmaxf(Mn, m[q]);
        }
        const float Mu = finite_or_0(Mn);
        const float rs = weight(M, Mu);
        L *= rs;
        O *= rs;
#pragma unroll
        for (int q = 1; q < NP; ++q) {
          const float f = weight(m[q], Mu);
          L += f * sml[(q * G + h) * 2 + 1];
          O += f * *reinterpret_cast<const f32x4*>(so + (q * E + e) * 4);
        }
        M = Mn;
      }
    }
    if (owner) store_out(O, L, M);
    if (tid == 0) __hip_atomic_store(&a.counters[(size_t)bg * kCounterStride], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };

  // ---- which pieces this workgroup attends to --------------------------------------------
  // The static decomposition: workgroup (split, g, b) takes groups [split * gps, + gps) of
  // pair (b, g), as partial `split`.  Its page list and query are staged before anything else
  // (the sequence length arrives meanwhile) and kept when the balanced decomposition below
  // hands this workgroup the same piece.
  const int split = blockIdx.x;
  const int g_s = blockIdx.y;
  const int b_s = blockIdx.z;
  const int g0_s = split * a.gps;
  const int cand_s = max(0, min(a.gps, a.max_groups - g0_s));
  stage(b_s, g_s, g0_s, cand_s);
  const int s_bs = a.seq_lens[b_s];
  if (DELTA_DEBUG && (s_bs < 1 || s_bs > a.max_seq_len) && tid == 0 && blockIdx.x == 0 && blockIdx.y == 0)
    debug_flag(a.status, DELTA_DEBUG_SEQ_LEN);
  const int sel_ns = (MODE == ROWS_DENSE) ? 0 : min(a.sel_cnt[b_s], a.sel_stride);
  // groups of a sequence of s tokens (dense) or n selected units; lengths beyond the host bound
  // are clamped so that no access leaves the buffers
  auto groups_of = [&](int s, int n) {
    const int x = MODE == ROWS_DENSE ? (s + 15) >> 4 : MODE == ROWS_SEL_PAGE ? n : (n + 15) >> 4;
    return max(0, min(x, a.max_groups));
  };

  int bal_chunk = 0;          // > 0: this launch takes the balanced decomposition
  int bal_w = 0, bal_x = 0, bal_xe = 0;   // this workgroup's run [bal_x, bal_xe)
  // lane l of every wave: sequence l's length, units of work, and units of work of sequences
  // 0 .. l - 1
  int bal_len = 0, bal_units = 0, bal_before = 0;
  // (one sequence that nearly fills the host's bound: the static pieces are even)
  if (BAL && (gridDim.z > 1 || 10 * groups_of(s_bs, 0) < 9 * a.max_groups)) {
    // Balanced decomposition (the work of a batch spread evenly over the CUs): every (sequence,
    // KV head) pair is kPieceCost units of work followed by its groups, and the pairs, in (b,
    // g) order, are cut into runs of `chunk` units, run w for workgroup w (the launch's linear
    // index, in dispatch order).  A run may span pairs; a pair is combined from the pieces the
    // run boundaries cut its groups into, in order.  An empty sequence counts as one group (its
    // piece writes the empty output).  Every wave derives the same cut from the sequence
    // lengths (one per lane: B <= 64).
    const int B = gridDim.z;
    if (lane < B) {
      bal_len = a.seq_lens[lane];
      bal_units = max(1, groups_of(bal_len, 0)) + kPieceCost;
    }
    const int incl = wave_incl_scan(bal_units);
    bal_before = incl - bal_units;
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int longest = (int)wave_max((uint32_t)bal_units) - kPieceCost;
    const int Hkv = a.n_kv_heads;
    // the host bounds the launch's work units below 2^26
    const int W = Hkv * total;
    // (and no pair is cut into more pieces than it has partial slots)
    const int chunk = max(max((W + a.n_runs - 1) / a.n_runs, a.chunk_min),
                          (longest + a.slots - 2) / (a.slots - 1));
    // Taken only when a CU's longest share gets shorter by a twentieth or more than with the
    // static pieces (a.static_rounds of them one after another, min(gps, longest) groups each).
    // Equal lengths that fill the device evenly keep the static pieces, which never straddle a
    // pair: otherwise the run boundaries would drift through successive pairs and leave slivers
    // of a few groups, each with a piece's fixed costs.
    if (20 * (chunk + kPieceCost) <= 19 * (min(a.gps, longest) + kPieceCost) * a.static_rounds) {
      bal_chunk = chunk;   // (uniform over the launch)
      bal_w = split + gridDim.x * (g_s + Hkv * b_s);
      bal_x = bal_w < a.n_runs ? min((int64_t)bal_w * chunk, (int64_t)W) : W;
      bal_xe = min((int64_t)W, (int64_t)bal_x + chunk);
    }
  }

  // ---- the pieces, one attention call site (the balanced runs, or the static piece) --------
  bool first = true;
  while (true) {
    // Lane-dependent values are recomputed per piece instead of being hoisted out of this loop
    // (where they would stay live, in registers, through the attention loop of every piece).
    if (BAL) asm volatile("" : "+v"(tid), "+v"(lane), "+v"(quad), "+v"(hcol));
    int b, g, g0, ng, slot, n_valid, s_b, sel_n, n_groups;
    if (BAL && bal_chunk > 0) {
      if (bal_x >= bal_xe) break;
      // sequence b: the last with Hkv * (units before b) <= x (lanes below B, in order)
      const int Hkv = a.n_kv_heads;
      const uint64_t le = __ballot(lane < (int)gridDim.z && Hkv * bal_before <= bal_x);
      b = __builtin_amdgcn_readfirstlane(__popcll(le) - 1);
      const int pb = __builtin_amdgcn_readlane(bal_before, b);
      const int ub = __builtin_amdgcn_readlane(bal_units, b);
      g = (bal_x - Hkv * pb) / ub;
      const int off = Hkv * pb + g * ub + kPieceCost;   // the pair's first group
      const int end = off + ub - kPieceCost;
      if (off >= bal_xe) break;   // the run ends before the pair's groups begin
      const int x = max(bal_x, off);
      const int first_run = off / bal_chunk;
      n_valid = (end - 1) / bal_chunk - first_run + 1;
      slot = bal_w - first_run;
      g0 = x - off;
      ng = min(bal_xe, end) - x;
      s_b = __builtin_amdgcn_readlane(bal_len, b);
      sel_n = 0;
      n_groups = groups_of(s_b, 0);
      bal_x = x + ng;
      if (!(first && b == b_s && g == g_s && g0 == g0_s && min(ng, kSeg) <= cand_s)) {
        if (!first) lds_barrier();   // the previous piece's merge is done with the LDS
        stage(b, g, g0, ng);
      }
    } else {
      if (!first) break;
      b = b_s;
      g = g_s;
      g0 = g0_s;
      s_b = s_bs;
      sel_n = sel_ns;
      n_groups = groups_of(s_b, sel_n);
      n_valid = (n_groups + a.gps - 1) / a.gps;
      slot = split;
      ng = n_valid > 0 ? min(a.gps, n_groups - g0) : 0;
      if (n_valid > 0 && split >= n_valid) break;
      if (n_valid == 0 && split > 0) break;
    }
    first = false;
    // the piece is the same in every lane: scalar registers for the walk's bounds and addresses
    b = __builtin_amdgcn_readfirstlane(b);
    g = __builtin_amdgcn_readfirstlane(g);
    g0 = __builtin_amdgcn_readfirstlane(g0);
    ng = __builtin_amdgcn_readfirstlane(ng);
    slot = __builtin_amdgcn_readfirstlane(slot);
    n_valid = __builtin_amdgcn_readfirstlane(n_valid);
    s_b = __builtin_amdgcn_readfirstlane(s_b);
    sel_n = __builtin_amdgcn_readfirstlane(sel_n);
    n_groups = __builtin_amdgcn_readfirstlane(n_groups);
    if (n_groups == 0) write_empty(b, g);
    else run(b, g, g0, ng, slot, n_valid, s_b, sel_n);
  }
}

template <int D, int G>
hipError_t launch_dg(int mode, const AttnArgs& a, int batch, hipStream_t stream) {
  const dim3 grid(a.n_split, a.n_kv_heads, batch), block(kAttnThreads);
  switch (mode) {
    case ROWS_DENSE:
      // the balanced decomposition is a separate instantiation, so that launches which cannot
      // take it run the static kernel's code (0.5-1 us of a launch of 8-12)
      if (a.logits && a.n_runs > 0) hipLaunchKernelGGL((attn_kernel<D, G, ROWS_DENSE, true, true>), grid, block, 0, stream, a);
      else if (a.logits) hipLaunchKernelGGL((attn_kernel<D, G, ROWS_DENSE, true, false>), grid, block, 0, stream, a);
      else if (a.n_runs > 0) hipLaunchKernelGGL((attn_kernel<D, G, ROWS_DENSE, false, true>), grid, block, 0, stream, a);
      else hipLaunchKernelGGL((attn_kernel<D, G, ROWS_DENSE, false, false>), grid, block, 0, stream, a);
      break;
    case ROWS_SEL_PAGE: hipLaunchKernelGGL((attn_kernel<D, G, ROWS_SEL_PAGE, false, false>), grid, block, 0, stream, a); break;
    case ROWS_SEL_TOKEN: hipLaunchKernelGGL((attn_kernel<D, G, ROWS_SEL_TOKEN, false, false>), grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_d(int group, int mode, const AttnArgs& a, int batch, hipStream_t stream) {
  switch (group) {
    case 1: return launch_dg<D, 1>(mode, a, batch, stream);
    case 2: return launch_dg<D, 2>(mode, a, batch, stream);
    case 3: return launch_dg<D, 3>(mode, a, batch, stream);
    case 4: return launch_dg<D, 4>(mode, a, batch, stream);
    case 5: return launch_dg<D, 5>(mode, a, batch, stream);
    case 6: return launch_dg<D, 6>(mode, a, batch, stream);
    case 7: return launch_dg<D, 7>(mode, a, batch, stream);
    case 8: return launch_dg<D, 8>(mode, a, batch, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_attention(int head_dim, int group, int mode, const AttnArgs& a, int batch,
                            hipStream_t stream) {
  if (head_dim == 128) return launch_d<128>(group, mode, a, batch, stream);
  if (head_dim == 64) return launch_d<64>(group, mode, a, batch, stream);
  return hipErrorInvalidValue;
}

}  // namespace delta
