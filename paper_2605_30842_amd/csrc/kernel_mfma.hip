// Matrix-core (MFMA) decode-attention kernel for bf16 caches on gfx950.
//
// One work item = one (split, KV head hk, sequence b), run by one workgroup.
// Three forms hand the items out: one workgroup per split (short calls), equal
// ranges over all sequences' tokens (long calls), and a queue (configured
// split sizes). The 4 waves take 32-token tiles of the split in turn. Per tile a wave computes
//   S^T[token, head] = K_tile . Q^T    with v_mfma_f32_16x16x32_bf16
// (16 tokens x 16 head columns per instruction; the G real heads of the GQA
// group occupy the first G columns), runs the online softmax on the scores
// in registers, and accumulates
//   O^T[d, head] += V_tile^T[d, token] . P^T[token, head]
// again with 16x16x32 MFMAs. P is split as P = P_hi + P_lo, both bf16, and
// both halves are multiplied (two MFMAs), so the weights keep about 17
// significant bits instead of bf16's 8.
//
// Operand layouts (lane = 16 * g + c, c in 0..15, g in 0..3):
//   MFMA 16x16x32 reads, for A, row c and reduction elements 8g..8g+7 of the
//   lane; for B, column c and the same reduction elements; it returns
//   D[4g + r][c] in accumulator register r.
//   QK:  A = K rows (token c of the sub-tile), reduction = head_dim slice
//        32kb + 8g .. +8 -> one 16-byte load per (sub-tile, kb).
//        B = Q rows (head c), same slice. Result: lane holds the score of
//        head c for tokens 4g + r of each 16-token sub-tile.
//   PV:  B = P^T: lane already holds head c's weights for the 8 tokens
//        {16s + 4g + r}; they become reduction elements e = 4s + r.
//        A = V^T: the same 8 tokens, row c standing for d = NT*c + n in
//        n-tile n (NT = D/16). Loading V row (16s + 4g + r), bytes
//        [2*NT*c, 2*NT*(c+1)) gives every n-tile's element at once, and
//        those loads read whole 256-byte rows with 16 consecutive lanes.
//        A v_perm per element pair regroups them into MFMA operands.
//        Result: lane holds head c at d = NT*(4g + r) + n, so its maximum,
//        sum and rescaling are those of its own head.
// The reduction index of an MFMA is a dummy index, so any consistent
// assignment of (lane, element) to tokens or head_dim positions is valid as
// long as A and B use the same one, which they do by construction above.
//
// FP8 caches (OCP E4M3 codes with a per-tensor scale) use the same tiles at
// one byte per element and widen the codes to bf16 in registers before the
// matrix-core steps (exact: every E4M3 value is a bf16 value). The scales
// are folded into the score scale (K) and the final output (V). For the QK
// step a lane's K slice is then its D / 4 consecutive codes (head_dim
// (D / 4) g onward, 16 per 16-byte load): k-block kb is head_dim
// (D / 4) g + 8 kb .. + 8, and the Q operand follows the same assignment.
#include "attn_common.h"

namespace comem {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int D>
struct VRow;  // per-lane slice of one V row: NT bf16 values
// V rows are read whole by consecutive lanes and never again: load them with
// the non-temporal (streaming) cache policy. K rows are read in two halves
// of a 128-byte line by consecutive instructions, so they keep the default
// policy and the second half hits the line the first half brought in.
constexpr int kStreaming = 2;

template <>
struct VRow<128> {
  u32x4 w;
  __device__ uint32_t word(int i) const { return w[i]; }
  __device__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    w = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, kStreaming));
  }
};
template <>
struct VRow<64> {
  u32x2 w;
  __device__ uint32_t word(int i) const { return w[i]; }
  __device__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    w = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, kStreaming));
  }
};

template <int D>
struct Tile {
  static constexpr int KB = D / 32;
  u32x4 k[2][KB];   // [sub-tile][k-block]
  VRow<D> v[2][4];  // [sub-tile][r]
};

__device__ inline bf16x8 as_bf16x8(u32x4 x) { return __builtin_bit_cast(bf16x8, x); }

// The V slice of a row in an FP8 cache: NT one-byte codes.
template <int D>
struct VRow8;
template <>
struct VRow8<128> {
  u32x2 w;
  __device__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    w = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, kStreaming));
  }
};
template <>
struct VRow8<64> {
  uint32_t w;
  __device__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    w = __builtin_amdgcn_raw_buffer_load_b32(r, voff, 0, kStreaming);
  }
};

template <int D>
struct Tile8 {
  u32x4 k[2][D / 64];  // [sub-tile][16 codes]: the lane's D / 4 codes of its K row
  VRow8<D> v[2][4];
};

template <int D, bool FP8>
struct TileOf {
  using type = Tile<D>;
};
template <int D>
struct TileOf<D, true> {
  using type = Tile8<D>;
};

// Two E4M3 codes (bytes 0-1, or 2-3 with HIGH) of w as a bf16 pair, low element first.
template <bool HIGH>
__device__ inline uint32_t e4m3_pair_to_bf16(uint32_t w) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HIGH));
}

// Widen an FP8 tile to the bf16 tile the matrix-core steps read.
template <int D>
__device__ inline void widen_tile(const Tile8<D>& R, Tile<D>& T) {
  constexpr int KB = D / 32;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const uint32_t w0 = R.k[s][kb >> 1][2 * (kb & 1)], w1 = R.k[s][kb >> 1][2 * (kb & 1) + 1];
      T.k[s][kb] = u32x4{e4m3_pair_to_bf16<false>(w0), e4m3_pair_to_bf16<true>(w0), e4m3_pair_to_bf16<false>(w1),
                         e4m3_pair_to_bf16<true>(w1)};
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (D == 128) {
        const u32x2 w = R.v[s][r].w;
        T.v[s][r].w = u32x4{e4m3_pair_to_bf16<false>(w[0]), e4m3_pair_to_bf16<true>(w[0]),
                            e4m3_pair_to_bf16<false>(w[1]), e4m3_pair_to_bf16<true>(w[1])};
      } else {
        T.v[s][r].w = u32x2{e4m3_pair_to_bf16<false>(R.v[s][r].w), e4m3_pair_to_bf16<true>(R.v[s][r].w)};
      }
    }
  }
}

// Largest batch the work-queue and the balanced kernel take (their
// per-sequence offsets live in LDS).
constexpr int kMaxQueueBatch = 4096;

enum class Layout { kContig, kPaged, kPagedFine };

template <int D, Layout LAYOUT, bool FP8>
struct Loader {
  using TileT = typename TileOf<D, FP8>::type;
  static constexpr int kElemBytes = FP8 ? 1 : 2;
  const char* kbase;  // K of this (b, hk): contiguous layout already offset to the sequence start
  const char* vbase;
  const int32_t* bt_row;  // the sequence's block-table row (paged layouts)
  uint32_t pool;          // pages in the pool; an entry at or past it (negative ones too) is outside
  uint32_t* errors;
  uint32_t stride_token;  // at most 2^26
  int64_t stride_page;
  int page_shift, page_mask;
  int t_first;  // the wave's first tile
  int t_step;   // tokens from one of its tiles to the next
  int t_end;
  int lane, c, g;
  uint32_t koff;     // c * stride_token + 16 g (FP8: + (D / 4) g)
  uint32_t voff[4];  // (4 g + r) * stride_token + (NT * c elements)

  // Block-table entries. They come as vector loads, requested well ahead of
  // the tiles that need them, and take no LDS and no barrier. (As scalar
  // loads they shared the counter of the cross-lane maximum's LDS
  // operations, which then waited for them: 8 x 131072 tokens took 661
  // instead of 630 us.)
  //
  // Pages of 16 tokens or more: lane l of `now` holds the entry of half l % 2
  // of the wave's tile 32 i + l / 2, that of `next` the entries of the 32
  // tiles after those. Smaller pages: lane l < 32 of `now` holds the entry of
  // token l of the tile to be requested, `next` those of the tile after it.
  // Entries are checked as they become `now`, once each. (Checked for every
  // row of the 10 a lane reads, with a branch to the error word: 1-token pages,
  // 8 KV heads, us before / after: 32768 tokens bf16 33.5 / 32.2, FP8 22.9 /
  // 17.9; 16 x 400-4000 FP8 30.2 / 23.8; 6 x 1200-12000 bf16 44.6 / 41.9.)
  int32_t now, next;

  // An entry outside the pool reads page 0.
  __device__ int32_t in_pool(int32_t entry) const {
    if (static_cast<uint32_t>(entry) >= pool) {
      if (errors != nullptr) atomicOr(errors, kErrBlockTable);
      return 0;
    }
    return entry;
  }
  __device__ int32_t entry_of(int t) const { return bt_row[min(t, t_end - 1) >> page_shift]; }
  // Entries of the wave's tiles n .. n + 31 (n a multiple of 32), or of its tile n.
  __device__ int32_t entries(int n) const {
    if constexpr (LAYOUT == Layout::kPaged) return entry_of(t_first + t_step * (n + (lane >> 1)) + 16 * (lane & 1));
    return entry_of(t_first + t_step * n + (lane & 31));
  }
  __device__ void first_entries() {
    if constexpr (LAYOUT == Layout::kPaged) {
      now = in_pool(entries(0));
      next = entries(32);
    } else if constexpr (LAYOUT == Layout::kPagedFine) {
      now = in_pool(entries(0));
      next = entries(1);
    }
  }
  // t tokens, in bytes (t >= 0).
  __device__ int64_t tokens(int t) const {
    return static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(t)) * stride_token);
  }

  // Before the request of the wave's tile n (n = 1, 2, ...).
  __device__ void next_entries(int n) {
    if constexpr (LAYOUT == Layout::kPaged) {
      if ((n & 31) == 0) {
        now = in_pool(next);
        next = entries(n + 32);
      }
    } else if constexpr (LAYOUT == Layout::kPagedFine) {
      now = in_pool(next);
      next = entries(n + 1);
    }
  }

  // Request the wave's tile n, at token t0. Contiguous caches and pages of 16
  // tokens or more: per 16-token half one buffer descriptor on the half's
  // first row (uniform, in SGPRs) and fixed 32-bit lane offsets. The
  // descriptor ends with the last row inside the split, so rows past it
  // arrive as zeros without a memory access; their weights are zero. Smaller
  // pages: per-lane rows, clamped to the last valid one. With `repeat` the
  // call only keeps the load count of the pipeline steady: it re-reads the
  // tile's K rows (still cached) into both halves and its data is unused.
  __device__ void load(TileT& T, int n, int t0, bool repeat) const {
    constexpr int KB = D / 32;
    const char* vsrc = repeat ? kbase : vbase;
    if constexpr (LAYOUT == Layout::kPagedFine) {
      constexpr int VBYTES = kElemBytes * D / 16;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const char* kr = kbase + lane_row(t0, 16 * s + c) + (FP8 ? (D / 4) * g : 16 * g);
        if constexpr (FP8) {
#pragma unroll
          for (int i = 0; i < D / 64; ++i) T.k[s][i] = *reinterpret_cast<const u32x4*>(kr + 16 * i);
        } else {
#pragma unroll
          for (int kk = 0; kk < KB; ++kk) T.k[s][kk] = *reinterpret_cast<const u32x4*>(kr + 64 * kk);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          T.v[s][r].w = *reinterpret_cast<const decltype(T.v[s][r].w)*>(vsrc + lane_row(t0, 16 * s + 4 * g + r) + VBYTES * c);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int t = t0 + 16 * s;
        int64_t base;
        if constexpr (LAYOUT == Layout::kContig) {
          base = tokens(t);
        } else {
          const int page = __builtin_amdgcn_readlane(now, 2 * (n & 31) + s);
          base = static_cast<int64_t>(page) * stride_page + tokens(t & page_mask);
        }
        base = uniform_i64(base);
        // Bytes from the half's first row to the end of its last one inside
        // the split (selects, not a clamp: the clamp became a vector
        // instruction whose register waited for tile loads in flight).
        const int left = t_end - t;
        const uint32_t some = left > 0 ? (static_cast<uint32_t>(left) - 1) * stride_token + kElemBytes * D : 0;
        const int extent = uniform_i32(static_cast<int>(left >= 16 ? 15 * stride_token + kElemBytes * D : some));
        const __amdgpu_buffer_rsrc_t rk =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(kbase + base), 0, extent, kBufferConfig);
        const __amdgpu_buffer_rsrc_t rv =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(vsrc + base), 0, extent, kBufferConfig);
        if constexpr (FP8) {
#pragma unroll
          for (int i = 0; i < D / 64; ++i)
            T.k[s][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, koff + 16 * i, 0, 0));
        } else {
#pragma unroll
          for (int kk = 0; kk < KB; ++kk)
            T.k[s][kk] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, koff + 64 * kk, 0, 0));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) T.v[s][r].load(rv, voff[r]);
      }
    }
  }

  // Small pages: byte offset of row i of the tile at t0, clamped to the last valid one.
  __device__ int64_t lane_row(int t0, int i) const {
    const int ic = min(i, t_end - 1 - t0);
    return static_cast<int64_t>(__shfl(now, ic)) * stride_page + tokens((t0 + ic) & page_mask);
  }
};

// The larger (or the sum) of the four lane groups' values of x, in every
// lane: row and half swaps in the vector unit, where a shuffle through LDS
// takes a round trip of about 100 cycles in the middle of a tile's one chain.
struct Max {
  __device__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
struct Add {
  __device__ float operator()(float a, float b) const { return a + b; }
};
template <typename Op>
__device__ inline float across_groups(float x, Op op) {
  const uint32_t u = __float_as_uint(x);
  const auto rows = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t v = __float_as_uint(op(__uint_as_float(rows[0]), __uint_as_float(rows[1])));
  const auto halves = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return op(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
}

// With one wave on a SIMD (short calls, and the balanced form) a tile's time
// is this chain's latency: scores, maximum, weights, products. So nothing in
// it goes through LDS, and the outputs are rescaled only when a maximum moved.
template <int D>
__device__ inline void compute_tile(const Tile<D>& T, int t0, int t_end, int g,
                                    const bf16x8 (&qop)[D / 32], float scale_log2, float& m_run,
                                    float& l_run, f32x4 (&acc)[D / 16]) {
  constexpr int KB = D / 32;
  constexpr int NT = D / 16;
  // Scores S^T: lane holds head c, tokens t0 + 16s + 4g + r.
  f32x4 sc[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    sc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KB; ++kk)
      sc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.k[s][kk]), qop[kk], sc[s], 0, 0, 0);
  }
  float x[8];
  float mt = -INFINITY;
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 16 * s + 4 * g + r;
      const float v = t < t_end ? sc[s][r] * scale_log2 : -INFINITY;
      x[4 * s + r] = v;
      mt = fmaxf(mt, v);
    }
  const float m_new = fmaxf(m_run, across_groups(mt, Max{}));
  if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
    const float alpha = fast_exp2(m_run - m_new);
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] *= alpha;
    l_run *= alpha;
    m_run = m_new;
  }
  float psum = 0.f;
  uint32_t ph[4], pl[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const float p0 = fast_exp2(x[e] - m_new);
    const float p1 = fast_exp2(x[e + 1] - m_new);
    psum += p0 + p1;
    split_bf16(p0, p1, ph[e / 2], pl[e / 2]);
  }
  l_run += psum;
  const bf16x8 p_hi = as_bf16x8(u32x4{ph[0], ph[1], ph[2], ph[3]});
  const bf16x8 p_lo = as_bf16x8(u32x4{pl[0], pl[1], pl[2], pl[3]});
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const uint32_t sel = (n & 1) ? 0x07060302u : 0x05040100u;
    const int wi = n >> 1;
    u32x4 va;
    va[0] = __builtin_amdgcn_perm(T.v[0][1].word(wi), T.v[0][0].word(wi), sel);
    va[1] = __builtin_amdgcn_perm(T.v[0][3].word(wi), T.v[0][2].word(wi), sel);
    va[2] = __builtin_amdgcn_perm(T.v[1][1].word(wi), T.v[1][0].word(wi), sel);
    va[3] = __builtin_amdgcn_perm(T.v[1][3].word(wi), T.v[1][2].word(wi), sel);
    acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(va), p_hi, acc[n], 0, 0, 0);
    acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(va), p_lo, acc[n], 0, 0, 0);
  }
}

// compute_tile on a tile as loaded (FP8 tiles are widened first).
template <int D, bool FP8>
__device__ inline void compute_loaded(const typename TileOf<D, FP8>::type& T, int t0, int t_end, int g,
                                      const bf16x8 (&qop)[D / 32], float scale_log2, float& m_run, float& l_run,
                                      f32x4 (&acc)[D / 16]) {
  if constexpr (FP8) {
    Tile<D> W;
    widen_tile<D>(T, W);
    compute_tile<D>(W, t0, t_end, g, qop, scale_log2, m_run, l_run, acc);
  } else {
    compute_tile<D>(T, t0, t_end, g, qop, scale_log2, m_run, l_run, acc);
  }
}

// ctx_lens[b] and, for the contiguous layout, seq_start[b]: both loads are
// issued before either value is used (the empty asm consumes both at once),
// so they share one memory round trip.
template <Layout LAYOUT>
__device__ inline void load_sequence(const AttnParams& p, int b, int& L, int64_t& seq_row) {
  b = uniform_i32(b);  // uniform in every caller
  L = uniform_i32(p.ctx_lens[b]);
  seq_row = LAYOUT == Layout::kContig ? uniform_i64(p.seq_start[b]) : 0;
  asm volatile("" : "+s"(L), "+s"(seq_row));
  L = checked_len(L, p.max_ctx, p.errors);
}

// Attention of the G query heads of KV head hk of sequence b over one split
// (its `ntiles` tiles of 32 tokens, `stride` tokens from one to the next, from
// token t_begin, a multiple of 32, on; the last may end early at t_end),
// ending with this split's share of the log-sum-exp merge. Called by every thread of the
// workgroup. seq_row is seq_start[b] for the contiguous layout (unused when
// paged); the callers load it together with ctx_lens[b], so the two loads
// cost one round trip before the first tile is requested.
//
// With next_item set (work-queue form), thread 0 takes the workgroup's next
// item from the queue once the token loop is done: issued earlier, the queue
// atomic would sit ahead of the tile loads in the in-order memory counter.
template <int D, Layout LAYOUT, bool FP8, typename Parts>
__device__ void attend_split(const AttnParams& p, WaveState<D>& ws, int b, int hk, const Parts& parts, int t_begin,
                             int stride, int ntiles, int t_end, int L, int64_t seq_row, int* next_item) {
  using TileT = typename TileOf<D, FP8>::type;
  using LoaderT = Loader<D, LAYOUT, FP8>;
  constexpr int KB = D / 32;
  constexpr int NT = D / 16;
  const int lane = threadIdx.x & 63;
  const int w = uniform_i32(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int G = p.group;

  LoaderT ld;
  ld.kbase = p.k + hk * p.stride_head;
  ld.vbase = p.v + hk * p.stride_head;
  ld.bt_row = nullptr;
  if constexpr (LAYOUT == Layout::kContig) {
    const int64_t seq0 = seq_row * p.stride_token;
    ld.kbase += seq0;
    ld.vbase += seq0;
  } else {
    ld.bt_row = p.block_table + static_cast<int64_t>(b) * p.max_pages;
  }
  ld.pool = static_cast<uint32_t>(min(p.num_pages, int64_t{1} << 31));
  ld.errors = p.errors;
  ld.stride_token = static_cast<uint32_t>(p.stride_token);
  ld.stride_page = p.stride_page;
  ld.page_shift = p.page_shift;
  ld.page_mask = p.page_mask;
  ld.t_end = t_end;
  ld.lane = lane;
  ld.c = c;
  ld.g = g;
  ld.koff = static_cast<uint32_t>(c * p.stride_token + (FP8 ? (D / 4) * g : 16 * g));
#pragma unroll
  for (int r = 0; r < 4; ++r)
    ld.voff[r] = static_cast<uint32_t>((4 * g + r) * p.stride_token + (FP8 ? NT : 2 * NT) * c);

  // Q operand: head c of the group (zero columns past G), slice 32kb + 8g
  // (FP8 caches: (D / 4) g + 8 kb, the slice the lane's K codes cover).
  bf16x8 qop[KB];
  {
    const char* qrow = p.q + (static_cast<int64_t>(b) * p.num_q_heads + hk * G + c) * D * 2;
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) {
      u32x4 qv = u32x4{0u, 0u, 0u, 0u};
      if (c < G) qv = *reinterpret_cast<const u32x4*>(qrow + (FP8 ? (D / 2) * g + 16 * kk : 64 * kk + 16 * g));
      qop[kk] = as_bf16x8(qv);
    }
  }

  float m_run = kLowest, l_run = 0.f;
  f32x4 acc[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Fused append: the wave that owns the tile of token L - 1 stores its rows
  // first (not when the length was clamped: that row is not the new token's).
  if (p.new_k != nullptr && L > 0 && t_begin + stride * (ntiles - 1) == ((L - 1) & ~31) &&
      w == (ntiles - 1) % kWaves && p.ctx_lens[b] == L) {
    int64_t row;
    if constexpr (LAYOUT == Layout::kContig) {
      row = (seq_row + static_cast<int64_t>(L - 1)) * p.stride_token;
    } else {
      row = checked_page_row(p, ld.bt_row[(L - 1) >> p.page_shift], L - 1);
    }
    store_new_token(p, b, hk, row, FP8 ? D / 16 : D / 8, lane);
  }
  // Tiles w, w + 4, ...: while one tile is computed the next is in flight.
  // The prefetch is issued unconditionally (past the wave's last tile it
  // re-reads cached K rows of that one) and pinned ahead of the compute, so
  // the compiler waits for exactly the older tile's loads.
  if (w < ntiles) {
    const int last = (ntiles - 1 - w) / kWaves;  // the wave's tiles 0 .. last
    ld.t_first = t_begin + stride * w;
    ld.t_step = stride * kWaves;
    auto token = [&](int n) { return ld.t_first + ld.t_step * n; };
    TileT A, B;
    ld.first_entries();
    ld.load(A, 0, token(0), false);
    for (int n = 0;;) {
      int nx = min(n + 1, last);
      if (n < last) ld.next_entries(nx);
      ld.load(B, nx, token(nx), n == last);
      __builtin_amdgcn_sched_barrier(0);
      compute_loaded<D, FP8>(A, token(n), t_end, g, qop, p.scale_log2, m_run, l_run, acc);
      if (n == last) break;
      n = nx;
      nx = min(n + 1, last);
      if (n < last) ld.next_entries(nx);
      ld.load(A, nx, token(nx), n == last);
      __builtin_amdgcn_sched_barrier(0);
      compute_loaded<D, FP8>(B, token(n), t_end, g, qop, p.scale_log2, m_run, l_run, acc);
      if (n == last) break;
      n = nx;
    }
  }

  if (next_item != nullptr && threadIdx.x == 0)
    *next_item = static_cast<int>(gridDim.x + atomicAdd(p.tickets + p.queue_slot, 1u));

  // Wave totals: l over the four lane groups; state to LDS.
  l_run = across_groups(l_run, Add{});
  if (g == 0 && c < G) {
    ws.m[w][c] = m_run;
    ws.l[w][c] = l_run;
  }
  // A lane holds head c at NT consecutive head_dim positions per r: 16-byte
  // stores.
  if (c < G) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int n = 0; n < NT; n += 4)
        *reinterpret_cast<float4*>(&ws.o[w][c][NT * (4 * g + r) + n]) =
            make_float4(acc[n][r], acc[n + 1][r], acc[n + 2][r], acc[n + 3][r]);
  }
  __syncthreads();
  finalize_split<D>(p, ws, b, hk, parts);
}

// a / d for a, d < 2^23 and rd = 1 / d to within two units in the last place:
// the float quotient is off by at most one.
__device__ inline uint32_t div_small(uint32_t a, uint32_t d, float rd) {
  const uint32_t q = static_cast<uint32_t>(static_cast<float>(a) * rd);
  const int r = static_cast<int>(a - q * d);
  return r < 0 ? q - 1 : (r >= static_cast<int>(d) ? q + 1 : q);
}

// Tiles of a sequence (an empty one has one, empty, tile).
__device__ inline int tiles_of(int L) { return L > 0 ? (L + 31) >> 5 : 1; }

// Tiles per range of a call of `total` tiles: an equal share of the ranges,
// but no less than a piece should have (see decode_mfma_balanced_kernel), and
// one sequence of at most p.whole_tiles whole.
__device__ inline int range_tiles(const AttnParams& p, int total) {
  if (total <= p.whole_tiles) return total;
  const int share = static_cast<int>(
      div_small(total + p.ranges - 1, p.ranges, __builtin_amdgcn_rcpf(static_cast<float>(p.ranges))));
  const float piece = __builtin_ceilf(__builtin_amdgcn_sqrtf(p.split_coef * static_cast<float>(total)));
  return uniform_i32(max(share, max(2, static_cast<int>(piece))));
}

// One workgroup per (split, KV head, sequence); splits past a sequence's end
// exit. Within a sequence the KV head varies fastest with the linear
// workgroup id, the order in which workgroups are dealt to the XCDs (round
// robin): with 8 KV heads all splits of a head run on one XCD, and the heads
// of a token range are read side by side. The batch-1 32K step with K and V
// in two allocations took 29.1 instead of 30.3 us (27.8 and 27.9 us with the
// recommended placement). Grids of more than 2^24 workgroups per sequence
// keep the direct order (the 32-bit index arithmetic stays exact).
//
// A planned call of one sequence comes here with p.ranges set: its balanced
// ranges are even splits whose size follows from L, and the balanced kernel's
// prefix sums and search cost 0.9 us (us, 1024-token splits / now, bf16,
// G = 4, 8 KV heads: 1000 tokens 13.8 / 7.2, 4000 17.1 / 10.0, 6001 17.4 / 11.0).
template <int D, Layout LAYOUT, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void decode_mfma_kernel(const AttnParams p) {
  int j = blockIdx.x, hk = blockIdx.y;
  const int b = blockIdx.z;
  if (static_cast<uint64_t>(gridDim.x) * gridDim.y <= (1u << 24)) {
    const uint32_t lin = blockIdx.x + gridDim.x * blockIdx.y;
    hk = static_cast<int>(lin % gridDim.y);
    j = static_cast<int>(lin / gridDim.y);
  }
  int L;
  int64_t seq_row;
  load_sequence<LAYOUT>(p, b, L, seq_row);
  const int chunk = p.ranges > 0 ? 32 * range_tiles(p, tiles_of(L)) : p.chunk;
  const EvenParts parts(p, b, hk, j, L, chunk);
  if (j >= parts.count) return;
  __shared__ WaveState<D> ws;
  int t0 = j * chunk, stride = 32, t_end = t0 + min(L - t0, chunk), ntiles = (t_end - t0 + 31) >> 5;
  if (p.ranges > 0) {
    // Split j of n takes the tiles j, j + n, ... (a call with ranges has fewer
    // than 2^23), not a run of them: the workgroups then read one moving window
    // of the cache, where runs of a power of two of tokens start whole MiB
    // apart (us per call, runs / strided, contiguous: 32768 tokens FP8 16.9 /
    // 15.9 eager, 18.6 / 17.5 with cold caches, bf16 25.1 / 25.0 and 27.8 /
    // 27.2; eager, 8192 12.8 / 12.6, 16384 16.8 / 16.6, 65536 48.7 / 46.5 and
    // FP8 28.5 / 26.4, 131072 86.3 / 83.7 and 49.0 / 48.7; 6001, 20000 and
    // 100001 within 0.7%). Pages lie scattered anyway (16 tokens: 16384 16.9 /
    // 16.8, 32768 26.0 / 25.8; 64: 25.7 / 25.9); they keep the same splits, so
    // that a paged call returns the contiguous call's bits.
    const int n = parts.count;
    t0 = 32 * j;
    stride = 32 * n;
    t_end = L;
    ntiles = L > 0 ? uniform_i32(static_cast<int>(div_small(tiles_of(L) - j + n - 1, n,
                                                            __builtin_amdgcn_rcpf(static_cast<float>(n)))))
                   : 0;
  }
  attend_split<D, LAYOUT, FP8>(p, ws, b, hk, parts, t0, stride, ntiles, t_end, L, seq_row, nullptr);
}

// In-place prefix sum by one wave: a[i + 1] (counts of sequences 0..n-1)
// becomes the total of the first i + 1 counts, and a[0] = 0.
__device__ inline void wave_prefix_sum(int* a, int n, int lane) {
  int carry = 0;
  for (int base = 0; base < n; base += 64) {
    const int i = base + lane;
    int v = i < n ? a[i + 1] : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    if (i < n) a[i + 1] = carry + v;
    carry += __shfl(v, 63);
  }
  if (lane == 0) a[0] = 0;
}

// Sequence b with first[b] <= index < first[b + 1] (first is a prefix sum).
__device__ inline int find_sequence(const int* first, int n, int index) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= index) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Persistent workgroups that take work items from a queue: the form for a
// configured split size with more items than workgroups. The items are the
// splits of every sequence in the order (b, j, hk), so that the heads of one
// token range are adjacent and sequences follow each other. Which workgroup
// runs an item depends on timing, but every item computes the same values
// and the merge order is fixed, so results do not. The queue counter and the
// count of finished workgroups live next to the tickets and return to zero
// when the last workgroup leaves. Faster XCDs and compute units simply take
// more items, and ragged batches need no empty workgroups.
template <int D, Layout LAYOUT, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void decode_mfma_queue_kernel(const AttnParams p, int batch) {
  __shared__ WaveState<D> ws;
  __shared__ int sm_first[kMaxQueueBatch + 1];  // prefix sums of splits per sequence
  __shared__ int sm_next;
  const int tid = threadIdx.x;
  uint32_t* queue = p.tickets + p.queue_slot;
  uint32_t* finished = queue + 1;

  for (int b = tid; b < batch; b += kThreads)  // a length out of bounds is reported by load_sequence
    sm_first[b + 1] = EvenParts::splits(checked_len(p.ctx_lens[b], p.max_ctx, nullptr), p.chunk);
  __syncthreads();
  if (tid < 64) wave_prefix_sum(sm_first, batch, tid);
  __syncthreads();
  const int total = sm_first[batch] * p.num_kv_heads;
  // Item blockIdx.x first; later items come from the queue, which hands out
  // gridDim.x, gridDim.x + 1, ... Without more items than workgroups the
  // queue is never touched.
  const bool queued = total > static_cast<int>(gridDim.x);

  int item = blockIdx.x;
  while (item < total) {
    const int index = item / p.num_kv_heads;
    const int hk = item - index * p.num_kv_heads;
    const int b = find_sequence(sm_first, batch, index);
    const int j = index - sm_first[b];
    int L;
    int64_t seq_row;
    load_sequence<LAYOUT>(p, b, L, seq_row);
    const int t0 = j * p.chunk, t_end = t0 + min(L - t0, p.chunk);
    attend_split<D, LAYOUT, FP8>(p, ws, b, hk, EvenParts(p, b, hk, j, L, p.chunk), t0, 32, (t_end - t0 + 31) >> 5, t_end, L,
                                 seq_row, queued ? &sm_next : nullptr);
    __syncthreads();
    item = queued ? sm_next : total;
    __syncthreads();
  }
  if (queued && tid == 0 && atomicAdd(finished, 1u) == gridDim.x - 1) {
    atomicExch(queue, 0u);
    atomicExch(finished, 0u);
  }
}

// The balanced form, for planned splits: the 32-token tiles of all sequences,
// one after the other, are cut into p.ranges equal ranges, and workgroup
// (hk, r) attends over range r of KV head hk, in one piece per sequence that
// the range touches. A sequence inside one range is written directly; the
// pieces of one that several ranges share are merged by the last to finish.
// A second piece costs a workgroup a merge and a pipeline to refill, about
// the time of kPieceTiles tiles, so each sequence counts that many units
// before its tiles (us without / with: 8 fp8 sequences of 1000-7000 tokens
// 18.5 / 16.7, 8 bf16 of 2000-8192 36.3 / 34.9, 4 of 5000-32768 63.0 / 61.4).
//
// HBM bandwidth bounds it, and one workgroup per CU with one long equal piece
// of work reads faster than more, shorter items: fewer times does a workgroup
// stop reading to merge its waves and publish (about 10 us under load), and
// no last round of items runs on a part of the chip. Measured (us, work queue
// of 1024- to 4096-token splits / balanced): 8 x 131072 tokens, G = 8, 4 GiB
// in 64-token pages 661 / 628 (6.8 TB/s); 16 x 4K-64K packed 380 / 357; 64 x
// 2K-16K in 16-token pages 382 / 363.
// With the heads of a range in adjacent workgroups, its rows are read side by
// side, and with 8 KV heads a head stays on one XCD.
//
// Short calls are bounded by latency instead: a longer range costs time per
// token on its one CU, a shorter one more partial results to merge. With a
// per token and m per split, a length n splits best into pieces of
// sqrt(m n / a) tokens; p.split_coef holds m / (32 a batch), and no range is
// shorter than that length for the mean sequence of the call (nor than 64
// tokens).
template <int D, Layout LAYOUT, bool FP8>
__global__ __launch_bounds__(kThreads, 2) void decode_mfma_balanced_kernel(const AttnParams p, int batch) {
  __shared__ WaveState<D> ws;
  __shared__ int sm_first[kMaxQueueBatch + 1];  // batches over 64: prefix sums of units per sequence
  constexpr int kPiece = FP8 || D == 64 ? kPieceTilesLight : kPieceTiles;
  const int hk = blockIdx.x, r = blockIdx.y;
  const int lane = threadIdx.x & 63;
  // Units per sequence as prefix sums: up to 64 sequences in the lanes of
  // every wave, else in LDS.
  const bool in_lanes = batch <= 64;
  int len = 0, incl = 0, total;
  int64_t row = 0;  // seq_start, requested together with the length
  if (in_lanes) {
    if (lane < batch) {
      len = p.ctx_lens[lane];
      if constexpr (LAYOUT == Layout::kContig) row = p.seq_start[lane];
      len = checked_len(len, p.max_ctx, p.errors);
      incl = kPiece + tiles_of(len);
    }
    for (int o = 1; o < batch; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    total = __builtin_amdgcn_readlane(incl, batch - 1);
  } else {
    for (int b = threadIdx.x; b < batch; b += kThreads)
      sm_first[b + 1] = kPiece + tiles_of(checked_len(p.ctx_lens[b], p.max_ctx, p.errors));
    __syncthreads();
    if (threadIdx.x < 64) wave_prefix_sum(sm_first, batch, lane);
    __syncthreads();
    total = uniform_i32(sm_first[batch]);
  }
  const int per = range_tiles(p, total);
  const float rper = __builtin_amdgcn_rcpf(static_cast<float>(per));
  int cur = r * per;
  if (cur >= total) return;
  const int stop = min(cur + per, total);
  int b = in_lanes ? __builtin_ctzll(__builtin_amdgcn_ballot_w64(lane < batch && incl > cur))
                   : uniform_i32(find_sequence(sm_first, batch, cur));
  for (;;) {
    const int first = in_lanes ? (b > 0 ? __builtin_amdgcn_readlane(incl, b - 1) : 0) : uniform_i32(sm_first[b]);
    const int end = in_lanes ? __builtin_amdgcn_readlane(incl, b) : uniform_i32(sm_first[b + 1]);
    int L;
    int64_t seq_row;
    if (in_lanes) {
      L = __builtin_amdgcn_readlane(len, b);
      const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(row), b);
      const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(row >> 32), b);
      seq_row = static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
    } else {
      load_sequence<LAYOUT>(p, b, L, seq_row);
    }
    const int piece_end = min(stop, end), begin = first + kPiece;
    if (piece_end > begin) {
      const int r0 = uniform_i32(static_cast<int>(div_small(begin, per, rper)));
      const int r1 = uniform_i32(static_cast<int>(div_small(end - 1, per, rper)));
      const int t0 = 32 * max(cur - begin, 0), t_end = min(L, 32 * (piece_end - begin));
      attend_split<D, LAYOUT, FP8>(p, ws, b, hk, RangeParts(p, hk, r, r0, r1), t0, 32, (t_end - t0 + 31) >> 5, t_end, L, seq_row,
                                   nullptr);
    }
    cur = piece_end;
    if (cur >= stop) return;
    ++b;
    __syncthreads();  // the wave states are rewritten
  }
}

}  // namespace

using KernelFn = void (*)(AttnParams);
using QueueKernelFn = void (*)(AttnParams, int);

template <int D, bool FP8>
KernelFn pick_layout(bool paged, int page_size) {
  if (!paged) return decode_mfma_kernel<D, Layout::kContig, FP8>;
  return page_size >= 16 ? decode_mfma_kernel<D, Layout::kPaged, FP8> : decode_mfma_kernel<D, Layout::kPagedFine, FP8>;
}

template <int D, bool FP8>
QueueKernelFn pick_queue_layout(bool paged, int page_size) {
  if (!paged) return decode_mfma_queue_kernel<D, Layout::kContig, FP8>;
  return page_size >= 16 ? decode_mfma_queue_kernel<D, Layout::kPaged, FP8>
                         : decode_mfma_queue_kernel<D, Layout::kPagedFine, FP8>;
}

template <int D, bool FP8>
QueueKernelFn pick_balanced_layout(bool paged, int page_size) {
  if (!paged) return decode_mfma_balanced_kernel<D, Layout::kContig, FP8>;
  return page_size >= 16 ? decode_mfma_balanced_kernel<D, Layout::kPaged, FP8>
                         : decode_mfma_balanced_kernel<D, Layout::kPagedFine, FP8>;
}

KernelFn select_mfma_kernel(int head_dim, bool paged, int page_size, bool fp8) {
  if (head_dim == 128) return fp8 ? pick_layout<128, true>(paged, page_size) : pick_layout<128, false>(paged, page_size);
  if (head_dim == 64) return fp8 ? pick_layout<64, true>(paged, page_size) : pick_layout<64, false>(paged, page_size);
  return nullptr;
}

QueueKernelFn select_mfma_queue_kernel(int head_dim, bool paged, int page_size, bool fp8) {
  if (head_dim == 128)
    return fp8 ? pick_queue_layout<128, true>(paged, page_size) : pick_queue_layout<128, false>(paged, page_size);
  if (head_dim == 64)
    return fp8 ? pick_queue_layout<64, true>(paged, page_size) : pick_queue_layout<64, false>(paged, page_size);
  return nullptr;
}

QueueKernelFn select_mfma_balanced_kernel(int head_dim, bool paged, int page_size, bool fp8) {
  if (head_dim == 128)
    return fp8 ? pick_balanced_layout<128, true>(paged, page_size) : pick_balanced_layout<128, false>(paged, page_size);
  if (head_dim == 64)
    return fp8 ? pick_balanced_layout<64, true>(paged, page_size) : pick_balanced_layout<64, false>(paged, page_size);
  return nullptr;
}

int mfma_max_queue_batch() { return kMaxQueueBatch; }

}  // namespace comem
