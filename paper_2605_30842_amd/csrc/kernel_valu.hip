// Vector-ALU decode-attention kernel (float32 or bf16 caches) on gfx950.
//
// One workgroup = one (split j, KV head hk, sequence b); its 4 waves take
// tiles of the split in turn. Within a wave, LPR = D / VEC consecutive lanes
// cover one K/V row with one 16-byte load each (VEC elements), so a load
// instruction reads RPL = 64 / LPR whole rows; a tile is U such loads per
// lane (RPL * U tokens). Each lane computes its slice of the G dot products,
// the slices are summed across the LPR lanes of the row, and every lane then
// runs the online softmax of its row slot and accumulates weight * V over its
// own head_dim slice. The row slots of a wave are merged by log-sum-exp at
// the end.
//
// Short calls are a chain of latencies, long ones are bound by the rate of the
// sums: a tile takes U G log2(LPR) of them per lane. So lanes are joined by
// data-parallel operands and row swaps of the vector unit, not by shuffles
// through LDS, and where that pays the first tile is requested before Q is
// waited for, and the next tile while one is computed. us, with shuffles and
// every tile requested when due -> now, f32, 8 x 8192 tokens, D = 128, 8 KV
// heads (4 at G = 16), contiguous and in 16-token pages: G = 1 95.3 -> 95.6 and
// 129 -> 114, G = 4 98.9 -> 95.4 and 132 -> 113, G = 8 150 -> 113 and 175 ->
// 135, G = 16 219 -> 137 and 378 -> 173.
#include "attn_common.h"

namespace comem {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Elem;
template <>
struct Elem<float> {
  static constexpr int kVec = 4;
  __device__ static void widen(const u32x4& x, float (&f)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(x[i]);
  }
};
struct Bf16 {};
template <>
struct Elem<Bf16> {
  static constexpr int kVec = 8;
  __device__ static void widen(const u32x4& x, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(x[i] << 16);
      f[2 * i + 1] = __uint_as_float(x[i] & 0xffff0000u);
    }
  }
};

template <int CTRL>
__device__ inline float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, static_cast<int>(__float_as_uint(x)), CTRL, 0xf, 0xf, true));
}

// The values of the lanes O apart (bit O of the lane clear, set); for O = 8
// the lane's own comes first.
template <int O>
__device__ inline void lane_pair(float x, float& x0, float& x1) {
  const uint32_t u = __float_as_uint(x);
  if constexpr (O == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    x0 = __uint_as_float(r[0]);
    x1 = __uint_as_float(r[1]);
  } else if constexpr (O == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    x0 = __uint_as_float(r[0]);
    x1 = __uint_as_float(r[1]);
  } else {
    x0 = x;
    x1 = __shfl_xor(x, O);
  }
}

// Sum over the LPR lanes of a row, in each of them: pairs and quads by quad
// permutation (lane ^ 1, lane ^ 2), then mirrored halves of 8 and 16 lanes,
// whose quads (halves) already hold one value.
template <int LPR>
__device__ inline float row_sum(float a) {
  a += dpp<0xb1>(a);
  a += dpp<0x4e>(a);
  if constexpr (LPR >= 8) a += dpp<0x141>(a);
  if constexpr (LPR >= 16) a += dpp<0x140>(a);
  if constexpr (LPR == 32) {
    float x0, x1;
    lane_pair<16>(a, x0, x1);
    a = x0 + x1;
  }
  return a;
}

// Merge the softmax states of the lanes O, 2 O, ... 32 apart.
template <int O, int G, int VEC>
__device__ inline void merge_slots(float (&m)[G], float (&l)[G], float (&acc)[G][VEC]) {
  if constexpr (O < 64) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float m0, m1, x0, x1;
      lane_pair<O>(m[h], m0, m1);
      const float M = fmaxf(m0, m1);
      const float a0 = fast_exp2(m0 - M);
      const float a1 = fast_exp2(m1 - M);
      lane_pair<O>(l[h], x0, x1);
      l[h] = x0 * a0 + x1 * a1;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        lane_pair<O>(acc[h][e], x0, x1);
        acc[h][e] = x0 * a0 + x1 * a1;
      }
      m[h] = M;
    }
    merge_slots<2 * O, G, VEC>(m, l, acc);
  }
}

template <typename T, int D, int G, bool PAGED>
__global__ __launch_bounds__(kThreads) void decode_valu_kernel(const AttnParams p) {
  constexpr int VEC = Elem<T>::kVec;
  constexpr int EB = 16 / VEC;    // element bytes
  constexpr int LPR = D / VEC;    // lanes per row
  constexpr int RPL = 64 / LPR;   // rows per load instruction
  constexpr int U = 4;            // loads per lane per tile
  constexpr int TT = RPL * U;     // tokens per tile
  // kEarly: the first tile before Q, later ones as soon as the last is done;
  // kAhead: the next tile while one is computed, where a second one fits the
  // registers. Contiguous caches gain from neither unless a tile's sums take
  // long (8 and 16 float32 heads); in pages a tile waits for its block-table
  // entries first. us, when due / early / ahead (8 x 8192 tokens, 8 KV heads, 4
  // at G = 16; D = 128, then 64). Contiguous: f32 G = 2 95.0 / 95.0 / 95.3 and
  // 50.3 / 51.7 / 51.9, G = 4 95.1 / 99.2 / 98.6 and 50.3 / 54.5 / 54.6, G = 8
  // 120 / 121 / 117 and 59.8 / 60.6 / 59.3, G = 16 140 / 143 / 130 and 74.5 /
  // 72.9 / 68.5; bf16 G = 4 53.4 / 55.6 / 57.7 and 31.1 / 34.2 / 34.7, G = 8
  // 77.7 / 79.2 / 97.8 and 46.0 / 47.9 / 58.2. 16-token pages: f32 G = 1 126 /
  // 115 / 114, G = 2 128 / 117 / 114, G = 4 130 / 123 / 114, G = 8 147 / 149 /
  // 147 and 76.5 / 75.1 / 72.9, G = 16 157 / 157 / 166 and 85.4 / 84.2 / 87.2;
  // bf16 G = 4 74.0 / 71.2 / 65.6, G = 8 92 / 147 / 128, G = 16 129 / 130 / 159
  // and 81.5 / 77.9 / 91.4.
  constexpr bool kWide = VEC == 4;  // float32
  constexpr bool kAhead = PAGED ? G <= 4 || (G == 8 && kWide) : G >= 8 && kWide;
  constexpr bool kEarly = kAhead || (PAGED && G == 16);
  // A row slot without a token of a tile has nothing to add for it: one branch
  // around all heads, or one for each where a tile of bf16 heads fills the
  // registers, which keeps the heads' sums from being scheduled together (G =
  // 16 contiguous 123 and 74.8 us with one branch, 110 and 70.5 with one each;
  // f32 G = 8 120 and 125, G = 16 140 and 157).
  constexpr bool kPerHead = !kWide && (G == 16 || (G == 8 && !PAGED));
  const int j = blockIdx.x, hk = blockIdx.y, b = blockIdx.z;
  int L = p.ctx_lens[b];
  int64_t seq0 = PAGED ? 0 : p.seq_start[b];
  asm volatile("" : "+s"(L), "+s"(seq0));  // one round trip for both
  L = checked_len(L, p.max_ctx, p.errors);
  const EvenParts parts(p, b, hk, j, L, p.chunk);
  if (j >= parts.count) return;
  const int t_begin = j * p.chunk;
  const int t_end = t_begin + min(L - t_begin, p.chunk);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int rho = lane / LPR, ds = lane % LPR;

  __shared__ WaveState<D> ws;

  u32x4 qraw[G];
  {
    const char* q0 = p.q + (static_cast<int64_t>(b) * p.num_q_heads + hk * G) * D * EB;
#pragma unroll
    for (int h = 0; h < G; ++h) qraw[h] = *reinterpret_cast<const u32x4*>(q0 + (h * D + ds * VEC) * EB);
  }
  const char* kb = p.k + hk * p.stride_head;
  const char* vb = p.v + hk * p.stride_head;

  float m[G], l[G], acc[G][VEC];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m[h] = kLowest;
    l[h] = 0.f;
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[h][e] = 0.f;
  }

  // Fused append: the wave whose tile holds token L - 1 (and every clamped
  // read of that row) stores the new rows first (not when the length was
  // clamped: that row is not the new token's).
  if (p.new_k != nullptr && t_end == L && L > 0 && w == ((L - 1 - t_begin) / TT) % kWaves && p.ctx_lens[b] == L) {
    int64_t row;
    if constexpr (PAGED) {
      row = checked_page_row(p, p.block_table[static_cast<int64_t>(b) * p.max_pages + ((L - 1) >> p.page_shift)],
                             L - 1);
    } else {
      row = (seq0 + L - 1) * p.stride_token;
    }
    store_new_token(p, b, hk, row, D * EB / 16, lane);
  }
  u32x4 kr[U], vr[U];
  auto request = [&](int base, u32x4 (&k)[U], u32x4 (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = min(base + u * RPL + rho, t_end - 1);
      const int64_t off = row_offset<PAGED>(p, b, seq0, t) + ds * 16;
      k[u] = *reinterpret_cast<const u32x4*>(kb + off);
      v[u] = *reinterpret_cast<const u32x4*>(vb + off);
    }
  };
  int base = t_begin + w * TT;
  if constexpr (kEarly) {
    if (base < t_end) request(base, kr, vr);
    __builtin_amdgcn_sched_barrier(0);
  }
  float qf[G][VEC];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    Elem<T>::widen(qraw[h], qf[h]);
#pragma unroll
    for (int e = 0; e < VEC; ++e) qf[h][e] *= p.scale_log2;
  }
  while (base < t_end) {
    const int next = base + kWaves * TT;
    u32x4 kn[U], vn[U];
    if constexpr (!kEarly) request(base, kr, vr);
    if constexpr (kAhead) {
      if (next < t_end) request(next, kn, vn);
      __builtin_amdgcn_sched_barrier(0);
    }
    float s[U][G];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[VEC];
      Elem<T>::widen(kr[u], kf);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) a += qf[h][e] * kf[e];
        a = row_sum<LPR>(a);
        if constexpr (kPerHead) a = a == a ? a : INFINITY;  // NaN: the maximum would pass over it (inf - inf is NaN too)
        s[u][h] = (base + u * RPL + rho < t_end) ? a : -INFINITY;
      }
    }
    float vf[U][VEC];
#pragma unroll
    for (int u = 0; u < U; ++u) Elem<T>::widen(vr[u], vf[u]);
    auto top = [&](int h) {
      float mt = m[h];
#pragma unroll
      for (int u = 0; u < U; ++u) mt = fmaxf(mt, s[u][h]);
      return mt;
    };
    auto fold = [&](int h, float m_new) {
      const float alpha = fast_exp2(m[h] - m_new);
      l[h] *= alpha;
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[h][e] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float pu = fast_exp2(s[u][h] - m_new);
        l[h] += pu;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[h][e] += pu * vf[u][e];
      }
      m[h] = m_new;
    };
    if constexpr (kPerHead) {
#pragma unroll
      for (int h = 0; h < G; ++h) {
        const float m_new = top(h);
        if (m_new == kLowest) continue;
        fold(h, m_new);
      }
    } else if (base + rho < t_end) {
#pragma unroll
      for (int h = 0; h < G; ++h) fold(h, top(h));
    }
    base = next;
    if constexpr (kAhead) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        kr[u] = kn[u];
        vr[u] = vn[u];
      }
    } else if constexpr (kEarly) {
      if (base < t_end) request(base, kr, vr);
    }
  }

  // Merge the RPL row slots of the wave (lanes that share ds).
  merge_slots<LPR, G, VEC>(m, l, acc);
  if (rho == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      if (ds == 0) {
        ws.m[w][h] = m[h];
        ws.l[w][h] = l[h];
      }
#pragma unroll
      for (int e = 0; e < VEC; ++e) ws.o[w][h][ds * VEC + e] = acc[h][e];
    }
  }
  __syncthreads();
  finalize_split<D>(p, ws, b, hk, parts);
}

template <typename T, int D, bool PAGED>
void (*pick_group(int G))(AttnParams) {
  switch (G) {
    case 1: return decode_valu_kernel<T, D, 1, PAGED>;
    case 2: return decode_valu_kernel<T, D, 2, PAGED>;
    case 4: return decode_valu_kernel<T, D, 4, PAGED>;
    case 8: return decode_valu_kernel<T, D, 8, PAGED>;
    case 16: return decode_valu_kernel<T, D, 16, PAGED>;
    default: return nullptr;
  }
}

template <typename T>
void (*pick_dim(int D, int G, bool paged))(AttnParams) {
  if (D == 128) return paged ? pick_group<T, 128, true>(G) : pick_group<T, 128, false>(G);
  if (D == 64) return paged ? pick_group<T, 64, true>(G) : pick_group<T, 64, false>(G);
  return nullptr;
}

}  // namespace

using KernelFn = void (*)(AttnParams);

KernelFn select_valu_kernel(bool bf16, int head_dim, int group, bool paged) {
  return bf16 ? pick_dim<Bf16>(head_dim, group, paged) : pick_dim<float>(head_dim, group, paged);
}

}  // namespace comem
