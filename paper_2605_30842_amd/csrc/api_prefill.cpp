// Host side of the prefill-attention C ABI (comem_prefill_attn.h): argument
// validation (before any HIP call) and launch of the prefill kernel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "attn_common.h"
#include "comem_decode_attn.h"
#include "comem_prefill_attn.h"
#include "plan.h"
#include "prefill.h"

using namespace comem::host;

namespace {

// A prefill call with no sequence or no new token reads and writes nothing,
// so, as for batch = 0 in the decode calls, it needs no buffers.
bool prefill_is_empty(int32_t batch, int32_t max_q_len) { return batch == 0 || max_q_len == 0; }

comem_status check_bounds(const comem_decode_attn_plan& p, int32_t batch, int32_t max_q_len, int64_t max_ctx_len) {
  if (batch < 0 || batch > p.cfg.max_batch) return COMEM_ERR_INVALID_SHAPE;
  if (max_ctx_len < 0 || max_ctx_len > p.cfg.max_ctx_len) return COMEM_ERR_INVALID_SHAPE;
  if (max_q_len < 0 || max_q_len > max_ctx_len) return COMEM_ERR_INVALID_SHAPE;
  return COMEM_OK;
}

// Checks of a prefill call shared by both layouts; fills the kernel arguments.
comem_status prepare_prefill(const comem_decode_attn_plan& p, const void* q, const int64_t* q_start,
                             const int32_t* q_lens, int32_t max_q_len, const void* k, const void* v,
                             int64_t stride_token, int64_t stride_head, const int32_t* ctx_lens, int32_t batch,
                             int64_t max_ctx_len, float* out, float* lse, const void* workspace,
                             comem::PrefillParams& a) {
  if (p.cfg.dtype != COMEM_BF16) return COMEM_ERR_UNSUPPORTED;
  comem_status st = check_bounds(p, batch, max_q_len, max_ctx_len);
  if (st != COMEM_OK || prefill_is_empty(batch, max_q_len)) return st;
  st = validate_common(p, q, k, v, stride_token, stride_head, ctx_lens, batch, max_ctx_len, out, lse, workspace);
  if (st != COMEM_OK) return st;
  if (q_start == nullptr || q_lens == nullptr) return COMEM_ERR_NULL_POINTER;
  if (!aligned(q_start, 8) || !aligned(q_lens, 4)) return COMEM_ERR_MISALIGNED;
  const int64_t e = elem_bytes(p.cfg);
  std::memset(&a, 0, sizeof(a));
  a.q = static_cast<const char*>(q);
  a.k = static_cast<const char*>(k);
  a.v = static_cast<const char*>(v);
  a.out = out;
  a.lse = lse;
  a.q_start = q_start;
  a.q_lens = q_lens;
  a.ctx_lens = ctx_lens;
  a.stride_token = stride_token * e;
  a.stride_head = stride_head * e;
  a.num_q_heads = p.cfg.num_q_heads;
  a.group = group_of(p.cfg);
  a.tokens_per_block = comem::kPrefillRows / a.group;
  a.scale_log2 = p.cfg.scale * 1.4426950408889634f;
  a.max_ctx = static_cast<int32_t>(max_ctx_len);
  a.max_q = max_q_len;
  return COMEM_OK;
}

// Workspace bytes of `items` (sequence, KV head, query block) items whose keys
// `splits` workgroups share.
size_t split_bytes(const comem_decode_attn_plan& p, int64_t items, int64_t splits) {
  if (splits <= 1) return 0;
  const size_t rows = static_cast<size_t>(items) * static_cast<size_t>(splits) * comem::kPrefillRows;
  return align256(rows * 4) + rows * static_cast<size_t>(p.cfg.head_dim) * 4;
}

// Estimated us of a call whose blocks' keys `splits` workgroups each share.
// One workgroup runs on a compute unit (its K and V tiles take 128 KB of LDS).
// A 64-key tile takes it 0.7 us on an idle GPU and 1.2 on a full one, whose
// clock the power limits (head_dim 64: 0.66 and 0.8), its start and end 12 us
// (9), and the partial results go out and come back once, at about 3 TB/s.
// Unsplit blocks differ: each sees the keys up to its own last token, so the
// units need the rounds of the largest blocks, or, where blocks are many and
// small, an even share of all tiles and half of the difference between the
// largest and the smallest block.
double prefill_us(const comem_decode_attn_plan& p, int64_t pairs, int64_t blocks, int64_t max_ctx_len,
                  int64_t splits) {
  const double units = p.num_cus, block_tiles = comem::kPrefillRows / group_of(p.cfg) / 64.0;
  const double items = static_cast<double>(pairs * blocks);
  const double most = static_cast<double>(ceil_div(max_ctx_len, comem::kPrefillTileKeys));
  const double least = std::max(1.0, most - block_tiles * static_cast<double>(blocks - 1));
  const double even = items * (most + least) / 2 / units;
  const double rounds = std::ceil(items * static_cast<double>(splits) / units);
  double steps = rounds * std::ceil(most / static_cast<double>(splits));
  if (splits == 1) {
    // Round r's largest block is (r - 1) units / pairs blocks from the largest.
    const double drop = block_tiles * units / static_cast<double>(pairs);
    const double r = std::min(rounds, std::max(1.0, std::floor((most + drop) / (2 * drop))));
    steps = std::max({most, r * (most - drop * (r - 1)), rounds * (most - drop * (rounds - 1)),
                      even + (most - least) / 2});
  }
  const double load = std::min(1.0, even / steps);
  const bool wide = p.cfg.head_dim == 128;
  const double us = (wide ? 12 : 9) + (wide ? 0.7 + 0.5 * load : 0.66 + 0.14 * load) * steps;
  return us + (splits > 1 ? 2 + 2 * static_cast<double>(split_bytes(p, pairs * blocks, splits)) / 3e6 : 0);
}

// Workgroups per query block. A few new tokens over a long prefix leave most
// units idle (300 tokens over 24300, G = 4, 8 KV heads: 80 workgroups). With
// the keys of every block shared by several workgroups the rounds are shorter
// and end more evenly; the count with the shortest rounds is taken, of those
// that leave a split at least 8 tiles, where the call is estimated to gain 5%.
// Measured over 43 shapes and both head_dims, every split count forced in turn
// (us, unsplit / taken; best where another count is): head_dim 128, 8 KV heads,
// G = 4: 300 tokens over 24300 317 / 167 (3 splits), 32 311 / 38.6, 1100 over
// 32768 1027 / 765 (5), 256 over 8000 113 / 57 (4), 500 over 4096 69 / 61; G =
// 2: 700 over 12000, twice, stays unsplit (189; 198 in 4), 5000 uncached tokens
// of 4 heads too (92; 106 in 2). head_dim 64: 300 over 24300 261 / 109, 1100
// over 32768 727 / 491 (490), 500 over 4096 55 / 42, the 5000 stay at 67 (77 in
// 2), the 700 take 128 (134 unsplit). With one round and a little, or many
// rounds, nothing is gained and nothing split (1024 over 32768: 639; 650 in 2).
int64_t plan_splits(const comem_decode_attn_plan& p, int64_t batch, int64_t max_q_len, int64_t max_ctx_len,
                    size_t bytes) {
  constexpr int64_t kMinTiles = 8, kMaxSplits = 64;
  const int64_t pairs = batch * p.cfg.num_kv_heads;
  const int64_t blocks = ceil_div(max_q_len, comem::kPrefillRows / group_of(p.cfg)), items = pairs * blocks;
  const int64_t tiles = ceil_div(max_ctx_len, comem::kPrefillTileKeys);
  if (items >= 8 * p.num_cus) return 1;  // rounds are many, the last one is a small part
  int64_t best = 1;
  double least = 0;
  for (int64_t n = 1; n <= kMaxSplits && n * kMinTiles <= tiles; ++n) {
    if (split_bytes(p, items, n) > bytes) break;
    double us = 1.2 * static_cast<double>(ceil_div(items * n, p.num_cus) * ceil_div(tiles, n));
    if (n > 1) us += 6 + 2 * static_cast<double>(split_bytes(p, items, n)) / 3e6;
    if (n == 1 || us < 0.95 * least) {
      best = n;
      least = us;
    }
  }
  if (best > 1 && prefill_us(p, pairs, blocks, max_ctx_len, best) > 0.95 * prefill_us(p, pairs, blocks, max_ctx_len, 1))
    return 1;
  return best;
}

comem_status launch_prefill(const comem_decode_attn_plan& p, const comem::PrefillParams& a, bool paged,
                            int32_t batch, int32_t max_q_len, void* workspace, size_t workspace_bytes, void* stream) {
  const int64_t blocks = ceil_div(max_q_len, a.tokens_per_block);
  comem::PrefillParams args = a;
  args.blocks = static_cast<int32_t>(blocks);
  args.splits = static_cast<int32_t>(
      plan_splits(p, batch, max_q_len, a.max_ctx, workspace == nullptr ? 0 : workspace_bytes));
  comem::PrefillKernelFn fn =
      comem::select_prefill_kernel(p.cfg.head_dim, paged ? a.page_mask + 1 : 0, args.splits > 1);
  comem::PrefillKernelFn merge = comem::select_prefill_merge_kernel(p.cfg.head_dim);
  if (fn == nullptr || merge == nullptr) return COMEM_ERR_UNSUPPORTED;
  if (args.splits > 1) {
    const size_t rows = static_cast<size_t>(batch * p.cfg.num_kv_heads * blocks) * static_cast<size_t>(args.splits) *
                        comem::kPrefillRows;
    args.lse_part = static_cast<float*>(workspace);
    args.o_part = reinterpret_cast<float*>(static_cast<char*>(workspace) + align256(rows * 4));
  }
  void* argv[] = {&args};
  const unsigned heads = static_cast<unsigned>(p.cfg.num_kv_heads), seqs = static_cast<unsigned>(batch);
  hipError_t err = hipLaunchKernel(reinterpret_cast<const void*>(fn),
                                   dim3(static_cast<unsigned>(blocks * args.splits), heads, seqs),
                                   dim3(comem::kPrefillThreads), argv, 0, static_cast<hipStream_t>(stream));
  if (err == hipSuccess && args.splits > 1) {
    err = hipLaunchKernel(
        reinterpret_cast<const void*>(merge),
        dim3(static_cast<unsigned>(blocks * (comem::kPrefillRows / comem::kPrefillMergeRows)), heads, seqs),
        dim3(comem::kPrefillMergeThreads), argv, 0, static_cast<hipStream_t>(stream));
  }
  return err == hipSuccess ? COMEM_OK : COMEM_ERR_HIP;
}

}  // namespace

extern "C" {

comem_status comem_prefill_attn_workspace(const comem_decode_attn_plan* plan, int32_t batch, int32_t max_q_len,
                                          int64_t max_ctx_len, size_t* workspace_bytes_out) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  if (workspace_bytes_out == nullptr) return COMEM_ERR_NULL_POINTER;
  *workspace_bytes_out = 0;
  if (p->cfg.dtype != COMEM_BF16) return COMEM_ERR_UNSUPPORTED;
  const comem_status st = check_bounds(*p, batch, max_q_len, max_ctx_len);
  if (st != COMEM_OK || prefill_is_empty(batch, max_q_len)) return st;
  const int64_t items =
      static_cast<int64_t>(batch) * p->cfg.num_kv_heads * ceil_div(max_q_len, comem::kPrefillRows / group_of(p->cfg));
  *workspace_bytes_out = split_bytes(*p, items, plan_splits(*p, batch, max_q_len, max_ctx_len, SIZE_MAX));
  return COMEM_OK;
}

comem_status comem_prefill_attn_split(const comem_decode_attn_plan* plan, const void* q, const int64_t* q_start,
                                      const int32_t* q_lens, int32_t max_q_len, const void* k, const void* v,
                                      int64_t stride_token, int64_t stride_head, const int64_t* seq_start,
                                      const int32_t* ctx_lens, int32_t batch, int64_t max_ctx_len, float* out,
                                      float* lse, void* workspace, size_t workspace_bytes, void* hip_stream) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  comem::PrefillParams a;
  comem_status st = prepare_prefill(*p, q, q_start, q_lens, max_q_len, k, v, stride_token, stride_head, ctx_lens,
                                    batch, max_ctx_len, out, lse, workspace, a);
  if (st != COMEM_OK || prefill_is_empty(batch, max_q_len)) return st;
  if (seq_start == nullptr) return COMEM_ERR_NULL_POINTER;
  if (!aligned(seq_start, 8)) return COMEM_ERR_MISALIGNED;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  a.seq_start = seq_start;
  return launch_prefill(*p, a, false, batch, max_q_len, workspace, workspace_bytes, hip_stream);
}

comem_status comem_prefill_attn(const comem_decode_attn_plan* plan, const void* q, const int64_t* q_start,
                                const int32_t* q_lens, int32_t max_q_len, const void* k, const void* v,
                                int64_t stride_token, int64_t stride_head, const int64_t* seq_start,
                                const int32_t* ctx_lens, int32_t batch, int64_t max_ctx_len, float* out,
                                float* lse, void* hip_stream) {
  return comem_prefill_attn_split(plan, q, q_start, q_lens, max_q_len, k, v, stride_token, stride_head, seq_start,
                                  ctx_lens, batch, max_ctx_len, out, lse, nullptr, 0, hip_stream);
}

comem_status comem_prefill_attn_split_paged(const comem_decode_attn_plan* plan, const void* q, const int64_t* q_start,
                                            const int32_t* q_lens, int32_t max_q_len, const void* k_pages,
                                            const void* v_pages, int64_t stride_page, int64_t stride_token,
                                            int64_t stride_head, int32_t page_size, int64_t num_pages,
                                            const int32_t* block_table, int32_t max_pages_per_seq,
                                            const int32_t* ctx_lens, int32_t batch, int64_t max_ctx_len, float* out,
                                            float* lse, void* workspace, size_t workspace_bytes, void* hip_stream) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  comem::PrefillParams a;
  comem_status st = prepare_prefill(*p, q, q_start, q_lens, max_q_len, k_pages, v_pages, stride_token, stride_head,
                                    ctx_lens, batch, max_ctx_len, out, lse, workspace, a);
  if (st != COMEM_OK || prefill_is_empty(batch, max_q_len)) return st;
  st = validate_paged(*p, stride_page, page_size, num_pages, block_table, max_pages_per_seq, max_ctx_len);
  if (st != COMEM_OK) return st;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  a.block_table = block_table;
  a.stride_page = stride_page * elem_bytes(p->cfg);
  a.max_pages = max_pages_per_seq;
  a.page_shift = log2_of(page_size);
  a.page_mask = page_size - 1;
  a.num_pages = num_pages;
  return launch_prefill(*p, a, true, batch, max_q_len, workspace, workspace_bytes, hip_stream);
}

comem_status comem_prefill_attn_paged(const comem_decode_attn_plan* plan, const void* q, const int64_t* q_start,
                                      const int32_t* q_lens, int32_t max_q_len, const void* k_pages,
                                      const void* v_pages, int64_t stride_page, int64_t stride_token,
                                      int64_t stride_head, int32_t page_size, int64_t num_pages,
                                      const int32_t* block_table, int32_t max_pages_per_seq,
                                      const int32_t* ctx_lens, int32_t batch, int64_t max_ctx_len, float* out,
                                      float* lse, void* hip_stream) {
  return comem_prefill_attn_split_paged(plan, q, q_start, q_lens, max_q_len, k_pages, v_pages, stride_page,
                                        stride_token, stride_head, page_size, num_pages, block_table,
                                        max_pages_per_seq, ctx_lens, batch, max_ctx_len, out, lse, nullptr, 0,
                                        hip_stream);
}

}  // extern "C"
