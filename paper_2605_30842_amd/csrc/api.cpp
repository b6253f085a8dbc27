// Host side of the decode-attention C ABI: argument validation (always before
// any HIP call), split planning, kernel selection and launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>

#include "attn_common.h"
#include "comem_decode_attn.h"
#include "kv_append.h"
#include "noalloc.h"
#include "plan.h"

namespace comem {
using KernelFn = void (*)(AttnParams);
using QueueKernelFn = void (*)(AttnParams, int);
KernelFn select_mfma_kernel(int head_dim, bool paged, int page_size, bool fp8);
QueueKernelFn select_mfma_queue_kernel(int head_dim, bool paged, int page_size, bool fp8);
QueueKernelFn select_mfma_balanced_kernel(int head_dim, bool paged, int page_size, bool fp8);
int mfma_max_queue_batch();
KernelFn select_valu_kernel(bool bf16, int head_dim, int group, bool paged);
}  // namespace comem

using namespace comem::host;

namespace {

constexpr int kAssumedCUs = 256;                        // gfx950 (MI355X) without a device query
constexpr int64_t kTargetWgsPerCu = 2;                  // workgroups per compute unit for one full round
constexpr int kQueueWgsPerCu = 2;                       // resident workgroups per compute unit (MFMA kernel)
constexpr int64_t kMinRangeTokens = 64;                 // shortest range of the balanced form
constexpr int64_t kMaxBalancedTiles = int64_t{1} << 23; // 32-token tiles the balanced form counts exactly
constexpr int64_t kMaxSplitPages = 2048;                // block-table entries of a configured split, upper bound
constexpr int64_t kMinChunk = 64;                       // tokens per split, lower bound
constexpr int64_t kMaxChunk = 2048;                     // tokens per split, upper bound (auto plan)

bool uses_mfma(const comem_decode_attn_plan& p);

// A workspace starts with the two work-queue counters and the device error
// word, then come the tickets [max_batch * Hkv], then the partial results.
constexpr int kCounterWords = 3;
constexpr int kErrorWord = 2;

// Words between two tickets (log2). Atomics on one 128-byte line take their
// turns, whichever word they name: with the tickets of 8 heads side by side,
// the 256 workgroups of a batch-1 call waited 1.2 us for their ticket, with
// a line each 0.4 us. So a call spreads its tickets as far as the region at
// the workspace's start has room for. All of that region is zero between
// calls, however far apart the last call's tickets lay.
constexpr int kMaxTicketShift = 5;

// Words before the first ticket.
int32_t ticket_base(int shift) { return std::max(shift > 0 ? 4 : kCounterWords, 1 << shift); }

size_t ticket_region_bytes(int64_t tickets, int shift) {
  return align256((static_cast<size_t>(ticket_base(shift)) + (static_cast<size_t>(tickets) << shift)) * 4);
}

int ticket_shift(int64_t tickets, size_t bytes) {
  int shift = kMaxTicketShift;
  while (shift > 0 && ticket_region_bytes(tickets, shift) > bytes) --shift;
  return shift;
}

// The region of a plan: a line for every ticket where all of them then fit
// the counter region of the allocation-free call (a plan it took with dense
// tickets it takes with spread ones too), closer for more sequences, whose
// workgroups reach their tickets at different times. With a configured
// chunk_tokens the tickets of max_batch sequences lie side by side: such a
// call is refused when its workspace is too small, so the size stays the one
// that the partial results need.
size_t plan_ticket_bytes(int64_t tickets, bool planned_chunk) {
  return ticket_region_bytes(tickets, planned_chunk ? ticket_shift(tickets, comem::kScratchTicketBytes) : 0);
}

// Bytes of that region in a workspace of ws_bytes. A smaller one than the plan
// reports gives up the room between tickets first, so that it holds the
// partial results of every call that dense tickets leave room for. The size
// must not depend on the call: a region that one call counts in would hold
// another's partial results.
size_t counter_region(const comem_decode_attn_plan& p, size_t ws_bytes) {
  const size_t least = p.dense_bytes + p.partial_bytes;
  return ws_bytes < least ? p.dense_bytes : std::min(p.ticket_bytes, p.dense_bytes + (ws_bytes - least) / 256 * 256);
}

// Where a call's tickets lie and its partial results begin.
struct Counters {
  size_t bytes;
  int shift;
  Counters(const comem_decode_attn_plan& p, int64_t batch, size_t region)
      : bytes(region), shift(ticket_shift(batch * p.cfg.num_kv_heads, region)) {}
};

bool debug_checks(const comem_decode_attn_plan& p) { return (p.cfg.flags & COMEM_FLAG_DEBUG_CHECKS) != 0; }

// With debug checks the error word lives in the workspace, so one is needed.
comem_status check_debug_workspace(const comem_decode_attn_plan& p, const void* workspace, size_t ws_bytes) {
  if (!debug_checks(p)) return COMEM_OK;
  if (workspace == nullptr) return COMEM_ERR_NULL_POINTER;
  return ws_bytes < p.dense_bytes ? COMEM_ERR_WORKSPACE_TOO_SMALL : COMEM_OK;
}

// Workspace bytes for `slots` (sequence, split) partial results: counters and
// tickets, then per-head lse values, then per-head partial outputs.
size_t slots_workspace_bytes(const comem_decode_attn_plan& p, size_t counter_bytes, int64_t slots) {
  const size_t rows = static_cast<size_t>(slots) * static_cast<size_t>(p.cfg.num_q_heads);
  return counter_bytes + align256(rows * 4) + rows * static_cast<size_t>(p.cfg.head_dim) * 4;
}

// Workspace bytes a call with `batch` sequences and `splits` splits needs.
// A single split writes the output directly and touches no workspace.
size_t call_workspace_bytes(const comem_decode_attn_plan& p, const Counters& c, int64_t batch, int64_t splits) {
  return splits <= 1 ? 0 : slots_workspace_bytes(p, c.bytes, batch * splits);
}

// Largest planned split, in tokens, of a paged call with pages of `page_size`
// tokens (a multiple of 32): it spans no more entries than a configured one
// may.
int64_t mfma_page_cap(int64_t page_size) {
  return std::max<int64_t>(32, (kMaxSplitPages - 2) * page_size / 32 * 32);
}

// Ranges of the balanced form (decode_mfma_balanced_kernel), for each KV head:
// one workgroup per compute unit; two where one would leave more than 15% of
// the units idle (43 heads: 5 ranges on 215 of 256).
int64_t max_ranges(const comem_decode_attn_plan& p) {
  const int64_t heads = p.cfg.num_kv_heads, one = p.num_cus / heads;
  return 20 * one * heads >= 17 * p.num_cus ? one : std::max<int64_t>(1, 2 * p.num_cus / heads);
}

// With many KV heads a head has so few ranges that they can't even out: the
// unequal sums of a unit's or an XCD's neighbours show. us, splits / ranges, G
// = 1: 4 x 8192 tokens, 40 heads D = 128 122 / 115, 64 178 / 172, 80 225 /
// 247, D = 64 96 139 / 154, 160 233 / 307; one sequence of 8192, 40 heads D =
// 128 38.5 / 31.3, 96 70.8 / 70.7, 128 94 / 87, 300 of 4096 D = 64 59 / 70,
// FP8 160 of 8192 72 / 80.
bool can_balance(const comem_decode_attn_plan& p, int64_t batch) {
  return uses_mfma(p) && p.cfg.variant != COMEM_VARIANT_MFMA_GRID && p.cfg.chunk_tokens == 0 &&
         batch <= comem::mfma_max_queue_batch() && p.cfg.num_kv_heads <= (batch == 1 ? 128 : 64);
}

// Workspace bytes of the balanced form past the tickets: two partial-result
// slots per range and KV head.
size_t balanced_bytes(const comem_decode_attn_plan& p) {
  const size_t rows = 2 * static_cast<size_t>(max_ranges(p)) * static_cast<size_t>(p.cfg.num_q_heads);
  return align256(rows * 4) + rows * static_cast<size_t>(p.cfg.head_dim) * 4;
}

// (Shortest piece worth a split, in 32-token tiles)^2 per tile of context
// and sequence: with a us per token on one CU and m us per part to merge, a
// length n splits best into pieces of sqrt(m n / a). From sweeps of batch-1
// calls (us): a = 0.0045 + 1.1e-5 per byte of a token's K and V of one head
// (0.0102 at 512 bytes, 0.006 at 256), m = 0.02 + 9e-5 per output value of
// the group (0.065 at G D = 512, 0.2 at 2048).
float split_coefficient(const comem_decode_attn_plan& p) {
  const float token_bytes = 2.f * static_cast<float>(p.cfg.head_dim * elem_bytes(p.cfg));
  const float a = 0.0045f + 1.1e-5f * token_bytes;
  const float m = 0.02f + 9e-5f * static_cast<float>(group_of(p.cfg) * p.cfg.head_dim);
  return m / (32.f * a);
}

// Most tokens of a sequence that are better left to one workgroup than shared
// by n: a second part costs a ticket and a merge, about 3 us (5 with the 2048
// output values of G = 16, D = 128), and n parts save (n - 1) / n of the time
// per token. Swept over one sequence and 2-30, 1-8 KV heads, G = 1, 4 and 16,
// contexts of 40 to 800 tokens (us, whole / split; one sequence of 8 heads, G =
// 4): 512-byte tokens 100 tokens 5.5 / 6.5, 280 6.9 / 6.6, 430 8.0 / 6.8; FP8
// 100 4.6 / 6.5, 430 6.4 / 6.7, 640 7.5 / 6.9; G = 16 430 8.7 / 8.6, FP8 640 7.8
// / 8.7; in two parts (16 sequences) 640 12.7 / 13.0, FP8 640 9.1 / 9.9.
int64_t whole_tokens(const comem_decode_attn_plan& p, int64_t n) {
  if (n <= 1) return kMaxContext;
  const int64_t tokens = p.cfg.head_dim * elem_bytes(p.cfg) <= 128 ? 440 : 280;
  return (group_of(p.cfg) * p.cfg.head_dim >= 2048 ? 3 * tokens / 2 : tokens) * n / (n - 1);
}

// Tokens per split of a long call in the grid and work-queue forms, from the
// host-side bounds (the device-side lengths are never read on the host). Splits of
// 4096 tokens keep contexts of 128k and more at <= 32 splits; otherwise 2048
// if that still leaves >= 16 work items per resident workgroup, else 1024.
// Smaller items end the work queue more evenly (the last items handed out
// finish at nearly the same time) at the cost of one more partial result
// per item; at 8 items of 2048 tokens per workgroup the even end still wins.
int64_t long_chunk(const comem_decode_attn_plan& p, int64_t batch, int64_t L) {
  if (L >= 32 * 4096) return 4096;
  const int64_t resident = static_cast<int64_t>(kQueueWgsPerCu) * p.num_cus;
  if (batch * p.cfg.num_kv_heads * ceil_div(L, 2048) >= 16 * resident) return 2048;
  return 1024;
}

// Long calls of several sequences take the balanced form, short ones one
// workgroup per split. The balanced kernel starts 1-2 us later, and a range
// pays for every piece it holds; its equal shares win that back once ranges
// are long.
//
// With fewer pairs of sequence and head than compute units, swept over 2-128
// sequences, 2-8 KV heads, bf16 and FP8, head_dim 64 and 128, lengths from
// 0.15, 0.5 and 1 of the bound up (best splits / balanced): at 900-1000 tokens
// of bound per range and sequence 0.87-1.05, at 1365 0.94-1.27, from 2700
// 0.97-1.35.
//
// With a pair for every unit, short calls run whole sequences, and a call then
// takes as long as its longest one on one unit (0.01 us a token) unless the
// others keep the units busy as long: with few sequences per range the line
// rises with them. With many, a range's pieces even out by themselves and the
// line falls towards the length at which whole sequences of about equal length
// stop being faster. Swept over 12-512 sequences, 2-32 KV heads, bounds 1100
// to 8192, lengths equal, uniform from 0.1 or 0.5 of the bound, and one or a
// sixteenth of them at the bound and the others at 0.02-0.1 of it (us, whole
// / balanced, equal lengths; uniform from 0.1; one long and the others a
// tenth): 32 x 8 heads 1100 tokens 25.0 / 25.8; 18.8 / 20.1; 16.8 / 13.0, 2000
// 39.9 / 41.4; 30.7 / 30.6; 26.0 / 14.9, 3100 64.1 / 65.2; 43.4 / 38.8; 37.6 /
// 17.0. 128 x 8 2048 168 / 166; 110 / 105; 32.1 / 32.9, 3100 244 / 246; 163 /
// 152; 52.6 / 45.5. 256 x 8 2048 326 / 324; 202 / 197; 39 / 55, 3100 482 / 485;
// 298 / 282; 64 / 80. Light tokens cost a range's pieces relatively more.
bool long_call(const comem_decode_attn_plan& p, int64_t batch, int64_t L) {
  const int64_t ranges = max_ranges(p);
  if (batch * p.cfg.num_kv_heads < p.num_cus) return batch * L >= 1200 * (ranges + batch);
  const bool light = p.cfg.head_dim * elem_bytes(p.cfg) <= 128;
  return L >= (light ? 1500 : 1000) + 260 * batch / ranges || batch * L >= (light ? 2048 : 1600) * (ranges + batch);
}

// Tokens per split of a short call: one split per compute unit, none shorter
// than a piece worth its merge; a whole sequence once the (sequence, head)
// pairs fill the chip (64 x 1024 tokens: 32.5 us; 128 x 2048: 120.9, 126 at
// 1024). Otherwise at most 1024: the bound may be far above the lengths, and
// one longer split would run alone.
int64_t short_chunk(const comem_decode_attn_plan& p, int64_t batch, int64_t L) {
  const int64_t pairs = batch * p.cfg.num_kv_heads;
  if (pairs >= p.num_cus) return ceil_div(L, 32) * 32;
  const int64_t parts = p.num_cus / pairs;
  if (parts > 1 && L <= whole_tokens(p, parts)) return ceil_div(L, 32) * 32;
  const int64_t share = ceil_div(L, parts);
  const double piece = 32.0 * std::sqrt(split_coefficient(p) * static_cast<double>(ceil_div(L, 32)));
  const int64_t chunk = std::max({kMinRangeTokens, share, static_cast<int64_t>(std::ceil(piece))});
  return std::min<int64_t>(1024, ceil_div(chunk, 32) * 32);
}

// Choose tokens per split and the split count for one call. page_size is 0
// for a contiguous cache; for a paged one the matrix-core kernel's planned
// splits stay within kMaxSplitPages entries.
comem_status plan_call(const comem_decode_attn_plan& p, const Counters& c, int64_t batch, int64_t max_ctx,
                       int64_t page_size, size_t ws_bytes, int64_t* chunk_out, int64_t* splits_out) {
  const int64_t L = max_ctx > 0 ? max_ctx : 1;
  const int64_t cap = page_size > 0 && uses_mfma(p) ? mfma_page_cap(page_size) : INT64_MAX;
  int64_t chunk;
  if (p.cfg.chunk_tokens > 0) {
    chunk = p.cfg.chunk_tokens;
    if (call_workspace_bytes(p, c, batch, ceil_div(L, chunk)) > ws_bytes) return COMEM_ERR_WORKSPACE_TOO_SMALL;
  } else {
    if (uses_mfma(p)) {
      const int64_t most = std::min(long_chunk(p, batch, L), cap);
      chunk = long_call(p, batch, L) ? most : std::min(short_chunk(p, batch, L), cap);
      // A workspace too small for these splits gets those of a long call.
      if (call_workspace_bytes(p, c, batch, ceil_div(L, chunk)) > ws_bytes) chunk = std::max(chunk, most);
    } else {
      const int64_t target = kTargetWgsPerCu * p.num_cus;
      const int64_t per = ceil_div(batch * p.cfg.num_kv_heads * L, target);
      chunk = kMinChunk;
      while (chunk < per && chunk < kMaxChunk) chunk *= 2;
    }
    while (call_workspace_bytes(p, c, batch, ceil_div(L, chunk)) > ws_bytes) {
      if (chunk >= L || chunk * 2 > cap) {
        if (L > cap) return COMEM_ERR_WORKSPACE_TOO_SMALL;
        chunk = cap;  // a whole sequence needs no partial results
        break;
      }
      chunk *= 2;
    }
  }
  *chunk_out = chunk;
  *splits_out = ceil_div(L, chunk);
  return COMEM_OK;
}

comem_status validate_config(const comem_decode_attn_config& c) {
  if (c.num_q_heads <= 0 || c.num_kv_heads <= 0 || c.num_q_heads % c.num_kv_heads != 0)
    return COMEM_ERR_INVALID_SHAPE;
  if (c.num_kv_heads > kGridYZLimit) return COMEM_ERR_INVALID_SHAPE;
  const int G = group_of(c);
  if (G != 1 && G != 2 && G != 4 && G != 8 && G != 16) return COMEM_ERR_UNSUPPORTED;
  if (c.head_dim != 64 && c.head_dim != 128) return COMEM_ERR_UNSUPPORTED;
  if (c.dtype != COMEM_F32 && c.dtype != COMEM_BF16 && c.dtype != COMEM_FP8_E4M3) return COMEM_ERR_UNSUPPORTED;
  if (!std::isfinite(c.scale) || !(c.scale > 0.f)) return COMEM_ERR_INVALID_SHAPE;
  if (c.max_batch <= 0 || c.max_batch > kGridYZLimit) return COMEM_ERR_INVALID_SHAPE;
  if (c.max_ctx_len <= 0 || c.max_ctx_len > kMaxContext) return COMEM_ERR_INVALID_SHAPE;
  if (c.chunk_tokens < 0 || c.chunk_tokens % 32 != 0 || c.chunk_tokens > kMaxContext)
    return COMEM_ERR_INVALID_SHAPE;
  if (c.variant != COMEM_VARIANT_AUTO && c.variant != COMEM_VARIANT_VALU && c.variant != COMEM_VARIANT_MFMA &&
      c.variant != COMEM_VARIANT_MFMA_GRID)
    return COMEM_ERR_UNSUPPORTED;
  if ((c.flags & ~COMEM_FLAG_DEBUG_CHECKS) != 0) return COMEM_ERR_UNSUPPORTED;
  if ((c.variant == COMEM_VARIANT_MFMA || c.variant == COMEM_VARIANT_MFMA_GRID) && c.dtype == COMEM_F32)
    return COMEM_ERR_UNSUPPORTED;
  if (c.dtype == COMEM_FP8_E4M3) {
    if (c.variant == COMEM_VARIANT_VALU) return COMEM_ERR_UNSUPPORTED;
    if (!std::isfinite(c.k_scale) || !(c.k_scale > 0.f) || !std::isfinite(c.v_scale) || !(c.v_scale > 0.f))
      return COMEM_ERR_INVALID_SHAPE;
  }
  return COMEM_OK;
}

bool uses_mfma(const comem_decode_attn_plan& p) {
  return p.cfg.variant == COMEM_VARIANT_MFMA || p.cfg.variant == COMEM_VARIANT_MFMA_GRID ||
         (p.cfg.variant == COMEM_VARIANT_AUTO && p.cfg.dtype != COMEM_F32);
}

// The work-queue form of the matrix-core kernel keeps two counters beside the
// tickets, so it needs a workspace (of at least that region).
bool uses_queue(const comem_decode_attn_plan& p, const Counters& c, int64_t batch, const void* workspace,
                size_t ws_bytes) {
  return uses_mfma(p) && p.cfg.variant != COMEM_VARIANT_MFMA_GRID && batch <= comem::mfma_max_queue_batch() &&
         workspace != nullptr && ws_bytes >= c.bytes;
}

// The balanced form of the matrix-core kernel needs a workspace for its partial
// results and a token count that its 24-bit arithmetic holds.
bool uses_balanced(const comem_decode_attn_plan& p, const Counters& c, int64_t batch, int64_t max_ctx,
                   const void* workspace, size_t ws_bytes) {
  return can_balance(p, batch) && (batch == 1 || long_call(p, batch, max_ctx)) && workspace != nullptr &&
         ws_bytes >= c.bytes + balanced_bytes(p) &&
         batch * (ceil_div(max_ctx + 1, 32) + comem::kPieceTilesLight) < kMaxBalancedTiles;
}

comem_status launch_balanced(const comem_decode_attn_plan& p, bool paged, comem::AttnParams& a, int64_t batch,
                             void* stream) {
  // No more ranges than the call's bound can fill.
  a.ranges = static_cast<int32_t>(
      std::min(max_ranges(p), batch * ceil_div(std::max<int64_t>(a.max_ctx, 1), kMinRangeTokens)));
  a.split_coef = split_coefficient(p) / static_cast<float>(batch);
  const unsigned heads = static_cast<unsigned>(p.cfg.num_kv_heads), ranges = static_cast<unsigned>(a.ranges);
  const int page = a.page_mask + 1;
  hipError_t err;
  if (batch == 1) {
    comem::KernelFn fn = comem::select_mfma_kernel(p.cfg.head_dim, paged, page, is_fp8(p.cfg));
    if (fn == nullptr) return COMEM_ERR_UNSUPPORTED;
    a.num_splits = a.ranges;
    a.whole_tiles = static_cast<int32_t>(whole_tokens(p, max_ranges(p)) / 32);
    void* args[] = {&a};
    err = hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3(ranges, heads), dim3(comem::kThreads), args, 0,
                          static_cast<hipStream_t>(stream));
  } else {
    comem::QueueKernelFn fn = comem::select_mfma_balanced_kernel(p.cfg.head_dim, paged, page, is_fp8(p.cfg));
    if (fn == nullptr) return COMEM_ERR_UNSUPPORTED;
    int nb = static_cast<int>(batch);
    void* args[] = {&a, &nb};
    err = hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3(heads, ranges), dim3(comem::kThreads), args, 0,
                          static_cast<hipStream_t>(stream));
  }
  return err == hipSuccess ? COMEM_OK : COMEM_ERR_HIP;
}

comem_status launch(const comem_decode_attn_plan& p, bool paged, comem::AttnParams& a, int64_t batch,
                    int64_t splits, bool queue, void* stream) {
  const bool bf16 = p.cfg.dtype == COMEM_BF16;
  const int64_t items = batch * p.cfg.num_kv_heads * splits;
  const int64_t resident = static_cast<int64_t>(kQueueWgsPerCu) * p.num_cus;
  // With no more (nominal) items than resident workgroups every item gets its
  // own workgroup anyway, and the grid form saves the queue's prologue; whole
  // sequences (short calls with a pair for every compute unit) start without it
  // too. Splits past the resident ones would wait in the grid for a unit of
  // their own XCD (2 x 8192 tokens, 33 heads, FP8: 30.1 us, queued 25.7).
  const bool whole = p.cfg.chunk_tokens == 0 && !long_call(p, batch, a.max_ctx) &&
                     batch * p.cfg.num_kv_heads >= p.num_cus;
  if (queue && items > resident && !whole) {
    comem::QueueKernelFn qfn = comem::select_mfma_queue_kernel(p.cfg.head_dim, paged, a.page_mask + 1, is_fp8(p.cfg));
    if (qfn == nullptr) return COMEM_ERR_UNSUPPORTED;
    dim3 grid(static_cast<unsigned>(items < resident ? items : resident));
    dim3 block(comem::kThreads);
    int nb = static_cast<int>(batch);
    void* args[] = {&a, &nb};
    const hipError_t err = hipLaunchKernel(reinterpret_cast<const void*>(qfn), grid, block, args, 0,
                                           static_cast<hipStream_t>(stream));
    return err == hipSuccess ? COMEM_OK : COMEM_ERR_HIP;
  }
  comem::KernelFn fn = uses_mfma(p) ? comem::select_mfma_kernel(p.cfg.head_dim, paged, a.page_mask + 1, is_fp8(p.cfg))
                                    : comem::select_valu_kernel(bf16, p.cfg.head_dim, group_of(p.cfg), paged);
  if (fn == nullptr) return COMEM_ERR_UNSUPPORTED;
  dim3 grid(static_cast<unsigned>(splits), static_cast<unsigned>(p.cfg.num_kv_heads),
            static_cast<unsigned>(batch));
  dim3 block(comem::kThreads);
  void* args[] = {&a};
  const hipError_t err = hipLaunchKernel(reinterpret_cast<const void*>(fn), grid, block, args, 0,
                                         static_cast<hipStream_t>(stream));
  return err == hipSuccess ? COMEM_OK : COMEM_ERR_HIP;
}

// Checks of an append call; fills the kernel arguments shared by both layouts.
comem_status prepare_append(const comem_decode_attn_plan& p, const void* new_k, const void* new_v, void* k,
                            void* v, int64_t stride_token, int64_t stride_head, const int32_t* ctx_lens,
                            int32_t batch, int64_t max_ctx_len, comem::AppendParams& a) {
  if (batch < 0 || batch > p.cfg.max_batch) return COMEM_ERR_INVALID_SHAPE;
  if (max_ctx_len < 0 || max_ctx_len > p.cfg.max_ctx_len) return COMEM_ERR_INVALID_SHAPE;
  if (batch == 0) return COMEM_OK;
  if (new_k == nullptr || new_v == nullptr || k == nullptr || v == nullptr || ctx_lens == nullptr)
    return COMEM_ERR_NULL_POINTER;
  if (stride_token <= 0 || stride_head < 0) return COMEM_ERR_INVALID_SHAPE;
  if (p.cfg.num_kv_heads > 1 && stride_head == 0) return COMEM_ERR_INVALID_SHAPE;
  const int64_t e = elem_bytes(p.cfg);
  if ((stride_token * e) % 16 != 0 || (stride_head * e) % 16 != 0) return COMEM_ERR_MISALIGNED;
  if (!aligned(new_k, 16) || !aligned(new_v, 16) || !aligned(k, 16) || !aligned(v, 16))
    return COMEM_ERR_MISALIGNED;
  std::memset(&a, 0, sizeof(a));
  a.new_k = static_cast<const char*>(new_k);
  a.new_v = static_cast<const char*>(new_v);
  a.k = static_cast<char*>(k);
  a.v = static_cast<char*>(v);
  a.ctx_lens = ctx_lens;
  a.stride_token = stride_token * e;
  a.stride_head = stride_head * e;
  a.max_ctx_len = max_ctx_len;
  a.num_kv_heads = p.cfg.num_kv_heads;
  a.chunks_per_head = static_cast<int32_t>(p.cfg.head_dim * e / 16);
  return COMEM_OK;
}

comem_status launch_append(const comem::AppendParams& a, bool paged, int32_t batch, void* stream) {
  comem::AppendParams args = a;
  void* argv[] = {&args};
  const hipError_t err = hipLaunchKernel(reinterpret_cast<const void*>(comem::select_append_kernel(paged)),
                                         dim3(static_cast<unsigned>(batch)), dim3(comem::kThreads), argv, 0,
                                         static_cast<hipStream_t>(stream));
  return err == hipSuccess ? COMEM_OK : COMEM_ERR_HIP;
}

void fill_common(const comem_decode_attn_plan& p, comem::AttnParams& a, const void* q, const void* k,
                 const void* v, int64_t stride_token, int64_t stride_head, const int32_t* ctx_lens,
                 float* out, float* lse, void* workspace, int64_t batch, int64_t max_ctx_len, int64_t chunk,
                 int64_t splits, bool queue, bool balanced, const Counters& c) {
  const int64_t e = elem_bytes(p.cfg);
  std::memset(&a, 0, sizeof(a));
  a.max_ctx = static_cast<int32_t>(max_ctx_len);
  if (debug_checks(p)) a.errors = static_cast<uint32_t*>(workspace) + kErrorWord;
  a.q = static_cast<const char*>(q);
  a.k = static_cast<const char*>(k);
  a.v = static_cast<const char*>(v);
  a.out = out;
  a.lse = lse;
  a.ctx_lens = ctx_lens;
  a.stride_token = stride_token * e;
  a.stride_head = stride_head * e;
  a.num_q_heads = p.cfg.num_q_heads;
  a.num_kv_heads = p.cfg.num_kv_heads;
  a.group = group_of(p.cfg);
  a.chunk = static_cast<int32_t>(chunk);
  a.num_splits = static_cast<int32_t>(splits);
  // An FP8 cache's K scale multiplies every score; its V scale every output.
  a.scale_log2 = p.cfg.scale * (is_fp8(p.cfg) ? p.cfg.k_scale : 1.f) * 1.4426950408889634f;
  a.out_scale = is_fp8(p.cfg) ? p.cfg.v_scale : 1.f;
  a.queue_slot = -ticket_base(c.shift);
  a.ticket_shift = c.shift;
  if (splits > 1 || queue || balanced) {
    char* ws = static_cast<char*>(workspace);
    const size_t slots = (balanced ? 2 * static_cast<size_t>(max_ranges(p))
                                   : static_cast<size_t>(batch) * static_cast<size_t>(splits)) *
                         static_cast<size_t>(p.cfg.num_q_heads);
    a.tickets = reinterpret_cast<uint32_t*>(ws) + ticket_base(c.shift);
    a.lse_part = reinterpret_cast<float*>(ws + c.bytes);
    a.o_part = reinterpret_cast<float*>(ws + c.bytes + align256(slots * 4));
  }
}

// The attention calls, with or without the fused append of the new rows.
comem_status decode_contiguous(const comem_decode_attn_plan* plan, const void* q, const void* new_k,
                               const void* new_v, const void* k, const void* v, int64_t stride_token,
                               int64_t stride_head, const int64_t* seq_start, const int32_t* ctx_lens,
                               int32_t batch, int64_t max_ctx_len, float* out, float* lse, void* workspace,
                               size_t workspace_bytes, void* hip_stream, bool fused, bool scratch = false) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  comem_status st = validate_common(*p, q, k, v, stride_token, stride_head, ctx_lens, batch, max_ctx_len,
                                    out, lse, workspace);
  if (st != COMEM_OK || batch == 0) return st;
  if (seq_start == nullptr) return COMEM_ERR_NULL_POINTER;
  if (!aligned(seq_start, 8)) return COMEM_ERR_MISALIGNED;
  if (fused) {
    if (new_k == nullptr || new_v == nullptr) return COMEM_ERR_NULL_POINTER;
    if (!aligned(new_k, 16) || !aligned(new_v, 16)) return COMEM_ERR_MISALIGNED;
  }
  int64_t chunk = 0, splits = 0;
  const size_t room = workspace == nullptr ? 0 : workspace_bytes;
  const Counters c(*p, batch, scratch ? comem::kScratchTicketBytes : counter_region(*p, room));
  st = plan_call(*p, c, batch, max_ctx_len, 0, room, &chunk, &splits);
  if (st != COMEM_OK) return st;
  st = check_debug_workspace(*p, workspace, workspace_bytes);
  if (st != COMEM_OK) return st;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  const bool balanced = uses_balanced(*p, c, batch, max_ctx_len, workspace, workspace_bytes);
  const bool queue = uses_queue(*p, c, batch, workspace, workspace_bytes);
  comem::AttnParams a;
  fill_common(*p, a, q, k, v, stride_token, stride_head, ctx_lens, out, lse, workspace, batch, max_ctx_len, chunk,
              splits, queue, balanced, c);
  a.seq_start = seq_start;
  if (fused) {
    a.new_k = static_cast<const char*>(new_k);
    a.new_v = static_cast<const char*>(new_v);
  }
  if (balanced) return launch_balanced(*p, false, a, batch, hip_stream);
  return launch(*p, false, a, batch, splits, queue, hip_stream);
}

comem_status decode_paged(const comem_decode_attn_plan* plan, const void* q, const void* new_k,
                          const void* new_v, const void* k_pages, const void* v_pages, int64_t stride_page,
                          int64_t stride_token, int64_t stride_head, int32_t page_size, int64_t num_pages,
                          const int32_t* block_table, int32_t max_pages_per_seq, const int32_t* ctx_lens,
                          int32_t batch, int64_t max_ctx_len, float* out, float* lse, void* workspace,
                          size_t workspace_bytes, void* hip_stream, bool fused) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  comem_status st = validate_common(*p, q, k_pages, v_pages, stride_token, stride_head, ctx_lens, batch,
                                    max_ctx_len, out, lse, workspace);
  if (st != COMEM_OK || batch == 0) return st;
  st = validate_paged(*p, stride_page, page_size, num_pages, block_table, max_pages_per_seq, max_ctx_len);
  if (st != COMEM_OK) return st;
  if (fused) {
    if (new_k == nullptr || new_v == nullptr) return COMEM_ERR_NULL_POINTER;
    if (!aligned(new_k, 16) || !aligned(new_v, 16)) return COMEM_ERR_MISALIGNED;
  }
  int64_t chunk = 0, splits = 0;
  const size_t room = workspace == nullptr ? 0 : workspace_bytes;
  const Counters c(*p, batch, counter_region(*p, room));
  st = plan_call(*p, c, batch, max_ctx_len, page_size, room, &chunk, &splits);
  if (st != COMEM_OK) return st;
  // A split's block-table entries are bounded (a planned split always fits; a
  // configured chunk_tokens may not).
  if (uses_mfma(*p) && (chunk - 1) / page_size + 2 > kMaxSplitPages) return COMEM_ERR_INVALID_SHAPE;
  st = check_debug_workspace(*p, workspace, workspace_bytes);
  if (st != COMEM_OK) return st;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  const bool balanced = uses_balanced(*p, c, batch, max_ctx_len, workspace, workspace_bytes);
  const bool queue = uses_queue(*p, c, batch, workspace, workspace_bytes);
  comem::AttnParams a;
  fill_common(*p, a, q, k_pages, v_pages, stride_token, stride_head, ctx_lens, out, lse, workspace, batch,
              max_ctx_len, chunk, splits, queue, balanced, c);
  a.block_table = block_table;
  a.stride_page = stride_page * elem_bytes(p->cfg);
  a.max_pages = max_pages_per_seq;
  a.num_pages = num_pages;
  a.page_shift = log2_of(page_size);
  a.page_mask = page_size - 1;
  if (fused) {
    a.new_k = static_cast<const char*>(new_k);
    a.new_v = static_cast<const char*>(new_v);
  }
  if (balanced) return launch_balanced(*p, true, a, batch, hip_stream);
  return launch(*p, true, a, batch, splits, queue, hip_stream);
}

}  // namespace

extern "C" {

const char* comem_status_string(comem_status s) {
  switch (s) {
    case COMEM_OK: return "ok";
    case COMEM_ERR_NULL_POINTER: return "a required pointer is NULL";
    case COMEM_ERR_INVALID_SHAPE: return "invalid shape, stride or bound";
    case COMEM_ERR_UNSUPPORTED: return "unsupported dtype, head_dim, GQA group, variant or device";
    case COMEM_ERR_MISALIGNED: return "pointer or byte stride not suitably aligned";
    case COMEM_ERR_WORKSPACE_TOO_SMALL: return "workspace too small for this call";
    case COMEM_ERR_BAD_HANDLE: return "NULL or invalid plan";
    case COMEM_ERR_HIP: return "HIP runtime error";
    case COMEM_ERR_NO_DEVICE: return "plan was made without a device";
    case COMEM_ERR_SCRATCH_LIMIT: return "call needs more than the library's fixed device scratch holds";
  }
  return "unknown status";
}

comem_status comem_decode_attn_init(const comem_decode_attn_config* cfg, int device,
                                    comem_decode_attn_plan** plan_out, size_t* workspace_bytes_out) {
  if (cfg == nullptr || plan_out == nullptr || workspace_bytes_out == nullptr) return COMEM_ERR_NULL_POINTER;
  *plan_out = nullptr;
  *workspace_bytes_out = 0;
  const comem_status st = validate_config(*cfg);
  if (st != COMEM_OK) return st;
  if (device < COMEM_NO_DEVICE) return COMEM_ERR_INVALID_SHAPE;
  int num_cus = kAssumedCUs;
  if (device != COMEM_NO_DEVICE) {
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess) return COMEM_ERR_HIP;
    if (device >= count) return COMEM_ERR_INVALID_SHAPE;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return COMEM_ERR_HIP;
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return COMEM_ERR_UNSUPPORTED;
    num_cus = prop.multiProcessorCount;
  }
  auto* p = new (std::nothrow) comem_decode_attn_plan;
  if (p == nullptr) return COMEM_ERR_HIP;
  p->magic = kPlanMagic;
  p->cfg = *cfg;
  p->device = device;
  p->num_cus = num_cus > 0 ? num_cus : kAssumedCUs;
  const int64_t tickets = static_cast<int64_t>(cfg->max_batch) * cfg->num_kv_heads;
  p->ticket_bytes = plan_ticket_bytes(tickets, cfg->chunk_tokens == 0);
  p->dense_bytes = ticket_region_bytes(tickets, 0);
  // Largest number of (sequence, split) slots any call within the limits plans
  // (for the matrix-core kernel: splits of 1024 tokens, or, of short calls, one
  // per compute unit);
  // calls with a smaller workspace get coarser splits.
  const int64_t B = cfg->max_batch, L = cfg->max_ctx_len;
  int64_t slots;
  if (cfg->chunk_tokens > 0) {
    slots = B * ceil_div(L, cfg->chunk_tokens);
  } else if (uses_mfma(*p)) {
    slots = std::max(B * ceil_div(L, 1024), ceil_div(static_cast<int64_t>(p->num_cus), cfg->num_kv_heads));
  } else {
    const int64_t target = kTargetWgsPerCu * p->num_cus;
    const int64_t a = ceil_div(target, cfg->num_kv_heads) + B;
    const int64_t b = B * ceil_div(L, kMaxChunk);
    slots = a > b ? a : b;
    const int64_t c = B * ceil_div(L, kMinChunk);
    if (c < slots) slots = c;
  }
  p->partial_bytes = slots_workspace_bytes(*p, 0, slots);
  p->workspace_bytes = p->ticket_bytes + p->partial_bytes;
  if (cfg->chunk_tokens == 0 && uses_mfma(*p) && cfg->variant != COMEM_VARIANT_MFMA_GRID)
    p->workspace_bytes = std::max(p->workspace_bytes, p->ticket_bytes + balanced_bytes(*p));
  // The allocation-free entry point's scratch on this device (looked up and
  // cleared once per device); the other entry points work without it.
  if (device != COMEM_NO_DEVICE) (void)comem::scratch_setup(device);
  *plan_out = p;
  *workspace_bytes_out = p->workspace_bytes;
  return COMEM_OK;
}

comem_status comem_decode_attn_destroy(comem_decode_attn_plan* plan) {
  if (plan == nullptr) return COMEM_OK;
  if (plan->magic != kPlanMagic) return COMEM_ERR_BAD_HANDLE;
  plan->magic = 0;
  delete plan;
  return COMEM_OK;
}

comem_status comem_decode_attn_device_errors(const comem_decode_attn_plan* plan, void* workspace,
                                             size_t workspace_bytes, uint32_t* errors_out, void* hip_stream) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  if (workspace == nullptr || errors_out == nullptr) return COMEM_ERR_NULL_POINTER;
  if (!aligned(workspace, 256)) return COMEM_ERR_MISALIGNED;
  if (workspace_bytes < p->dense_bytes) return COMEM_ERR_WORKSPACE_TOO_SMALL;
  *errors_out = 0;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  uint32_t* word = static_cast<uint32_t*>(workspace) + kErrorWord;
  uint32_t host = 0;
  if (hipMemcpyAsync(&host, word, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess) return COMEM_ERR_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return COMEM_ERR_HIP;
  if (host != 0) {
    if (hipMemsetAsync(word, 0, sizeof(host), s) != hipSuccess) return COMEM_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return COMEM_ERR_HIP;
  }
  *errors_out = host;
  return COMEM_OK;
}

comem_status comem_decode_attn_plan_splits(const comem_decode_attn_plan* plan, int32_t batch,
                                           int64_t max_ctx_len, size_t workspace_bytes,
                                           int32_t* chunk_tokens_out, int32_t* num_splits_out) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  if (chunk_tokens_out == nullptr || num_splits_out == nullptr) return COMEM_ERR_NULL_POINTER;
  if (batch < 0 || batch > p->cfg.max_batch) return COMEM_ERR_INVALID_SHAPE;
  if (max_ctx_len < 0 || max_ctx_len > p->cfg.max_ctx_len) return COMEM_ERR_INVALID_SHAPE;
  int64_t chunk = 0, splits = 0;
  const Counters c(*p, batch, counter_region(*p, workspace_bytes));
  const comem_status st = plan_call(*p, c, batch, max_ctx_len, 0, workspace_bytes, &chunk, &splits);
  if (st != COMEM_OK) return st;
  *chunk_tokens_out = static_cast<int32_t>(chunk);
  *num_splits_out = static_cast<int32_t>(splits);
  return COMEM_OK;
}

comem_status comem_decode_attn(const comem_decode_attn_plan* plan, const void* q, const void* k,
                               const void* v, int64_t stride_token, int64_t stride_head,
                               const int64_t* seq_start, const int32_t* ctx_lens, int32_t batch,
                               int64_t max_ctx_len, float* out, float* lse, void* workspace,
                               size_t workspace_bytes, void* hip_stream) {
  return decode_contiguous(plan, q, nullptr, nullptr, k, v, stride_token, stride_head, seq_start, ctx_lens, batch,
                           max_ctx_len, out, lse, workspace, workspace_bytes, hip_stream, false);
}

comem_status comem_decode_attn_noalloc(const comem_decode_attn_plan* plan, const void* q, const void* k,
                                       const void* v, int64_t stride_token, int64_t stride_head,
                                       const int64_t* seq_start, const int32_t* ctx_lens, int32_t batch,
                                       int64_t max_ctx_len, float* out, float* lse, void* hip_stream) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  if (debug_checks(*p)) return COMEM_ERR_UNSUPPORTED;
  comem_status st = validate_common(*p, q, k, v, stride_token, stride_head, ctx_lens, batch, max_ctx_len, out, lse,
                                    nullptr);
  if (st != COMEM_OK || batch == 0) return st;
  if (seq_start == nullptr) return COMEM_ERR_NULL_POINTER;
  if (!aligned(seq_start, 8)) return COMEM_ERR_MISALIGNED;
  // The splits a call with the plan's own workspace would use, and what they
  // need past the scratch's fixed counter region.
  if (p->dense_bytes > comem::kScratchTicketBytes) return COMEM_ERR_SCRATCH_LIMIT;
  int64_t chunk = 0, splits = 0;
  const Counters c(*p, batch, p->ticket_bytes);
  st = plan_call(*p, c, batch, max_ctx_len, 0, p->workspace_bytes, &chunk, &splits);
  if (st != COMEM_OK) return st;
  // (A short call's splits never need more than those of 1024 tokens and up
  // that decide here.)
  if (uses_mfma(*p) && p->cfg.chunk_tokens == 0)
    splits = std::max(splits, ceil_div(max_ctx_len > 0 ? max_ctx_len : 1, long_chunk(*p, batch, max_ctx_len)));
  const size_t partials = call_workspace_bytes(*p, c, batch, splits);
  const size_t need = comem::kScratchTicketBytes + (partials > 0 ? partials - c.bytes : 0);
  if (need > comem::kScratchBytes) return COMEM_ERR_SCRATCH_LIMIT;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  void* scratch = comem::scratch_pointer(p->device);
  if (scratch == nullptr) return COMEM_ERR_HIP;
  return decode_contiguous(plan, q, nullptr, nullptr, k, v, stride_token, stride_head, seq_start, ctx_lens, batch,
                           max_ctx_len, out, lse, scratch, comem::kScratchBytes, hip_stream, false, true);
}

comem_status comem_decode_attn_paged(const comem_decode_attn_plan* plan, const void* q,
                                     const void* k_pages, const void* v_pages, int64_t stride_page,
                                     int64_t stride_token, int64_t stride_head, int32_t page_size,
                                     int64_t num_pages, const int32_t* block_table,
                                     int32_t max_pages_per_seq, const int32_t* ctx_lens,
                                     int32_t batch, int64_t max_ctx_len, float* out, float* lse,
                                     void* workspace, size_t workspace_bytes, void* hip_stream) {
  return decode_paged(plan, q, nullptr, nullptr, k_pages, v_pages, stride_page, stride_token, stride_head,
                      page_size, num_pages, block_table, max_pages_per_seq, ctx_lens, batch, max_ctx_len, out, lse,
                      workspace, workspace_bytes, hip_stream, false);
}

comem_status comem_append_decode_attn(const comem_decode_attn_plan* plan, const void* q, const void* new_k,
                                      const void* new_v, void* k, void* v, int64_t stride_token,
                                      int64_t stride_head, const int64_t* seq_start, const int32_t* ctx_lens,
                                      int32_t batch, int64_t max_ctx_len, float* out, float* lse,
                                      void* workspace, size_t workspace_bytes, void* hip_stream) {
  return decode_contiguous(plan, q, new_k, new_v, k, v, stride_token, stride_head, seq_start, ctx_lens, batch,
                           max_ctx_len, out, lse, workspace, workspace_bytes, hip_stream, true);
}

comem_status comem_append_decode_attn_paged(const comem_decode_attn_plan* plan, const void* q,
                                            const void* new_k, const void* new_v, void* k_pages,
                                            void* v_pages, int64_t stride_page, int64_t stride_token,
                                            int64_t stride_head, int32_t page_size, int64_t num_pages,
                                            const int32_t* block_table, int32_t max_pages_per_seq,
                                            const int32_t* ctx_lens, int32_t batch, int64_t max_ctx_len,
                                            float* out, float* lse, void* workspace, size_t workspace_bytes,
                                            void* hip_stream) {
  return decode_paged(plan, q, new_k, new_v, k_pages, v_pages, stride_page, stride_token, stride_head, page_size,
                      num_pages, block_table, max_pages_per_seq, ctx_lens, batch, max_ctx_len, out, lse, workspace,
                      workspace_bytes, hip_stream, true);
}

comem_status comem_kv_append(const comem_decode_attn_plan* plan, const void* new_k, const void* new_v,
                             void* k, void* v, int64_t stride_token, int64_t stride_head,
                             const int64_t* seq_start, const int32_t* ctx_lens, int32_t batch,
                             int64_t max_ctx_len, void* hip_stream) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  comem::AppendParams a;
  comem_status st = prepare_append(*p, new_k, new_v, k, v, stride_token, stride_head, ctx_lens, batch,
                                   max_ctx_len, a);
  if (st != COMEM_OK || batch == 0) return st;
  if (seq_start == nullptr) return COMEM_ERR_NULL_POINTER;
  if (!aligned(seq_start, 8)) return COMEM_ERR_MISALIGNED;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  a.seq_start = seq_start;
  return launch_append(a, false, batch, hip_stream);
}

comem_status comem_kv_append_paged(const comem_decode_attn_plan* plan, const void* new_k,
                                   const void* new_v, void* k_pages, void* v_pages, int64_t stride_page,
                                   int64_t stride_token, int64_t stride_head, int32_t page_size,
                                   int64_t num_pages, const int32_t* block_table,
                                   int32_t max_pages_per_seq, const int32_t* ctx_lens, int32_t batch,
                                   int64_t max_ctx_len, void* hip_stream) {
  const comem_decode_attn_plan* p = checked(plan);
  if (p == nullptr) return COMEM_ERR_BAD_HANDLE;
  comem::AppendParams a;
  comem_status st = prepare_append(*p, new_k, new_v, k_pages, v_pages, stride_token, stride_head, ctx_lens,
                                   batch, max_ctx_len, a);
  if (st != COMEM_OK || batch == 0) return st;
  st = validate_paged(*p, stride_page, page_size, num_pages, block_table, max_pages_per_seq, max_ctx_len);
  if (st != COMEM_OK) return st;
  if (p->device == COMEM_NO_DEVICE) return COMEM_ERR_NO_DEVICE;
  a.block_table = block_table;
  a.stride_page = stride_page * elem_bytes(p->cfg);
  a.num_pages = num_pages;
  a.max_pages = max_pages_per_seq;
  a.page_shift = log2_of(page_size);
  a.page_mask = page_size - 1;
  return launch_append(a, true, batch, hip_stream);
}

}  // extern "C"
