// Host-side validation, plan selection and workspace layout (no HIP calls).
#include "host_plan.h"

#include <algorithm>

namespace egmla {

namespace {
constexpr int kMaxRowDim = 640;     // d_c + d_r handled by the VALU kernel's LDS tile
constexpr int kMaxHeadDim = 1024;   // d_h and d_v
constexpr int kTargetWorkItems = 1024;
// Token-split MFMA kernel: one 4-wave work-group per compute unit streams
// longest without gaps between its loads (256 compute units).
constexpr int kTargetWorkItemsTok = 256;
// ... and its smallest automatic split, one unit for each of its four waves
// (measured with few sequences: 8 of 1000 tokens 13.8 us per call with 64-token
// splits, 16.3 with 256), while the partials of a sequence stay few (1 x 32768:
// 18.7 us with 128 partials, 19.8 with 256).
constexpr int kMaxPartialsTok = 128;
constexpr int kMergeValueDim = 128;  // value dim of the MFMA merge kernels (run_decode)
constexpr int kMinSplitTok = 64;
// The d_c 128 kernel takes the balanced schedule from this capacity on, where a
// (sequence, split) item is long enough to pay for the schedule and the second
// work-group per compute unit (up to 2 us):
// from kTokBalancedUneven tokens if the items do not fit one per compute unit
// (some then run two, and the balanced pieces win at equal lengths too), else
// only from kTokBalancedEven, where the longest sequences set the time.
// Measured, us per call without / with, lengths n / 16 to n and all n:
//   72 x 1900 (544-token items, 288 of them)  29.4 / 25.7, 32.9 / 30.7
//   200 x 1900 (two items a sequence, 400)    53.0 / 36.5, 59.2 / 50.8
//   96 x 1000 (384, 288)                      25.2 / 21.3, 27.3 / 27.3
//   64 x 4000 (1024, 256)                     29.8 / 29.9, 35.3 / 37.0
//   128 x 1000 (512, 256)                     23.3 / 25.0, 26.6 / 27.6
//   256 x 1900 (1920, 256)                    45.5 / 41.3, 55.3 / 56.7
constexpr int kTokBalancedMinCap = 1024;
constexpr int kTokBalancedUneven = 448;
constexpr int kTokBalancedEven = 1920;
// fp32 matrix-core kernel: 4-wave work-groups, two per compute unit up to
// d_c 64; above, a work-group's LDS leaves room for one (measured at batch 32,
// d_c 256, lengths to 3003: 384-token splits 42.0 us per call, 192-token 48.7).
constexpr int kTargetWorkItemsF32 = 512;

// Single-launch form: W_UK (and W_UV) bytes of a block of heads, at most.
constexpr int64_t kOneMaxWeightBytes = 128 * 1024;

int ceil_div(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }
bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }
}  // namespace

bool mfma_shape_supported(const eg_mla_dims& d) {
  if (d.dtype != EG_MLA_BF16) return false;
  if (d.num_heads % 16 != 0) return false;
  if (d.rope_dim != 64) return false;
  return d.latent_dim == 128 || d.latent_dim == 320 || d.latent_dim == 512;
}

bool tok_kernel_shape(const eg_mla_dims& d) { return d.latent_dim == 128 && d.rope_dim == 64; }
bool rows_kernel_shape(const eg_mla_dims& d) { return d.latent_dim == 320 && d.rope_dim == 64; }
bool heads_kernel_shape(const eg_mla_dims& d) {
  return d.latent_dim == 512 && d.rope_dim == 64 && d.head_dim == 128 && d.v_head_dim == 128 &&
         d.num_heads % kHeadsPerItemWide == 0;
}

bool f32_kernel_shape(const eg_mla_dims& d) { return d.latent_dim <= 320 && d.rope_dim <= 64; }

eg_mla_status check_dims(const eg_mla_dims* d) {
  if (!d) return EG_MLA_ERR_INVALID_ARG;
  if (d->dtype != EG_MLA_FP32 && d->dtype != EG_MLA_BF16) return EG_MLA_ERR_INVALID_ARG;
  if (d->num_heads < 1 || d->head_dim < 1 || d->v_head_dim < 1 || d->latent_dim < 1 || d->rope_dim < 0 ||
      d->vocab_size < 1 || d->page_size < 1 || d->gate_dim < 1)
    return EG_MLA_ERR_INVALID_ARG;
  if (d->softmax_scale != d->softmax_scale) return EG_MLA_ERR_INVALID_ARG;  // NaN
  if (d->gate_dim != d->latent_dim) return EG_MLA_ERR_UNSUPPORTED;
  // 16-byte vector access to latent rows, gate rows and query rows.
  const int vec = d->dtype == EG_MLA_BF16 ? 8 : 4;
  if (d->latent_dim % vec != 0 || d->rope_dim % vec != 0 || d->head_dim % vec != 0)
    return EG_MLA_ERR_UNSUPPORTED;
  if (d->latent_dim + d->rope_dim > kMaxRowDim) return EG_MLA_ERR_UNSUPPORTED;
  if (d->head_dim > kMaxHeadDim || d->v_head_dim > kMaxHeadDim) return EG_MLA_ERR_UNSUPPORTED;
  return EG_MLA_OK;
}

eg_mla_status make_decode_plan(const eg_mla_dims& d, int32_t batch, int32_t max_pages_per_seq,
                               const eg_mla_plan* plan, DecodePlan* out, PlanRows rows_rule) {
  DecodePlan p;
  const int forced = plan ? plan->path : EG_MLA_PATH_AUTO;
  if (forced != EG_MLA_PATH_AUTO && forced != EG_MLA_PATH_VALU && forced != EG_MLA_PATH_MFMA)
    return EG_MLA_ERR_INVALID_ARG;
  const bool mfma_ok = mfma_shape_supported(d);
  if (forced == EG_MLA_PATH_MFMA && !mfma_ok) return EG_MLA_ERR_UNSUPPORTED;
  p.path = (forced == EG_MLA_PATH_VALU || !mfma_ok) ? EG_MLA_PATH_VALU : EG_MLA_PATH_MFMA;

  const int64_t cap64 = static_cast<int64_t>(max_pages_per_seq) * d.page_size;
  if (cap64 > (1 << 30)) return EG_MLA_ERR_INVALID_ARG;
  p.capacity = static_cast<int>(cap64);

  // The vector kernel stays for the shapes the fp32 matrix-core kernel does
  // not take, for explicit splits past its token list, and when asked for.
  p.f32_mfma = rows_rule != PlanRows::kMost && p.path == EG_MLA_PATH_VALU && forced == EG_MLA_PATH_AUTO &&
               f32_kernel_shape(d) && (plan == nullptr || plan->split_tokens <= kMaxSplitTokens);
  if (p.path == EG_MLA_PATH_MFMA) {
    p.heads_per_group = heads_kernel_shape(d) ? kHeadsPerItemWide : 16;
  } else if (p.f32_mfma) {
    p.heads_per_group = 16;
  } else {
    // Heads per VALU work item: at most 8192 latent accumulators per workgroup.
    p.heads_per_group = std::max(1, std::min({d.num_heads, 8192 / d.latent_dim, 256}));
  }
  p.head_groups = ceil_div(d.num_heads, p.heads_per_group);

  const int req_slices = plan ? plan->id_slices : 0;
  if (req_slices != 0 && req_slices != 1 && req_slices != kIdSlices) return EG_MLA_ERR_INVALID_ARG;
  const bool sliced_kernel = p.path == EG_MLA_PATH_MFMA && tok_kernel_shape(d);
  // automatic: no slices (measured faster on MI355X: a sliced work item must
  // resolve its token ids before its first cache-row load)
  p.slices = sliced_kernel && req_slices == kIdSlices ? kIdSlices : 1;
  const bool rows_kernel = p.path == EG_MLA_PATH_MFMA && rows_kernel_shape(d);
  // kernels whose waves own whole units of tokens take short splits
  const bool unit_kernel = rows_rule == PlanRows::kFast && ((sliced_kernel && p.slices == 1) || rows_kernel);
  const int max_split = sliced_kernel ? kMaxSliceSplitTokens : kMaxSplitTokens;

  int split = plan ? plan->split_tokens : 0;
  if (split < 0 || split % kTile != 0) return EG_MLA_ERR_INVALID_ARG;
  if (p.path == EG_MLA_PATH_MFMA && split > max_split) return EG_MLA_ERR_UNSUPPORTED;
  if (split == 0) {
    // Work items (splits x slices) to fill the chip: each work item of the
    // sliced kernel handles 1/slices of its split's tokens.
    const int64_t work =
        static_cast<int64_t>(std::max(batch, 1)) * std::max(p.capacity, 1) * p.head_groups * p.slices;
    const int64_t target =
        p.path == EG_MLA_PATH_MFMA && (tok_kernel_shape(d) || heads_kernel_shape(d)) ? kTargetWorkItemsTok
        // (measured: 256 x 2048 117 us per call against 122 with two work-groups
        // per compute unit, 32 x 4096 42.5 against 47.9)
        : rows_kernel && rows_rule != PlanRows::kMost ? kTargetWorkItemsTok
        : p.f32_mfma ? (d.latent_dim <= 64 ? kTargetWorkItemsF32 : kTargetWorkItemsF32 / 2)
                     : kTargetWorkItems;
    int64_t s = (work + target - 1) / target;
    const int gran = p.slices > 1 ? 256 : kTile;  // sliced kernel: whole 256-position scan rows
    s = (s + gran - 1) / gran * gran;
    const int min_split = unit_kernel ? kMinSplitTok
                          : p.path == EG_MLA_PATH_MFMA || p.f32_mfma ? 256
                                                                     : 128;
    s = std::max<int64_t>(s, min_split);
    if (unit_kernel) s = std::max<int64_t>(s, (p.capacity / kMaxPartialsTok + kTile - 1) / kTile * kTile);
    // the general merge reads a sequence's partials one after the other: no more
    // than 16 for the sake of short splits (d_v 64, 1 x 4096: 64 partials 21.6 us
    // per call, 16 18.4; 1 x 2048: 32 18.0, 16 17.0)
    if (unit_kernel && d.v_head_dim != kMergeValueDim && s < 256)
      s = std::max<int64_t>(s, std::min(256, ceil_div(p.capacity, 16 * kTile) * kTile));
    if (sliced_kernel && unit_kernel && s < 256) {
      const int64_t per_split = static_cast<int64_t>(std::max(batch, 1)) * p.head_groups;
      const int cap = std::max(p.capacity, 1);
      auto cut = [&](int n) { return std::max(kMinSplitTok, ceil_div(cap, n * kTile) * kTile); };
      // Short splits only where the items still run one per compute unit (48 x
      // 1000: 288 items of 192 tokens 18.8 us per call, 192 of 256 17.1); up to
      // 4 sequences of 4096 no more than 32 a sequence, which the kernel can
      // absorb the query with (below; 4 x 4096: 32 splits of 128 15.1 us in a
      // graph, 64 of 64 and a launch more 14.5, but a host needs 13 to 17 to
      // enqueue its three launches, 10.5 to 12 for two).  With 17 to 32 sequences 8 a
      // sequence rather than some number between 8 and 16: the absorption is
      // then shared evenly, and 8 partials merge in small work-groups; up to 192
      // tokens each (us per call: as above / 8 splits / of 256 tokens):
      //   20 x 1300  17.6 / 16.1 / 17.2    24 x 1500  18.3 / 16.6 / 17.3
      //   28 x 1100  18.0 / 16.5 / 17.3    20 x 900   16.6 / 15.9 / 17.0
      // and 256 tokens from there to 2048 (24 x 1600 18.2 / 17.7 / 17.3, 28 x
      // 1800 19.9 / 18.6 / 18.7); above, more than 8 splits are due anyway
      // (20 x 2300 18.1 / 18.7 / 19.1).
      if (per_split <= 4 && cap <= 32 * 128)
        s = std::max<int64_t>(s, cut(32));
      else if (per_split > 16 && 8 * per_split <= kTargetWorkItemsTok && cap <= 8 * 256)
        s = cut(8) <= 192 ? cut(8) : 256;
      else if (per_split * ceil_div(cap, static_cast<int>(s)) > kTargetWorkItemsTok)
        s = per_split <= 16 && cut(16) < 256 ? cut(16) : 256;  // (12 x 2048, not 264 items: 16 splits 15.7, 256 tokens 17.0)
    }
    s = std::min<int64_t>(s, max_split);
    split = static_cast<int>(s);
  }
  p.split_tokens = split;
  p.s_max = std::max(1, ceil_div(std::max(p.capacity, 1), split));
  // One launch instead of three where a work-group can afford its heads'
  // weights (read whole by every sequence) and its whole context, and all
  // work-groups are resident at once.
  p.one_launch = p.f32_mfma && (plan == nullptr || plan->split_tokens == 0) && p.capacity > 0 &&
                 p.capacity <= kOneMaxTokens && d.latent_dim <= kOneMaxLatent &&
                 static_cast<int64_t>(std::min(d.num_heads, 16)) * std::max(d.head_dim, d.v_head_dim) * d.latent_dim *
                         elem_bytes(d) <= kOneMaxWeightBytes &&
                 static_cast<int64_t>(std::max(batch, 0)) * p.head_groups <= kTargetWorkItemsF32;
  // The head-split kernel balances tokens over its work-groups whatever the
  // length mix; its split size only caps the token list it stages at a time.
  p.balanced = p.path == EG_MLA_PATH_MFMA && heads_kernel_shape(d);
  if (p.balanced && (plan == nullptr || plan->split_tokens == 0)) p.split_tokens = kMaxSplitTokens;

  const size_t B = static_cast<size_t>(std::max(batch, 0));
  const size_t H = static_cast<size_t>(d.num_heads);
  const size_t DQ = static_cast<size_t>(d.latent_dim + d.rope_dim);
  // The split kernel absorbs the query itself when that costs each work-group
  // at most 2 heads' W_UK (8 or more splits per sequence, the first 16 of them
  // producers) and every work-group is resident at once (2 per compute unit);
  // otherwise (many splits, whose extra work-groups only wait, or a batch of
  // several rounds of work-groups each reading 4 or more heads' W_UK) the
  // absorption kernel runs first (measured: B32 L4096 25.2 against 25.7 us
  // per call; B4 L32768 28.9 against 27.8; B256 L2048 70.8 against 59.4).  Of
  // 17 to 32 splits the short ones take it, where waiting for the producers
  // costs no more than the launch they save: the two run about as long (2 x
  // 1856 13.6 / 13.7 us in a graph, 12 x 1280 14.7 / 14.5; 8 x 3000, 256 items,
  // 16.0 / 15.4), but a step of append and decode is then four launches, not
  // five, and a host has to enqueue them: 2 x 1856 22.9 us against 25.7.
  const int64_t nblk = static_cast<int64_t>(std::max(batch, 0)) * p.s_max * p.head_groups;
  const bool short_splits = unit_kernel && (plan == nullptr || plan->split_tokens == 0) && p.s_max <= 32 &&
                            (p.split_tokens <= kMinSplitTok || (p.split_tokens <= 128 && nblk <= 224));
  p.fused_absorb = sliced_kernel && p.slices == 1 && d.head_dim == 128 && p.s_max >= 8 &&
                   (p.s_max <= 16 || short_splits) && nblk <= 2 * kTargetWorkItemsTok;
  auto layout = [&]() {
    const size_t rows = p.balanced       ? kWideMaxGroups + B
                        : p.tok_balanced ? static_cast<size_t>(p.pieces)
                                         : B * static_cast<size_t>(p.s_max) * static_cast<size_t>(p.slices);
    size_t off = 0;
    p.off_q = off;
    off = align_up(off + B * H * DQ * 4);
    p.off_ml = off;
    off = align_up(off + rows * H * 2 * 4);
    // partial outputs: fp32 sums, or (wide kernel) fp16 rows normalised by their sums
    p.off_o = off;
    off = align_up(off + rows * H * static_cast<size_t>(d.latent_dim) * (p.balanced ? 2 : 4));
    if (p.balanced || p.tok_balanced) {
      p.off_sched = off;
      off = align_up(off + 16 + (p.balanced ? kWideMaxGroups * 8 : static_cast<size_t>(p.pieces) * 16) + B * 8);
    }
    if (p.fused_absorb) {
      p.off_flags = off;
      off = align_up(off + B * static_cast<size_t>(p.head_groups) * static_cast<size_t>(p.s_max) * 8);
    }
    return off;
  };
  size_t off = layout();
  // Few splits per sequence: a work-group's time follows its sequence's
  // length, so the d_c 128 kernel takes the balanced schedule, two
  // work-groups per compute unit.  Not beyond the batch where the dispatcher
  // itself evens out the work-groups, nor where the search's largest piece (about
  // N / (pieces - batch), see tok_sizes) could outgrow the token list, nor where the extra partial rows would take a call that fits
  // the workspace-free entry's scratch out of it.
  if (rows_rule == PlanRows::kFast && sliced_kernel && p.slices == 1 && !p.fused_absorb && d.head_dim == 128 && batch > 32 && p.s_max < 8 &&
      (plan == nullptr || plan->split_tokens == 0) && p.capacity >= kTokBalancedMinCap &&
      p.split_tokens >= (nblk > kTargetWorkItemsTok ? kTokBalancedUneven : kTokBalancedEven) &&
      batch <= kTokMaxBatch) {
    const int pieces = kTokMaxPieces / p.head_groups / 8 * 8;
    if (pieces > batch &&
        static_cast<int64_t>(batch) * p.capacity / (pieces - batch) < max_split - 128) {
      const size_t plain = off;
      p.tok_balanced = true;
      p.pieces = pieces;
      off = layout();
      if (off > plain && off > EG_MLA_NOALLOC_SCRATCH_BYTES && plain <= EG_MLA_NOALLOC_SCRATCH_BYTES) {
        p.tok_balanced = false;
        p.pieces = 0;
        off = layout();
      }
    }
  }
  p.bytes = std::max<size_t>(off, kAlign);
  *out = p;
  return EG_MLA_OK;
}

eg_mla_status fit_decode_plan(const eg_mla_dims& d, int32_t batch, int32_t max_pages_per_seq, const eg_mla_plan* plan,
                              size_t workspace_bytes, DecodePlan* out) {
  eg_mla_status st = make_decode_plan(d, batch, max_pages_per_seq, plan, out);
  if (st != EG_MLA_OK || out->bytes <= workspace_bytes) return st;
  st = make_decode_plan(d, batch, max_pages_per_seq, plan, out, PlanRows::kFew);
  return st != EG_MLA_OK || out->bytes <= workspace_bytes ? st : EG_MLA_ERR_WORKSPACE;
}

size_t decode_workspace_bytes(const eg_mla_dims& d, int32_t batch, int32_t max_pages_per_seq, const eg_mla_plan* plan) {
  size_t bytes = 0;
  for (const PlanRows rows : {PlanRows::kFast, PlanRows::kFew, PlanRows::kMost}) {
    DecodePlan p;
    if (make_decode_plan(d, batch, max_pages_per_seq, plan, &p, rows) != EG_MLA_OK) return 0;
    bytes = std::max(bytes, p.bytes);
  }
  return bytes;
}

eg_mla_status validate_decode(const eg_mla_dims* d, int32_t batch, const void* q, const void* latent_cache,
                              const int32_t* token_id_cache, const void* gate_table, const void* w_uk,
                              const void* w_uv, const int32_t* seq_lens, int32_t max_pages_per_seq,
                              int64_t num_slots, const int32_t* page_table, const void* workspace,
                              size_t workspace_bytes, const void* out, const eg_mla_plan* plan, DecodePlan* p) {
  eg_mla_status st = check_dims(d);
  if (st != EG_MLA_OK) return st;
  if (batch < 0 || max_pages_per_seq < 0 || num_slots < 0) return EG_MLA_ERR_INVALID_ARG;
  if (num_slots >= (int64_t{1} << 31)) return EG_MLA_ERR_UNSUPPORTED;  // 32-bit row indices in the kernels
  const eg_mla_status fit = fit_decode_plan(*d, batch, max_pages_per_seq, plan, workspace_bytes, p);
  if (fit != EG_MLA_OK && fit != EG_MLA_ERR_WORKSPACE) return fit;
  if (batch == 0) return EG_MLA_OK;
  if (!q || !gate_table || !w_uk || !w_uv || !seq_lens || !out) return EG_MLA_ERR_INVALID_ARG;
  if (max_pages_per_seq > 0 && (!latent_cache || !token_id_cache)) return EG_MLA_ERR_INVALID_ARG;
  if (!page_table) {
    // contiguous rows: every sequence's capacity must fit in the cache
    const int64_t need = static_cast<int64_t>(batch) * max_pages_per_seq * d->page_size;
    if (need > num_slots) return EG_MLA_ERR_INVALID_ARG;
  } else if (num_slots < d->page_size && max_pages_per_seq > 0) {
    return EG_MLA_ERR_INVALID_ARG;
  }
  // 16-byte vector loads of rows and weights
  if (!aligned16(q) || !aligned16(latent_cache) || !aligned16(gate_table) || !aligned16(w_uk) || !aligned16(w_uv))
    return EG_MLA_ERR_INVALID_ARG;
  if (!workspace || fit != EG_MLA_OK) return EG_MLA_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0) return EG_MLA_ERR_WORKSPACE;
  return EG_MLA_OK;
}

eg_mla_status validate_append(const eg_mla_dims* d, int32_t n_tokens, int32_t hidden, const void* x,
                              const int32_t* token_ids, const int32_t* positions, const int32_t* slots,
                              const void* w_dkv, const void* latent_cache, const int32_t* token_id_cache,
                              int64_t num_slots) {
  eg_mla_status st = check_dims(d);
  if (st != EG_MLA_OK) return st;
  if (n_tokens < 0 || hidden < 1 || num_slots < 0) return EG_MLA_ERR_INVALID_ARG;
  if (hidden > 32768) return EG_MLA_ERR_UNSUPPORTED;  // x row staged in LDS
  if (d->rope_dim % 2 != 0) return EG_MLA_ERR_INVALID_ARG;
  if (n_tokens == 0) return EG_MLA_OK;
  if (!x || !token_ids || !positions || !slots || !w_dkv || !latent_cache || !token_id_cache)
    return EG_MLA_ERR_INVALID_ARG;
  return EG_MLA_OK;
}

eg_mla_status validate_gate_rows(const eg_mla_dims* d, int32_t emb_dim, int32_t emb_vocab, int64_t n,
                                 const int32_t* ids, const void* emb, const void* w_ue, const void* out) {
  eg_mla_status st = check_dims(d);
  if (st != EG_MLA_OK) return st;
  if (emb_dim < 1 || emb_vocab < 1 || n < 0) return EG_MLA_ERR_INVALID_ARG;
  if (emb_dim > 16384) return EG_MLA_ERR_UNSUPPORTED;  // one embedding row staged in LDS (VALU kernel)
  if (n == 0) return EG_MLA_OK;
  if (!ids || !emb || !w_ue || !out) return EG_MLA_ERR_INVALID_ARG;
  return EG_MLA_OK;
}

size_t prefill_workspace_bytes(const eg_mla_dims& d, int32_t seq_len) {
  const size_t T = static_cast<size_t>(std::max(seq_len, 0));
  const size_t H = static_cast<size_t>(d.num_heads);
  // fp32 explicit keys [H, T, d_h + d_r] and values [H, T, d_v]
  size_t k = align_up(H * T * static_cast<size_t>(d.head_dim + d.rope_dim) * 4);
  size_t v = align_up(H * T * static_cast<size_t>(d.v_head_dim) * 4);
  return std::max<size_t>(k + v, kAlign);
}

eg_mla_status validate_prefill(const eg_mla_dims* d, int32_t seq_len, const void* q, const void* latent,
                               const int32_t* token_ids, const void* gate_table, const void* w_uk,
                               const void* w_uv, const void* workspace, size_t workspace_bytes,
                               const void* out) {
  eg_mla_status st = check_dims(d);
  if (st != EG_MLA_OK) return st;
  if (seq_len < 0) return EG_MLA_ERR_INVALID_ARG;
  if (seq_len > 32768) return EG_MLA_ERR_UNSUPPORTED;  // one score row staged in LDS
  if (seq_len == 0) return EG_MLA_OK;
  if (!q || !latent || !token_ids || !gate_table || !w_uk || !w_uv || !out) return EG_MLA_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < prefill_workspace_bytes(*d, seq_len)) return EG_MLA_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0) return EG_MLA_ERR_WORKSPACE;
  return EG_MLA_OK;
}

bool prefill_varlen_absorbed(const eg_mla_dims& d) {
  return d.dtype == EG_MLA_BF16 && d.num_heads == 16 && d.head_dim == 128 && d.v_head_dim == 128 &&
         d.latent_dim == 128 && d.rope_dim == 64 && d.gate_dim == d.latent_dim;
}

bool prefill_varlen_shape_ok(const eg_mla_dims& d) {
  if (prefill_varlen_absorbed(d)) return true;
  // the explicit form: any head count, d_c a multiple of 64
  return d.dtype == EG_MLA_BF16 && d.head_dim == 128 && d.v_head_dim == 128 && d.rope_dim == 64 &&
         d.latent_dim % 64 == 0 && d.gate_dim == d.latent_dim;
}

PrefillVarlenLayout prefill_varlen_layout(const eg_mla_dims& d, int32_t total_tokens) {
  const size_t T = static_cast<size_t>(std::max(total_tokens, 0));
  const size_t H = static_cast<size_t>(d.num_heads);
  PrefillVarlenLayout L;
  L.off_seq_start = 0;  // int32 [T]
  if (prefill_varlen_absorbed(d)) {
    // the size is that of query rows of d_c + d_r, whose RoPE part the attention reads from
    // the query: the blocks' order lies in the part of them that is left
    L.off_qf = align_up(T * 4);                                                    // fp16 [T][H][d_c]
    L.off_order = L.off_qf + align_up(T * H * static_cast<size_t>(d.latent_dim) * 2);  // int2 [ceil(T / 8)]
    L.off_olat = L.off_qf + align_up(T * H * static_cast<size_t>(d.latent_dim + d.rope_dim) * 2);  // fp16 [T][H][d_c]
    L.off_ct = L.off_olat + align_up(T * H * static_cast<size_t>(d.latent_dim) * 2);   // fp16 [T][d_c]
    L.bytes = std::max<size_t>(L.off_ct + align_up(T * static_cast<size_t>(d.latent_dim) * 2), kAlign);
  } else {
    L.off_qf = align_up(T * 4);                                                  // K^C: fp16 [H][T][d_h]
    L.off_olat = L.off_qf + align_up(T * H * static_cast<size_t>(d.head_dim) * 2);  // V: fp16 [H][T][d_v]
    L.off_ct = L.off_olat + align_up(T * H * static_cast<size_t>(d.v_head_dim) * 2);  // bf16 hi, lo [2][T][d_c]
    L.bytes = std::max<size_t>(L.off_ct + 2 * align_up(T * static_cast<size_t>(d.latent_dim) * 2), kAlign);
  }
  return L;
}

eg_mla_status validate_prefill_varlen(const eg_mla_dims* d, int32_t batch, int32_t total_tokens,
                                      const int32_t* cu_seqlens, const void* q, const void* latent,
                                      const int32_t* token_ids, const void* gate_table, const void* w_uk,
                                      const void* w_uv, const void* workspace, size_t workspace_bytes,
                                      const void* out) {
  eg_mla_status st = check_dims(d);
  if (st != EG_MLA_OK) return st;
  if (batch < 1 || total_tokens < 0) return EG_MLA_ERR_INVALID_ARG;
  if (!prefill_varlen_shape_ok(*d)) return EG_MLA_ERR_UNSUPPORTED;
  if (total_tokens == 0) return EG_MLA_OK;
  if (!cu_seqlens || !q || !latent || !token_ids || !gate_table || !w_uk || !w_uv || !out)
    return EG_MLA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(latent) || !aligned16(gate_table) || !aligned16(w_uk) || !aligned16(w_uv) ||
      !aligned16(out))
    return EG_MLA_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < prefill_varlen_layout(*d, total_tokens).bytes) return EG_MLA_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0) return EG_MLA_ERR_WORKSPACE;
  return EG_MLA_OK;
}

bool literal_tile_shape(const eg_mla_dims& d) {
  return d.dtype == EG_MLA_BF16 && d.latent_dim == 128 && d.head_dim == 128 && d.v_head_dim == 128 &&
         d.rope_dim == 64 && d.num_heads <= 160 && literal_lds_bytes(d.num_heads, 1) <= 160 * 1024;
}

size_t literal_generic_lds_bytes(const eg_mla_dims& d) {
  // latents of a group of 8 tokens, key dots and weights [8][H], moment sums
  // [4][8][2], per-token figures [3][8], per-head sums [2][H] and softmax
  // state [3][H], value sums [H][d_v] (all fp32)
  const size_t H = static_cast<size_t>(d.num_heads);
  return 4 * (8 * static_cast<size_t>(d.latent_dim) + 16 * H + 64 + 24 + 5 * H +
              H * static_cast<size_t>(d.v_head_dim));
}

size_t literal_lds_bytes(int num_heads, int groups) {
  // per head group: weight / gate-tile region, value sums [4][d_v] and, for two
  // groups, the tokens' moments [3][4][32]; per-wave scores [4][H][32], two
  // sums per head, per-wave figures per head, token means [4][32] (all fp32)
  return static_cast<size_t>(groups) * (272 * 256 + 4 * 128 * 4 + (groups > 1 ? 3 * 4 * 32 * 4 : 0)) +
         4 * static_cast<size_t>(num_heads) * 32 * 4 + static_cast<size_t>(num_heads) * (2 + 12) * 4 + 4 * 32 * 4;
}

int literal_head_groups(int num_heads) {
  return num_heads % 2 == 0 && literal_lds_bytes(num_heads, 2) <= 160 * 1024 ? 2 : 1;
}

size_t literal_workspace_bytes(const eg_mla_dims& d, int32_t batch, int32_t max_pages_per_seq) {
  const int64_t cap = static_cast<int64_t>(std::max(max_pages_per_seq, 0)) * d.page_size;
  const int64_t tiles = (cap + 127) / 128;
  return std::max<size_t>(align_up(static_cast<size_t>(std::max(batch, 0)) * static_cast<size_t>(tiles) *
                                   d.num_heads * (d.v_head_dim + 4) * sizeof(float)),
                          kAlign);
}

eg_mla_status validate_literal(const eg_mla_dims* d, int32_t batch, const void* q, const void* latent_cache,
                               const int32_t* token_id_cache, const void* gate_full, const void* w_uk,
                               const void* w_uv, const void* ln_w, const void* ln_b, uint32_t flags,
                               const int32_t* seq_lens, const int32_t* page_table, int32_t max_pages_per_seq,
                               int64_t num_slots, const void* workspace, size_t workspace_bytes, const void* out) {
  eg_mla_status st = check_dims(d);
  if (st != EG_MLA_OK) return st;
  if (batch < 0 || max_pages_per_seq < 0 || num_slots < 0) return EG_MLA_ERR_INVALID_ARG;
  if ((flags & ~(EG_MLA_LITERAL_NO_LN | EG_MLA_LITERAL_ADD)) != 0) return EG_MLA_ERR_INVALID_ARG;
  if (literal_tile_shape(*d)) {
    // gate rows are addressed by 32-bit byte offsets in the tile kernel
    if (static_cast<int64_t>(d->vocab_size) * d->num_heads * (d->head_dim + d->v_head_dim) * 2 >=
        (int64_t{1} << 32))
      return EG_MLA_ERR_UNSUPPORTED;
  } else if (literal_generic_lds_bytes(*d) > 160 * 1024) {
    return EG_MLA_ERR_UNSUPPORTED;  // the generic kernel's tile state does not fit in LDS
  }
  if (static_cast<int64_t>(max_pages_per_seq) * d->page_size > (int64_t{1} << 30)) return EG_MLA_ERR_UNSUPPORTED;
  if (num_slots >= (int64_t{1} << 31)) return EG_MLA_ERR_UNSUPPORTED;
  if (batch == 0) return EG_MLA_OK;
  if (!q || !gate_full || !w_uk || !w_uv || !seq_lens || !out || !latent_cache || !token_id_cache)
    return EG_MLA_ERR_INVALID_ARG;
  if (max_pages_per_seq < 1 || num_slots < 1) return EG_MLA_ERR_INVALID_ARG;
  if (!page_table && static_cast<int64_t>(batch) * max_pages_per_seq * d->page_size > num_slots)
    return EG_MLA_ERR_INVALID_ARG;  // contiguous rows: every sequence's capacity must fit in the cache
  if ((flags & EG_MLA_LITERAL_NO_LN) == 0 && (!ln_w || !ln_b)) return EG_MLA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(latent_cache) || !aligned16(gate_full) || !aligned16(w_uk) || !aligned16(w_uv))
    return EG_MLA_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < literal_workspace_bytes(*d, batch, max_pages_per_seq))
    return EG_MLA_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign != 0) return EG_MLA_ERR_WORKSPACE;
  return EG_MLA_OK;
}

}  // namespace egmla

extern "C" {

const char* eg_mla_status_string(eg_mla_status s) {
  switch (s) {
    case EG_MLA_OK: return "EG_MLA_OK";
    case EG_MLA_ERR_INVALID_ARG: return "EG_MLA_ERR_INVALID_ARG: invalid argument";
    case EG_MLA_ERR_UNSUPPORTED: return "EG_MLA_ERR_UNSUPPORTED: shape or option not supported";
    case EG_MLA_ERR_WORKSPACE: return "EG_MLA_ERR_WORKSPACE: workspace missing, misaligned or too small";
    case EG_MLA_ERR_HIP: return "EG_MLA_ERR_HIP: HIP runtime or launch failure";
  }
  return "EG_MLA_ERR_UNKNOWN";
}

eg_mla_status eg_mla_check_dims(const eg_mla_dims* dims) { return egmla::check_dims(dims); }

size_t eg_mla_decode_workspace_size(const eg_mla_dims* dims, int32_t batch, int32_t max_pages_per_seq,
                                    const eg_mla_plan* plan) {
  if (egmla::check_dims(dims) != EG_MLA_OK || batch < 0 || max_pages_per_seq < 0) return 0;
  return egmla::decode_workspace_bytes(*dims, batch, max_pages_per_seq, plan);
}

size_t eg_mla_prefill_workspace_size(const eg_mla_dims* dims, int32_t seq_len) {
  if (egmla::check_dims(dims) != EG_MLA_OK || seq_len < 0) return 0;
  return egmla::prefill_workspace_bytes(*dims, seq_len);
}

size_t eg_mla_prefill_varlen_workspace_size(const eg_mla_dims* dims, int32_t total_tokens) {
  if (egmla::check_dims(dims) != EG_MLA_OK || total_tokens < 0 || !egmla::prefill_varlen_shape_ok(*dims)) return 0;
  return egmla::prefill_varlen_layout(*dims, total_tokens).bytes;
}

}  // extern "C"
