// Causal GQA flash attention over the paged KV cache for packed varlen query chunks
// (sp_attn_prefill): the attention each GPU runs on its head shard in the sequence-parallel
// mode after the sequence->head exchange, and for chunked prefill against a cached prefix.
// Per the paper's section "Introducing Shift Parallelism" this computation and its data
// mapping are the same in both parallel modes; only the query count per sequence differs.
//
// Decomposition.  One workgroup (8 waves) owns a tile of 256 query COLUMNS of one
// (sequence, KV head).  The G = Hq/Hkv query heads that share the KV head are stacked into the
// column dimension (column = token * G + head), so a K/V tile staged in LDS is reused by all
// G heads and all columns of a wave have nearly the same causal bound.  Each wave owns 32
// columns; the workgroup walks the visible keys in tiles of KVT tokens (KVT/16 pages, looked
// up in the block table), double-buffered in LDS.
//
// Bound: bf16 MFMA (4 * head_dim flops per visible (query, key) pair per head).  K/V HBM
// traffic is ~1/(8*columns) of that in bytes and is served mostly from L2.  Next to the matrix
// pipe the kernel keeps the VALU (softmax: 3.5 instructions per score, the exponential at half
// rate) and LDS (every MFMA takes one 1 KiB operand from it) busy at the same time.  Measured on
// a 32 k-token prefill, a tile max in every tile (a reduction plus a cross-lane step in front of
// every exponential) costs a quarter more cycles, and so do VALU instructions between the MFMAs
// of a matrix phase, while one plain instruction per score more or less in the softmax phase
// changes nothing at head_dim 128: so the softmax is a single pass without a tile max and the
// matrix phases carry no address arithmetic.  The matrix pipe is then busy in about 85 % of the
// cycles a CU is busy, and what limits the kernel beyond that is the clock the chip grants under
// this load (it is power-limited from the first tile on).
#include "decode_block.h"
#include "prefill_solo.h"

namespace sp {

// Launch-shape overrides of the calling thread (sp_debug_set_tuning); 0 = built-in heuristic.
static thread_local int g_split_mode = 0;
static thread_local int g_kv_splits = 0;
static thread_local int g_short_chunk_mode = 0;
static thread_local int g_order_mode = 0;
static thread_local int g_cut_mode = 0;
void set_prefill_cut(int mode) { g_cut_mode = mode; }
void set_prefill_order(int mode) { g_order_mode = mode; }
void set_prefill_short_chunk(int mode) { g_short_chunk_mode = mode; }
void set_prefill_split(int mode) { g_split_mode = mode; }
void set_prefill_kv_splits(int n) { g_kv_splits = n; }

// Mixed batch?  Decided from the host-side hints alone: chunks too long for the short-chunk path
// exist (max_q_len), and the tokens besides the longest chunk are so few that at least one other
// sequence must be short — those sequences are then routed to the split kernel (which reads a
// long cached prefix once, in pieces, at memory speed) and the rest to the prefill kernel, inside
// the one call.  Returns the token bound of "short" (one column tile of the split kernel), or 0.
static int mixed_route_cap(int batch, int total_q, int max_q_len, int num_q_heads, int num_kv_heads) {
  if (g_short_chunk_mode == 1 || batch < 2) return 0;
  const int cap = decode_route_cap(num_q_heads, num_kv_heads);
  if (cap <= 0 || max_q_len <= cap) return 0;  // no long chunk: the whole batch takes the short-chunk path
  const long rest = (long)total_q - max_q_len;
  if (rest <= 0 || rest >= (long)(batch - 1) * (cap + 1)) return 0;
  return cap;
}

// Slots for partials of the CUT form (0: not taken), from the host-side hints alone.
static int cut_slots(int batch, int total_q, int max_q_len, int max_kv_len, int num_q_heads, int num_kv_heads, int head_dim) {
  // Mixed batches: their chunk is short next to what a launch costs (2048 tokens: 64.2 us against 63.7).
  if (g_cut_mode == 1 || (g_cut_mode == 0 && mixed_route_cap(batch, total_q, max_q_len, num_q_heads, num_kv_heads) > 0)) return 0;
  return cut_form_slots(batch, total_q, max_q_len, max_kv_len, num_q_heads, num_kv_heads, head_dim, g_cut_mode == 2);
}

static size_t cut_bytes(int slots, int head_dim) {
  return slots == 0 ? 0 : 256 + (size_t)slots * (sizeof(CutEntry) + 256 * (head_dim + 2) * sizeof(float));
}

size_t prefill_workspace_bytes(int batch, int total_q_tokens, int max_q_len, int max_kv_len, int num_q_heads,
                               int num_kv_heads, int head_dim) {
  const long rows = (long)total_q_tokens * num_q_heads;
  const int cap = kv_split_cap(rows);
  const size_t pieces = cap >= 2 ? (size_t)rows * cap * (head_dim + 2) * sizeof(float) : 0;
  size_t shortq = g_short_chunk_mode == 1 ? 0
                                          : decode_multi_workspace_bytes(batch, total_q_tokens, max_q_len, max_kv_len,
                                                                         num_q_heads, num_kv_heads, head_dim);
  if (mixed_route_cap(batch, total_q_tokens, max_q_len, num_q_heads, num_kv_heads) > 0)
    shortq = decode_routed_workspace_bytes(batch, max_kv_len, num_q_heads, num_kv_heads, head_dim);
  const size_t cut = cut_bytes(cut_slots(batch, total_q_tokens, max_q_len, max_kv_len, num_q_heads, num_kv_heads, head_dim), head_dim);
  const size_t most = pieces > shortq ? pieces : shortq;
  return cut > most ? cut : most;
}

template <int D>
static int launch_prefill_d(const PrefillArgs &a, bool split, int batch, int max_q_len, hipStream_t stream) {
  constexpr size_t smem = kPrefillSmem<D>;
  static bool set[3] = {false, false, false};
  // Key ranges are only cut into pieces on small grids, which take the 128-column form anyway;
  // the 256-column form with partial outputs is not instantiated (it would not fit the register
  // budget of two workgroups per CU).
  if (a.kv_splits > 1) return launch_cfg(prefill_kernel<D, KVT, PFD, true, true, 0>, &set[0], 2 * smem, 128, a, batch, max_q_len, stream);
  if (split) return launch_cfg(prefill_kernel<D, KVT, PFD, true, false, 0>, &set[1], 2 * smem, 128, a, batch, max_q_len, stream);
  if constexpr (D == 64) return launch_cfg(solo_prefill_kernel<PrefillArgs>, &set[2], kSoloSmem, kSoloCols, a, batch, max_q_len, stream, kSoloThreads, kSoloLayers);
  else return launch_cfg(prefill_kernel<D, KVT, PFD, false, false, 0>, &set[2], smem, 256, a, batch, max_q_len, stream);
}

static int prefill_chunks(const sp_cache_desc &c, const void *k_new, const void *v_new, const void *q, void *out, const int32_t *cu_q,
                          const int32_t *ctx_lens, const int32_t *block_table, int batch, int max_pages, int total_q, int max_q_len,
                          int max_kv_len, int num_q_heads, float scale, void *workspace, size_t workspace_bytes, hipStream_t stream);

int launch_chunk_step(const sp_cache_desc &c, const void *k_new, const void *v_new, const void *q, void *out,
                      const int32_t *cu_q, const int32_t *ctx_lens, const int32_t *block_table, int batch,
                      int max_pages, int total_q, int max_q_len, int max_kv_len, int num_q_heads, float scale,
                      void *workspace, size_t workspace_bytes, hipStream_t stream) {
  if (g_short_chunk_mode != 1) {
    // short chunks: the decode kernels append the rows themselves
    int rc = launch_decode_multi(c, k_new, v_new, q, out, cu_q, ctx_lens, block_table, batch, max_pages, total_q,
                                 max_q_len, max_kv_len, num_q_heads, scale, workspace, workspace_bytes, stream);
    if (rc != 1) return rc;
  }
  return prefill_chunks(c, k_new, v_new, q, out, cu_q, ctx_lens, block_table, batch, max_pages, total_q, max_q_len, max_kv_len, num_q_heads,
                        scale, workspace, workspace_bytes, stream);
}

int launch_prefill(const sp_cache_desc &c, const void *q, void *out, const int32_t *cu_q,
                   const int32_t *ctx_lens, const int32_t *block_table, int batch, int max_pages,
                   int total_q, int max_q_len, int max_kv_len, int num_q_heads, float scale,
                   void *workspace, size_t workspace_bytes, hipStream_t stream) {
  if (g_short_chunk_mode != 1) {
    // Every chunk is a few tokens long: the bandwidth-bound split kernel of the decode path reads
    // each sequence's keys once for all of its query tokens.
    int rc = launch_decode_multi(c, nullptr, nullptr, q, out, cu_q, ctx_lens, block_table, batch, max_pages, total_q, max_q_len,
                                 max_kv_len, num_q_heads, scale, workspace, workspace_bytes, stream);
    if (rc != 1) return rc;
  }
  return prefill_chunks(c, nullptr, nullptr, q, out, cu_q, ctx_lens, block_table, batch, max_pages, total_q, max_q_len, max_kv_len, num_q_heads,
                        scale, workspace, workspace_bytes, stream);
}

// The prefill kernels; k_new / v_new non-NULL: the chunks' rows are appended here.
static int prefill_chunks(const sp_cache_desc &c, const void *k_new, const void *v_new, const void *q, void *out, const int32_t *cu_q,
                          const int32_t *ctx_lens, const int32_t *block_table, int batch, int max_pages, int total_q, int max_q_len,
                          int max_kv_len, int num_q_heads, float scale, void *workspace, size_t workspace_bytes, hipStream_t stream) {
  PrefillArgs a;
  a.k_pages = (const char *)c.k_pages;
  a.v_pages = (const char *)c.v_pages;
  a.q = (const char *)q;
  a.out = (char *)out;
  a.cu_q = cu_q;
  a.ctx_lens = ctx_lens;
  a.block_table = block_table;
  a.max_pages = max_pages;
  a.num_pages = c.num_pages;
  a.Hq = num_q_heads;
  a.Hkv = c.num_kv_heads;
  int group = num_q_heads / c.num_kv_heads;
  // Stack the heads of a group into the column dimension when the group size is a power of
  // two (<= 32); otherwise every query head gets its own tiles.
  int gshift = 0;
  if ((group & (group - 1)) == 0)
    while ((1 << gshift) < group && gshift < 5) ++gshift;
  a.gshift = gshift;
  a.n_hgroups = num_q_heads >> gshift;
  a.ntiles_x = 0;
  a.sl2e = scale * 1.44269504088896340736f;
  a.tau = 8.0f / a.sl2e;

  // ---- shape of the launch, from host-side counts only
  const long rows = (long)total_q * num_q_heads;
  const long wg128 = estimate_wg128(rows, batch, a.n_hgroups);
  const bool small_grid = g_split_mode == 0 ? is_small_grid(wg128) : g_split_mode == 2;
  // Pieces of the key ranges, bounded by what the caller's workspace holds.
  const size_t slot_bytes = (size_t)(c.head_dim + 2) * sizeof(float);
  int kvs = 1;
  if (workspace && rows > 0) {
    if (g_kv_splits > 0) {
      kvs = g_kv_splits;
    } else if (small_grid) {
      kvs = kv_pieces(wg128, max_kv_len);
    }
    const int cap = kv_split_cap(rows);
    if (kvs > cap) kvs = cap;
    const size_t fit = workspace_bytes / ((size_t)rows * slot_bytes);
    if ((size_t)kvs > fit) kvs = (int)fit;
    if (kvs < 1) kvs = 1;
  }
  // Mixed batch: short sequences go to the split kernel (launched last, below) when the workspace
  // holds their partials; the prefill kernel then skips them, and its key ranges stay uncut (the
  // longest key range of the batch, which sizes the pieces, belongs to a short sequence as a rule).
  a.route_cap = 0;
  {
    const int cap = mixed_route_cap(batch, total_q, max_q_len, num_q_heads, c.num_kv_heads);
    const size_t need = cap > 0 ? decode_routed_workspace_bytes(batch, max_kv_len, num_q_heads, c.num_kv_heads, c.head_dim) : 0;
    if (need > 0 && workspace && workspace_bytes >= need) {
      a.route_cap = cap;
      if (g_kv_splits == 0) kvs = 1;
    }
  }
  a.kv_splits = kvs;
  // Heaviest-first dispatch when the static (tile, sequence) order is not already that: several
  // sequences with cached prefixes (without prefixes the last query tiles of all sequences are
  // the heaviest items, and they are first in the static order too).
  a.batch = batch;
  a.total_q = total_q;
  const bool can_rank = batch <= 64 * kRankSlots;
  // Without prefixes too where the static order hands every XCD its own sequences (a multiple of 8 (sequence, head
  // group) streams, not all head groups of a sequence spread over the XCDs) and their lengths differ, i.e. fill less than
  // 0.9 of the batch's longest: the XCDs with the longer ones finish last.  8 sequences of up to 7473 tokens, 8q/1kv
  // d 128, filled 0.62: 646 us, ranked 336; 8 of up to 1868, 16q/2kv d 64, 0.73: 75 and 53; 8 of up to 2853, 12q/3kv d 64,
  // 0.75: 94 and 87; filled 0.94 and more: 2 to 9 % slower ranked (the search, and K/V tiles from other XCDs' L2s).
  // Below 512 tokens the search's microsecond shows (35.6 us, ranked 38.2), and where the longest sequences together give
  // an XCD no more workgroups than its 32 CUs there is nothing to even out (8 of up to 985 at 2q/1kv d 64: 14.7 and 15.6).
  const long streams = (long)batch * a.n_hgroups;
  const bool uneven = a.n_hgroups % 8 != 0 && streams % 8 == 0 && max_q_len >= 512 && 10L * total_q < 9L * batch * max_q_len &&
                      streams / 8 * (((long)max_q_len << a.gshift) / 128) > 32;
  a.ranked = can_rank && (g_order_mode == 0 ? batch >= 2 && (max_kv_len > max_q_len || uneven) : g_order_mode == 2);
  a.rank_shift = 6;
  while (a.rank_shift < 24 && (max_kv_len >> a.rank_shift) > 63) ++a.rank_shift;
  a.part_o = (float *)workspace;
  a.part_ml = a.part_o + (size_t)rows * kvs * c.head_dim;
#ifdef SP_PREFILL_TRACE
  if (kvs == 1 && (a.route_cap > 0 || workspace_bytes < kTraceBytes)) a.part_o = nullptr;  // no room for the timeline
#endif

  // Batches whose items may be of very different lengths: the CUT form.
  a.cut_slots = 0;
  {
    const int slots = g_split_mode == 0 && g_kv_splits == 0 && g_order_mode == 0 ? cut_slots(batch, total_q, max_q_len, max_kv_len, num_q_heads, c.num_kv_heads, c.head_dim) : 0;
    if (slots > 0 && workspace && workspace_bytes >= cut_bytes(slots, c.head_dim)) {
      a.cut_slots = slots;
      a.kv_splits = kvs = 1;
      a.ranked = 1;
      a.cut_used = (int32_t *)workspace;
      a.cut_tab = (CutEntry *)((char *)workspace + 256);
      a.part_ml = (float *)(a.cut_tab + slots);
      a.part_o = a.part_ml + (size_t)slots * 512;
    }
  }
  const bool split = kvs > 1 || (small_grid && !(g_split_mode == 0 && a.route_cap == 0 && whole_tiles_pay(rows, streams, max_kv_len)));
  // Append and prefill in one launch: where the hints let it expect prompts without cached tokens.  Sequences of max_q_len tokens
  // at most that together have batch x max_q_len are all that long, and with max_kv_len no larger have no prefix.  The hints may
  // also stand for more tokens than there are (a sub-range, padded buffers), so that sequences do have prefixes, which may lie on
  // pages that the call appends: a workgroup that meets one sees to it that what it reads is there (fresh_plan.h).
  // An `out` that reuses the new rows' buffers would be written while others still read them; and the loads to LDS take 16 bytes of
  // the new rows at a time, which the append kernel does from any address.
  // The heads of a KV head have to share query tiles, of few enough rows that a thread moves a few chunks of them, and row offsets
  // are products of 24 bits.
  if (k_new) {
    const int tile = (split || c.head_dim == 64 ? 128 : 256) >> gshift;
    if ((group & (group - 1)) == 0 && tile * (c.head_dim / 8) <= kFreshChunks && (long)batch * max_q_len == total_q && max_kv_len <= max_q_len &&
        kvs == 1 && a.cut_slots == 0 && a.route_cap == 0 && (long)c.num_kv_heads * c.head_dim * 2 < (1L << 23) &&
        apart(out, rows * c.head_dim * 2, k_new, rows / group * c.head_dim * 2) && apart(out, rows * c.head_dim * 2, v_new, rows / group * c.head_dim * 2) &&
        (((uintptr_t)k_new | (uintptr_t)v_new) & 15) == 0) {
      FreshArgs f;
      static_cast<PrefillArgs &>(f) = a;
      f.k_new = (const char *)k_new;
      f.v_new = (const char *)v_new;
      f.new_pages = most_new_pages(max_q_len);
      return launch_prefill_fresh(f, split, c.head_dim, batch, max_q_len, stream);
    }
    if (int rc = launch_kv_append(c, k_new, v_new, cu_q, ctx_lens, block_table, batch, max_pages, total_q, stream)) return rc;
  }
  // Mixed batch: both kinds of workgroups in one launch where the prefill ones take items by rank and the cached keys are
  // up to kMixedBytes, all sequences taken as long as the longest.  Beyond that the decode half alone saturates HBM
  // with all CUs, and starting on a part of them costs more than it hides (0.66 GB of keys: 148 us as two launches, 157 as one;
  // 1.3 GB: 234 and 250; 0.17 GB: 51.6 and 45.9; smaller shares for the CUs that come late: the same there, and 8q/1kv
  // batches of 30 MB 21 -> 25 us).
  constexpr long kMixedBytes = 640L << 20;
  if (a.route_cap > 0 && (long)batch * c.num_kv_heads * max_kv_len * c.head_dim * 4 <= kMixedBytes && a.ranked && a.cut_slots == 0 && kvs == 1 && g_split_mode == 0 && g_kv_splits == 0 && g_order_mode == 0) {
    DecodeArgs d;
    int shares, pieces;
    if (plan_decode_routed(d, c, q, out, cu_q, ctx_lens, block_table, batch, max_pages, max_kv_len, num_q_heads, scale, workspace,
                           workspace_bytes, &shares, &pieces)) {
      const int rc = launch_mixed(a, d, shares, pieces, split, c.head_dim, batch, max_q_len, stream);
      if (rc != 1) return rc;
    }
  }
  int rc = a.cut_slots > 0 ? launch_prefill_cut(a, c.head_dim, batch, max_q_len, cut_merge_groups(batch, total_q, max_kv_len, num_q_heads, a.n_hgroups, g_cut_mode == 2), stream)
           : c.head_dim == 128 ? launch_prefill_d<128>(a, split, batch, max_q_len, stream)
                             : launch_prefill_d<64>(a, split, batch, max_q_len, stream);
  if (rc != SP_OK) return rc;
  if (kvs > 1) {
    rc = launch_combine(a.part_o, a.part_ml, out, rows, kvs, c.head_dim, stream, cu_q, batch, num_q_heads);
    if (rc != SP_OK) return rc;
  }
  if (a.route_cap > 0) {
    // ... and the short sequences of a mixed batch on the split kernel, in the same stream: it runs
    // after the launches above, so it may reuse the workspace, and its rows are its own.
    rc = launch_decode_multi(c, nullptr, nullptr, q, out, cu_q, ctx_lens, block_table, batch, max_pages, total_q, max_q_len,
                             max_kv_len, num_q_heads, scale, workspace, workspace_bytes, stream, true);
    if (rc == 1) return fail(SP_ERR_WORKSPACE, "sp_attn_prefill: workspace too small for the routed short sequences");
  }
  return rc;
}

}  // namespace sp
