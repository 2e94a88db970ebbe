// The arithmetic of the prefill form that cuts long work items (CUT in prefill_tile.h): which launches take it, how many
// workgroups and partial slots they get, and from which length on the items are cut.  Plain integer code that
// compiles for the host as well: the kernel runs it with a wave's lanes and their reductions, the CPU tests with one
// "lane" that holds the whole batch.
#pragma once

#ifdef __HIP__
#define SP_HD __host__ __device__ __forceinline__
#else
#define SP_HD inline
#endif

namespace sp {

constexpr int kRankSlots = 4;       // sequences per lane: ranked batches hold up to 64 * kRankSlots
constexpr int kMaxCutPieces = 16;   // pieces of an item at most
constexpr int kMinCutTiles = 8;     // key tiles that are never cut further
constexpr int kCutShare = 256;      // CUs the key tiles are shared out to
constexpr int kMostExtraPieces = 205;  // workgroups beyond one per item: fewer than total tiles / limit <= 256 / 1.25
constexpr int kMostCutSlots = 416;     // pieces of cut items: at most 2 * 256 / 1.25, rounded up
constexpr int kMostSeqTiles = 1 << 22;  // key tiles of one sequence's items that cut_limit's sum can hold

SP_HD int imin(int a, int b) { return a < b ? a : b; }
SP_HD int imax(int a, int b) { return a > b ? a : b; }

// first query tile of a sequence (c cached and q new keys, nt tiles) that sees at least `keys` keys; nt if none does
SP_HD int first_tile_ge(int c, int q, int nt, int keys, int tpt_shift) {
  if (nt == 0 || c + q < keys) return nt;
  const int d = imax(keys - c, 0);
  const int j0 = ((d + (1 << tpt_shift) - 1) >> tpt_shift) - 1;
  return imin(imax(j0, 0), nt - 1);
}

constexpr int kMaxKvSplits = 16;
constexpr long kMaxPartialSlots = 1L << 17;  // (row, split) pairs the workspace is ever sized for

// Largest number of key-range pieces a batch of `rows` (token, head) rows may be cut into.
inline int kv_split_cap(long rows) {
  if (rows <= 0) return 1;
  long cap = kMaxPartialSlots / rows;
  return (int)(cap < 1 ? 1 : cap > kMaxKvSplits ? kMaxKvSplits : cap);
}

// Up to about one 256-column workgroup per CU: let the two wave groups split the key range of
// 128 columns instead (halves the critical path of the longest work item; measured faster up
// to that grid size, slower beyond it because every K/V tile is then staged for half the
// columns).
constexpr int kSmallGrid = 576;  // 128-column workgroups
inline bool is_small_grid(long wg128) { return wg128 <= kSmallGrid; }

// ... unless the halves are more than one round of workgroups, and short: a second round costs 5 to 8 us of starts, merges and
// stores, where whole tiles of 256 columns (or several workgroups a CU at head_dim 64) are one round and take 0.35 us longer per
// key tile.  The line over the longest key range in tiles and n = rows / 128, measured on 150 batches of 20 to 2350 tokens
// (us in halves and whole): 24 x 79..132 tokens at 16q/2kv 21.8 and 13.7; 8 x 800..1200 at 8q/1kv (n 500, 19 tiles) 39.9 and
// 29.7; 4 x 562..937 at 16q/2kv (375, 15) 27.5 and 24.2; 8 x 602 at 12q/3kv d 64 (451, 10) 16.0 and 13.8; 24 x 138 at 16q/2kv
// d 64 12.3 and 9.3; on the other side 1 x 1032 at 32q/8kv (258, 17) 21.5 and 24.3, 2 x 2037 at 12q/3kv d 64 (382, 32) 23.1 and
// 29.9, chunks of 256 tokens on prefixes of 1300 at 16q/2kv (512, 34) 57.0 and 76.2.  At the edge of the second round
// (3 x 688 at 16q/2kv d 64, 258 workgroups) 11.8 and 12.2, so it starts a little past 256.
inline bool whole_tiles_pay(long rows, long streams, long max_kv_len) {
  const long n = rows / 128, tiles = (max_kv_len + 63) / 64;
  return n + streams / 2 > 264 && tiles <= (n > 512 ? 40 : 13 + (n - 256) * 23 / 512);
}

// How many pieces the key range of a query tile of a small grid is cut into (1 = none): only when even the
// 128-column workgroups leave most CUs idle and the key ranges are long.  A piece's partial costs about as much HBM time
// as 500 keys cost matrix time, so pieces stay around 1500 keys or longer.
inline int kv_pieces(long wg128, long max_kv_len) {
  const long by_grid = 256 / (wg128 > 0 ? wg128 : 1);
  const long by_len = max_kv_len / 1536;
  return (int)(by_grid < by_len ? by_grid : by_len);
}

// 128-column workgroups that find work, estimated: rows / 128 plus half a partial tile per sequence and head group.
inline long estimate_wg128(long rows, int batch, long n_hgroups) { return rows / 128 + ((long)batch * n_hgroups + 1) / 2; }

// Whether a batch on cached prefixes takes the form, from the hints: batch sequences of `columns` query columns (tokens x
// heads in the column dimension) per head group on average, `streams` head groups of all sequences, keys up to
// max_kv_len.  narrow: the launch has 128-column workgroups otherwise, in `pieces` pieces each (else whole 256-column ones).
// Times are compared in key tiles of a workgroup.  The lengths are not known here: a sequence is taken to be 0.6 of the
// longest (narrow) or 0.4 (one alone: all of it), and what a whole launch waits for beyond the mean load of a CU to be 0.2 or
// 0.4 of its longest item.  Pieces by the hints leave partials of all rows, row_values each, which their merge reads; the
// form itself costs a merge and the search, 4 tiles in place of the narrow form and 20 in place of whole items (5-8 us even
// where the device finds nothing to cut).  The numbers are those that leave the least behind on 420 batches (equal, uniform,
// cubed and lognormal lengths, 1..200 sequences, 40..8192 columns, up to 60000 keys, nine head shards; both forms timed):
// 13.3 % of the time is gained over never cutting, 24 batches lose more than 3 %, 9 % on average and 25 % at most (5 chunks of
// up to 741 tokens at 16q/2kv: 216-229 and 269 us).  Without the merge of the pieces by hints it was 12.8 %: 7 x 137 tokens on up
// to 4660 keys at 16q/2kv 51.2 us in pieces, 30.6 cut; 13 chunks of up to 222 at 6q/2kv 50.3 and 33.0.
// Both sides of it:
//   1 x 64 tokens on 20000 keys, 8q/1kv: 30.4 us in 13 pieces of 128 columns, 39.6 cut; on 5500 keys 28.4 and 21.9 (an item
//   has kMaxCutPieces at most, each walked by one workgroup, where two wave groups share the narrow form's);
//   64 x 37 tokens of up to 6000 keys, 12q/3kv (columns for 1.2 tiles of 256): 92.6 and 124.5;
//   32 chunks of 512 tokens on up to 8192 keys: 164 whole, 106 cut; 549 items, longest 484 tiles: 518 and 359; 600 items, longest
//   27 tiles: 61.6 and 69 (nothing to gain: all items are short next to what a CU does).
inline bool cut_pays(int batch, long streams, double columns, long max_kv_len, bool narrow, int pieces, double row_values) {
  const double tiles = (double)((max_kv_len + 63) / 64), mean = batch == 1 ? 1.0 : narrow ? 0.6 : 0.4;
  const double share = streams * (double)(long)((columns + 255.99) / 256) * tiles * mean / kCutShare;
  double cut = 1.25 * share;
  if (cut < tiles / kMaxCutPieces) cut = tiles / kMaxCutPieces;
  if (cut < kMinCutTiles) cut = kMinCutTiles;
  const double longest = narrow ? tiles / (2 * pieces) : tiles;
  const double load = narrow ? 1.1 * streams * (double)(long)((columns + 127.99) / 128) * tiles * mean / (2 * kCutShare) + 0.2 * longest
                             : share + 0.4 * longest;
  const double merge = narrow && pieces > 1 ? 2 + 0.5e-6 * row_values * pieces : 0;
  return cut + (narrow ? 4 : 20) < (load > longest ? load : longest) + merge;
}

// Whether a batch without cached prefixes takes it: its items are of all lengths already, so that few are long next to a CU's
// share.  Not below kCutNoPrefixItems or kCutNoPrefixKeys (201 items of up to 3484 keys 58 us, cut 63; 258 of 2048 60 and 68), not
// where the 128-column form serves sequences of one length (257 items, 4097 tokens at 16q/2kv d 64: 52 and 64; of
// different lengths 99 and 87), and beyond 390 items, where heaviest first evens them out alone, only for different lengths
// (412 items, 4 x 3281 at 8q/1kv: 102 and 108; filled 0.45 of the longest, 431 items: 305 and 198).  In between: 9 to 36 % faster.
constexpr int kCutNoPrefixItems = 240, kCutNoPrefixEvenMost = 390, kCutNoPrefixMost = 448, kCutNoPrefixKeys = 3072;
inline bool cut_pays_no_prefix(long items, int batch, long total_q, long max_q_len, long max_kv_len, bool narrow) {
  if (items < kCutNoPrefixItems || items > kCutNoPrefixMost || max_kv_len < kCutNoPrefixKeys) return false;
  const long full = batch * max_q_len;
  return narrow ? 20 * total_q < 19 * full : items <= kCutNoPrefixEvenMost || 10 * total_q < 9 * full;
}

// Up to this many items on fewer keys the pieces of 128 columns serve nearly as well, and the form is not worth its workspace.
constexpr int kCutFewItems = 8, kCutFewKeys = 4096;

// Whether the key tiles of a sequence of up to max_q_len new and max_kv_len visible keys stay within what cut_limit's
// sum can hold.  Beyond that its limit is too small: it cuts into more pieces than it should.
inline bool cut_countable(long max_q_len, int tpt, long max_kv_len) {
  return (max_q_len + tpt - 1) / tpt * (max_kv_len / 64 + 1) <= kMostSeqTiles;
}

inline long cut_pieces_by_tiles(int max_kv_len) { return (max_kv_len + 64 * kMinCutTiles - 1) / (64 * kMinCutTiles); }
inline int cut_cap(long slots) { return (int)(slots < kMostCutSlots ? slots : kMostCutSlots); }

// Slots for partials of the form (0: not taken), from the hints; forced: wherever it can be computed.
inline int cut_form_slots(int batch, int total_q, int max_q_len, int max_kv_len, int num_q_heads, int num_kv_heads, int head_dim,
                          bool forced) {
  if (batch <= 0 || batch > 64 * kRankSlots || total_q <= 0 || max_kv_len > (1 << 24)) return 0;
  const int group = num_q_heads / num_kv_heads;
  const int cols = (group & (group - 1)) == 0 ? (group < 32 ? group : 32) : 1;  // heads in the column dimension
  const long rows = (long)total_q * num_q_heads, streams = (long)batch * (num_q_heads / cols);
  const long items = rows / 256 + (streams + 1) / 2, most = rows / 256 + streams;
  if (most > (1 << 20) || !cut_countable(max_q_len, 256 / cols, max_kv_len)) return 0;
  if (!forced) {
    const long wg128 = estimate_wg128(rows, batch, num_q_heads / cols);
    if (max_kv_len <= max_q_len) {
      if (!cut_pays_no_prefix(items, batch, total_q, max_q_len, max_kv_len, is_small_grid(wg128))) return 0;
    } else {
      if (items <= kCutFewItems && max_kv_len < kCutFewKeys) return 0;
      const int by_hints = kv_pieces(wg128, max_kv_len), cap = kv_split_cap(rows);
      const int pieces = by_hints < 1 ? 1 : by_hints < cap ? by_hints : cap;
      if (!cut_pays(batch, streams, (double)total_q * cols / batch, max_kv_len, is_small_grid(wg128), pieces, (double)rows * head_dim)) return 0;
    }
  }
  // an item has ceil(tiles / kMinCutTiles) pieces at most, and kMaxCutPieces
  const long pieces = forced ? kMaxCutPieces : cut_pieces_by_tiles(max_kv_len);
  return cut_cap(most * (pieces < kMaxCutPieces ? pieces : kMaxCutPieces));
}

// Workgroups that the merge is wide: slots for a piece per kMinCutTiles key tiles, also where an item has fewer.
inline int cut_merge_groups(int batch, int total_q, int max_kv_len, int num_q_heads, int n_hgroups, bool forced) {
  const long most = (long)total_q * num_q_heads / 256 + (long)batch * n_hgroups;
  return cut_cap(most * (forced ? kMaxCutPieces : cut_pieces_by_tiles(max_kv_len)));
}

// Workgroups of a ranked launch: every sequence has at most q_len / tpt + 1 query tiles, and the cut items add their
// further pieces.
inline long ranked_workgroups(long total_q, int tpt, int batch, int n_hgroups, int kv_splits, int cut_slots) {
  return (total_q / tpt + batch) * n_hgroups * kv_splits + (cut_slots < kMostExtraPieces ? cut_slots : kMostExtraPieces);
}

// Items of more than the returned number of key tiles are cut; p: pieces of this lane's cut items, *total_pieces: of the
// batch's (each once per head group).  Called by all lanes; a lane holds the sequences u < nslot with c cached, q new
// tokens and nt query tiles.  slots, launched: partial slots and workgroups there are.
template <int N, typename Sum, typename Max>
SP_HD int cut_limit(const int (&c)[N], const int (&q)[N], const int (&nt)[N], int nslot, int tpt_shift, int n_hgroups, int slots,
                    int launched, Sum sum, Max most, int (&p)[N], int *total_pieces) {
  // key tiles of the whole launch and of its longest item
  const int tpt = 1 << tpt_shift;
  int w = 0, longest = 0;
#pragma unroll
  for (int u = 0; u < N; ++u)
    if (u < nslot && nt[u] > 0) {
      const float keys = (float)nt[u] * (float)c[u] + (float)tpt * 0.5f * (float)nt[u] * (float)(nt[u] - 1) + (float)q[u];
      const float tiles = keys * (1.0f / 64);
      w += (int)(tiles < (float)kMostSeqTiles ? tiles : (float)kMostSeqTiles) + 1;  // 256 sequences of at most 2^22 fit the sum
      longest = imax(longest, (c[u] + q[u] + 63) >> 6);
    }
  w = sum(w);
  longest = most(longest);
  const int base = imax((int)((float)w * (float)n_hgroups * (1.25f / kCutShare)) + 1, imax(kMinCutTiles, (longest + kMaxCutPieces - 1) / kMaxCutPieces));
  int limit = base;
  bool settled = false;
  for (;;) {
    int wgs = 0, total = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      p[u] = 0;
      if (u >= nslot) continue;
      wgs += nt[u];
      // an item of t tiles has one piece for every n >= 0 with t > n * limit
      for (int n = 1; n * limit < longest; ++n) {
        const int more = nt[u] - first_tile_ge(c[u], q[u], nt[u], 64 * n * limit + 1, tpt_shift);
        p[u] += (n == 1 ? 2 : 1) * more;
        wgs += more;
      }
      total += p[u];
    }
    total = sum(total);
    wgs = sum(wgs);
    // Whatever the estimate above says, nothing is dealt out that was not launched: a piece without a workgroup would leave its
    // rows unwritten and its slot's table entry stale.  Longer pieces are fewer, and a limit of `longest` cuts nothing.
    if (total > 0 && (total * n_hgroups > slots || wgs * n_hgroups > launched)) {
      limit *= 2;
      settled = true;
      continue;
    }
    *total_pieces = total;
    if (settled || wgs * n_hgroups <= kCutShare) break;
    // One round of workgroups, with pieces up to 1.2 times as long, before a second round of a few (6 chunks at 8q/1kv,
    // 114 items: 66 -> 55 us; 8 at 16q/2kv, 144 items: 62 -> 55.5; of 450 batches 18 are 4 to 47 % faster for it; where the second
    // round is full of short items it is the better one: 28 at 8q/1kv, 118 items: 62 and 59), unless the whole items
    // alone are more than one round.
    int items = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) items += nt[u];
    if (limit == base && sum(items) * n_hgroups > kCutShare) break;
    if (5 * limit >= 6 * base) {
      limit = base;
      settled = true;
    } else {
      limit += imax(1, base / 10);
    }
  }
  return limit;
}

}  // namespace sp
