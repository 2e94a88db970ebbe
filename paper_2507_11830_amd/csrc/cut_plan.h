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

// Whether the key tiles of a sequence of up to max_q_len new and max_kv_len visible keys stay within what cut_limit's
// sum can hold.  Beyond that its limit is too small: it cuts into more pieces than it should.
inline bool cut_countable(long max_q_len, int tpt, long max_kv_len) {
  return (max_q_len + tpt - 1) / tpt * (max_kv_len / 64 + 1) <= kMostSeqTiles;
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
  int items = 0;
#pragma unroll
  for (int u = 0; u < N; ++u) items += nt[u];
  bool settled = sum(items) * n_hgroups > kCutShare;
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
    // 114 items: 66 -> 55 us; 8 at 16q/2kv, 144 items: 62 -> 55.5; 2 at 32q/4kv, 206 items: 134 -> 129; where the second
    // round is full of short items it had been the better one: 28 at 8q/1kv, 118 items: 57 -> 60; up to 1 us elsewhere).
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
