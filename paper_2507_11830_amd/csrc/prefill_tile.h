// The prefill attention kernel (attn_prefill.hip says what it computes and what bounds it), shared by the files that
// instantiate it: attn_prefill.hip and attn_prefill_cut.hip.
#pragma once
#include <type_traits>

#include "attn_tile.h"
#include "cut_plan.h"
#include "fresh_plan.h"

namespace sp {

// Scheduling pattern of a software-pipelined MFMA sequence of N operands starting at fused
// index I0 (indices below NPV are V^T operands = 2 LDS reads, the rest K operands = 1 read):
// PFD operand reads up front, then "read operand i+PFD, MFMA i".  The group sizes must be
// compile-time constants, hence the recursion.
template <int I, int N, int I0, int NPV, int PFD>
__device__ __forceinline__ void sgb_prologue() {
  if constexpr (I < PFD && I < N) {
    if constexpr (I0 + I < NPV) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    else __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    sgb_prologue<I + 1, N, I0, NPV, PFD>();
  }
}
template <int I, int N, int I0, int NPV, int PFD, int VPM, int NE = N>
__device__ __forceinline__ void sgb_steady() {  // MFMAs [I, NE) of a sequence of N
  if constexpr (I < NE) {
    if constexpr (I + PFD < N) {
      if constexpr (I0 + I + PFD < NPV) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      else __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    // VPM plain VALU instructions ride behind every PV MFMA (the row sums of the weights it multiplies)
    if constexpr (VPM > 0 && I0 + I < NPV) __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
    sgb_steady<I + 1, N, I0, NPV, PFD, VPM, NE>();
  }
}

// Measurement switches (compile-time, all off in the product build; the profiles record what each
// costs): -DSP_PREFILL_ALWAYS_FULL computes the tile max in every tile (the full softmax pass
// everywhere); -DSP_PREFILL_SUM_DOT2 sums the bf16-rounded weight pairs with the dot-product
// instruction and -DSP_PREFILL_SUM_MFMA with 4x4x4 MFMAs against an all-ones operand, instead of
// adding the fp32 weights (both go through the matrix pipe, where they queue behind the other
// wave's 32-cycle MFMAs: a third more cycles for the whole kernel); -DSP_PREFILL_SUM_IN_MATRIX_PHASE
// moves the row sum out of the softmax phase, behind the PV MFMAs of the next matrix phase (unpack
// the rounded weights by shift / mask, add: four plain VALU instructions per MFMA, which a lone
// wave hides behind its MFMAs in an issue probe — in this kernel they cost 13 % more time);
// -DSP_PREFILL_PRIO raises the wave priority during the matrix phases; -DSP_PREFILL_QSCALED folds
// scale * log2(e) into the resident Q operand and anchors the running max at 0 where the first
// tile allows it, so that the common softmax pass is exp2, add and half a convert per score (2.5
// VALU instructions instead of 3.5) — no change in time at head_dim 128, 9 % faster at head_dim
// 64 while this kernel served its whole tiles (those are prefill_solo.h's now; here head_dim 64 is the halved, cut and mixed forms),
// at the price of a score error that grows with the score; -DSP_PREFILL_BARRIER_IN_SEQ puts the
// second group's barrier before the last four MFMAs of its matrix phase, so that the first
// group's operand reads after the barrier run behind them — no change in time either.
// -DSP_PREFILL_TRACE makes launches that do not use the workspace otherwise (no key-range pieces,
// no routed short sequences) write a timeline into it: per workgroup the 100 MHz wall clock at its
// start, after the prologue's barrier, at the end of either wave group's tile loop and at its end,
// its tile count and the CU it ran on, and for every eighth tile period of the first group the
// wall clock and the shader clock (paper_2507_11830_amd/trace_prefill.py reads it).
#ifdef SP_PREFILL_TRACE
constexpr int kTraceWgs = 8192, kTraceRec = 8, kTracePer = 64;  // workgroups covered, longs per record, period stamps
constexpr size_t kTraceBytes = (size_t)kTraceWgs * (kTraceRec + 2 * kTracePer) * sizeof(long);
#define SP_TRACE_STAMP(slot, tid)                                                  \
  do {                                                                             \
    if (trace_rec && threadIdx.x == (tid)) trace_rec[slot] = (long)wall_clock64(); \
  } while (0)
#else
#define SP_TRACE_STAMP(slot, tid)
#endif
#ifdef SP_PREFILL_PRIO
#define SP_MATRIX_PHASE_BEGIN() __builtin_amdgcn_s_setprio(3)
#define SP_MATRIX_PHASE_END() __builtin_amdgcn_s_setprio(0)
#else
#define SP_MATRIX_PHASE_BEGIN()
#define SP_MATRIX_PHASE_END()
#endif
#ifdef SP_PREFILL_ALWAYS_FULL
constexpr bool kAlwaysFullSoftmax = true;
#else
constexpr bool kAlwaysFullSoftmax = false;
#endif
#ifdef SP_PREFILL_BARRIER_IN_SEQ
constexpr bool kBarrierInSeq = true;
#else
constexpr bool kBarrierInSeq = false;
#endif
#ifdef SP_PREFILL_QSCALED
constexpr bool kScaledQSwitch = true;
#else
constexpr bool kScaledQSwitch = false;
#endif

constexpr int KVT = 64, PFD = 4;  // keys per tile; operands read ahead of the MFMAs

// What the merge of a cut work item has to know; one per partial slot.
struct CutEntry {
  int32_t q0, q_len, tile, hg;
  int32_t pieces;  // partials of the item, which starts at this slot; 0: the slot belongs to an item before it
  int32_t stride;  // slots between two partials of the item
  int32_t pad[2];
};

struct PrefillArgs {
  const char *k_pages, *v_pages, *q;
  char *out;
  const int32_t *cu_q, *ctx_lens, *block_table;
  int max_pages, num_pages, Hq, Hkv, gshift, n_hgroups, ntiles_x;
  float sl2e;  // scale * log2(e)
  float tau;   // lazy-rescale threshold in raw score units (8 / sl2e)
  // PART kernels: blockIdx.z of kv_splits workgroups share a query tile's key range and write
  // un-normalised partials [row][kv_splits][D] and (max in log2 units, sum) [row][kv_splits][2]
  float *part_o, *part_ml;
  int kv_splits;
  int batch;
  int total_q;     // host count of query tokens (bounds the number of work items)
  int ranked;      // workgroups take their work items heaviest first (ranked_item below)
  int rank_shift;  // log2 of the weight unit in keys
  int route_cap;   // mixed batches: sequences with at most this many query tokens belong to the split kernel (0: none)
  // CUT kernels: up to cut_slots partials [slot][register-order D x 256 columns] in part_o, [slot][256][2] in part_ml
  int cut_slots;
  CutEntry *cut_tab;
  int32_t *cut_used;  // number of slots in use
};

// FreshArgs: the chunks' rows are not in the cache yet.  A workgroup takes its new keys from the new rows themselves, its
// cached ones from the pool (fresh_plan.h), and appends the rows of its own query tile.
struct FreshArgs : PrefillArgs {
  const char *k_new, *v_new;  // bf16 [total_q][Hkv][D]
  int new_pages;              // pages that the new rows of a sequence reach into, at most
};
constexpr int kFreshChunks = 1024;  // 16-byte chunks of K (and of V) in the rows of a query tile, at most: a few per thread

__device__ __forceinline__ int wave_total(int x) { return __builtin_amdgcn_readlane(wave_scan_incl(x), 63); }
// Wave-wide max of non-negative values, wave-uniform (same DPP steps; a lane without a source lane
// contributes 0).
__device__ __forceinline__ int wave_max_i(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false));
  return __builtin_amdgcn_readlane(x, 63);
}

// Ranked dispatch.  The hardware starts workgroups in linear id order and a CU takes the next one
// when it has room, so the launch is a list schedule and its makespan depends on the list's
// order: longest items first is the classic 4/3 rule, and a chunked-prefill batch whose sequences
// sit on cached prefixes of very different lengths is far from it in (tile, sequence) order (the
// early query tiles of the sequence with the longest prefix are as heavy as anything in the batch
// but would start last).  Here the workgroup with linear id r finds the r-th heaviest (sequence,
// query tile) item by itself: the weight of an item is its number of visible keys in units of
// 2^rank_shift keys (the host picks the unit so that the heaviest item weighs at most 63: finer
// classes would not change the makespan, and every doubling costs a probe), the number of items at
// least as heavy as x is a sum over sequences of a closed form, so a binary search over x and one
// prefix sum over the ties select the item in a few hundred instructions, from the same two
// length arrays every workgroup reads anyway.  Ties are taken sequence by sequence, later tiles first.  One
// sequence per lane and slot: batches of up to 64 * kRankSlots sequences.  The search is a chain
// of dependent cross-lane operations in a single wave (about 0.2 us per probe), which is why the
// probes are few and DPP, not LDS permutes, carries them.
struct RankedItem {
  int seq, tile;
  int q0, q_len, ctx;  // the sequence's entries of the length arrays, so that nobody has to load them again
  int piece, pieces;   // CUT: which piece of the item's key range, of how many
};

// CUT: items longer than `limit` key tiles are cut into ceil(tiles / limit) equal pieces, and the pieces come
// before all uncut items in the order.  limit is 5/4 of what a CU's equal share of the launch's key tiles is: an item
// beyond that would still run when every other CU has finished, while a shorter one is cheaper whole (a piece
// repeats the prologue, 5 us or three key tiles, and writes a partial).  Pieces are half a limit long at
// least, so they number at most 2 x 256 / 1.25.
template <bool CUT>
__device__ __forceinline__ bool ranked_item(const PrefillArgs &a, int tpt_shift, int r, int lane, RankedItem *out) {
  const int tpt = 1 << tpt_shift;
  int c[kRankSlots], q[kRankSlots], nt[kRankSlots], qs[kRankSlots], q_all[kRankSlots];
  const int nslot = (a.batch + 63) >> 6;  // uniform
#pragma unroll
  for (int u = 0; u < kRankSlots; ++u) {
    const int s = u * 64 + lane;
    c[u] = q[u] = nt[u] = qs[u] = 0;
    if (u < nslot && s < a.batch) {
      const int q0 = a.cu_q[s];
      qs[u] = q0;
      q[u] = max(a.cu_q[s + 1] - q0, 0);
      if (q[u] <= a.route_cap) q[u] = 0;  // served by the split kernel (route_cap = 0: nothing is)
      c[u] = max(a.ctx_lens[s], 0);
      nt[u] = (q[u] + tpt - 1) >> tpt_shift;
    }
    q_all[u] = q[u];
  }
  out->piece = 0;
  out->pieces = 1;
  int wsh = a.rank_shift;
  if (CUT) {
    int p[kRankSlots], total;  // pieces of cut items
    const int limit = cut_limit(c, q, nt, nslot, tpt_shift, a.n_hgroups, a.cut_slots, (int)gridDim.x, wave_total, wave_max_i, p, &total);
    if (r == 0 && out->tile == 0 && threadIdx.x == 0) *a.cut_used = total * a.n_hgroups;  // out->tile: the caller's head group
    if (r < total) {
      int k = r, at = -1;
#pragma unroll
      for (int u = 0; u < kRankSlots; ++u) {
        if (u >= nslot || at >= 0) continue;
        const int incl = wave_scan_incl(p[u]);
        const int tot = __builtin_amdgcn_readlane(incl, 63);
        if (k >= tot) {
          k -= tot;
          continue;
        }
        const int ln = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl > k));
        k -= __builtin_amdgcn_readlane(incl - p[u], ln);
        at = u * 64 + ln;
        out->q0 = __builtin_amdgcn_readlane(qs[u], ln);
        out->q_len = __builtin_amdgcn_readlane(q[u], ln);
        out->ctx = __builtin_amdgcn_readlane(c[u], ln);
      }
      out->seq = at;
      // the sequence's items from its last tile down: first those of most pieces
      const int tiles = (out->q_len + tpt - 1) >> tpt_shift;
      int hi = tiles;
      for (int n = ((out->ctx + out->q_len + 63) / 64 + limit - 1) / limit; n >= 2; --n) {
        const int lo = first_tile_ge(out->ctx, out->q_len, tiles, 64 * (n - 1) * limit + 1, tpt_shift);
        if (k < (hi - lo) * n) {
          out->tile = hi - 1 - k / n;
          out->piece = k % n;
          out->pieces = n;
          return true;
        }
        k -= (hi - lo) * n;
        hi = lo;
      }
      return false;  // not reached
    }
    r -= total;
    // the uncut items: every sequence's tiles up to `limit` key tiles
#pragma unroll
    for (int u = 0; u < kRankSlots; ++u) {
      const int n = first_tile_ge(c[u], q[u], nt[u], 64 * limit + 1, tpt_shift);
      if (n < nt[u]) {
        nt[u] = n;
        q[u] = n << tpt_shift;
      }
    }
    wsh = 6;
    while ((limit >> (wsh - 6)) > 63) ++wsh;
  }
  // first tile of slot u's sequence whose weight is >= x units (nt[u] if none); x never exceeds the heaviest item's weight + 1
  auto first_ge = [&](int u, int x) { return first_tile_ge(c[u], q[u], nt[u], x << wsh, tpt_shift); };
  auto total_ge = [&](int x) {
    int n = 0;
#pragma unroll
    for (int u = 0; u < kRankSlots; ++u)
      if (u < nslot) n += nt[u] - first_ge(u, x);
    return wave_total(n);
  };
  int n_items = 0, wmax = 0;
#pragma unroll
  for (int u = 0; u < kRankSlots; ++u) {
    n_items += nt[u];
    wmax = max(wmax, nt[u] ? (c[u] + q[u]) >> wsh : 0);
  }
  if (r >= wave_total(n_items)) return false;  // more workgroups than items
  wmax = wave_max_i(wmax);
  int lo = 0, hi = wmax + 1, n_hi = 0;  // total_ge(lo) > r >= total_ge(hi) = n_hi
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    const int n = total_ge(mid);
    if (n > r) {
      lo = mid;
    } else {
      hi = mid;
      n_hi = n;
    }
  }
  // the item weighs exactly lo units; it is number k among those, counted in sequence order
  int k = r - n_hi;
  bool found = false;
#pragma unroll
  for (int u = 0; u < kRankSlots; ++u) {
    if (u >= nslot || found) continue;
    const int j0 = first_ge(u, lo);
    const int ties = first_ge(u, lo + 1) - j0;  // this sequence's items of weight lo: tiles j0 .. j0 + ties - 1
    const int incl = wave_scan_incl(ties);
    const int tot = __builtin_amdgcn_readlane(incl, 63);
    if (k < tot) {
      const unsigned long long at = __builtin_amdgcn_ballot_w64(incl > k);
      const int ln = __builtin_ctzll(at);
      const int before = __builtin_amdgcn_readlane(incl - ties, ln);
      out->seq = u * 64 + ln;
      const int t_ln = __builtin_amdgcn_readlane(ties, ln);
      out->tile = __builtin_amdgcn_readlane(j0, ln) + (t_ln - 1 - (k - before));  // the sequence's later (heavier) tiles first
      out->q0 = __builtin_amdgcn_readlane(qs[u], ln);
      out->q_len = __builtin_amdgcn_readlane(q_all[u], ln);
      out->ctx = __builtin_amdgcn_readlane(c[u], ln);
      found = true;
    } else {
      k -= tot;
    }
  }
  return found;
}

// The work item of a workgroup of 2^cols_shift query columns, wave-uniform; false: there is none for it.
// Workgroups are dispatched in blockIdx.x-major order: the longest key ranges of ALL sequences
// go first, the short ones fill in behind them.
// Consecutive workgroup ids go round-robin over the 8 XCDs; with the (sequence, head group)
// index rotated by the tile index, the workgroups of one sequence spread over all XCDs even
// when the batch size is a multiple of 8 (unrotated, each sequence would sit on one XCD and a
// batch of unequal lengths would leave most of the chip idle).
struct WorkItem {
  int seq, hg, tile, q0, q_len, ctx;
  int piece, pieces;  // which piece of the key range; CUT: of how many
  int slot;           // CUT: partial slot of the piece
};
template <int CUT, bool SNAKE = false>
__device__ __forceinline__ bool take_item(const PrefillArgs &a, int cols_shift, int lane, WorkItem *o) {
  o->pieces = 1;
  o->slot = 0;
  unsigned lid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), bx = blockIdx.x, by = blockIdx.y;
  if constexpr (SNAKE) {
    // Several workgroups are resident on a CU: each round of 256 gives every CU one.  The second round goes from the lightest of
    // its items up, so that no CU has the heaviest item of both (head_dim 64, without and with: 4 x 1500 tokens at 16q/2kv 30.7 and
    // 28.8 us, 4 x 3000 at 12q/3kv 71.5 and 69.2, 8 x 1200 38.6 and 39.0; more rounds even themselves out, 2 x 16k 774 and 775).
    if (lid >= 256 && lid < 512) {
      const unsigned xcd = lid & 7, p = (lid >> 3) - 32, total = gridDim.x * gridDim.y * gridDim.z;
      const unsigned n = ((total < 512 ? total : 512) - 256 - xcd + 7) >> 3;  // this XCD's of the round
      lid = ((32 + n - 1 - p) << 3) | xcd;
      by = lid / gridDim.x;
      bx = lid - by * gridDim.x;
    }
  }
  if (CUT || a.ranked) {
    // linear id -> (item rank, head group, piece): the pieces and head groups of an item are
    // neighbours in the dispatch order, i.e. they start together and spread over the XCDs
    const unsigned per_item = (unsigned)(a.n_hgroups * a.kv_splits);
    const int r = (int)(lid / per_item);
    const int sub = (int)(lid - (unsigned)r * per_item);
    o->hg = sub / a.kv_splits;
    o->piece = sub - o->hg * a.kv_splits;
    RankedItem it;
    it.tile = o->hg;
    if (!ranked_item<CUT>(a, cols_shift - a.gshift, r, lane, &it)) return false;
    if (CUT) {
      o->piece = __builtin_amdgcn_readfirstlane(it.piece);
      o->pieces = __builtin_amdgcn_readfirstlane(it.pieces);
      o->slot = (int)lid;  // pieces of cut items come first: the launch index is the partial's slot
    }
    o->seq = __builtin_amdgcn_readfirstlane(it.seq);
    o->tile = __builtin_amdgcn_readfirstlane(it.tile);
    o->q0 = __builtin_amdgcn_readfirstlane(it.q0);
    o->q_len = __builtin_amdgcn_readfirstlane(it.q_len);
    o->ctx = __builtin_amdgcn_readfirstlane(it.ctx);
    return true;
  }
  int sh, row;
  if ((gridDim.x & 7) == 0) {
    // A multiple of 8 (sequence, head group) streams: every XCD gets its own streams with ALL their
    // query tiles (workgroup ids go round-robin over the XCDs, so XCD x sees the ids = x mod 8),
    // heaviest tiles first.  The workgroups an XCD runs at any moment then belong to a few
    // streams and sit at neighbouring query tiles, so they walk the same K/V pages nearly in
    // step and the XCD's L2 serves most of their tile loads (rotating streams over the XCDs
    // instead puts about one workgroup per stream on an XCD, and every tile load misses L2).
    const unsigned xcd = lid & 7, p = lid >> 3, spx = gridDim.x >> 3;
    row = (int)(p / spx);
    sh = (int)((p - (unsigned)row * spx) * 8 + xcd);
  } else {
    sh = (int)((bx + by + blockIdx.z) % gridDim.x);
    row = (int)(by + gridDim.y * blockIdx.z);
  }
  o->seq = sh / a.n_hgroups;
  o->hg = sh - o->seq * a.n_hgroups;
  o->piece = SNAKE ? 0 : row / (int)gridDim.y;  // SNAKE kernels have no pieces: their blockIdx.z is the second half of many tiles
  o->tile = a.ntiles_x - 1 - (row - o->piece * (int)gridDim.y);
  if (SNAKE && o->tile < 0) return false;
  o->ctx = a.ctx_lens[o->seq];
  o->q0 = a.cu_q[o->seq];
  o->q_len = a.cu_q[o->seq + 1] - o->q0;
  return o->q_len > a.route_cap;  // mixed batch: the split kernel serves the others
}

// What lane l of load instruction j of a page brings in: the 16-byte chunk `chunk` of the page's row `row`, as the swizzle of K's, or V's,
// tile has it.
struct PageChunk {
  int row, chunk;
};
template <int D>
__device__ __forceinline__ PageChunk page_chunk(bool is_v, int j, int l) {
  using Z = SwzTile<D>;
  const int lp = 4 * j + (l >> 4);  // line inside the page
  const int cl = (l & 15) ^ (is_v ? Z::gv(lp) : Z::gk(lp));
  return D == 128 ? PageChunk{lp, cl} : PageChunk{2 * lp + (cl >> 3), cl & 7};
}

// Instruction j of a page load: 1 KiB of the page whose block begins at pb to LDS at dst, both 1024 j further on; off: the lane's rest.
// M0 stays what the first instruction of a page sets it to until the page's last: between these statements nothing else may write
// it, and the build refuses a listing in which anything does.
__device__ __forceinline__ void page_load(const char *pb, unsigned dst, unsigned off, int j) {
  if (j == 0) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(pb));
  else if (j == 1) asm volatile("global_load_lds_dwordx4 %0, %1 offset:1024" ::"v"(off), "s"(pb));
  else if (j == 2) asm volatile("global_load_lds_dwordx4 %0, %1 offset:2048" ::"v"(off), "s"(pb));
  else asm volatile("global_load_lds_dwordx4 %0, %1 offset:3072" ::"v"(off), "s"(pb));
}

// FRESH, a sequence with cached tokens: appends what the call appends to the pages that the workgroup reads from the pool
// (fresh_plan.h), for one KV head.  set: kPageBits / 8 bytes of LDS.  Off the common path (a prompt has no cached tokens); bound
// by its dependent round trips, so all that depends on nothing is requested first.  Measured against an append of its own in front
// (hints for N tokens a sequence): 4 x 1024 tokens on 1024 at 8q/1kv, N 2048, 40.3 -> 38.2 us; 1 x 2000 on 6000, N 8192, 85.2 and 84.5;
// 64 x 64 on 64, N 128, 21.1 -> 15.4; 64 x 100 on 100 at 16q/2kv d 64, N 256, 27.4 -> 29.3.
template <int D, int THREADS>
__device__ __forceinline__ void append_to_pool_pages(const FreshArgs &a, lds_char *set, const int32_t *bt_row, const WorkItem &it, int kvh) {
  constexpr int ROWB = 2 * D, CPR = ROWB / 16, WAVES = THREADS / 64, N = (128 * CPR + THREADS - 1) / THREADS;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const size_t row_step = (size_t)a.Hkv * ROWB, head = (size_t)kvh * ROWB, page_head = (size_t)kvh * (kPage * ROWB);
  auto copy = [&](int page, int row, int chunk, u32x4 k, u32x4 v) __attribute__((always_inline)) {
    const size_t to = (size_t)page * (kPage * row_step) + page_head + row * ROWB + chunk * 16;
    *reinterpret_cast<u32x4 *>(const_cast<char *>(a.k_pages) + to) = k;
    *reinterpret_cast<u32x4 *>(const_cast<char *>(a.v_pages) + to) = v;
  };
  // the sequence's own rows: fewer than 128, behind its cached tokens
  const int own = min(it.q_len, pool_pages(it.ctx) * kPage - it.ctx) * CPR;
  u32x4 k[N], v[N];
  int page[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int i = tid + THREADS * u, t = i / CPR;
    page[u] = -1;
    if (i >= own) continue;
    const size_t from = (size_t)(it.q0 + t) * row_step + head + (i % CPR) * 16;
    k[u] = *reinterpret_cast<const u32x4 *>(a.k_new + from);
    v[u] = *reinterpret_cast<const u32x4 *>(a.v_new + from);
    if (((it.ctx + t) >> 4) < a.max_pages) page[u] = bt_row[(it.ctx + t) >> 4];
  }
  auto store_own = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (page[u] >= 0 && page[u] < a.num_pages) copy(page[u], (it.ctx + (tid + THREADS * u) / CPR) & 15, (tid + THREADS * u) % CPR, k[u], v[u]);
  };
  if (a.batch == 1) {
    store_own();
    return;
  }
  // other sequences' rows in these pages
  typedef __attribute__((address_space(3))) unsigned lds_word;
  typedef __attribute__((address_space(3))) u32x4 lds_quad;
  lds_word *const words = (lds_word *)set;
  const int pairs = a.batch * a.new_pages, mine = min(pool_pages(it.ctx), a.max_pages);
  NewRows r = {-1, 0, 0, 0, 0};
  auto pair = [&](int base) __attribute__((always_inline)) {
    const int i = base + lane * WAVES + w;  // the pages of one sequence go to all waves in turn
    return i < pairs && new_rows_of_pair(i, a.new_pages, a.cu_q, a.ctx_lens, a.max_pages, &r) && r.seq != it.seq ? a.block_table[r.entry] : -1;
  };
  for (int i = tid; i < kPageBits / 128; i += THREADS) ((lds_quad *)set)[i] = (u32x4){0, 0, 0, 0};
  __syncthreads();
  for (int i = tid; i < mine; i += THREADS) {
    const int pg = bt_row[i];
    __hip_atomic_fetch_or(words + page_word(pg), page_bit(pg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  int pg = pair(0);
  store_own();
  __syncthreads();
  for (int base = 0;;) {
    const bool hit = pg >= 0 && pg < a.num_pages && (words[page_word(pg)] & page_bit(pg)) != 0;
    for (unsigned long long m = __builtin_amdgcn_ballot_w64(hit); m != 0; m &= m - 1) {
      const int l = __builtin_ctzll(m);
      const int to = __builtin_amdgcn_readlane(pg, l), src = __builtin_amdgcn_readlane(r.src, l);
      const int lo = __builtin_amdgcn_readlane(r.lo, l), n = __builtin_amdgcn_readlane(r.n, l);
      for (int c = lane; c < n * CPR; c += 64) {
        const size_t from = (size_t)(src + c / CPR) * row_step + head + (c % CPR) * 16;
        copy(to, lo + c / CPR, c % CPR, *reinterpret_cast<const u32x4 *>(a.k_new + from), *reinterpret_cast<const u32x4 *>(a.v_new + from));
      }
    }
    if ((base += THREADS) >= pairs) break;
    pg = pair(base);
  }
}

// FRESH: the rows of a query tile, on their way from the caller's buffer to their pages; one head group per KV head does it.
template <int D, int THREADS>
struct TileRows {
  static constexpr int ROWB = 2 * D, CPR = ROWB / 16, N = kFreshChunks / THREADS;  // 16-byte chunks per row, and of a thread
  u32x4 k[N], v[N];
  int page[N];
  __device__ __forceinline__ void request(const FreshArgs &a, const int32_t *bt_row, const WorkItem &it, int kvh, int tok0, int tpt) {
    const bool mine = (it.hg << a.gshift) == kvh * (a.Hq / a.Hkv);
    const int chunks = mine ? min(tpt, it.q_len - tok0) * CPR : 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int i = threadIdx.x + THREADS * u, tok = tok0 + i / CPR, pos = it.ctx + tok;
      page[u] = -1;
      if (i >= chunks) continue;
      const size_t src = ((size_t)(it.q0 + tok) * a.Hkv + kvh) * ROWB + (i % CPR) * 16;
      k[u] = *reinterpret_cast<const u32x4 *>(a.k_new + src);
      v[u] = *reinterpret_cast<const u32x4 *>(a.v_new + src);
      if (pos >= 0 && (pos >> 4) < a.max_pages) page[u] = bt_row[pos >> 4];
    }
  }
  __device__ __forceinline__ void store(const FreshArgs &a, const WorkItem &it, int kvh, int tok0) const {
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (page[u] >= 0 && page[u] < a.num_pages) {  // rows without a page are skipped, as in kv_append_kernel
        const int i = threadIdx.x + THREADS * u, pos = it.ctx + tok0 + i / CPR;
        const size_t dst = ((size_t)page[u] * a.Hkv + kvh) * (kPage * ROWB) + (pos & 15) * ROWB + (i % CPR) * 16;
        *reinterpret_cast<u32x4 *>(const_cast<char *>(a.k_pages) + dst) = k[u];
        *reinterpret_cast<u32x4 *>(const_cast<char *>(a.v_pages) + dst) = v[u];
      }
  }
};

// The waves form two groups of four, one wave of each group per SIMD (waves w and w+4 share a
// SIMD).  Inside every tile period the groups run the same two phases in opposite order: one
// multiplies (PV of the previous tile, then QK^T of the current one) while the other runs its
// softmax on the VALU, then they swap; one workgroup barrier per tile.  Barrier-synchronised
// waves that all do the same phase at the same time leave the matrix pipe idle during every
// softmax and the VALU idle during every MFMA burst.
//
// LDS: K[2] and V[2] tile buffers in the swizzled layout of SwzTile, filled by direct
// global -> LDS loads (no register staging, no LDS write instructions).  The loads for the
// next K tile and the current V tile are issued right after the barrier that frees their
// slots and are waited for right before the next barrier, so each has a full tile period to
// land.  The load instruction is written as inline assembly: issued through the compiler
// builtin, every later LDS read is preceded by a full vmcnt(0) wait, because the compiler
// cannot tell the slot being filled from the slot being read.  M0 (the LDS destination) is
// used by nothing else in this kernel.
//
// The running max is only moved when some column's tile max exceeds it by more than 2^8 in
// the exponent (tau); otherwise weights are taken against the stale max (bounded by 2^8,
// harmless in fp32/bf16) and the O accumulators need no rescale.
//
// SPLIT = false is the arrangement described above: the groups own neighbouring sets of 128
// columns and share every K/V tile (the first group issues all tile loads).  SPLIT = true
// is for small grids, where a few hundred workgroups with a triangular causal profile leave
// most CUs waiting for the one with the longest key range: both groups then own the SAME 128
// columns and take alternate key tiles (group g the tiles 2i + g, each with its own K and V
// stream in its own LDS region), so the critical path of the longest work item halves while
// the ping-pong stays intact; the two running states are merged through LDS at the end like
// the splits of the decode path.
//
// PART = true additionally cuts a query tile's key range into kv_splits contiguous pieces, one
// workgroup each (blockIdx.z), which write un-normalised partials for the combine pass: the way
// out when a batch has few query tokens on long cached prefixes (late chunks of a chunked
// prefill), where one workgroup per query tile would walk thousands of keys alone.  Only
// instantiated together with SPLIT (such launches are small grids).
//
// CUT = true (with SPLIT = PART = false) is for batches of few rounds of workgroups whose items are of
// different lengths: items longer than a CU's share of the launch are cut into pieces by the lengths found on
// the device (ranked_item), and only those leave partials, for cut_combine_kernel.
//
// Args = MixedArgs (attn_mixed.hip): the launch also holds workgroups of another kernel, behind the prefill ones.
// Args = FreshArgs (attn_prefill_fresh.hip): the append happens here.
template <int D, int KVT, int PFD, bool SPLIT, bool PART, int CUT, typename Args = PrefillArgs>
__global__ __launch_bounds__(512, 2) void prefill_kernel(Args a) {
  using G = TileGeom<D>;
  using Z = SwzTile<D>;
  constexpr int COLS = SPLIT ? 128 : 256, KB = KVT / 32;
  constexpr bool FRESH = std::is_same<Args, FreshArgs>::value;
  constexpr int ROWB = D * 2;               // bytes of one K or V row
  constexpr int TBYTES = KVT * ROWB;        // one tile in LDS
  constexpr int REGION = 4 * TBYTES;        // K[2] at 0 and TBYTES, V[2] at 2 and 3 TBYTES
  constexpr int NIW = TBYTES / 1024 / 4;    // 1 KiB load instructions per wave and tile
  static_assert(KVT == 4 * kPage, "each of a group's four waves brings in one page of a tile");
  static_assert((TBYTES & (TBYTES - 1)) == 0, "slot toggling flips one address bit");
  extern __shared__ __align__(16) char smem_raw[];
  lds_char *smem = (lds_char *)smem_raw;
#ifdef SP_PREFILL_TRACE
  const unsigned trace_wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  long *trace_rec = !PART && !CUT && a.part_o && trace_wg < (unsigned)kTraceWgs ? (long *)a.part_o + (size_t)trace_wg * kTraceRec : nullptr;
  long *trace_per = trace_rec ? (long *)a.part_o + (size_t)kTraceWgs * kTraceRec + (size_t)trace_wg * kTracePer : nullptr;
  SP_TRACE_STAMP(0, 0);
#endif

  const int tid = threadIdx.x, lane = tid & 63;
  if constexpr (!FRESH && !std::is_same<Args, PrefillArgs>::value) {
    if (blockIdx.x >= a.first_other) {
      a.template run_other<D>(smem, lane);
      return;
    }
  }
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps branches on it scalar
  const int col = lane & 31, half = lane >> 5;
  const int grp = w >> 2;  // wave-uniform; waves w and w+4 share a SIMD: one wave of each group per SIMD
  const int wq = w & 3;    // wave inside its group
  const int rb = SPLIT ? grp * REGION : 0;  // this group's tile buffers
  WorkItem it;
  if (!take_item<CUT>(a, SPLIT ? 7 : 8, lane, &it)) return;
  const int seq = it.seq, hg = it.hg, tile = it.tile, piece = it.piece, q0 = it.q0, q_len = it.q_len, ctx = it.ctx, pieces = it.pieces, slot = it.slot;
  const int tpt = COLS >> a.gshift;
  const int tok0 = tile * tpt;
  if (tok0 >= q_len) return;
  const int kv_end = ctx + min(q_len, tok0 + tpt);
  const int kvh = (hg << a.gshift) / (a.Hq / a.Hkv);
  const int32_t *bt_row = a.block_table + (long)seq * a.max_pages;
  const int gmask = (1 << a.gshift) - 1;
  // FRESH, but the sequence has cached tokens after all (the hints do not rule it out where they are larger than the batch).  Looked
  // at when the queries have been requested, so that nobody waits for ctx first (1 x 128 tokens at 2q/1kv d 64: 6.97 -> 6.89 us), but
  // at head_dim 128, where the queries kept over the branch cost spills in the tile loop.
  auto cached_tokens_after_all = [&]() __attribute__((always_inline)) {
    if constexpr (FRESH) {
      if (__builtin_expect(ctx > 0, 0)) {
        append_to_pool_pages<D, 512>(a, smem, bt_row, it, kvh);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the stores
        __syncthreads();
      }
    }
  };
  if (D == 128) cached_tokens_after_all();

  // ---- this lane's column and the resident Q^T operands
  bf16x8 qreg[G::kDSteps];
  const int wc = SPLIT ? wq : w;  // wave's 32-column block inside the workgroup's columns
  const int C = wc * 32 + col;
  const int token = tok0 + (C >> a.gshift);
  const int head = (hg << a.gshift) | (C & gmask);
  const bool valid = token < q_len;
  // A column without a query (past the sequence's end) has scores of 0 and is not stored, so it takes any limit: with one of 1 key
  // its wave went through the mask in every tile instead of the last ones (1 x 5003 tokens, 8q/1kv: 77 -> 65 us).
  const int lim = valid ? ctx + token + 1 : kv_end;
  const long out_off = ((long)(q0 + token) * a.Hq + head) * (D * 2);
#pragma unroll
  for (int s = 0; s < G::kDSteps; ++s) {
    if (valid) {
      qreg[s] = *reinterpret_cast<const bf16x8 *>(a.q + out_off + 32 * s + 16 * half);
    } else {
      u32x4 z = {0, 0, 0, 0};
      qreg[s] = *reinterpret_cast<bf16x8 *>(&z);
    }
  }
  if (D == 64) cached_tokens_after_all();
  // Rows with at most kPreciseKeys keys get hi + lo weights (see pv_residual below); the workgroups
  // that hold such rows run their own copy of the tile loop.
  constexpr int kPreciseKeys = 256;
  const bool precise_wg = ctx + tok0 < kPreciseKeys;  // group-uniform
  // The scaled-Q form (measurement switch): 2.5 instead of 3.5 VALU instructions per score.  At
  // head_dim 64, where halving the MFMAs per score leaves the softmax phase longer than the other
  // wave's matrix phase, it was 9 % faster on whole tiles (prefill_solo.h's now); at head_dim 128 it changes nothing.  It is not the
  // product form at either: Q * scale * log2(e) is rounded to bf16 again, so the error of a score
  // grows with the score (relative 2^-9 per term), which is invisible on unit-variance inputs and
  // several per cent of a weight once scores reach the tens — the product keeps Q's products exact.
  constexpr bool kScaledQ = kScaledQSwitch && !SPLIT && !PART;
  if (kScaledQ && !precise_wg) {
    // Fold scale * log2(e) into the resident Q operand: the scores then leave the MFMAs in the
    // exponent's units and the softmax needs no multiply.  The product is rounded to bf16 again
    // (relative 2^-9 per component, a perturbation of each score far below the rounding of the
    // weights themselves).
#pragma unroll
    for (int s = 0; s < G::kDSteps; ++s) {
      union {
        bf16x8 v;
        uint32_t w[4];
        bf16x2 h[4];
      } u;
      u.v = qreg[s];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lo = __uint_as_float(u.w[i] << 16) * a.sl2e;
        const float hi = __uint_as_float(u.w[i] & 0xffff0000u) * a.sl2e;
        u.h[i] = __builtin_convertvector((f32x2){lo, hi}, bf16x2);
      }
      qreg[s] = u.v;
    }
  }
  const int wtok_first = tok0 + ((wc * 32) >> a.gshift);
  const int wlim_min = min(ctx + wtok_first + 1, kv_end);  // keys that all of the wave's columns see

  f32x16 o[G::kDBlocks];
#pragma unroll
  for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  // A column of the second SPLIT group may see only masked keys in its first tiles, or none at
  // all: its running max starts at a large finite value so that "all masked" gives weights
  // exp2(-inf) = 0 instead of exp2(-inf + inf).  Tile 0 always holds a visible key otherwise.
  float m_used = (SPLIT || PART || CUT) ? -1e30f : -INFINITY, l = 0.f, l2 = 0.f;  // row sum in two chains
  bool m_zero = false;  // wave-uniform: every column's running max is the anchor 0 (scaled-Q form only)
  f32x16 sacc[KB];
  bf16x8 pop[KB][2];

  // key tiles [t_begin, T) of the query tile's range belong to this workgroup
  const int T_all = (kv_end + KVT - 1) / KVT;
  int t_begin = 0, T = T_all;
  if (PART) {
    const int per = (T_all + a.kv_splits - 1) / a.kv_splits;
    t_begin = piece * per;
    T = min(T_all, t_begin + per);
  }
  if (CUT && pieces > 1) {  // no piece is empty: (pieces - 1) * per < T_all
    const int per = (T_all + pieces - 1) / pieces;
    t_begin = piece * per;
    T = min(T_all, t_begin + per);
  }
  const long prow = ((long)(q0 + token) * a.Hq + head) * a.kv_splits + (PART ? piece : 0);  // partial slot
  if (PART && t_begin >= T) {  // nothing left for this piece: an empty partial
    if (valid && half == 0) *reinterpret_cast<f32x2 *>(a.part_ml + prow * 2) = (f32x2){-INFINITY, 0.f};
    return;
  }
  const int ntl = T - t_begin;
  const int Tl = SPLIT ? (ntl - grp + 1) / 2 : ntl;  // tiles this group computes on
  const int P = SPLIT ? (ntl + 1) / 2 : ntl;         // tile periods (= barriers) of the workgroup
  auto gtile = [&](int i) __attribute__((always_inline)) { return t_begin + (SPLIT ? 2 * i + grp : i); };  // local tile number -> key tile of the sequence

  // ---- tile loads, all issued by the first group during its MFMA phase (the one phase that
  // starts right after a barrier AND has issue slots to spare; the same instructions placed in
  // a softmax phase measurably lengthen it).  In SPLIT mode the first group therefore also
  // feeds the second group's private K/V stream.  Wave wq brings in page wq of every tile
  // (16 rows = NIW instructions of 1 KiB): lane l of instruction j fills chunk slot l % 16 of
  // line 4j + l / 16 of that page and fetches whichever global chunk the swizzle assigns to
  // that slot.  Page ids are wave-uniform and read from the block table one period ahead.
  // A load instruction's offset field is added on both sides, to the global address and to the LDS address, and
  // instruction j of a page lies 1024 j further on both: M0 is set once per page, and the lane offsets hold
  // only what is left, the swizzle (set per instruction, with the page's clamped offsets looked up for K as well, the matrix
  // phase of the wave that loads was 40 scalar instructions longer: 4 x 2048 tokens 51.8 -> 49.5 us, 1 x 32768 1654 -> 1632).
  // Rows past the end of the sequence: their scores are masked, so K takes what the page holds; V is
  // redirected to the last valid row (a weight of 0 does not cover a NaN).  That concerns the pages from the
  // one with the sequence's last key on, which a stream reaches with its last tile and repeats from then
  // on: the offsets are switched once, outside the MFMA sequences, when that tile's V comes up.
  // New rows (FRESH, fresh_plan.h) are no page: they have the stride of a token, and end where the caller's buffer may end, so K is
  // redirected too.  The streams turn to them once.
  constexpr int NSTREAM = SPLIT ? 2 : 1;  // K/V tile streams of the workgroup
  constexpr int NLD = NSTREAM * 2 * NIW;  // load instructions per wave and period
  const int last_kv = kv_end - 1, last_page = last_kv >> 4;
  int new_tile = 0x7fffffff;  // FRESH: tiles from here on are read from the new rows
  if (FRESH && first_new_tile(ctx) < T) new_tile = first_new_tile(ctx);
  auto stream_tile = [&](int g, int i) __attribute__((always_inline)) { return t_begin + (SPLIT ? 2 * i + g : i); };  // local tile i of stream g
  constexpr int VBIAS = (NIW - 1) * 1024;  // keeps the V offsets of clamped rows from going below zero
  auto lane_off = [&](bool is_v, int j, int rip_lim, int row_stride, int l) __attribute__((always_inline)) {  // instruction j of a page load: lane l's source offset
    const PageChunk c = page_chunk<D>(is_v, j, l);
    return (unsigned)((FRESH ? __mul24(min(c.row, rip_lim), row_stride) : min(c.row, rip_lim) * row_stride) + c.chunk * 16 - 1024 * j + (is_v || FRESH ? VBIAS : 0));
  };
  constexpr int NK = FRESH ? NSTREAM : 1;
  unsigned koff[NK][NIW], voff[NSTREAM][NIW];  // of every stream; K's are the same for all unless redirected
  const int new_stride = a.Hkv * ROWB, first_stride = FRESH && new_tile == 0 ? new_stride : ROWB, last_stride = FRESH && new_tile < T ? new_stride : ROWB;
#pragma unroll
  for (int g = 0; g < NK; ++g)
#pragma unroll
    for (int j = 0; j < NIW; ++j) koff[g][j] = lane_off(false, j, 15, first_stride, lane);
#pragma unroll
  for (int g = 0; g < NSTREAM; ++g)
#pragma unroll
    for (int j = 0; j < NIW; ++j) voff[g][j] = lane_off(true, j, 15, first_stride, lane);
  // This KV head's block of page 0 and the number of pages; of new rows, the row that would be the first of page 0.
  const char *kpool, *vpool;
  int most_pages = FRESH && new_tile == 0 ? 0x7fffffff : a.num_pages;
  const size_t pool_block = (size_t)kvh * (kPage * ROWB);
  const long new_block = FRESH ? ((long)(q0 - ctx) * a.Hkv + kvh) * ROWB - VBIAS : 0;
  kpool = a.k_pages + pool_block - (FRESH ? VBIAS : 0);
  vpool = a.v_pages + pool_block - VBIAS;
  if constexpr (FRESH) {
    if (new_tile == 0) {
      kpool = a.k_new + new_block;
      vpool = a.v_new + new_block;
    }
  }
  auto clamp_v = [&](int g, int gt, int l) __attribute__((always_inline)) {  // before the loads of V of key tile gt of stream g
    if (gt < T - 1 || (T - 1) * (KVT / kPage) + wq < last_page) return;
#pragma unroll
    for (int j = 0; j < NIW; ++j) voff[g][j] = lane_off(true, j, last_kv & 15, last_stride, l);
  };
  auto clamp_k = [&](int g, int gt, int l) __attribute__((always_inline)) {  // the same for K
    if (!FRESH || gt < T - 1 || (T - 1) * (KVT / kPage) + wq < last_page) return;
#pragma unroll
    for (int j = 0; j < NIW; ++j) koff[FRESH ? g : 0][j] = lane_off(false, j, last_kv & 15, last_stride, l);
  };
  // FRESH: V, or K, comes to the new rows.  What the offsets move by is computed on the spot: kept over the tile loop it would cost registers.
  auto new_offset = [&](bool is_v, int j) __attribute__((always_inline)) {
    int l = lane;
    if constexpr (FRESH) asm volatile("" : "+v"(l));
    return (unsigned)__mul24(page_chunk<D>(is_v, j, l).row, new_stride - ROWB);
  };
  auto new_offsets_v = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NIW; ++j) voff[g][j] += new_offset(true, j);
  };
  auto new_offsets_k = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NIW; ++j) koff[FRESH ? g : 0][j] += new_offset(false, j);
  };
  auto turn_v = [&]() __attribute__((always_inline)) {
    if constexpr (FRESH) vpool = a.v_new + new_block;
  };
  auto turn_k = [&]() __attribute__((always_inline)) {
    if constexpr (FRESH) {
      kpool = a.k_new + new_block;
      most_pages = 0x7fffffff;
    }
  };
  // FRESH: the first period whose end has anything to aim (K is two tiles ahead)
  constexpr int STEP = SPLIT ? 2 : 1;
  const int calm = FRESH ? min(new_tile == 0 ? T : new_tile, T - STEP) / STEP - 2 : 0;
  const unsigned page_bytes = (unsigned)a.Hkv * (kPage * ROWB);  // sixteen new rows are as far apart
  auto page_idx = [&](int gt) __attribute__((always_inline)) { return min(min(gt, T - 1) * (KVT / kPage) + wq, last_page); };  // this wave's page of a tile
  // The inline assembly below makes the compiler treat every later load as possibly clobbered,
  // so block-table reads are vector loads; the value stays in a VGPR until the load that needs
  // it is issued one period later, and only then moves to an SGPR.
  auto page_of = [&](int gt) __attribute__((always_inline)) {  // all lanes read the same entry
    if constexpr (FRESH) {
      if (min(gt, T - 1) >= new_tile) return page_idx(gt);
    }
    return bt_row[page_idx(gt)];
  };
  auto page_pos = [&](int pg, int most) __attribute__((always_inline)) {  // where the page begins in the pool; no wild loads on bad metadata
    return (size_t)(unsigned)min(max(__builtin_amdgcn_readfirstlane(pg), 0), most - 1) * page_bytes;
  };
  const unsigned wave_dst = (unsigned)(wq * (NIW * 1024));
  static_assert(NIW <= 4, "an offset field holds up to 4095");
  using std::false_type;
  using std::integral_constant;
  using std::true_type;
  // The loads of period i, prepared right after the barrier that opens it: for every stream, K
  // of local tile i+1 and V of local tile i go into the slots whose last readers finished
  // before that barrier (K(i+1) into slot (i+1) & 1, V(i) into slot i & 1).  Past a stream's
  // last tile the loads repeat the sequence's last tile into a slot nobody reads.  The NLD
  // instructions are then emitted one at a time, spread over the MFMA sequence: issued back to
  // back by four waves at once they queue up at the CU's one texture address unit, and since a
  // wave issues in order, everything behind them waits too.
  int pg_k[NSTREAM];      // page ids of the next K loads (kept in VGPRs)
  size_t pos_v[NSTREAM];  // where the pages of the next V loads begin in the pool
  const char *ld[NSTREAM][2];
  auto issue_prep = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < NSTREAM; ++g) {
      const size_t pos = page_pos(pg_k[g], most_pages);
      ld[g][0] = kpool + pos;
      ld[g][1] = vpool + pos_v[g];
      pos_v[g] = pos;
      pg_k[g] = page_of(stream_tile(g, i + 2));
    }
  };
  auto slot_dst = [&](int g, int m, int slot) __attribute__((always_inline)) {  // LDS address of this wave's page in a tile slot
    return (unsigned)(g * REGION + (2 * m + slot) * TBYTES) + wave_dst;
  };
  auto issue_emit = [&](int n, int par) __attribute__((always_inline)) {  // n-th instruction of the period, n < NLD: streams and matrices in turn
    const int j = n % NIW, u = n / NIW, g = u % NSTREAM, m = u / NSTREAM;
    page_load(ld[g][m], slot_dst(g, m, m ? par : 1 - par), m ? voff[g][j] : koff[FRESH ? g : 0][j], j);
  };
  auto wait_loads = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0x0F70); };  // vmcnt(0) only

  // ---- LDS operand addresses of this lane: absolute LDS byte addresses for slot 0 of the K and
  // of the V buffers.  Everything else an operand read adds — the slot (TBYTES), the 32-key block
  // and the 16-key step — is a compile-time constant that goes into the instruction's offset
  // field, so the matrix phases contain no address arithmetic at all; the tile loop is unrolled
  // by two for that, one copy per slot parity.
  const unsigned lds0 = (unsigned)(size_t)smem + (unsigned)rb;
  unsigned kadr[G::kDSteps], vadr[G::kDBlocks];
#pragma unroll
  for (int s = 0; s < G::kDSteps; ++s) kadr[s] = lds0 + Z::template offset<false>(col, 2 * s + half);
  {
    const int n = lane & 15, dg = (lane >> 4) & 1;
#pragma unroll
    for (int db = 0; db < G::kDBlocks; ++db)
      vadr[db] = lds0 + 2 * TBYTES + Z::template offset<true>(4 * half + (n >> 2), 4 * db + 2 * dg + ((n & 3) >> 1)) +
                 8 * (n & 1);
  }
  static_assert(TBYTES + (KVT - 8) * ROWB < 65536, "operand offsets must fit the 16-bit offset field");

  // ---- the phases of a tile, per wave.  The MFMA phases are written software-pipelined ("read
  // operand i+PFD, MFMA i") and pinned to that issue order with sched_group_barrier, so that LDS
  // reads run a fixed distance ahead of the MFMAs that consume them (left alone, the scheduler
  // places each read right before its use and the matrix pipe waits on LDS latency).
  constexpr int NPV = KB * 2 * G::kDBlocks, NQK = KB * G::kDSteps;
  // Operand i of the fused sequence "PV of one tile, then QK^T of the next": i < NPV is a V^T
  // operand (two transposing reads: key rows 32b + 16ks + 4*half + 0..3 and the same + 8, in the
  // row order the score accumulator dictates) from V slot VS, the rest are K operands (one
  // 16-byte read) from K slot KS.
  auto load_op = [&](int i, int KS, int VS) __attribute__((always_inline)) -> bf16x8 {
    if (i < NPV) {
      int db = i % G::kDBlocks, ks = (i / G::kDBlocks) & 1, b = i / (2 * G::kDBlocks);
      return lds_read_vt((const lds_char *)(size_t)(vadr[db] + (unsigned)(VS * TBYTES + (32 * b + 16 * ks) * ROWB)), ROWB);
    }
    int j = i - NPV;
    int s = j % G::kDSteps, b = j / G::kDSteps;
    return *(const lds_bf16x8 *)(size_t)(kadr[s] + (unsigned)(KS * TBYTES + 32 * b * ROWB));
  };
  // Measurement switch SP_PREFILL_SUM_IN_MATRIX_PHASE: the row sum behind the PV MFMAs (unpack the
  // bf16 weights of 16 / NPV packed registers of P by shift / mask, two chains of adds).
  constexpr int RPM = (KB * 2 * 4) / NPV;  // packed registers of P per PV MFMA
  auto do_mfma = [&](int i, bf16x8 op) __attribute__((always_inline)) {
    if (i < NPV) {
      int db = i % G::kDBlocks, ks = (i / G::kDBlocks) & 1, b = i / (2 * G::kDBlocks);
      o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op, pop[b][ks], o[db], 0, 0, 0);
#ifdef SP_PREFILL_SUM_IN_MATRIX_PHASE
#pragma unroll
      for (int e = 0; e < RPM; ++e) {
        const int pr = i * RPM + e;  // packed register pr of the tile's 16: pop[pr / 8][(pr / 4) & 1], word pr % 4
        union {
          bf16x8 v;
          uint32_t w[4];
        } u;
        u.v = pop[pr / 8][(pr / 4) & 1];
        l += __uint_as_float(u.w[pr % 4] << 16);
        l2 += __uint_as_float(u.w[pr % 4] & 0xffff0000u);
      }
#endif
    } else {
      int j = i - NPV;
      int s = j % G::kDSteps, b = j / G::kDSteps;
      if (s == 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[b][r] = 0.f;
      }
      sacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op, qreg[s], sacc[b], 0, 0, 0);
    }
  };
  // TAILB: the workgroup barrier sits inside the sequence, before its last PFD MFMAs.  All LDS
  // reads of the sequence are done by then (their operands wait in registers), so the waves on
  // the other side of the barrier may overwrite the slots, and their first operand reads run
  // behind these trailing MFMAs instead of leaving the matrix pipe idle.
  auto mfma_seq = [&](auto I0c, auto I1c, auto stagec, auto ksc, auto vsc, auto tailc) __attribute__((always_inline)) {
    constexpr bool TAILB = decltype(tailc)::value;
    constexpr int I0 = decltype(I0c)::value, I1 = decltype(I1c)::value, N = I1 - I0;
    constexpr int KS = decltype(ksc)::value, VS = decltype(vsc)::value;  // K and V slots read
    constexpr bool STAGE = decltype(stagec)::value;  // emit this period's tile loads along the way
    constexpr int GAP = N >= NLD ? N / NLD : 1, PER = N >= NLD ? 1 : NLD / N;  // loads per MFMA slot
    bf16x8 ops[N];
#pragma unroll
    for (int i = 0; i < PFD && i < N; ++i) ops[i] = load_op(I0 + i, KS, VS);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (TAILB && i == N - PFD) {
        sgb_prologue<0, N, I0, NPV, PFD>();
        sgb_steady<0, N, I0, NPV, PFD, 0, N - PFD>();
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (i + PFD < N) ops[i + PFD] = load_op(I0 + i + PFD, KS, VS);
      do_mfma(I0 + i, ops[i]);
      if (STAGE && i % GAP == 0 && i / GAP * PER < NLD) {
#pragma unroll
        for (int e = 0; e < PER; ++e) issue_emit(i / GAP * PER + e, KS);
      }
    }
#ifdef SP_PREFILL_SUM_IN_MATRIX_PHASE
    // the row sums are only read at the very end of the kernel: without a use here the compiler
    // sinks their adds out of the matrix phase into the softmax that follows
    if (I0 < NPV) asm volatile("" : "+v"(l), "+v"(l2));
#endif
    if (!TAILB) {
      sgb_prologue<0, N, I0, NPV, PFD>();
#ifdef SP_PREFILL_SUM_IN_MATRIX_PHASE
      sgb_steady<0, N, I0, NPV, PFD, 4 * RPM>();
#else
      sgb_steady<0, N, I0, NPV, PFD, 0>();
#endif
    }
  };
  using slot0 = integral_constant<int, 0>;
  using slot1 = integral_constant<int, 1>;
  auto qk0 = [&]() __attribute__((always_inline)) {  // QK^T of a stream's first tile (K slot 0); its loads went out in the prologue
    mfma_seq(integral_constant<int, NPV>{}, integral_constant<int, NPV + NQK>{}, false_type{}, slot0{}, slot0{}, false_type{});
  };
  auto pv = [&](auto vsc) __attribute__((always_inline)) {  // PV of the tile in V slot vsc
    mfma_seq(integral_constant<int, 0>{}, integral_constant<int, NPV>{}, false_type{}, slot0{}, vsc, false_type{});
  };
  auto pv_qk = [&](auto stagec, auto parc, auto tailc) __attribute__((always_inline)) {  // period i of parity parc: PV of tile i-1 (V slot 1 - par), QK^T of tile i (K slot par)
    constexpr int PAR = decltype(parc)::value;
    mfma_seq(integral_constant<int, 0>{}, integral_constant<int, NPV + NQK>{}, stagec, parc, integral_constant<int, 1 - PAR>{}, tailc);
  };
  // Softmax of tile t.  The common case (FIRST = false, and the tile's scores stay within 2^8 of
  // the running max) is one pass of 3.5 VALU instructions per score: weight = exp2(score * c -
  // max * c), added to the row sum (two independent chains), rounded to bf16 in pairs.  No tile
  // max is computed: if a score had exceeded the running max by more than the threshold, its
  // weight and hence the lane's tile sum would exceed 2^8, and the wave falls back to the full
  // pass (tile max, lazy rescale of O and l, weights again from the raw scores, which the fast
  // pass leaves untouched).  The first tile always takes the full pass (the running max starts at
  // -inf), which also leaves the fp32 weights in sacc for the residual pass of short rows.
  // (Summing the rounded pairs with the bf16 dot-product instruction instead would be half the
  // additions, but measured it costs a third more cycles for the whole kernel: next to MFMAs that
  // instruction is far from full rate.)
  auto softmax = [&](int t, auto firstc, bool keep_fp32, auto qsc) __attribute__((always_inline)) {
    constexpr bool QS = decltype(qsc)::value;  // scores arrive in the exponent's units (Q was prescaled)
    constexpr bool FIRST = decltype(firstc)::value;  // keep_fp32 (wave-uniform): take the full pass, the residual pass follows
    const int base = gtile(t) * KVT;
    if (base + KVT > wlim_min) {
#pragma unroll
      for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          int kv = base + 32 * b + 8 * (r >> 2) + 4 * half + (r & 3);
          if (kv >= lim) sacc[b][r] = -INFINITY;
        }
    }
    float lsum = 0.f;
    bool full = FIRST || keep_fp32 || kAlwaysFullSoftmax;
    const float sc = QS ? 1.0f : a.sl2e;
    if (!full) {
      const float msc = m_used * sc;
#ifdef SP_PREFILL_SUM_IN_MATRIX_PHASE
      uint32_t pmax = 0;  // weights are >= 0, so their bit patterns order like their values (and NaN sorts above all)
#pragma unroll
      for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          union {
            bf16x2 h[4];
            bf16x8 v;
          } u;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[b][8 * ks + 2 * i], a.sl2e, -msc));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[b][8 * ks + 2 * i + 1], a.sl2e, -msc));
            u.h[i] = __builtin_convertvector((f32x2){p0, p1}, bf16x2);
            pmax = max(pmax, max(__float_as_uint(p0), __float_as_uint(p1)));  // one v_max3_u32 per pair
          }
          pop[b][ks] = u.v;
        }
      // NaN (a masked score against a running max that is still -inf) must take the full pass too
      full = __builtin_amdgcn_ballot_w64(pmax > 0x43800000u) != 0;  // some weight above 2^8: wave-uniform, rare
#else
      float ls0 = 0.f, ls1 = 0.f;
#ifdef SP_PREFILL_SUM_MFMA
      f32x4 lacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#endif
      if (QS && m_zero) {
        // no running max to subtract: 2.5 VALU instructions per score
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            union {
              bf16x2 h[4];
              bf16x8 v;
            } u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float p0 = __builtin_amdgcn_exp2f(sacc[b][8 * ks + 2 * i]);
              const float p1 = __builtin_amdgcn_exp2f(sacc[b][8 * ks + 2 * i + 1]);
              u.h[i] = __builtin_convertvector((f32x2){p0, p1}, bf16x2);
              ls0 += p0;
              ls1 += p1;
            }
            pop[b][ks] = u.v;
          }
      } else
#pragma unroll
      for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          union {
            bf16x2 h[4];
            bf16x8 v;
          } u;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[b][8 * ks + 2 * i], sc, -msc));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[b][8 * ks + 2 * i + 1], sc, -msc));
            u.h[i] = __builtin_convertvector((f32x2){p0, p1}, bf16x2);
#if defined(SP_PREFILL_SUM_DOT2)
            ls0 = __builtin_amdgcn_fdot2_f32_bf16(u.h[i], (bf16x2){(__bf16)1.0f, (__bf16)1.0f}, ls0, false);
#elif !defined(SP_PREFILL_SUM_MFMA)
            ls0 += p0;
            ls1 += p1;
#endif
          }
          pop[b][ks] = u.v;
#ifdef SP_PREFILL_SUM_MFMA
          {
            // row sums on the matrix pipe: a 4x4x4 MFMA (16 blocks) with an all-ones A operand adds up
            // the four bf16 values each lane holds in B; two of them cover this operand's eight
            union {
              bf16x8 v;
              s16x4 q[2];
            } w;
            w.v = u.v;
            const s16x4 ones4 = {0x3F80, 0x3F80, 0x3F80, 0x3F80};
            lacc[ks] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, w.q[0], lacc[ks], 0, 0, 0);
            lacc[ks] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, w.q[1], lacc[ks], 0, 0, 0);
          }
#endif
        }
#ifdef SP_PREFILL_SUM_MFMA
      lsum = lacc[0][0] + lacc[1][0];
#else
      lsum = ls0 + ls1;
#endif
      // NaN (a masked score against a running max that is still -inf) must take the full pass too
      full = __builtin_amdgcn_ballot_w64(!(lsum <= (QS ? 0x1p40f : 256.0f))) != 0;  // wave-uniform, rare
#endif
    }
    if (full) {
      float mx = sacc[0][0];
#pragma unroll
      for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[b][r]);
      mx = fmaxf(mx, other_half(mx));
      if (__builtin_amdgcn_ballot_w64(mx > m_used + (QS ? 8.0f : a.tau)) != 0) {  // wave-uniform
        float m_new = fmaxf(m_used, mx);
        // scaled-Q form: a first max within 2^+-32 anchors the column at 0, and while every column
        // of the wave sits there the fast pass skips the subtraction
        if (QS && FIRST && fabsf(mx) <= 32.0f) m_new = 0.f;
        const float alpha = __builtin_amdgcn_exp2f((m_used - m_new) * sc);
        m_used = m_new;
        if (QS) m_zero = __builtin_amdgcn_ballot_w64(m_used != 0.f) == 0;
        l *= alpha;
        l2 *= alpha;
#pragma unroll
        for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      }
      const float msc = m_used * sc;
      lsum = 0.f;
#pragma unroll
      for (int b = 0; b < KB; ++b) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sacc[b][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[b][r], sc, -msc));
#ifndef SP_PREFILL_SUM_IN_MATRIX_PHASE
          lsum += sacc[b][r];
#endif
        }
        pop[b][0] = pack8(sacc[b], 0);
        pop[b][1] = pack8(sacc[b], 8);
      }
    }
    l += lsum;
  };
  // Rows with at most kPreciseKeys keys take their weights as hi + lo: a second PV pass over the
  // tile with the bf16 residuals of P, so that the rounding of the weights (which only averages
  // out over many keys) stays out of the output tolerance there.  That concerns the first
  // kPreciseKeys / KVT key tiles of the workgroups whose first query sits below position
  // kPreciseKeys.  The pass needs the fp32 weights (the softmax's full pass leaves them in sacc)
  // and V of that tile in LDS: it runs at the start of the following period, before QK^T
  // overwrites sacc.
  auto precise = [&](int i) __attribute__((always_inline)) { return precise_wg && i >= 0 && gtile(i) * KVT < kPreciseKeys; };
  auto pv_residual = [&](auto vsc) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) pop[b][ks] = pack8_residual(sacc[b], 8 * ks, pop[b][ks]);
    pv(vsc);
#pragma unroll
    for (int b = 0; b < KB; ++b)  // back to the rounded weights (cheaper than keeping a copy live)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) pop[b][ks] = pack8(sacc[b], 8 * ks);
  };

  // prologue: K of every stream's first tile must be in LDS before anything is multiplied.  V of
  // that tile and K of the second one are requested in the same round trip (their slots are
  // free), so the first period has no load to wait for: a memory latency per workgroup that
  // small grids cannot hide behind other work.
  if (grp == 0) {
    size_t pos0[NSTREAM];
    if (FRESH && new_tile == 0) {  // nothing to look up
#pragma unroll
      for (int g = 0; g < NSTREAM; ++g) {
        pos0[g] = (size_t)(unsigned)page_idx(stream_tile(g, 0)) * page_bytes;
        pos_v[g] = (size_t)(unsigned)page_idx(stream_tile(g, 1)) * page_bytes;
      }
    } else {
      int pg0[NSTREAM], pg1[NSTREAM];
#pragma unroll
      for (int g = 0; g < NSTREAM; ++g) {
        pg0[g] = page_of(stream_tile(g, 0));
        pg1[g] = page_of(stream_tile(g, 1));
        pg_k[g] = page_of(stream_tile(g, 2));
      }
#pragma unroll
      for (int g = 0; g < NSTREAM; ++g) {
        pos0[g] = page_pos(pg0[g], a.num_pages);
        pos_v[g] = page_pos(pg1[g], FRESH && stream_tile(0, 1) == new_tile ? 0x7fffffff : a.num_pages);
      }
    }
    const bool turn1 = FRESH && stream_tile(0, 1) == new_tile, turn2 = FRESH && stream_tile(0, 2) == new_tile;
#pragma unroll
    for (int g = 0; g < NSTREAM; ++g) {
      clamp_v(g, stream_tile(g, 0), lane);
      clamp_k(g, stream_tile(g, 0), lane);
#pragma unroll
      for (int j = 0; j < NIW; ++j) page_load(kpool + pos0[g], slot_dst(g, 0, 0), koff[FRESH ? g : 0][j], j);
#pragma unroll
      for (int j = 0; j < NIW; ++j) page_load(vpool + pos0[g], slot_dst(g, 1, 0), voff[g][j], j);
      const char *k1 = kpool;
      if constexpr (FRESH) {
        if (__builtin_expect(turn1, 0)) {
          k1 = a.k_new + new_block;
          new_offsets_k(g);
        }
      }
      clamp_k(g, stream_tile(g, 1), lane);
#pragma unroll
      for (int j = 0; j < NIW; ++j) page_load(k1 + pos_v[g], slot_dst(g, 0, 1), koff[FRESH ? g : 0][j], j);
      if (__builtin_expect(turn1, 0)) new_offsets_v(g);
      if (__builtin_expect(turn2, 0)) new_offsets_k(g);
      clamp_v(g, stream_tile(g, 1), lane);
      clamp_k(g, stream_tile(g, 2), lane);
    }
    if (__builtin_expect(turn1, 0)) turn_v();
    if (__builtin_expect(turn1 || turn2, 0)) turn_k();
  }
  // FRESH: the rows of this query tile.  The requests go out behind those of the first tiles, the stores behind the barrier: they
  // are under way during the first period, whose end waits for them with its tile loads.
  TileRows<D, 512> rows;
  if constexpr (FRESH) rows.request(a, bt_row, it, kvh, tok0, tpt);
  wait_loads();
  __syncthreads();
  if constexpr (FRESH) {
    rows.store(a, it, kvh, tok0);
    if (new_tile == 0) {  // as a page id, and here, where no load is under way that the register could wait for
#pragma unroll
      for (int g = 0; g < NSTREAM; ++g) pg_k[g] = page_idx(stream_tile(g, 2));
    }
  }
  SP_TRACE_STAMP(1, 0);

  // One barrier per key tile.  Inside a tile period the two groups run the same two phases in
  // OPPOSITE order: the first group multiplies (PV of tile t-1, QK^T of tile t) and then
  // exponentiates tile t; the second group first exponentiates tile t-1 and then multiplies.
  // One wave of each group sits on every SIMD, so the matrix pipe and the VALU are both busy
  // through the whole period, and since nothing forces the phase boundary to line up, a short
  // softmax simply lets the next MFMA phase start early.  Wave priorities are left alone: raising
  // the multiplying wave (or the other one) measured 5 % more cycles for the whole kernel.
  // Buffer hand-off: from period 1 on, K(t+1) and V(t) are requested in the first group's MFMA
  // phase of period t into the slots last read in period t-1, have landed before the barrier
  // that ends period t, and are first read in period t+1.  Periods alternate between two copies
  // of the loop body, one per slot parity.
  // The tile loop exists twice: the few workgroups that hold rows of at most kPreciseKeys keys
  // (at most eight key tiles long) take the copy with the residual passes, everything else the
  // copy without them, whose registers and schedule the rare case then cannot disturb.
  auto tile_loop = [&](auto precc) __attribute__((always_inline)) {
    constexpr bool PREC = decltype(precc)::value;
    if (grp == 0) {  // always has Tl == P >= 1
      qk0();  // the loads of period 0 went out in the prologue
      softmax(0, true_type{}, false, integral_constant<bool, kScaledQ && !PREC>{});
      __syncthreads();
      auto period = [&](int t, auto parc) __attribute__((always_inline)) {
        constexpr int PAR = decltype(parc)::value;
#ifdef SP_PREFILL_TRACE
        if (trace_per && threadIdx.x == 0 && (t & 7) == 0 && t < 8 * kTracePer) {
          trace_per[t >> 3] = (long)wall_clock64();
          trace_per[(size_t)kTraceWgs * kTracePer + (t >> 3)] = (long)clock64();
        }
#endif
        if (PREC && precise(t - 1)) pv_residual(integral_constant<int, 1 - PAR>{});  // V(t-1) became visible at the barrier
        issue_prep(t);
        SP_MATRIX_PHASE_BEGIN();
        pv_qk(true_type{}, parc, false_type{});
        SP_MATRIX_PHASE_END();
        softmax(t, false_type{}, PREC && precise(t), integral_constant<bool, kScaledQ && !PREC>{});
        if (!FRESH || __builtin_expect(t >= calm, 0)) {
          int l = lane;
          if constexpr (FRESH && (PREC || (SPLIT && D == 128))) asm volatile("" : "+v"(l));  // rare copy of the loop: its swizzles are not kept in registers over it
          const bool v = FRESH && stream_tile(0, t + 1) == new_tile, k = FRESH && stream_tile(0, t + 2) == new_tile;
          if (__builtin_expect(v, 0)) turn_v();
          if (__builtin_expect(k, 0)) turn_k();
#pragma unroll
          for (int g = 0; g < NSTREAM; ++g) {
            if (__builtin_expect(v, 0)) new_offsets_v(g);
            if (__builtin_expect(k, 0)) new_offsets_k(g);
            clamp_v(g, stream_tile(g, t + 1), l);
            clamp_k(g, stream_tile(g, t + 2), l);
          }
        }
        wait_loads();
        __syncthreads();
      };
      int t = 1;
      for (; t + 1 < Tl; t += 2) {  // single-exit loop over pairs of periods; an odd one out follows it
        period(t, slot1{});
        period(t + 1, slot0{});
      }
      if (t < Tl) {
        period(t, slot1{});
        if (PREC && precise(t)) pv_residual(slot1{});
        pv(slot1{});
      } else {
        if (PREC && precise(t - 1)) pv_residual(slot0{});
        pv(slot0{});
      }
    } else {  // SPLIT: may have one tile less than the first group, or none
      if (Tl > 0) qk0();
      __syncthreads();
      if (Tl > 0) {
        softmax(0, true_type{}, false, integral_constant<bool, kScaledQ && !PREC>{});
        auto period = [&](int t, auto parc) __attribute__((always_inline)) {
          constexpr int PAR = decltype(parc)::value;
          if (PREC && precise(t - 1)) pv_residual(integral_constant<int, 1 - PAR>{});
          SP_MATRIX_PHASE_BEGIN();
          pv_qk(false_type{}, parc, integral_constant<bool, kBarrierInSeq>{});  // the period's barrier is inside
          SP_MATRIX_PHASE_END();
          if (!kBarrierInSeq) __syncthreads();
          softmax(t, false_type{}, PREC && precise(t), integral_constant<bool, kScaledQ && !PREC>{});
        };
        int t = 1;
        for (; t + 1 < Tl; t += 2) {
          period(t, slot1{});
          period(t + 1, slot0{});
        }
        if (t < Tl) {
          period(t, slot1{});
          if (PREC && precise(t)) pv_residual(slot1{});
          pv(slot1{});
        } else {
          if (PREC && precise(t - 1)) pv_residual(slot0{});
          pv(slot0{});
        }
      }
      for (int t = max(Tl, 1); t < P; ++t) __syncthreads();  // keep the barrier count of the first group
    }
  };

  if (precise_wg) tile_loop(true_type{});
  else tile_loop(false_type{});
  SP_TRACE_STAMP(2, 0);
  SP_TRACE_STAMP(3, 256);

  // The channel blocks this wave writes, db0 and on: with SPLIT each group finishes one half of them.
  constexpr int HB = SPLIT ? G::kDBlocks / 2 : G::kDBlocks;
  f32x16 fin[HB];
  const int db0 = SPLIT ? grp * HB : 0;
  if constexpr (SPLIT) {
    // ---- merge of the two groups' running states (same columns, same lane layout: wave w and wave w+4 hold
    // the same (column, channel) positions): each group hands over the half of O that the other one finishes,
    // in 16-byte pieces, so that both share the merge and the stores (4 x 2048 tokens, 8q/1kv, two such workgroups a
    // CU: 57.5 us when the first group did all of it in 4-byte pieces, 55.7 so).
    constexpr int NQ = 4 * HB;  // 16-byte pieces of half a state per lane
    static_assert(2 * 256 * (NQ * 16 + 8) <= 2 * REGION, "states must fit the tile buffers");
    lds_f32x4 *xch = (lds_f32x4 *)smem + wq * 64 + lane;                        // [group][piece][wave][lane]
    lds_f32x2 *xml = (lds_f32x2 *)(smem + 2 * 256 * NQ * 16) + wq * 64 + lane;  // [group][wave][lane]
    __syncthreads();  // every wave is done reading tiles
    // values are selected, not indices: an index that depends on the group would put o into memory
#pragma unroll
    for (int n = 0; n < HB; ++n)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a0 = o[n][4 * r4 + e], a1 = o[G::kDBlocks - HB + n][4 * r4 + e];
          x[e] = grp == 0 ? a1 : a0;
          fin[n][4 * r4 + e] = grp == 0 ? a0 : a1;
        }
        xch[(grp * NQ + 4 * n + r4) * 256] = x;
      }
    xml[grp * 256] = (f32x2){m_used, l + l2};
    __syncthreads();
    const f32x2 ml = xml[(1 - grp) * 256];
    const float m_new = fmaxf(m_used, ml[0]);  // the first group always saw a key: finite
    const float fa = __builtin_amdgcn_exp2f((m_used - m_new) * a.sl2e);  // 0 for a group that had no tile
    const float fb = __builtin_amdgcn_exp2f((ml[0] - m_new) * a.sl2e);
    l = (l + l2) * fa + ml[1] * fb;
    l2 = 0.f;
#pragma unroll
    for (int n = 0; n < HB; ++n)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 x = xch[((1 - grp) * NQ + 4 * n + r4) * 256];
#pragma unroll
        for (int e = 0; e < 4; ++e) fin[n][4 * r4 + e] = fin[n][4 * r4 + e] * fa + x[e] * fb;
      }
    m_used = m_new;  // what l and fin now refer to (a partial carries it along)
  } else {
#pragma unroll
    for (int db = 0; db < HB; ++db) fin[db] = o[db];
  }

  l += l2;
  float lt = l + other_half(l);
  if (PART) {  // un-normalised partial for the combine pass
    if (valid) {
      float *po = a.part_o + prow * D + 32 * db0;
#pragma unroll
      for (int db = 0; db < HB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *reinterpret_cast<f32x4 *>(po + 32 * db + 8 * r4 + 4 * half) =
              (f32x4){fin[db][4 * r4], fin[db][4 * r4 + 1], fin[db][4 * r4 + 2], fin[db][4 * r4 + 3]};
      if (half == 0 && db0 == 0) *reinterpret_cast<f32x2 *>(a.part_ml + prow * 2) = (f32x2){m_used * a.sl2e, lt};
    }
    return;
  }
  if (CUT && pieces > 1) {  // un-normalised partial in register order: every store instruction writes 1 KiB in a row
    float *po = a.part_o + ((size_t)slot * 8 + w) * (32 * D) + lane * 4;
#pragma unroll
    for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        *reinterpret_cast<f32x4 *>(po + (4 * db + r4) * 256) = (f32x4){o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]};
    if (half == 0) *reinterpret_cast<f32x2 *>(a.part_ml + ((size_t)slot * 256 + C) * 2) = (f32x2){m_used * a.sl2e, lt};
    if (tid == 0) a.cut_tab[slot] = CutEntry{q0, q_len, tile, hg, piece == 0 ? pieces : 0, a.n_hgroups, {0, 0}};
    return;
  }
  // ---- normalise and store
  float inv = 1.0f / lt;
  if (valid) {
    char *dst = a.out + out_off + 64 * db0;
#pragma unroll
    for (int db = 0; db < HB; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        store4_bf16(dst + (32 * db + 8 * r4 + 4 * half) * 2, fin[db][4 * r4] * inv, fin[db][4 * r4 + 1] * inv,
                    fin[db][4 * r4 + 2] * inv, fin[db][4 * r4 + 3] * inv);
  }
#ifdef SP_PREFILL_TRACE
  SP_TRACE_STAMP(4, 0);
  if (trace_rec && threadIdx.x == 0) {
    trace_rec[5] = T_all;
    // HW_ID (wave, SIMD, CU, shader array, shader engine) and XCC_ID of the wave
    trace_rec[6] = (long)__builtin_amdgcn_s_getreg((31 << 11) | 4) | ((long)__builtin_amdgcn_s_getreg((3 << 11) | 20) << 32);
    trace_rec[7] = ((long)seq << 32) | (unsigned)tile;
  }
#endif
}


template <int D>
constexpr size_t kPrefillSmem = 4 * (size_t)KVT * D * 2;  // K[2] V[2], unpadded

// Launch index space of `cols` query columns per workgroup; completes a.  SP_ERR_BAD_SHAPE if it exceeds the limits.
inline int prefill_grid(PrefillArgs &a, int cols, int batch, int max_q_len, int layers, dim3 *grid) {
  int tpt = cols >> a.gshift;
  a.ntiles_x = (max_q_len + tpt - 1) / tpt;
  long gx = (long)batch * a.n_hgroups;
  if (gx > 0x7fffffffL || a.ntiles_x > 65535 * layers)
    return fail(SP_ERR_BAD_SHAPE, "sp_attn_prefill: grid %ld x %d exceeds the launch limits", gx, a.ntiles_x);
  const int z = a.ntiles_x > 65535 ? layers : 1;
  *grid = dim3((unsigned)gx, (unsigned)((a.ntiles_x + z - 1) / z), (unsigned)(a.kv_splits * z));
  if (a.ranked) {
    // Ranked workgroups take items by linear id, so the launch only needs as many workgroups as
    // there can be items (ranked_workgroups).  (The grid of
    // the static order is batch x tiles of the LONGEST chunk; in a ragged batch most of it is
    // empty, and an empty workgroup still holds a CU for a microsecond.)
    const long wgs = ranked_workgroups(a.total_q, tpt, batch, a.n_hgroups, a.kv_splits, a.cut_slots);
    if (wgs > 0x7fffffffL) a.ranked = 0;  // workgroups are numbered in 32 bits
    else *grid = dim3((unsigned)wgs, 1, 1);
  }
  return SP_OK;
}

// Dynamic LDS of a kernel, asked for once.
inline int grant_smem(const void *fn, bool *done, size_t smem) {
  if (*done) return SP_OK;  // benign if two threads race
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return fail(SP_ERR_HIP, "prefill smem attribute: %s", hipGetErrorString(e));
  *done = true;
  return SP_OK;
}

// Launches one prefill kernel instantiation with `cols` query columns per workgroup.  layers: how many times 65535 query tiles of a
// sequence it takes (a kernel without pieces: blockIdx.z is theirs).
template <typename Args>
inline int launch_cfg(void (*fn)(Args), bool *attr_set, size_t smem, int cols, const Args &a0, int batch, int max_q_len,
                      hipStream_t stream, int threads = 512, int layers = 1) {
  Args a = a0;
  dim3 grid;
  if (int rc = prefill_grid(a, cols, batch, max_q_len, layers, &grid)) return rc;
  if (int rc = grant_smem((const void *)fn, attr_set, smem)) return rc;
  hipLaunchKernelGGL(fn, grid, dim3((unsigned)threads), smem, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SP_ERR_HIP, "prefill launch: %s", hipGetErrorString(e));
  return SP_OK;
}

// attn_prefill_cut.hip: the CUT form and its combine pass, which is `groups` workgroups wide (at least cut_slots, as far as it matters).
int launch_prefill_cut(const PrefillArgs &a, int head_dim, int batch, int max_q_len, int groups, hipStream_t stream);
// attn_prefill_fresh.hip: append and prefill in one launch; split: 128-column workgroups.
int launch_prefill_fresh(const FreshArgs &a, bool split, int head_dim, int batch, int max_q_len, hipStream_t stream);
struct DecodeArgs;
// attn_mixed.hip: ranked prefill workgroups of 128 (split) or 256 columns and `shares` workgroups of the equal-share decode.
int launch_mixed(const PrefillArgs &a, const DecodeArgs &d, int shares, int pieces, bool split, int head_dim, int batch, int max_q_len, hipStream_t stream);

}  // namespace sp
