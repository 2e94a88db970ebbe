// Which keys a workgroup of the launch that also appends (FRESH in prefill_tile.h) takes from where.  Nothing orders the
// workgroups of one launch, so none may read a row of the cache that this call appends, unless it has appended the row itself:
//   - from the first pair of key tiles on that holds new rows only, keys are read from the step's new rows themselves;
//   - new rows in the pages below that, the sequence's own next to its last cached tokens and those that another sequence of
//     the call appends to a page of the prefix (two prompts in one step, the second on the first one's pages), the workgroup appends
//     itself before it reads them.  Others write the same rows at the same time, with the same bytes.
// Plain integer code that compiles for the host as well, for the CPU tests.
#pragma once

#ifndef SP_HD
#ifdef __HIP__
#define SP_HD __host__ __device__ __forceinline__
#else
#define SP_HD inline
#endif
#endif

namespace sp {

constexpr int kFreshPage = 16;  // tokens

// The first key tile (64 tokens) that is read from the new rows, of a sequence with ctx cached tokens.  Even, so that two
// streams of alternate tiles turn to them in the same period.
constexpr int kFreshTilePages = 4;
SP_HD int first_new_tile(int ctx) { return ctx < 0 ? 0x7ffffff0 / kFreshTilePages : (int)(((long)ctx + 127) / 128 * 2); }
// Pages below it, which are read from the pool.
SP_HD int pool_pages(int ctx) { return first_new_tile(ctx) * kFreshTilePages; }

// Pages that the new rows of one sequence reach into, at most.
SP_HD int most_new_pages(int max_q_len) { return (int)(((long)max_q_len + 2 * (kFreshPage - 1)) / kFreshPage); }

// The set of the pages that are read from the pool, one bit per page id modulo its size: exact for pools of up to that many pages, beyond
// it some pages are appended to for nothing.
constexpr int kPageBits = 1 << 18;
SP_HD int page_word(int page) { return (page & (kPageBits - 1)) >> 5; }
SP_HD unsigned page_bit(int page) { return 1u << (page & 31); }

// What the call appends to one page.
struct NewRows {
  int seq;
  long entry;  // of the block table: which page
  int src;     // the first of the new rows
  int lo, n;   // rows lo .. lo + n - 1 of the page
};

// The i-th of the batch x per pairs of a sequence and one of the pages (per = most_new_pages) its new rows may reach into; false: they do not.
SP_HD bool new_rows_of_pair(int i, int per, const int *cu_q, const int *ctx_lens, int max_pages, NewRows *o) {
  const int s = i / per, ctx = ctx_lens[s], src = cu_q[s], end = ctx + cu_q[s + 1] - src;
  if (ctx < 0) return false;
  const int page = ctx / kFreshPage + (i - s * per), from = page * kFreshPage;
  const int first = from > ctx ? from : ctx, last = from + kFreshPage < end ? from + kFreshPage : end;
  if (first >= last || page >= max_pages) return false;
  o->seq = s;
  o->entry = (long)s * max_pages + page;
  o->src = src + (first - ctx);
  o->lo = first - from;
  o->n = last - first;
  return true;
}

// Whether n bytes at p and m bytes at q have none in common.
inline bool apart(const void *p, long n, const void *q, long m) {
  const unsigned long a = (unsigned long)p, b = (unsigned long)q;
  return a < b ? b - a >= (unsigned long)n : a - b >= (unsigned long)m;
}

}  // namespace sp
