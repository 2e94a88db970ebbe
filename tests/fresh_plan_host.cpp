// The choice of sources of the launch that also appends (csrc/fresh_plan.h) for the CPU tests: what one workgroup appends before
// it reads, in the kernel's order, with one thread.
#include "fresh_plan.h"

#include <vector>

extern "C" {

int apart(const void *p, long n, const void *q, long m) { return sp::apart(p, n, q, m); }

int pool_pages(int ctx) { return sp::pool_pages(ctx); }

// Rows (page, row of it, new row) that a workgroup of sequence seq appends to the pages it reads from the pool; returns their number.
int appended(int batch, int max_q_len, const int *cu_q, const int *ctx_lens, const int *table, int max_pages, int num_pages, int seq, int *rows) {
  std::vector<unsigned> set(sp::kPageBits / 32, 0u);
  for (int i = 0; i < sp::pool_pages(ctx_lens[seq]) && i < max_pages; ++i) {
    const int page = table[(long)seq * max_pages + i];
    set[sp::page_word(page)] |= sp::page_bit(page);
  }
  int n = 0;
  const int len = cu_q[seq + 1] - cu_q[seq], room = sp::pool_pages(ctx_lens[seq]) * sp::kFreshPage - ctx_lens[seq];
  for (int t = 0; t < len && t < room; ++t, ++n) {  // its own
    const int pos = ctx_lens[seq] + t;
    rows[3 * n] = table[(long)seq * max_pages + pos / 16];
    rows[3 * n + 1] = pos % 16;
    rows[3 * n + 2] = cu_q[seq] + t;
  }
  const int per = sp::most_new_pages(max_q_len);
  for (int i = 0; i < batch * per; ++i) {
    sp::NewRows r = {-1, 0, 0, 0, 0};
    if (!sp::new_rows_of_pair(i, per, cu_q, ctx_lens, max_pages, &r) || r.seq == seq) continue;
    const int page = table[r.entry];
    if (page < 0 || page >= num_pages || !(set[sp::page_word(page)] & sp::page_bit(page))) continue;
    for (int k = 0; k < r.n; ++k, ++n) {
      rows[3 * n] = page;
      rows[3 * n + 1] = r.lo + k;
      rows[3 * n + 2] = r.src + k;
    }
  }
  return n;
}

}
