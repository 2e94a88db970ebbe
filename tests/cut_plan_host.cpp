// The cut form's arithmetic (csrc/cut_plan.h) for the CPU tests: one "lane" that holds the whole batch.
#include "cut_plan.h"

extern "C" {

int form_slots(int batch, int total_q, int max_q_len, int max_kv_len, int num_q_heads, int num_kv_heads, int head_dim) {
  return sp::cut_form_slots(batch, total_q, max_q_len, max_kv_len, num_q_heads, num_kv_heads, head_dim, false);
}

int merge_groups(int batch, int total_q, int max_kv_len, int num_q_heads, int n_hgroups) {
  return sp::cut_merge_groups(batch, total_q, max_kv_len, num_q_heads, n_hgroups, false);
}

int launched_workgroups(long total_q, int tpt, int batch, int n_hgroups, int slots) {
  return (int)sp::ranked_workgroups(total_q, tpt, batch, n_hgroups, 1, slots);
}

int limit_of(int batch, const int *ctx, const int *new_tokens, int tpt_shift, int n_hgroups, int slots, int launched, int *total_pieces) {
  static int c[256], q[256], nt[256], p[256];
  for (int s = 0; s < 256; ++s) {
    c[s] = s < batch ? ctx[s] : 0;
    q[s] = s < batch ? new_tokens[s] : 0;
    nt[s] = (q[s] + (1 << tpt_shift) - 1) >> tpt_shift;
  }
  auto same = [](int x) { return x; };
  return sp::cut_limit(c, q, nt, batch, tpt_shift, n_hgroups, slots, launched, same, same, p, total_pieces);
}

}
