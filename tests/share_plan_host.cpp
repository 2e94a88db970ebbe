// How the equal-share decode deals rows to workgroups (csrc/share_plan.h), for the CPU tests.
#include "share_plan.h"

extern "C" {

int share_of(int total, long wgs) { return sp::share_blocks(total, sp::share_inverse(wgs)); }
int one_wave(long rows, int geff, int max_len, int head_dim, long splits) {
  return sp::one_wave_pays(rows, geff, max_len, head_dim, splits, head_dim == 128 ? 256 : 512);
}
int pieces_of(int last, int share, int wg) { return sp::share_pieces(last, share, wg); }

}
