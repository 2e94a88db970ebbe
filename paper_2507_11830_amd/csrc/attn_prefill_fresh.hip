// Append and prefill in one launch (FreshArgs in prefill_tile.h), for whole prompts.
//
// Why.  As two launches the append comes first and costs a launch and three dependent memory round trips, 5 to 7 us, before the
// prefill kernel spends as much again on its own first tiles.  A prompt's keys are the step's own new rows, so a workgroup takes
// its tiles from them (which also saves the page ids' round trip) and stores the rows of its query tile to their pages while it works.
// Where the hints say that sequences have cached tokens the two launches are kept.  Where they say that there are none, they may
// still stand for more tokens than the call has, and nothing orders the workgroups of a launch: fresh_plan.h says how a sequence
// with cached tokens then gets the rows that the call appends, its own and those that other sequences append under its prefix.
// Measured (append and prefill, 8q/1kv d 128 where not said otherwise): 1 x 128 tokens at 2q/1kv d 64 9.2 -> 6.8 us, 1 x 300
// 14.7 -> 12.3, 1 x 1500 23.9 -> 22.0, 4 x 2048 51.6 -> 46.1, 1 x 9000 at 16q/2kv d 64 199 -> 193, 4 x 8192 at 32q/8kv 1822 -> 1800.
// Bound: as attn_prefill.hip; small prompts are a chain of the lengths, the first tiles and the stores.
#include "prefill_solo.h"

namespace sp {

template <int D>
static int launch_fresh_d(const FreshArgs &a, bool split, int batch, int max_q_len, hipStream_t stream) {
  constexpr size_t smem = kPrefillSmem<D>;
  static_assert(kPageBits / 8 <= smem && kPageBits / 8 <= kSoloSmem, "the set of pages lies where the tiles will");
  static bool set[2] = {false, false};
  if (split) return launch_cfg(prefill_kernel<D, KVT, PFD, true, false, 0, FreshArgs>, &set[0], 2 * smem, 128, a, batch, max_q_len, stream);
  if constexpr (D == 64) return launch_cfg(solo_prefill_kernel<FreshArgs>, &set[1], kSoloSmem, kSoloCols, a, batch, max_q_len, stream, kSoloThreads, kSoloLayers);
  else return launch_cfg(prefill_kernel<D, KVT, PFD, false, false, 0, FreshArgs>, &set[1], smem, 256, a, batch, max_q_len, stream);
}

int launch_prefill_fresh(const FreshArgs &a, bool split, int head_dim, int batch, int max_q_len, hipStream_t stream) {
  return head_dim == 128 ? launch_fresh_d<128>(a, split, batch, max_q_len, stream) : launch_fresh_d<64>(a, split, batch, max_q_len, stream);
}

}  // namespace sp
