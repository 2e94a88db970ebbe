// Mixed batches in one launch: the prefill workgroups of the sequences with long chunks and, behind them in the
// dispatch order, the equal-share decode workgroups of the sequences with a few query tokens.
//
// Why.  One after the other, the two leave half of the chip idle: the prefill workgroups are few and bound by the
// matrix pipe and their own length, the decode ones are bound by HBM.  A CU takes one workgroup of either kind at a time
// (LDS, registers), so the CUs without a prefill item start on the keys of the decoding sequences at once, and the others
// join them as their items end.  The two halves touch disjoint rows of `out`; only the decode one uses the workspace.
// Measured (63 sequences of 512..8192 keys and a 2048-token chunk, 8q/1kv d 128, append and combine included):
// 63.0 -> 47.8 us (append 5.5, the launch 36, combine 4.5; before: append 5.5, prefill 31.4, decode 23.9, combine 4.5);
// 36 sequences of up to 3586 keys and 197 tokens: 30.5 -> 22; 23 of up to 5059 and 1586, 16q/2kv: 51.3 -> 44.
#include "decode_stream.h"
#include "prefill_tile.h"

namespace sp {

struct MixedArgs : PrefillArgs {
  DecodeArgs d;
  unsigned first_other;  // first launch index of the decode workgroups
  template <int D>
  __device__ __forceinline__ void run_other(lds_char *smem, int lane) const {
    if (threadIdx.x >= 64 * kWaves) return;  // barriers do not wait for waves that have ended
    decode_share<D, false, true, 1>(d, smem, lane, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), (int)(blockIdx.x - first_other));
  }
};

template <int D, bool SPLIT>
static int launch_mixed_d(const PrefillArgs &a, const DecodeArgs &d, int shares, int pieces, int batch, int max_q_len, hipStream_t stream) {
  static bool set = false;
  constexpr size_t own = (SPLIT ? 2 : 1) * kPrefillSmem<D>, other = kDecodeShareSmem<D, true>;
  constexpr size_t smem = own > other ? own : other;
  auto fn = prefill_kernel<D, KVT, PFD, SPLIT, false, 0, MixedArgs>;
  MixedArgs m;
  static_cast<PrefillArgs &>(m) = a;
  m.d = d;
  dim3 grid;
  if (int rc = prefill_grid(m, SPLIT ? 128 : 256, batch, max_q_len, 1, &grid)) return rc;
  if (!m.ranked || grid.x > 0x7fffffffu - (unsigned)shares) return 1;
  m.first_other = grid.x;
  grid.x += (unsigned)shares;
  if (int rc = grant_smem((const void *)fn, &set, smem)) return rc;
  hipLaunchKernelGGL(fn, grid, dim3(512), smem, stream, m);
  launch_decode_combine(d, pieces, D, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SP_ERR_HIP, "mixed launch: %s", hipGetErrorString(e));
  return SP_OK;
}

int launch_mixed(const PrefillArgs &a, const DecodeArgs &d, int shares, int pieces, bool split, int head_dim, int batch, int max_q_len, hipStream_t stream) {
  if (head_dim == 128)
    return split ? launch_mixed_d<128, true>(a, d, shares, pieces, batch, max_q_len, stream)
                 : launch_mixed_d<128, false>(a, d, shares, pieces, batch, max_q_len, stream);
  return split ? launch_mixed_d<64, true>(a, d, shares, pieces, batch, max_q_len, stream)
               : launch_mixed_d<64, false>(a, d, shares, pieces, batch, max_q_len, stream);
}

}  // namespace sp
