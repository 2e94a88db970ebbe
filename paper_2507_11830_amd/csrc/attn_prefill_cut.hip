// The form of the prefill kernel that cuts long work items (CUT in prefill_tile.h) and the pass that merges their
// partials.
//
// Why.  A work item is one (sequence, head group, 256-column query tile) and a CU runs one at a time.  In a launch
// of one or two rounds of items over cached prefixes of very different lengths the time is that of the longest item:
// 32 chunks of up to 512 tokens at half-cached contexts (median 1500 tokens, longest 8704) at 8 query heads / 1 KV
// head are 432 items of 1 to 136 key tiles, 39 tiles a CU on average, and the 136 tiles decided.  The host
// does not know the lengths, so the kernel finds by itself which items are longer than a CU's share and cuts them.
// Measured, append included: that batch 164 -> 106 us (765 TFLOP/s; kernel 163 -> 96-104, combine 6.5); 34 chunks of
// 64 tokens on prefixes of up to 8192, 93 -> 55 us; 3 chunks on 4370, 2q/1kv d 64, 34 -> 24 us (before: pieces of 128 columns).
// Bound: the matrix pipe as in the plain form, then how evenly pieces of half to one share fill 256 CUs.
#include "prefill_tile.h"

namespace sp {

// Merge of the partials of cut items.  A workgroup takes 32 columns of the tiles of every kCombineGroups-th slot and,
// where a slot is the first of an item, adds the item's pieces: wave v the channels v * D/4 .. in the lane
// order of the prefill kernel's accumulators, so that loads are 1 KiB in a row.  The kernel is a chain of
// memory round trips: one for the table (all of the workgroup's entries together), then one per item and four pieces.
// (How the workgroups that have work fall on the CUs changes with the launch's width by up to 4 us for small batches, without a
// rule: 16 items of 7 pieces, one head group, 119 wide 26.2 us, 121 wide 29.8; 6 of 16, 162 wide 26.9, 144 wide 35.8.  The width
// is that of a piece per kMinCutTiles key tiles, which was the best of those tried on most batches.)
constexpr int kCombineGroups = 208;
template <int D>
__global__ __launch_bounds__(256) void cut_combine_kernel(PrefillArgs a) {
  constexpr int NC = D / 32;  // 1 KiB chunks of a wave
  constexpr int NS = (kMostCutSlots + kCombineGroups - 1) / kCombineGroups;
  const int wb = blockIdx.y, wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 31, half = lane >> 5;
  const int used = *a.cut_used;
  CutEntry entry[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) entry[i] = a.cut_tab[min((int)blockIdx.x + i * kCombineGroups, a.cut_slots - 1)];
  const int C = wb * 32 + col;
#pragma unroll
  for (int si = 0; si < NS; ++si) {
    const CutEntry e = entry[si];
    const int slot = blockIdx.x + si * kCombineGroups;
    if (slot >= used || e.pieces <= 0) continue;  // uniform, like the next
    const int tok0 = e.tile * (256 >> a.gshift), token = tok0 + (C >> a.gshift);
    if (tok0 + ((wb * 32) >> a.gshift) >= e.q_len) continue;
    const float *po = a.part_o + ((size_t)slot * 8 + wb) * (32 * D) + (wv * NC) * 256 + lane * 4;
    const float *pml = a.part_ml + ((size_t)slot * 256 + C) * 2;
    float M = -INFINITY, den = 0.f;
    f32x4 acc[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto add = [&](int b, auto nc) __attribute__((always_inline)) {  // the pieces b .. b + N - 1
      constexpr int N = decltype(nc)::value;
      f32x2 ml[N];
      f32x4 v[N][NC];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const size_t at = (size_t)min(b + u, e.pieces - 1) * e.stride;  // past the end: the last one again, weight 0
        ml[u] = *reinterpret_cast<const f32x2 *>(pml + at * 512);
#pragma unroll
        for (int i = 0; i < NC; ++i) v[u][i] = *reinterpret_cast<const f32x4 *>(po + at * (256 * D) + i * 256);
      }
      __builtin_amdgcn_sched_barrier(0);  // all of it in flight before anything is used
      float Mn = M;
#pragma unroll
      for (int u = 0; u < N; ++u) Mn = fmaxf(Mn, ml[u][0]);
      const float alpha = __builtin_amdgcn_exp2f(M - Mn);  // the maxima are finite: 0 the first time
      M = Mn;
      den *= alpha;
#pragma unroll
      for (int i = 0; i < NC; ++i) acc[i] *= alpha;
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const float f = b + u < e.pieces ? __builtin_amdgcn_exp2f(ml[u][0] - M) : 0.f;
        den += f * ml[u][1];
#pragma unroll
        for (int i = 0; i < NC; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] += f * v[u][i][j];
      }
    };
    if (e.pieces == 2) {  // the usual case
      add(0, std::integral_constant<int, 2>{});
    } else {
      for (int b = 0; b < e.pieces; b += 4) add(b, std::integral_constant<int, 4>{});
    }
    if (token < e.q_len) {
      const float inv = 1.0f / den;
      const int head = (e.hg << a.gshift) | (C & ((1 << a.gshift) - 1));
      char *dst = a.out + ((long)(e.q0 + token) * a.Hq + head) * (D * 2);
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int n = wv * NC + i;  // chunk: 32-channel block n / 4, register quad n % 4
        store4_bf16(dst + (32 * (n >> 2) + 8 * (n & 3) + 4 * half) * 2, acc[i][0] * inv, acc[i][1] * inv, acc[i][2] * inv, acc[i][3] * inv);
      }
    }
  }
}

template <int D>
static int launch_cut_d(const PrefillArgs &a, int batch, int max_q_len, int groups, hipStream_t stream) {
  static bool set = false;
  int rc = launch_cfg(prefill_kernel<D, KVT, PFD, false, false, 1>, &set, kPrefillSmem<D>, 256, a, batch, max_q_len, stream);
  if (rc != SP_OK) return rc;
  hipLaunchKernelGGL(cut_combine_kernel<D>, dim3((unsigned)(groups < kCombineGroups ? groups : kCombineGroups), 8), dim3(256), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SP_ERR_HIP, "prefill combine launch: %s", hipGetErrorString(e));
  return SP_OK;
}

int launch_prefill_cut(const PrefillArgs &a, int head_dim, int batch, int max_q_len, int groups, hipStream_t stream) {
  return head_dim == 128 ? launch_cut_d<128>(a, batch, max_q_len, groups, stream) : launch_cut_d<64>(a, batch, max_q_len, groups, stream);
}

}  // namespace sp
