// Shared by the two decode split kernels (attn_decode.hip: one wave per split of fixed length;
// attn_decode_stream.hip: workgroups of four waves with equal shares of the batch's keys): launch
// arguments, ordering helpers and the work on one 32-key block.
#pragma once
#include "attn_tile.h"

namespace sp {

struct DecodeArgs {
  const char *k_pages, *v_pages, *q;
  const char *k_new, *v_new;  // APPEND kernels: this step's K/V rows, bf16 [tokens][Hkv][D] (one token per sequence unless MQ)
  const int32_t *seq_lens, *block_table;
  const int32_t *cu_q, *ctx_lens;  // MQ kernels: query-token prefix sums [batch + 1], cached lengths [batch]
  float *part_o;   // [row][nsplit][D], row = token * Hq + head (one token per sequence unless MQ)
  float *part_ml;  // [row][nsplit][2]  (m in log2 units, l)
  int max_pages, num_pages, Hq, Hkv, group, geff, n_hgroups, chunk, nsplit;
  int q_cap;  // MQ kernels: query tokens per tile (32 / geff)
  int route_cap;  // MQ kernels: 0, or (mixed batches) only sequences with at most this many query tokens are
                  // served, and the partials are indexed [sequence][route_cap tokens][head] instead of by token row
  int32_t *arrive;  // FUSE kernels: one arrival counter per (sequence, head group), zero between launches
  char *out;        // FUSE kernels: bf16 [batch][Hq][D]
  // stream kernels (attn_decode_stream.hip): row_splits splits of `chunk` keys per row, or (0) the rows dealt in equal
  // runs; partials [slot][cols][D], cols = query tokens x geff; equal runs: per row its first slot and number of slots
  int batch, cols, row_splits, hg_per_kv, q_max;
  int32_t *row_tab;
  unsigned inv_wgs;  // share_inverse of the number of workgroups
  float sl2e;
  float tau;  // lazy-rescale threshold in raw score units (8 / sl2e)
};

// Orders a wave's own LDS writes before its later LDS reads without a workgroup barrier: the
// hardware runs one wave's LDS operations in order, so only the compiler has to be stopped from
// moving them across this point.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// s_waitcnt on the vector-memory counter only (the other counters are not named, so they are
// left alone).  The "memory" clobber keeps the compiler from moving LDS reads of the awaited
// block above it.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// One 32-key block (keys base .. base + 31, of which those at kv1 and beyond are masked; MQ: per column
// those at its causal limit and beyond) against the wave's column tiles: S^T = K Q^T, online softmax,
// O^T += V^T P^T.  sbk / sbv: the block's K and V in LDS; precise: weights as hi + lo.
template <int D, bool MQ, int NT, typename BeforePv>
__device__ __forceinline__ void attend_block(const lds_char *sbk, const lds_char *sbv, const int (&kofs)[D / 16], const int (&vofs)[D / 32],
                                             const bf16x8 (&qreg)[NT][D / 16], f32x16 (&o)[NT][D / 32], float (&m)[NT],
                                             float (&l)[NT], int base, int kv1, int lim_min, const int (&lim_col)[NT], int half,
                                             float sl2e, float tau, bool precise, BeforePv before_pv) {
  using G = TileGeom<D>;
  constexpr int ROWB = D * 2;
  f32x16 sacc[NT], sacc1[NT];  // two accumulators per tile halve the dependent MFMA chain a lone wave sits through
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[nt][r] = sacc1[nt][r] = 0.f;
#pragma unroll
  for (int s = 0; s < G::kDSteps; s += 2) {
    bf16x8 kop0 = *(const lds_bf16x8 *)(sbk + kofs[s]);
    bf16x8 kop1 = *(const lds_bf16x8 *)(sbk + kofs[s + 1]);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      sacc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop0, qreg[nt][s], sacc[nt], 0, 0, 0);
      sacc1[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop1, qreg[nt][s + 1], sacc1[nt], 0, 0, 0);
    }
  }
  bf16x8 pop[NT][2];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[nt][r] += sacc1[nt][r];
    if (MQ) {
      if (base + 32 > min(lim_min, kv1)) {  // the block reaches into the chunk: per-column causal limit
        const int lim = min(lim_col[nt], kv1);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          int kv = base + 8 * (r >> 2) + 4 * half + (r & 3);
          if (kv >= lim) sacc[nt][r] = -INFINITY;
        }
      }
    } else if (base + 32 > kv1) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        int kv = base + 8 * (r >> 2) + 4 * half + (r & 3);
        if (kv >= kv1) sacc[nt][r] = -INFINITY;
      }
    }
    float mx = sacc[nt][0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sacc[nt][r]);
    mx = fmaxf(mx, other_half(mx));
    // The running max only moves when some column's block max exceeds it by more than 2^8 in
    // the exponent (tau); otherwise weights are taken against the stale max (bounded by 2^8,
    // harmless in fp32/bf16) and the O accumulators need no rescale.
    if (__builtin_amdgcn_ballot_w64(mx > m[nt] + tau) != 0) {  // wave-uniform, rare after the first block
      const float m_new = fmaxf(m[nt], mx);
      const float alpha = __builtin_amdgcn_exp2f((m[nt] - m_new) * sl2e);
      m[nt] = m_new;
      l[nt] *= alpha;
#pragma unroll
      for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[nt][db][r] *= alpha;
    }
    const float msc = m[nt] * sl2e;
    float lsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[nt][r], sl2e, -msc));
      sacc[nt][r] = p;
      lsum += p;
    }
    l[nt] += lsum;
    pop[nt][0] = pack8(sacc[nt], 0);
    pop[nt][1] = pack8(sacc[nt], 8);
  }
  before_pv();
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int db = 0; db < G::kDBlocks; ++db) {
      bf16x8 vop = lds_read_vt(sbv + vofs[db] + 16 * ks * ROWB, ROWB);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        o[nt][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop, pop[nt][ks], o[nt][db], 0, 0, 0);
    }
  if (precise) {  // short sequences: weights as hi + lo, so the bf16 rounding of P (which only averages out over many keys) stays out of the tolerance
    bf16x8 plo[NT][2];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      plo[nt][0] = pack8_residual(sacc[nt], 0, pop[nt][0]);
      plo[nt][1] = pack8_residual(sacc[nt], 8, pop[nt][1]);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < G::kDBlocks; ++db) {
        bf16x8 vop = lds_read_vt(sbv + vofs[db] + 16 * ks * ROWB, ROWB);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          o[nt][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop, plo[nt][ks], o[nt][db], 0, 0, 0);
      }
  }
}

constexpr int kMaxShareSeqs = 512;  // longest batch of the equal-share decode (its rows' ends and lengths are held in LDS)

// Equal-share decode.  a: everything but the workspace pointers and the split fields is set.  max_q: query tokens per
// sequence at most, tiles: column tiles per wave.  Returns 1 without launching when the shape or the workspace
// does not qualify.  form: 0 built-in choice, 2 equal shares, 3 fixed splits.
int launch_decode_stream(DecodeArgs &a, int batch, int max_q, int tiles, int max_len, int head_dim, void *workspace,
                         size_t workspace_bytes, int form, hipStream_t stream);
// Its parts: everything but the launches (returns 1 if launch_decode_stream would; alone = false: the workgroups run next
// to prefill workgroups), and the merge of the partials of a plan with row_splits 0 over query chunks.
int plan_decode_stream(DecodeArgs &a, int batch, int max_q, int tiles, int max_len, int head_dim, void *workspace,
                       size_t workspace_bytes, int form, bool alone, dim3 *grid, int *pieces);
void launch_decode_combine(const DecodeArgs &a, int max_pieces, int head_dim, hipStream_t stream);
// Equal shares for the short sequences of a mixed batch (launch_decode_multi with routed = true): arguments, number of
// shares and of partials per row.  False where they cannot be taken.
bool plan_decode_routed(DecodeArgs &a, const sp_cache_desc &c, const void *q, void *out, const int32_t *cu_q,
                        const int32_t *ctx_lens, const int32_t *block_table, int batch, int max_pages, int max_kv_len,
                        int num_q_heads, float scale, void *workspace, size_t workspace_bytes, int *shares, int *pieces);

}  // namespace sp
