// Decode attention with equal shares: the batch's keys, laid end to end in 32-key blocks, are dealt to
// the workgroups in equal contiguous runs, whatever the lengths of the sequences are.
//
// Why.  Splits of a fixed length leave the chip unevenly loaded: the grid has to be sized for the
// longest possible sequence (most of its workgroups then find no keys, yet hold a CU's LDS for the
// two microseconds it takes them to read the length), the last split of every sequence is short,
// and whether the batch happens to fill a whole number of rounds decides the time (measured on 64
// sequences of 512..8192 keys at 8 query heads / 1 KV head: 31 to 47 us over split lengths of 1024 to
// 4096 keys).  Here one launch of as many workgroups as the chip holds at once reads every key exactly
// once, and every workgroup reads the same number of keys.
//
// A row is one (sequence, head group).  Every workgroup reads the batch's length array (one memory
// round trip, the one that a workgroup of the other kernel spends on its own length), scans it with DPP
// shifts, takes its run of the concatenated rows and walks the row segments in it.  Inside a segment
// wave w of the four takes the blocks w, w + 4, ... through a private ring of two LDS slots (as in
// attn_decode.hip), and the four states are merged through LDS.  A row that lies in one run is written to
// `out` at once; a row that is cut leaves one un-normalised partial per workgroup it touches, and
// the combine kernel below merges those (the other rows' waves find nothing to do).
//
// A segment costs more than its keys: page ids, query rows and the first block are three dependent
// memory round trips, and the merge is a fourth.  Every row is therefore dealt with kRowCost blocks in
// front of its own, so that a workgroup with two segments gets fewer keys.
//
// Batches that fit one round of resident workgroups at up to 1024 keys each take the same kernel with fixed
// splits instead (launch_decode_stream says why), and sequences of up to 512 keys one workgroup per
// row, with no partial and no combine launch.
//
// Bound: HBM bandwidth, 4 * head_dim bytes per cached token per KV head; on small batches the chain of memory round
// trips.  Measured (split + combine, one-wave splits of fixed length before -> here): 64 sequences of 512..8192 keys,
// 8q/1kv, d 128: 37.5 -> 31.9 us (the key loop moves 157 MB in 20 us; 5 us pass before the first block is there, 3 us
// in the tail and the merge); 128 sequences of 1024..16384 keys, 32q/8kv (4.9 GB): 803 -> 728 us (6.7 TB/s);
// 64 x 4 query tokens: 35.4 -> 31.1 us; one sequence of 32900 keys: 12.5 -> 11.6 us; one of 137 keys: 11.2 -> 7.5 us.
#include "decode_block.h"

namespace sp {

constexpr int kWaves = 4;          // waves per workgroup
constexpr int kMaxSeqs = 512;      // longest batch (its rows' ends and lengths are held in LDS)
constexpr int kRowCost = 8;        // blocks that a segment's fixed cost amounts to (64-sequence batch: 4 blocks 34.5 us, 8 and 12 33.5)
constexpr int kMinShare = 12;      // blocks per workgroup below which a further cut costs more than it gives

typedef __attribute__((address_space(3))) int32_t lds_int;

// Inclusive prefix sum over the 64 lanes (gfx9 DPP: shifts inside rows of 16, then the two row
// broadcasts).
__device__ __forceinline__ int scan_incl(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
  return x;
}

// Page ids of the blocks i0 .. i0 + 31 of wave w in a segment that begins at the row's block p0: two per block,
// one per lane; -1 past the table row.  Bad metadata must not become a wild access: loads go through the clamped
// id, the fused-append stores through the raw one and are skipped when it lies outside the pool (the
// same rows sp_kv_append skips).
__device__ __forceinline__ int load_pages(const DecodeArgs &a, int seq, int p0, int i0, int w, int lane) {
  const int idx = 2 * (p0 + kWaves * (i0 + (lane >> 1)) + w) + (lane & 1);
  const int pg = a.block_table[(long)seq * a.max_pages + min(idx, a.max_pages - 1)];
  return idx < a.max_pages ? pg : -1;
}

// Key blocks [p0, p1) of one row, by the whole workgroup.  pages: load_pages of the segment's first blocks.
// whole: they are all of the row's, so the result is the output row; otherwise it goes to partial slot `slot`.
template <int D, bool APPEND, bool MQ, int NT>
__device__ __forceinline__ void row_segment(const DecodeArgs &a, lds_char *smem, int lane, int w, int seq, int hg, int L, int ctx,
                                            int tok_base, int p0, int p1, int pages, bool whole, int slot) {
  using G = TileGeom<D>;
  using Z = SwzTile<D>;
  constexpr int ROWB = D * 2;           // bytes of one K or V row
  constexpr int MBYTES = 32 * ROWB;     // one 32-key block of K or of V in LDS (swizzled, unpadded)
  constexpr int SLOT = 2 * MBYTES;      // K block, then V block
  constexpr int NI = MBYTES / 1024;     // 1 KiB load instructions per matrix and block
  constexpr int RPI = 1024 / ROWB;      // key rows per load instruction
  constexpr int LPB = 2 * NI;           // load instructions per block
  constexpr int CPR = D / 8;            // 16-byte chunks per row
  const int col = lane & 31, half = lane >> 5;
  const int head0 = hg * a.geff;
  const int kvh = a.hg_per_kv == 1 ? hg : hg / a.hg_per_kv;
  const bool writer = a.hg_per_kv == 1 || hg == kvh * a.hg_per_kv;  // fused append: one writer per (position, KV head)
  const float inv_geff = 1.0f / (float)a.geff;                      // (int)((x + 0.5) / geff) is x / geff for the x < 64 it is used on
  const int kv1 = min(L, 32 * p1);
  const int nb = (p1 - p0 + kWaves - 1 - w) / kWaves;             // blocks of this wave, may be 0
  auto base_of = [&](int i) __attribute__((always_inline)) { return 32 * (p0 + kWaves * i + w); };  // first key of its block i
  const int qn = MQ ? min(L - ctx, a.q_max) : 1;  // query tokens (no more than the caller's hint: the partial slots hold no more)
  // Column -> (query token, head) of the tile.
  const int t0 = MQ ? (int)(((float)col + 0.5f) * inv_geff) : 0, h_col = col - t0 * a.geff;
  bool col_valid[NT];
  int lim_col[NT];
  bf16x8 qreg[NT][G::kDSteps];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int t = nt * a.q_cap + t0;  // tile nt holds the tokens nt * q_cap .. (nt + 1) * q_cap - 1
    col_valid[nt] = MQ ? t0 < a.q_cap && t < qn : col < a.geff;
    lim_col[nt] = MQ ? (col_valid[nt] ? ctx + t + 1 : L) : 0;
    const char *qrow = a.q + ((long)(tok_base + t) * a.Hq + head0 + h_col) * (D * 2);
#pragma unroll
    for (int s = 0; s < G::kDSteps; ++s) {
      if (col_valid[nt]) {
        qreg[nt][s] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * s + 16 * half);
      } else {
        u32x4 z = {0, 0, 0, 0};
        qreg[nt][s] = *reinterpret_cast<bf16x8 *>(&z);
      }
    }
  }
  // single-token fused append: the new K/V row, one 16-byte chunk per lane
  u32x4 knew = {0, 0, 0, 0}, vnew = {0, 0, 0, 0};
  if (APPEND && !MQ) {
    const size_t noff = (((size_t)seq * a.Hkv + kvh) * CPR + (lane % CPR)) * 16;
    knew = *reinterpret_cast<const u32x4 *>(a.k_new + noff);
    vnew = *reinterpret_cast<const u32x4 *>(a.v_new + noff);
  }

  int pages_before = pages, pages_next = pages;
  if (nb > 32) pages_next = load_pages(a, seq, p0, 32, w, lane);

  // ---- block loads: as in attn_decode.hip
  const int dq = lane >> 4, dslot = lane & 15;
  constexpr int IPP = NI / 2;  // load instructions per page and matrix
  unsigned voff_k[IPP], voff_v[IPP];  // this lane's byte offset inside a (page, kv head) block, per instruction
#pragma unroll
  for (int jj = 0; jj < IPP; ++jj) {
    const int line = 4 * jj + dq;
    const int clk = dslot ^ Z::gk(line), clv = dslot ^ Z::gv(line);
    voff_k[jj] = (unsigned)(((D == 128 ? line : 2 * line + (clk >> 3)) & 15) * ROWB + (D == 128 ? clk : (clk & 7)) * 16);
    voff_v[jj] = (unsigned)(((D == 128 ? line : 2 * line + (clv >> 3)) & 15) * ROWB + (D == 128 ? clv : (clv & 7)) * 16);
  }
  const size_t page_stride = (size_t)a.Hkv * (kPage * ROWB);
  const char *kpool = a.k_pages + (size_t)kvh * (kPage * ROWB), *vpool = a.v_pages + (size_t)kvh * (kPage * ROWB);
  auto page_base = [&](const char *pool, int ln) __attribute__((always_inline)) {
    const int pg = min(max(__builtin_amdgcn_readlane(pages, ln), 0), a.num_pages - 1);
    return pool + (size_t)(unsigned)pg * page_stride;
  };
  auto issue_mat = [&](int bi, bool isv, unsigned dst0) __attribute__((always_inline)) {
    const char *pool = isv ? vpool : kpool;
    const int last = kv1 - 1 - base_of(bi);  // last valid row of the block
    const int ln = 2 * (bi & 31);
    if (last >= 31) {
#pragma unroll
      for (int pp = 0; pp < 2; ++pp) {
        const char *pb = page_base(pool, ln + pp);
#pragma unroll
        for (int jj = 0; jj < IPP; ++jj) {
          const unsigned dst = dst0 + (pp * IPP + jj) * 1024;
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(dst),
                       "v"(isv ? voff_v[jj] : voff_k[jj]), "s"(pb)
                       : "memory");
        }
      }
      return;
    }
    // the row's last, partial block: rows past the end are redirected to the last row
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int pslot = min(RPI * j, last) >> 4;  // uniform
      const int rip_lim = pslot == (last >> 4) ? (last & 15) : 15;
      const char *pb = page_base(pool, ln + pslot);
      const int line = 4 * j + dq;  // line inside the block
      const int cl = dslot ^ (isv ? Z::gv(line) : Z::gk(line));
      const int rip = (D == 128 ? line : 2 * line + (cl >> 3)) & 15;
      const int chunk16 = D == 128 ? cl : (cl & 7);
      const unsigned voff = (unsigned)(min(rip, rip_lim) * ROWB + chunk16 * 16);
      const unsigned dst = dst0 + j * 1024;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(dst), "v"(voff), "s"(pb)
                   : "memory");
    }
  };
  auto issue_block = [&](int bi) __attribute__((always_inline)) {
    if ((bi & 31) == 0 && bi > 0) {  // the next 32 blocks' page ids, requested 32 blocks ago
      pages_before = pages;
      pages = pages_next;
      if (bi + 32 < nb) pages_next = load_pages(a, seq, p0, bi + 32, w, lane);
    }
    const unsigned slot_base = (unsigned)((2 * w + (bi & 1)) * SLOT);
    issue_mat(bi, false, slot_base);
    issue_mat(bi, true, slot_base + MBYTES);
  };

  int kofs[G::kDSteps], vofs[G::kDBlocks];
#pragma unroll
  for (int s = 0; s < G::kDSteps; ++s) kofs[s] = Z::template offset<false>(col, 2 * s + half);
  {
    const int n = lane & 15, dg = (lane >> 4) & 1;
#pragma unroll
    for (int db = 0; db < G::kDBlocks; ++db)
      vofs[db] = Z::template offset<true>(4 * half + (n >> 2), 4 * db + 2 * dg + ((n & 3) >> 1)) + 8 * (n & 1);
  }
  f32x16 o[NT][G::kDBlocks];
  float m[NT], l[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    m[nt] = MQ ? -1e30f : -INFINITY;  // MQ: a column may see none of the first blocks' keys; exp2(m - m) stays defined
    l[nt] = 0.f;
#pragma unroll
    for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[nt][db][r] = 0.f;
  }

  if (nb > 0) issue_block(0);
  for (int i = 0; i < nb; ++i) {
    if (i + 1 < nb) {  // the slot of block i - 1 is free again
      issue_block(i + 1);
      wait_vmcnt<LPB>();
    } else {
      wait_vmcnt<0>();
    }
    const lds_char *sbk = smem + (2 * w + (i & 1)) * SLOT, *sbv = sbk + MBYTES;
    const int base = base_of(i);
    if (APPEND && MQ && base + 32 > ctx) {
      // Rows of this block at positions >= ctx are not in the cache yet: every lane fetches its 16-byte
      // pieces of the new rows, patches the block in LDS and, for positions of the row, stores them to their
      // pages.  Rows past the end take the chunk's last row.
      const int c = lane % CPR;
      const int pages_i = i + 1 < nb && ((i + 1) & 31) == 0 ? pages_before : pages;  // block i + 1 may have moved on to its 32 page ids
#pragma unroll
      for (int j = 0; j < 32 * CPR / 64; ++j) {
        const int row = j * (64 / CPR) + lane / CPR;
        const int pos = base + row;
        const int pg = __shfl(pages_i, 2 * (i & 31) + (row >> 4));  // by all lanes: a cross-lane read must not sit in the branch
        if (pos >= ctx) {
          const int t = min(pos, L - 1) - ctx;
          const size_t noff = (((size_t)(tok_base + t) * a.Hkv + kvh) * CPR + c) * 16;
          const u32x4 kn = *reinterpret_cast<const u32x4 *>(a.k_new + noff);
          const u32x4 vn = *reinterpret_cast<const u32x4 *>(a.v_new + noff);
          *(lds_u32x4 *)(const_cast<lds_char *>(sbk) + Z::template offset<false>(row, c)) = kn;
          *(lds_u32x4 *)(const_cast<lds_char *>(sbv) + Z::template offset<true>(row, c)) = vn;
          if (writer && pos < kv1 && pg >= 0 && pg < a.num_pages) {
            const size_t dst = (size_t)(unsigned)pg * page_stride + (size_t)(pos & 15) * ROWB + c * 16;
            *reinterpret_cast<u32x4 *>(const_cast<char *>(kpool) + dst) = kn;
            *reinterpret_cast<u32x4 *>(const_cast<char *>(vpool) + dst) = vn;
          }
        }
      }
      wave_lds_fence();
    }
    if (APPEND && !MQ && base + 32 >= L) {
      // The row's last block, which holds position L - 1: its row for that position and the rows after it
      // (redirected to it) are stale cache bytes; overwrite them in LDS and store the new row to its page.
      const int r_new = (L - 1) & 31, c = lane % CPR;
#pragma unroll
      for (int j = 0; j < 32 * CPR / 64; ++j) {
        const int row = j * (64 / CPR) + lane / CPR;
        if (row >= r_new) {
          *(lds_u32x4 *)(const_cast<lds_char *>(sbk) + Z::template offset<false>(row, c)) = knew;
          *(lds_u32x4 *)(const_cast<lds_char *>(sbv) + Z::template offset<true>(row, c)) = vnew;
        }
      }
      const int pg = __builtin_amdgcn_readlane(pages, 2 * (i & 31) + (r_new >> 4));
      if (lane < CPR && writer && pg >= 0 && pg < a.num_pages) {
        const size_t dst = (size_t)(unsigned)pg * page_stride + (size_t)((L - 1) & 15) * ROWB + c * 16;
        *reinterpret_cast<u32x4 *>(const_cast<char *>(kpool) + dst) = knew;
        *reinterpret_cast<u32x4 *>(const_cast<char *>(vpool) + dst) = vnew;
      }
      wave_lds_fence();
    }
    attend_block<D, MQ, NT>(sbk, sbv, kofs, vofs, qreg, o, m, l, base, kv1, ctx + 1, lim_col, half, a.sl2e, a.tau, L <= 256, [] {});
  }

  // ---- merge of the four waves' states: every wave leaves its o, m and l in LDS (rows padded by 16
  // bytes, so that the 16 lanes of a store hit all banks), then a thread sums four channels of a column.
  constexpr int OROW = D + 4;
  static_assert(kWaves * 32 * (OROW + 2) * 4 <= kWaves * 2 * SLOT, "the states must fit the rings");
  lds_float *xo = (lds_float *)smem, *xml = xo + kWaves * 32 * OROW;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float lt = l[nt] + other_half(l[nt]);
    __syncthreads();  // every wave is done with its ring (and, later on, with the tile before)
    if (col_valid[nt]) {
      lds_float *dst = xo + (w * 32 + col) * OROW + 4 * half;
#pragma unroll
      for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *(lds_f32x4 *)(dst + 32 * db + 8 * r4) =
              (f32x4){o[nt][db][4 * r4], o[nt][db][4 * r4 + 1], o[nt][db][4 * r4 + 2], o[nt][db][4 * r4 + 3]};
      if (half == 0) *(lds_f32x2 *)(xml + (w * 32 + col) * 2) = (f32x2){lt == 0.f ? -INFINITY : m[nt] * a.sl2e, lt};
    }
    __syncthreads();
    const int tile_cols = MQ ? min(max(qn - nt * a.q_cap, 0), a.q_cap) * a.geff : a.geff;
    for (int i = threadIdx.x; i < tile_cols * (D / 4); i += 64 * kWaves) {
      const int c = i / (D / 4), ch = 4 * (i - c * (D / 4));
      float M = -INFINITY, den = 0.f;
      f32x2 wml[kWaves];
#pragma unroll
      for (int u = 0; u < kWaves; ++u) {
        wml[u] = *(lds_f32x2 *)(xml + (u * 32 + c) * 2);
        M = fmaxf(M, wml[u][0]);
      }
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < kWaves; ++u) {
        const float f = wml[u][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(wml[u][0] - M);
        den += f * wml[u][1];
        const f32x4 ou = *(lds_f32x4 *)(xo + (u * 32 + c) * OROW + ch);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += f * ou[e];
      }
      const int tc = nt * a.q_cap * a.geff + c;  // token * geff + head
      if (whole) {  // at least one key: M is finite
        const int t = MQ ? (int)(((float)tc + 0.5f) * inv_geff) : 0;
        const float inv = 1.0f / den;
        *reinterpret_cast<bf16x4 *>(a.out + (((long)(tok_base + t) * a.Hq + head0 + tc - t * a.geff) * D + ch) * 2) =
            __builtin_convertvector(acc * inv, bf16x4);
      } else {
        const long pidx = (long)slot * a.cols + tc;
        *reinterpret_cast<f32x4 *>(a.part_o + pidx * D + ch) = acc;
        if (ch == 0) *reinterpret_cast<f32x2 *>(a.part_ml + pidx * 2) = (f32x2){M, den};
      }
    }
  }
}

// out row of a sequence without keys
template <int D>
__device__ __forceinline__ void zero_row(const DecodeArgs &a, int seq, int hg) {
  char *dst = a.out + ((long)seq * a.Hq + hg * a.geff) * (D * 2);
  for (int i = threadIdx.x; i < a.geff * (D / 8); i += 64 * kWaves) *reinterpret_cast<u32x4 *>(dst + 16 * i) = (u32x4){0, 0, 0, 0};
}

template <int D, bool APPEND, bool MQ, int NT>
__global__ __launch_bounds__(64 * kWaves, NT > 1 ? 1 : 2) void decode_stream_kernel(DecodeArgs a) {
  constexpr int RING = kWaves * 2 * 2 * 32 * D * 2;
  extern __shared__ __align__(16) char smem_raw[];
  lds_char *smem = (lds_char *)smem_raw;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Blocks of a sequence's row plus the row's fixed cost; 0 for a sequence that has no output row here.
  auto weight = [&](int L, int qn) __attribute__((always_inline)) {
    if (MQ && (qn <= 0 || (a.route_cap > 0 && qn > a.route_cap))) return 0;
    return ((max(L, 0) + 31) >> 5) + kRowCost;
  };
  if (a.row_splits) {  // fixed splits of a.chunk keys
    const int hg = blockIdx.x, seq = blockIdx.y, split = blockIdx.z;
    int L, ctx = 0, tok = seq, qn = 1;
    const int p0 = split * (a.chunk >> 5);
    const int pages = load_pages(a, seq, p0, 0, w, lane);  // in the same round trip as the lengths
    if (MQ) {
      tok = a.cu_q[seq];
      qn = a.cu_q[seq + 1] - tok;
      ctx = a.ctx_lens[seq];
      L = ctx + qn;
      if (weight(L, qn) == 0) return;
    } else {
      L = a.seq_lens[seq];
    }
    const int p1 = min((L + 31) >> 5, p0 + (a.chunk >> 5)), slot = (seq * a.n_hgroups + hg) * a.row_splits + split;
    if (p1 <= p0) {  // no keys: a row of zeros if there is no other split, else an empty partial
      if (a.row_splits == 1) {
        if (!MQ) zero_row<D>(a, seq, hg);
      } else if ((int)threadIdx.x < a.cols) {
        *reinterpret_cast<f32x2 *>(a.part_ml + 2 * ((long)slot * a.cols + threadIdx.x)) = (f32x2){-INFINITY, 0.f};
      }
      return;
    }
    row_segment<D, APPEND, MQ, NT>(a, smem, lane, w, seq, hg, L, ctx, tok, p0, p1, pages, a.row_splits == 1, slot);
    return;
  }
  // ---- the batch's rows, laid end to end: s_end[s] = end of sequence s's rows.  Every wave computes and
  // writes the same values, so none has to wait for another.
  lds_int *s_end = (lds_int *)(smem + RING), *s_len = s_end + kMaxSeqs, *s_ctx = s_len + kMaxSeqs, *s_tok = s_ctx + kMaxSeqs;
  const int nslot = (a.batch + 63) >> 6;  // uniform
  int total = 0;
#pragma unroll 1
  for (int u = 0; u < nslot; ++u) {
    const int s = u * 64 + lane;
    int len = 0, qn = 1, wt = 0;
    if (s < a.batch) {
      if (MQ) {
        const int tok = a.cu_q[s], ctx = a.ctx_lens[s];
        qn = a.cu_q[s + 1] - tok;
        len = ctx + qn;
        s_ctx[s] = ctx;
        s_tok[s] = tok;
      } else {
        len = a.seq_lens[s];
      }
      wt = weight(len, qn);
    }
    const int end = total + scan_incl(wt * a.n_hgroups);
    total = __builtin_amdgcn_readlane(end, 63);
    s_end[s] = end;
    s_len[s] = len;
  }
  wave_lds_fence();
  int share = (int)(((unsigned long long)(unsigned)total * a.inv_wgs) >> 32) + 1;  // >= total / workgroups
  share = (max(share, kMinShare + kRowCost) + kWaves - 1) & -kWaves;
  const int lo = blockIdx.x * share, hi = min(total, lo + share);
  if (lo >= hi) return;
  auto uni = [&](lds_int *p) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(*p); };
  int seq = 0;
#pragma unroll 1
  for (int u = 0; u < nslot; ++u) {
    const int s = u * 64 + lane;
    seq += __builtin_popcountll(__builtin_amdgcn_ballot_w64(s < a.batch && s_end[s] <= lo));
  }
  int row0 = seq > 0 ? uni(s_end + seq - 1) : 0, hg = 0;  // where the row begins, and its head group
  int end = uni(s_end + seq), L = uni(s_len + seq);
  int v = ((max(L, 0) + 31) >> 5) + kRowCost;             // the row's weight
#pragma unroll 1
  while (row0 + v <= lo) {
    row0 += v;
    ++hg;
  }
  for (;;) {
    const int ctx = MQ ? uni(s_ctx + seq) : 0, tok = MQ ? uni(s_tok + seq) : seq;
    const int first = row0 + kRowCost, last = row0 + v;  // the row's key blocks
    const int p0 = max(lo - first, 0), p1 = min(hi, last) - first;
    const int row = seq * a.n_hgroups + hg;
    if (first == last) {
      if (!MQ && row0 >= lo) zero_row<D>(a, seq, hg);
      if (row0 >= lo && threadIdx.x == 0) *reinterpret_cast<u32x2 *>(a.row_tab + 2 * (long)row) = (u32x2){0, 1};
    } else if (p1 > p0) {
      const bool whole = p0 == 0 && p1 == v - kRowCost;
      if (p0 == 0 && threadIdx.x == 0) {  // the row's first partial slot and its number of partials
        const uint32_t pieces = whole ? 1 : (uint32_t)((last - 1) / share - (int)blockIdx.x + 1);
        *reinterpret_cast<u32x2 *>(a.row_tab + 2 * (long)row) = (u32x2){(uint32_t)(blockIdx.x + row), pieces};
      }
      row_segment<D, APPEND, MQ, NT>(a, smem, lane, w, seq, hg, L, ctx, tok, p0, p1, load_pages(a, seq, p0, 0, w, lane), whole, blockIdx.x + row);
    }
    if (last >= hi) return;
    if (p1 > p0) __syncthreads();  // the next segment's loads go where this one's states are
    row0 = last;
    ++hg;
    if (row0 == end) {  // on to the next sequence that has rows
      hg = 0;
      do {
        ++seq;
        end = uni(s_end + seq);
      } while (end == row0);
      L = uni(s_len + seq);
      v = ((max(L, 0) + 31) >> 5) + kRowCost;
    }
  }
}

// Merge of the partials of the rows that were cut: one workgroup per (row, column), one wave per 32-channel
// slice; eight lanes x 16 bytes cover the slice of one partial, so a load instruction covers eight
// partials and NB of them are in flight together.  Lane group g adds the partials g, g + 8, ... in order,
// the eight groups are added in a fixed butterfly.
//
// PG > 1 (rows in many pieces): PG such workgroups in one, each merging a contiguous run of the row's
// partials; the PG results meet in LDS.
template <int D, int NB, int PG, bool MQ>
__global__ __launch_bounds__(2 * D * PG) void combine_rows_kernel(DecodeArgs a) {
  const int tc = blockIdx.x, row = blockIdx.y;
  const int pg = threadIdx.x / (2 * D), lane = threadIdx.x & 63, g = lane >> 3;
  const int ch = ((threadIdx.x & (2 * D - 1)) >> 6) * 32 + (lane & 7) * 4;
  u32x2 tab = {(uint32_t)(row * a.row_splits), (uint32_t)a.row_splits};
  if (a.row_splits == 0) tab = *reinterpret_cast<const u32x2 *>(a.row_tab + 2 * (long)row);
  long orow = (long)row * a.geff + tc;  // a.Hq = head groups x geff
  if (MQ) {
    const int seq = row / a.n_hgroups, hg = row - seq * a.n_hgroups;
    const int tok = a.cu_q[seq], qn = a.cu_q[seq + 1] - tok;
    const int t = tc / a.geff;
    orow = (long)(tok + t) * a.Hq + hg * a.geff + tc - t * a.geff;
    if (t >= qn || (a.route_cap > 0 && qn > a.route_cap)) return;
  }
  int n = (int)tab[1];
  if (n <= 1) return;  // written by the split kernel
  long p0 = (long)tab[0] * a.cols + tc;
  if (PG > 1) {
    const int per = (n + PG - 1) / PG, from = min(pg * per, n);
    p0 += (long)from * a.cols;
    n = min(per, n - from);
  }
  float M = -INFINITY, den = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int b = 0; b < n; b += 8 * NB) {
    f32x2 ml[NB];
    f32x4 v[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const long p = p0 + (long)min(b + 8 * u + g, n - 1) * a.cols;  // past the end: the last one again, weight 0
      ml[u] = *reinterpret_cast<const f32x2 *>(a.part_ml + 2 * p);
      v[u] = *reinterpret_cast<const f32x4 *>(a.part_o + p * D + ch);
    }
    __builtin_amdgcn_sched_barrier(0);  // all of it in flight before anything is used
    float mb = -INFINITY;
#pragma unroll
    for (int u = 0; u < NB; ++u) mb = fmaxf(mb, b + 8 * u + g < n ? ml[u][0] : -INFINITY);
#pragma unroll
    for (int o = 8; o <= 32; o <<= 1) mb = fmaxf(mb, __shfl_xor(mb, o));
    const float Mn = fmaxf(M, mb);
    const float alpha = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
    acc *= alpha;
    den *= alpha;
    M = Mn;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const bool live = b + 8 * u + g < n && ml[u][0] != -INFINITY;  // a column may see none of a partial's keys
      const float f = live ? __builtin_amdgcn_exp2f(ml[u][0] - M) : 0.f;
      den += live ? f * ml[u][1] : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += live ? f * v[u][e] : 0.f;
    }
  }
#pragma unroll
  for (int o = 8; o <= 32; o <<= 1) {
    den += __shfl_xor(den, o);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o);
  }
  if constexpr (PG > 1) {
    __shared__ f32x4 x_acc[PG][D / 4];
    __shared__ f32x2 x_ml[PG];
    if (g == 0) x_acc[pg][ch / 4] = acc;
    if ((threadIdx.x & (2 * D - 1)) == 0) x_ml[pg] = (f32x2){M, den};
    __syncthreads();
    if (threadIdx.x >= D / 4) return;
    M = -INFINITY;
#pragma unroll
    for (int u = 0; u < PG; ++u) M = fmaxf(M, x_ml[u][0]);
    acc = (f32x4){0.f, 0.f, 0.f, 0.f};
    den = 0.f;
#pragma unroll
    for (int u = 0; u < PG; ++u) {
      const float f = x_ml[u][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x_ml[u][0] - M);
      den += f * x_ml[u][1];
      const f32x4 au = x_acc[u][threadIdx.x];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += f * au[e];
    }
  } else if (g != 0) {
    return;
  }
  const int och = PG > 1 ? 4 * (int)threadIdx.x : ch;
  const float inv = M == -INFINITY ? 0.f : 1.0f / den;  // no keys at all: zeros
  *reinterpret_cast<bf16x4 *>(a.out + (orow * D + och) * 2) = __builtin_convertvector(acc * inv, bf16x4);
}

template <int D, bool APPEND, bool MQ, int NT>
static int launch_stream(const DecodeArgs &a, dim3 wgs, int max_pieces, hipStream_t stream) {
  static bool attr_set = false;  // benign if two threads race
  constexpr int smem = kWaves * 2 * 2 * 32 * D * 2 + (MQ ? 4 : 2) * kMaxSeqs * 4;
  auto fn = decode_stream_kernel<D, APPEND, MQ, NT>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return fail(SP_ERR_HIP, "decode smem attribute: %s", hipGetErrorString(e));
    attr_set = true;
  }
  hipLaunchKernelGGL(fn, wgs, dim3(64 * kWaves), smem, stream, a);
  if (a.row_splits != 1) {
    const dim3 grid((unsigned)a.cols, (unsigned)(a.batch * a.n_hgroups)), block(2 * D);
    if (max_pieces <= 16) hipLaunchKernelGGL((combine_rows_kernel<D, 2, 1, MQ>), grid, block, 0, stream, a);
    else if (max_pieces <= 64) hipLaunchKernelGGL((combine_rows_kernel<D, 8, 1, MQ>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((combine_rows_kernel<D, 8, 4, MQ>), grid, dim3(8 * D), 0, stream, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SP_ERR_HIP, "decode launch: %s", hipGetErrorString(e));
  return SP_OK;
}

int launch_decode_stream(DecodeArgs &a, int batch, int max_q, int tiles, int max_len, int head_dim, void *workspace,
                         size_t workspace_bytes, int form, hipStream_t stream) {
  const long rows = (long)batch * a.n_hgroups;
  const bool mq = a.cu_q != nullptr;
  if (rows > 65535) return 1;
  // Single tokens on little data (up to 32 MB of K at most) and middling lengths: one wave per 128 keys writes its
  // partial without the merge's barriers, and its combine pass is not long yet (16 sequences of
  // 512..8192 keys at 8q/1kv: 13.0 us against 13.8; from 32 such sequences on, 20.8 against 19.4).
  if (form == 0 && !mq && max_len > 512 && max_len <= 8192 && rows * max_len * head_dim <= 8192L * 16 * 128) return 1;
  a.batch = batch;
  a.hg_per_kv = a.group / a.geff;
  a.q_max = max_q;
  a.cols = max_q * a.geff;
  // Workgroups that are resident at once: one per CU at head_dim 128 and two at 64 (LDS; one with two
  // column tiles: registers).
  const long resident = head_dim == 128 || tiles == 2 ? 256 : 512;
  const size_t slot_bytes = (size_t)a.cols * (head_dim + 2) * sizeof(float);
  const size_t ws = workspace ? workspace_bytes : 0;
  dim3 wgs;
  int max_pieces;
  // Fixed splits where the shortest that fit one round of resident workgroups, all sequences taken as long
  // as the longest, are at most 1024 keys: a workgroup's start is then one memory round trip shorter
  // than with equal shares, and so is the combine pass.
  int chunk = max_len <= 512 && form == 0 ? 512 : 256;
  while (chunk <= 1024 && rows * ((max_len + chunk - 1) / chunk) > resident && (max_len > 512 || form != 0)) chunk += 128;
  long splits = (max_len + chunk - 1) / chunk;
  if (chunk > 1024 || form == 2 || (splits > 1 && ws < rows * splits * slot_bytes)) splits = 0;
  // Equal shares: a partial slot per (workgroup, row) pair along the concatenated rows, and the table of rows.
  const size_t tab = (size_t)(rows * 8 + 15) / 16 * 16;
  const long least = kMinShare + kRowCost;
  const long useful = (rows * ((max_len + 31) / 32 + kRowCost) + least - 1) / least;
  const long want = resident < useful ? resident : useful;
  if (splits == 0 && (batch > kMaxSeqs || ws < tab + (rows + want) * slot_bytes)) {
    if (max_len > 1024) return 1;
    chunk = 1024;
    splits = 1;
  }
  a.row_splits = (int)splits;
  a.chunk = chunk;
  if (splits > 0) {
    wgs = dim3((unsigned)a.n_hgroups, (unsigned)batch, (unsigned)splits);
    max_pieces = (int)splits;
    a.part_o = (float *)workspace;
    a.part_ml = a.part_o + (size_t)rows * splits * a.cols * head_dim;
  } else {
    wgs = dim3((unsigned)want);
    max_pieces = (int)((max_len + 31) / 32 / least + 2);
    if (max_pieces > want) max_pieces = (int)want;
    a.inv_wgs = (unsigned)((0x100000000ull + want - 1) / want);
    a.row_tab = (int32_t *)workspace;
    a.part_o = (float *)((char *)workspace + tab);
    a.part_ml = a.part_o + (size_t)(rows + want) * a.cols * head_dim;
  }
#define SP_STREAM(D_)                                                                                                    \
  (!mq ? (a.k_new ? launch_stream<D_, true, false, 1>(a, wgs, max_pieces, stream) : launch_stream<D_, false, false, 1>(a, wgs, max_pieces, stream)) \
   : tiles == 1                                                                                                          \
       ? (a.k_new ? launch_stream<D_, true, true, 1>(a, wgs, max_pieces, stream) : launch_stream<D_, false, true, 1>(a, wgs, max_pieces, stream))   \
       : (a.k_new ? launch_stream<D_, true, true, 2>(a, wgs, max_pieces, stream) : launch_stream<D_, false, true, 2>(a, wgs, max_pieces, stream)))
  return head_dim == 128 ? SP_STREAM(128) : SP_STREAM(64);
#undef SP_STREAM
}

}  // namespace sp
