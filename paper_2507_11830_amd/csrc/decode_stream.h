// The work of one workgroup of the equal-share decode (attn_decode_stream.hip says how the keys are dealt and why), shared
// by the files that launch it: attn_decode_stream.hip and attn_mixed.hip.
#pragma once
#include "decode_block.h"
#include "share_plan.h"

namespace sp {

constexpr int kMaxSeqs = kMaxShareSeqs;

typedef __attribute__((address_space(3))) int32_t lds_int;

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
      // Computed anew for every block: hoisted out of the loop, the offsets of a rare block would hold 16 registers (with two
      // column tiles the kernel then keeps others in scratch memory, and reloads them for every block).
      int ln = lane;
      asm("" : "+v"(ln));
      const int c = ln % CPR;
      const int pages_i = i + 1 < nb && ((i + 1) & 31) == 0 ? pages_before : pages;  // block i + 1 may have moved on to its 32 page ids
#pragma unroll
      for (int j = 0; j < 32 * CPR / 64; ++j) {
        const int row = j * (64 / CPR) + ln / CPR;
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

// Share number wg of the batch's rows, by kWaves waves (further threads of the workgroup have ended).
template <int D, bool APPEND, bool MQ, int NT>
__device__ __forceinline__ void decode_share(const DecodeArgs &a, lds_char *smem, int lane, int w, int wg) {
  constexpr int RING = kWaves * 2 * 2 * 32 * D * 2;
  // Blocks of a sequence's row plus the row's fixed cost; 0 for a sequence that has no output row here.
  auto weight = [&](int L, int qn) __attribute__((always_inline)) {
    if (MQ && (qn <= 0 || (a.route_cap > 0 && qn > a.route_cap))) return 0;
    return ((max(L, 0) + 31) >> 5) + kRowCost;
  };
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
    const int end = total + wave_scan_incl(wt * a.n_hgroups);
    total = __builtin_amdgcn_readlane(end, 63);
    s_end[s] = end;
    s_len[s] = len;
  }
  wave_lds_fence();
  const int share = share_blocks(total, a.inv_wgs);
  const int lo = wg * share, hi = min(total, lo + share);
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
        const uint32_t pieces = whole ? 1 : (uint32_t)share_pieces(last, share, wg);
        *reinterpret_cast<u32x2 *>(a.row_tab + 2 * (long)row) = (u32x2){(uint32_t)(wg + row), pieces};
      }
      row_segment<D, APPEND, MQ, NT>(a, smem, lane, w, seq, hg, L, ctx, tok, p0, p1, load_pages(a, seq, p0, 0, w, lane), whole, wg + row);
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

// LDS of a workgroup: the waves' rings and the rows' ends.
template <int D, bool MQ>
constexpr int kDecodeShareSmem = kWaves * 2 * 2 * 32 * D * 2 + (MQ ? 4 : 2) * kMaxSeqs * 4;

}  // namespace sp
