// The prefill attention kernel for head_dim 64 on grids that fill the chip: workgroups of four waves and 128 query columns, three of
// them resident on a CU (attn_prefill.hip says what is computed; prefill_tile.h has the two-group kernel, the choice of work items
// and the reasons for the operand layouts).
//
// Why.  At head_dim 64 a score has half the MFMAs and as much softmax, so the VALU is the longer pipe: 32 MFMAs (1024 cycles)
// against 224 softmax instructions (1200) per SIMD, 64 keys and 256 columns; an issue probe of both takes 1497 cycles.  The
// two-group kernel takes 2075: one wave's softmax is a serial stream of 112 instructions at 7 to 8 cycles each next to the other
// wave's MFMAs, and at every change of phase both wait.  Here a wave interleaves its own multiplications and softmax (QK^T of one
// 32-key block and PV of another around the exponentials of a third), needs 166 registers, and so three waves share a SIMD; as they
// belong to different workgroups, one wave's barriers and dependent steps are covered by the others: 1880 cycles (counters, 2 x 9001..16384
// tokens: 1.30 M cycles that a CU is busy, 692 units of 64 keys and 256 columns).  Bound: instruction issue.  In 78 % of the busy cycles a
// SIMD issues a VALU or MFMA instruction (271 VALU per unit), the matrix pipe is busy in 54 %, the waves wait for memory or a barrier in
// 15 %; the launch takes 1.37 to 1.42 M cycles at 1.6 to 1.8 GHz.
// Measured (two-group kernel with 256 columns -> here): 2 sequences of 9001..16384 tokens at 16q/2kv 802 -> 758 us (972 TFLOP/s),
// 4 x 1500 29.4 -> 26.8, 2 x 2500 42.0 -> 37.5, 8 x 1200 41.6 -> 37.2, 4 x 3000 at 12q/3kv 75.0 -> 67.8, 40 chunks of 400 on up to 1300
// keys 65.1 -> 57.7; 6 x 600..900 24.7 (halves) -> 20.9.  Rows of few keys, which take the block by block part below, are the least:
// 17 chunks of 422 on up to 595 keys 31.9 -> 32.9, 24 x 320..527 at 12q/3kv 32.3 -> 33.0.  Smaller grids stay
// with 128 columns on two wave groups: one such workgroup alone on a CU takes half as long per tile as this one (1 x 2000 tokens 20.6 us, here 25.7).
// Tried on the way: the same loop with eight waves and 256 columns, two waves per SIMD and one barrier for all (2250
// cycles; 797 -> 834 us on 2 x 16k tokens), with 64-key blocks (1950 cycles, 773 us); at head_dim 128, where two such waves share a SIMD, 2250
// cycles instead of 2380, but twice the tile loads: 1677 -> 1849 us on 1 x 32768 tokens.
//
// LDS: K[3] and V[2] tile slots in the swizzled layout of SwzTile.  In the period of tile t the waves read K(t) and V(t-1), and
// the loads of K(t+2) and V(t) are issued into the slots last read in period t-1; they have landed when the period ends.  K is
// one tile ahead of its use, so that the first operands of period t+1 are read before the barrier that opens it.
#pragma once
#include "prefill_tile.h"

namespace sp {

constexpr int kSoloThreads = 256, kSoloCols = 128, kSoloKSlots = 3, kSoloVSlots = 2;
constexpr int kSoloLayers = 2;  // half as many columns as the two-group kernel: twice as many query tiles, for the same longest chunk
constexpr size_t kSoloSmem = (kSoloKSlots + kSoloVSlots) * (size_t)KVT * 64 * 2;

template <typename Args>
__global__ __launch_bounds__(kSoloThreads, 3) void solo_prefill_kernel(Args a) {
  constexpr int D = 64;
  using G = TileGeom<D>;
  using Z = SwzTile<D>;
  using std::integral_constant;
  constexpr bool FRESH = std::is_same<Args, FreshArgs>::value;
  constexpr int WAVES = kSoloThreads / 64;
  constexpr int ROWB = D * 2;                     // bytes of one K or V row
  constexpr int TBYTES = KVT * ROWB;              // one tile in LDS
  constexpr int VBASE = kSoloKSlots * TBYTES;     // V slots behind the K slots
  constexpr int NIW = TBYTES / 1024 / WAVES;      // 1 KiB load instructions per wave, matrix and tile
  static_assert(KVT == 4 * kPage, "each of the four waves brings in one page of a tile");
  extern __shared__ __align__(16) char smem_raw[];
  lds_char *smem = (lds_char *)smem_raw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int col = lane & 31, half = lane >> 5;
  WorkItem it;
  if (!take_item<0, true>(a, 7, lane, &it)) return;
  const int tpt = kSoloCols >> a.gshift, tok0 = it.tile * tpt, q0 = it.q0, q_len = it.q_len, ctx = it.ctx, hg = it.hg;
  if (tok0 >= q_len) return;
  const int kv_end = ctx + min(q_len, tok0 + tpt);
  const int kvh = (hg << a.gshift) / (a.Hq / a.Hkv);
  const int32_t *bt_row = a.block_table + (long)it.seq * a.max_pages;

  // ---- FRESH: a sequence with cached tokens after all (prefill_tile.h)
  if constexpr (FRESH) {
    if (__builtin_expect(ctx > 0, 0)) {
      append_to_pool_pages<D, kSoloThreads>(a, smem, bt_row, it, kvh);
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    }
  }

  // ---- this lane's column and the resident Q^T operands
  const int C = w * 32 + col, token = tok0 + (C >> a.gshift);
  const bool valid = token < q_len;
  const int lim = valid ? ctx + token + 1 : kv_end;  // a column without a query has scores of 0 and is not stored: any limit will do
  const int wlim_min = min(ctx + tok0 + ((w * 32) >> a.gshift) + 1, kv_end);  // keys that all of the wave's columns see
  const long out_off = ((long)(q0 + token) * a.Hq + ((hg << a.gshift) | (C & ((1 << a.gshift) - 1)))) * (D * 2);
  bf16x8 qreg[G::kDSteps];
#pragma unroll
  for (int s = 0; s < G::kDSteps; ++s) {
    if (valid) {
      qreg[s] = *reinterpret_cast<const bf16x8 *>(a.q + out_off + 32 * s + 16 * half);
    } else {
      u32x4 z = {0, 0, 0, 0};
      qreg[s] = *reinterpret_cast<bf16x8 *>(&z);
    }
  }
  f32x16 o[G::kDBlocks];
#pragma unroll
  for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_used = -INFINITY, l = 0.f, l2 = 0.f;  // running max; row sum in two chains
  const int T = (kv_end + KVT - 1) / KVT;       // key tiles

  // ---- tile loads (prefill_tile.h): wave w brings in page w of every tile
  const int last_kv = kv_end - 1, last_page = last_kv >> 4;
  int new_tile = 0x7fffffff;  // FRESH: tiles from here on are read from the new rows
  if (FRESH && first_new_tile(ctx) < T) new_tile = first_new_tile(ctx);
  constexpr int BIAS = (NIW - 1) * 1024;  // keeps the offsets of clamped rows from going below zero
  auto lane_off = [&](bool is_v, int j, int rip_lim, int row_stride) __attribute__((always_inline)) {  // instruction j of a page: this lane's source offset
    int ln = lane;
    if constexpr (FRESH) asm volatile("" : "+v"(ln));  // not kept in registers over the tile loop
    const PageChunk c = page_chunk<D>(is_v, j, ln);
    return (unsigned)((FRESH ? __mul24(min(c.row, rip_lim), row_stride) : min(c.row, rip_lim) * row_stride) + c.chunk * 16 - 1024 * j + BIAS);
  };
  const int new_stride = a.Hkv * ROWB, first_stride = FRESH && new_tile == 0 ? new_stride : ROWB, last_stride = FRESH && new_tile < T ? new_stride : ROWB;
  unsigned koff[NIW], voff[NIW];
#pragma unroll
  for (int j = 0; j < NIW; ++j) {
    koff[j] = lane_off(false, j, 15, first_stride);
    voff[j] = lane_off(true, j, 15, first_stride);
  }
  // This KV head's block of page 0; of new rows, the row that would be the first of page 0.
  const size_t block = (size_t)kvh * (kPage * ROWB);
  const long new_block = FRESH ? ((long)(q0 - ctx) * a.Hkv + kvh) * ROWB - BIAS : 0;
  const char *kpool = a.k_pages + block - BIAS, *vpool = a.v_pages + block - BIAS;
  if constexpr (FRESH) {
    if (new_tile == 0) {
      kpool = a.k_new + new_block;
      vpool = a.v_new + new_block;
    }
  }
  const bool my_last = (T - 1) * (KVT / kPage) + w >= last_page;  // the last tile's page of this wave holds the last key, or lies behind it
  auto clamp_v = [&](int t) __attribute__((always_inline)) {  // before the load of V of tile t
    if constexpr (FRESH) {
      if (__builtin_expect(t == new_tile, 0)) {
        vpool = a.v_new + new_block;
#pragma unroll
        for (int j = 0; j < NIW; ++j) voff[j] = lane_off(true, j, 15, new_stride);
      }
    }
    if (t < T - 1 || !my_last) return;
#pragma unroll
    for (int j = 0; j < NIW; ++j) voff[j] = lane_off(true, j, last_kv & 15, last_stride);
  };
  auto clamp_k = [&](int t) __attribute__((always_inline)) {  // new rows end where the caller's buffer may end
    if constexpr (FRESH) {
      if (__builtin_expect(t == new_tile, 0)) {
        kpool = a.k_new + new_block;
#pragma unroll
        for (int j = 0; j < NIW; ++j) koff[j] = lane_off(false, j, 15, new_stride);
      }
    }
    if (!FRESH || t < T - 1 || !my_last) return;
#pragma unroll
    for (int j = 0; j < NIW; ++j) koff[j] = lane_off(false, j, last_kv & 15, last_stride);
  };
  const unsigned page_bytes = (unsigned)a.Hkv * (kPage * ROWB);  // sixteen new rows are as far apart
  auto page_idx = [&](int t) __attribute__((always_inline)) { return min(min(t, T - 1) * (KVT / kPage) + w, last_page); };  // this wave's page of a tile
  auto page_of = [&](int t) __attribute__((always_inline)) {  // all lanes read the same entry
    if constexpr (FRESH) {
      if (min(t, T - 1) >= new_tile) return 0;
    }
    return bt_row[page_idx(t)];
  };
  auto page_pos = [&](int t, int pg) __attribute__((always_inline)) {  // where the page begins in the pool; no wild loads on bad metadata
    int n = 0;
    if (FRESH && min(t, T - 1) >= new_tile) n = page_idx(t);
    else n = min(max(__builtin_amdgcn_readfirstlane(pg), 0), a.num_pages - 1);
    return (size_t)(unsigned)n * page_bytes;
  };
  static_assert(NIW == 2, "two instructions per page");
  const unsigned wave_dst = (unsigned)(w * (NIW * 1024));
  // Every load of this wave has landed; then all waves'.  Not __syncthreads: that would also wait for the operands of the next
  // period that are on their way from LDS (their slot is not written before the period after).  The clobber keeps the
  // compiler from carrying LDS contents across.
  auto next_period = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory"); };

  // ---- LDS operand addresses of this lane in the slots that are being read
  const unsigned lds0 = (unsigned)(size_t)smem;
  unsigned kadr[G::kDSteps], vadr[G::kDBlocks];
#pragma unroll
  for (int s = 0; s < G::kDSteps; ++s) kadr[s] = lds0 + Z::template offset<false>(col, 2 * s + half);
  {
    const int n = lane & 15, dg = (lane >> 4) & 1;
#pragma unroll
    for (int db = 0; db < G::kDBlocks; ++db)
      vadr[db] = lds0 + VBASE + Z::template offset<true>(4 * half + (n >> 2), 4 * db + 2 * dg + ((n & 3) >> 1)) + 8 * (n & 1);
  }
  int kslot = 0, vslot = 0;
  auto k_next = [&]() __attribute__((always_inline)) {  // what the K addresses move by, to the next slot
    const int d = kslot == kSoloKSlots - 1 ? -(kSoloKSlots - 1) * TBYTES : TBYTES;
    kslot = kslot == kSoloKSlots - 1 ? 0 : kslot + 1;
    return (unsigned)d;
  };
  auto v_next = [&]() __attribute__((always_inline)) {
    const int d = vslot ? -TBYTES : TBYTES;
    vslot ^= 1;
    return (unsigned)d;
  };

  // Operands of a block: NK of K, each for one 16-channel step of QK^T, then NV of V^T (two transposing reads), each for one
  // 32-channel block and 16-key step of PV.
  constexpr int NK = G::kDSteps, NV = 2 * G::kDBlocks, NOP = NK + NV;
  constexpr int PFD = 4;   // operands read ahead
  auto k_op = [&](int b, int s) __attribute__((always_inline)) -> bf16x8 { return *(const lds_bf16x8 *)(size_t)(kadr[s] + (unsigned)(32 * b * ROWB)); };
  auto v_op = [&](int b, int i) __attribute__((always_inline)) -> bf16x8 {
    return lds_read_vt((const lds_char *)(size_t)(vadr[i % G::kDBlocks] + (unsigned)((32 * b + 16 * (i / G::kDBlocks)) * ROWB)), ROWB);
  };
  f32x16 sc[2];     // raw scores of the blocks being multiplied and exponentiated
  bf16x8 pw[2][2];  // their weights
  auto qk = [&](int s, bf16x8 x, f32x16 &dst) __attribute__((always_inline)) {
    if (s == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[r] = 0.f;
    }
    dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qreg[s], dst, 0, 0, 0);
  };
  auto pv = [&](int i, bf16x8 x, const bf16x8 (&p)[2]) __attribute__((always_inline)) {
    o[i % G::kDBlocks] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, p[i / G::kDBlocks], o[i % G::kDBlocks], 0, 0, 0);
  };
  auto mask = [&](int base, f32x16 &s) __attribute__((always_inline)) {  // keys base .. base + 31
    if (base + 32 <= wlim_min) return;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (base + 8 * (r >> 2) + 4 * half + (r & 3) >= lim) s[r] = -INFINITY;
  };
  // The general softmax of a block: its max, the lazy rescale of O and l, weights from the raw scores and their sums.  keep: they
  // stay in s.
  auto full = [&](f32x16 &s, bf16x8 (&p)[2], float (&ls)[2], bool keep) __attribute__((always_inline)) {
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(mx, other_half(mx));
    if (__builtin_amdgcn_ballot_w64(mx > m_used + a.tau) != 0) {  // wave-uniform
      const float m_new = fmaxf(m_used, mx);
      const float alpha = __builtin_amdgcn_exp2f((m_used - m_new) * a.sl2e);
      m_used = m_new;
      l *= alpha;
      l2 *= alpha;
#pragma unroll
      for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    }
    const float msc = m_used * a.sl2e;
    ls[0] = ls[1] = 0.f;
    f32x16 x;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      x[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], a.sl2e, -msc));
      ls[r & 1] += x[r];
    }
    p[0] = pack8(x, 0);
    p[1] = pack8(x, 8);
    if (keep) s = x;
  };

  // ---- the first tiles
  int pg = 0;        // page id of the next K load
  size_t pos_v = 0, pos_w = 0;  // where the pages of the next two V loads begin
  constexpr int kPreciseKeys = 256;
  const bool precise = ctx + (it.tile & ~1) * tpt < kPreciseKeys;  // some rows of this tile or its neighbour, as with 256 columns, have at most that many keys
  {
    int pg0 = 0, pg1 = 0;
    if (!FRESH || new_tile != 0) {
      pg0 = page_of(0);
      pg1 = page_of(1);
      pg = page_of(2);
    }
    clamp_k(0);
    clamp_v(0);
    const size_t pos0 = page_pos(0, pg0);
    pos_v = page_pos(1, pg1);
#pragma unroll
    for (int j = 0; j < NIW; ++j) page_load(kpool + pos0, wave_dst, koff[j], j);
    clamp_k(1);
#pragma unroll
    for (int j = 0; j < NIW; ++j) page_load(kpool + pos_v, TBYTES + wave_dst, koff[j], j);
#pragma unroll
    for (int j = 0; j < NIW; ++j) page_load(vpool + pos0, VBASE + wave_dst, voff[j], j);
    clamp_k(2);
    clamp_v(1);
    TileRows<D, kSoloThreads> rows;
    if constexpr (FRESH) rows.request(a, bt_row, it, kvh, tok0, tpt);
    next_period();
    if constexpr (FRESH) rows.store(a, it, kvh, tok0);
  }

  // Tile 0 sets the running max, both blocks of it: a weight of 1 is exact, and the more keys, the more rows have their
  // largest one there
#pragma unroll
  for (int s = 0; s < NK; ++s) qk(s, k_op(0, s), sc[0]);
#pragma unroll
  for (int s = 0; s < NK; ++s) qk(s, k_op(1, s), sc[1]);
  mask(0, sc[0]);
  mask(32, sc[1]);
#pragma unroll
  for (int r = 0; r < 16; ++r) m_used = fmaxf(m_used, fmaxf(sc[0][r], sc[1][r]));
  m_used = fmaxf(m_used, other_half(m_used));
  if (precise) {
    // Rows with at most kPreciseKeys keys take their weights as hi + lo: a second PV with what bf16 rounded away, so that the
    // rounding of the weights (which only averages out over many keys) stays out of the output tolerance there.  The
    // workgroups that hold such rows are at most eight tiles long and go through them block by block.
    for (int t = 0; t < T; ++t) {
      if (t + 1 < T) {  // K of tile 1 is there already
        if (t + 2 < T) {
          const size_t pos = page_pos(t + 2, pg);
          const int to = kslot == 0 ? 2 : kslot - 1;
#pragma unroll
          for (int j = 0; j < NIW; ++j) page_load(kpool + pos, (unsigned)(to * TBYTES) + wave_dst, koff[j], j);
          pos_w = pos;
        }
        const unsigned to = (unsigned)(VBASE + (1 - vslot) * TBYTES) + wave_dst;
#pragma unroll
        for (int j = 0; j < NIW; ++j) page_load(vpool + pos_v, to, voff[j], j);
        pos_v = pos_w;
        pg = page_of(t + 3);
        clamp_k(t + 3);
        clamp_v(t + 2);
      }
#pragma unroll 1
      for (int b = 0; b < 2; ++b) {
        const int base = t * KVT + 32 * b;
        const unsigned rows = (unsigned)(32 * b * ROWB);
#pragma unroll
        for (int s = 0; s < NK; ++s) {
          qk(s, *(const lds_bf16x8 *)(size_t)(kadr[s] + rows), sc[0]);
        }
        mask(base, sc[0]);
        float ls[2];
        full(sc[0], pw[0], ls, true);
        l += ls[0];
        l2 += ls[1];
        const bool lo = base < kPreciseKeys;
#pragma unroll 1
        for (int pass = 0; pass < (lo ? 2 : 1); ++pass) {
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            pv(i, lds_read_vt((const lds_char *)(size_t)(vadr[i % G::kDBlocks] + rows + (unsigned)(16 * (i / G::kDBlocks) * ROWB)), ROWB), pw[0]);
          }
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) pw[0][ks] = pack8_residual(sc[0], 8 * ks, pw[0][ks]);
        }
      }
      const unsigned dk = k_next(), dv = v_next();
#pragma unroll
      for (int s = 0; s < NK; ++s) kadr[s] += dk;
#pragma unroll
      for (int db = 0; db < G::kDBlocks; ++db) vadr[db] += dv;
      next_period();
    }
  } else {
    bf16x8 ops[PFD];  // the first operands of the next block
    // One 32-key block of the pipeline: QK^T of block B of the K slot into sc[B] and PV of block B of the V slot with pw[B],
    // while the scores in sc[1 - B] become weights in pw[1 - B].  QKV: 3 both, 2 PV only (the end).  AFTER: reads the first operands
    // of the block that follows.  emit: called behind every operand.
    auto block = [&](auto bc, auto whatc, int base, auto emit, auto first_of_next) __attribute__((always_inline)) {
      constexpr int B = decltype(bc)::value, I0 = decltype(whatc)::value == 3 ? 0 : NK, N = NOP - I0;
      constexpr int NS = 16, SPO = NS / N;        // scores of a lane, and behind each multiplication
      static_assert(NS % N == 0 && SPO % 2 == 0, "scores go in pairs");
      mask(base, sc[1 - B]);
      const float msc = m_used * a.sl2e;
      float ls[2] = {0.f, 0.f}, x[NS];
      union {
        bf16x2 h[4];
        bf16x8 v;
      } u[2];
      auto step = [&](int i) __attribute__((always_inline)) {  // each operation one step behind the one that feeds it
#pragma unroll
        for (int r = SPO * i; r < SPO * (i + 1) && r < NS; ++r) x[r] = __builtin_fmaf(sc[1 - B][r], a.sl2e, -msc);
#pragma unroll
        for (int e = 0; e < SPO; ++e) {
          const int r = SPO * (i - 1) + e;
          if (r >= 0 && r < NS) x[r] = __builtin_amdgcn_exp2f(x[r]);
        }
#pragma unroll
        for (int e = 0; e < SPO; e += 2) {
          const int r = SPO * (i - 2) + e;
          if (r < 0 || r >= NS) continue;
          ls[0] += x[r];
          ls[1] += x[r + 1];
          u[r / 8].h[r / 2 % 4] = __builtin_convertvector((f32x2){x[r], x[r + 1]}, bf16x2);
        }
      };
      auto op = [&](int i) __attribute__((always_inline)) -> bf16x8 { return i < NK ? k_op(B, i) : v_op(B, i - NK); };
      bf16x8 q[N];
#pragma unroll
      for (int i = 0; i < PFD; ++i) q[i] = I0 == 0 ? ops[i] : op(I0 + i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < N + 2; ++i) {
        if (i + PFD < N) q[i + PFD] = op(I0 + i + PFD);
        else if (i < N) first_of_next(i + PFD - N);
        if (i < N) {
          if (I0 + i < NK) qk(I0 + i, q[i], sc[B]);
          else pv(I0 + i - NK, q[i], pw[B]);
          emit(i);
        }
        step(i);
        __builtin_amdgcn_sched_barrier(0);
      }
      pw[1 - B][0] = u[0].v;
      pw[1 - B][1] = u[1].v;
      // some weight above 2^8, or NaN (a masked score against a running max that is still -inf): wave-uniform
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(ls[0] + ls[1] <= 256.0f)) != 0, 0)) full(sc[1 - B], pw[1 - B], ls, false);
      l += ls[0];
      l2 += ls[1];
    };
    using I0 = integral_constant<int, 0>;
    using I1 = integral_constant<int, 1>;
    using Both = integral_constant<int, 3>;
    using PvOnly = integral_constant<int, 2>;
    auto nothing = [](int) {};
    float ls[2];  // period 0
    full(sc[0], pw[0], ls, false);
    l += ls[0];
    l2 += ls[1];
    if (T > 1) {
      pos_w = page_pos(2, pg);
#pragma unroll
      for (int j = 0; j < NIW; ++j) page_load(kpool + pos_w, 2 * TBYTES + wave_dst, koff[j], j);
      pg = page_of(3);
      clamp_k(3);
      {
        const unsigned dk = k_next();
#pragma unroll
        for (int s = 0; s < NK; ++s) kadr[s] += dk;
      }
#pragma unroll
      for (int i = 0; i < PFD; ++i) ops[i] = k_op(0, i);
      next_period();
      for (int t = 1; t < T; ++t) {
        const size_t pos = page_pos(t + 2, pg);
        const char *kb = kpool + pos, *vb = vpool + pos_v;
        pos_v = pos_w;
        pos_w = pos;
        pg = page_of(t + 3);
        const unsigned kto = (unsigned)((kslot == 0 ? 2 : kslot - 1) * TBYTES) + wave_dst, vto = (unsigned)(VBASE + (1 - vslot) * TBYTES) + wave_dst;
        const int base = t * KVT;
        const unsigned dk = k_next(), dv = v_next();
        bf16x8 nx[PFD];
        block(I0{}, Both{}, base - 32, [&](int i) __attribute__((always_inline)) {
          if (i % 2 && i / 2 < NIW) page_load(kb, kto, koff[i / 2], i / 2);
        }, [&](int i) __attribute__((always_inline)) { nx[i] = k_op(1, i); });
#pragma unroll
        for (int i = 0; i < PFD; ++i) ops[i] = nx[i];
        block(I1{}, Both{}, base, [&](int i) __attribute__((always_inline)) {
          if (i % 2 && i / 2 < NIW) page_load(vb, vto, voff[i / 2], i / 2);
          if (i == NK - 1) {  // the last K operand of the tile has been read: on to the next slot
#pragma unroll
            for (int s = 0; s < NK; ++s) kadr[s] += dk;
          }
        }, [&](int i) __attribute__((always_inline)) { nx[i] = k_op(0, i); });
#pragma unroll
        for (int i = 0; i < PFD; ++i) ops[i] = nx[i];
#pragma unroll
        for (int db = 0; db < G::kDBlocks; ++db) vadr[db] += dv;
        clamp_k(t + 3);
        clamp_v(t + 1);
        next_period();
      }
    }
    block(I0{}, PvOnly{}, (T - 1) * KVT + 32, nothing, nothing);
#pragma unroll
    for (int i = 0; i < NV; ++i) pv(i, v_op(1, i), pw[1]);
  }

  // ---- normalise and store
  const float ln = l + l2, inv = 1.0f / (ln + other_half(ln));
  if (valid) {
    char *dst = a.out + out_off;
#pragma unroll
    for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        store4_bf16(dst + (32 * db + 8 * r4 + 4 * half) * 2, o[db][4 * r4] * inv, o[db][4 * r4 + 1] * inv, o[db][4 * r4 + 2] * inv,
                    o[db][4 * r4 + 3] * inv);
  }
}

}  // namespace sp
