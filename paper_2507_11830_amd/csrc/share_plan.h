// How the equal-share decode (decode_stream.h) deals a batch's rows to its workgroups, and which batches are left to
// one-wave splits.  Plain code that compiles for the host as well: the CPU tests run it.
#pragma once
#include <stdint.h>

#ifdef __HIP__
#define SP_HD __host__ __device__ __forceinline__
#else
#define SP_HD inline
#endif

namespace sp {

constexpr int kWaves = 4;          // waves per workgroup
constexpr int kRowCost = 8;        // blocks that a segment's fixed cost amounts to (64-sequence batch: 4 blocks 34.5 us, 8 and 12 33.5)
constexpr int kMinShare = 12;      // blocks per workgroup below which a further cut costs more than it gives

// 2^32 / workgroups, rounded up and, for a single one, down to what 32 bits hold.
inline unsigned share_inverse(long wgs) {
  const unsigned long long inv = (0x100000000ull + (unsigned long long)wgs - 1) / (unsigned long long)wgs;
  return inv > 0xffffffffull ? 0xffffffffu : (unsigned)inv;
}

// Blocks per workgroup of rows that weigh `total` blocks together.  share * workgroups >= total for every inverse, that
// of one workgroup too (total - 1 + 1): whatever lengths the device finds, the last share reaches the last row's end, and no
// row is recorded with partials of workgroups that there are not.
SP_HD int share_blocks(int total, unsigned inverse) {
  const int share = (int)(((unsigned long long)(unsigned)total * inverse) >> 32) + 1;
  return ((share > kMinShare + kRowCost ? share : kMinShare + kRowCost) + kWaves - 1) & -kWaves;
}

// Partials of a row that ends at `last` and whose first key block lies in workgroup wg's share.
SP_HD int share_pieces(int last, int share, int wg) { return (last - 1) / share - wg + 1; }

// Single tokens that one-wave splits (attn_decode.hip) serve faster: a wave writes its partial without the merge's barriers and
// four of them share a CU (ten at head_dim 64), where a workgroup of decode_stream.h has it alone (two at 64).  splits: that
// kernel's per row, 0: equal shares.
inline bool one_wave_pays(long rows, int geff, int max_len, int head_dim, long splits, long resident) {
  if (max_len <= 512) {
    // One workgroup per row: every round of resident ones costs 4 us however short the rows are, while a wave reads up to
    // 128 keys in one split (1024 rows 14 us against 20, 3752 of up to 121 keys at 8q/8kv 36 and 61; head_dim 64, 2676 of up to
    // 95: 16 and 20; 704 rows of up to 109: 12.8 each).  With one or two heads per KV head the partials of a few splits
    // are small too (1024 rows of up to 300 keys: 21.3 and 24.5; of up to 512 keys 33.7 and 30.8; four heads 33 and 31).
    return (max_len <= 128 && rows > (head_dim == 128 ? 3 : 4) * resident) ||
           (geff <= 2 && max_len <= 320 && rows > (head_dim == 128 ? 2 : 6) * resident);
  }
  // Little data (keys x channels of the batch, all sequences taken as long as the longest): up to 16 M in every form (16 sequences of
  // 512..8192 keys at 8q/1kv: 13.0 us against 13.8; from 32 such sequences on, 20.8 against 19.4), up to 32 M where equal
  // shares or an unfilled round of splits compete (300 rows of up to 600 keys 16.2 and 20; 200 of up to 1500 at
  // head_dim 64 10.5 and 13; 256 of up to 900 keys, one round: 28 % slower), twice that with one or two heads (384 rows of up to
  // 900 keys 21.0 and 22.7; 512 of 900..2000 at head_dim 64 31.9 and 33.6).
  const double data = (double)rows * max_len * head_dim;
  if (max_len > 8192) return false;
  if (data <= 8192.0 * 16 * 128) return true;
  return data <= (geff <= 2 ? 64e6 : 32e6) && (splits == 0 || (splits >= 2 && 20 * rows * splits <= 19 * resident));
}

}  // namespace sp
