// How the equal-share decode (decode_stream.h) deals a batch's rows to its workgroups.  Plain integer code that compiles
// for the host as well: the CPU tests run it.
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

}  // namespace sp
