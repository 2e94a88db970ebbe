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
// 8q/1kv, d 128: 37.5 -> 31.5 us (157 MB; a batch of 138 MB, all read once: kernel 25.6 us, 5.4 TB/s with the ramp to the first
// block and the tail, merge 4.2); 128 sequences of 1024..16384 keys, 32q/8kv (4.9 GB): 808 -> 734 us (6.7 TB/s);
// 64 x 4 query tokens: 35.5 -> 31.1 us; one sequence of 32900 keys: 12.5 -> 11.6-12.1 us; one of 137 keys: 10 -> 7.3 us.
#include "decode_stream.h"

namespace sp {

template <int D, bool APPEND, bool MQ, int NT>
__global__ __launch_bounds__(64 * kWaves, NT > 1 ? 1 : 2) void decode_stream_kernel(DecodeArgs a) {
  extern __shared__ __align__(16) char smem_raw[];
  lds_char *smem = (lds_char *)smem_raw;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
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
      if (qn <= 0 || (a.route_cap > 0 && qn > a.route_cap)) return;
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
  decode_share<D, APPEND, MQ, NT>(a, smem, lane, w, blockIdx.x);
}

// Merge of the partials of the rows that were cut: one workgroup per (row, column), one wave per 32-channel
// slice; eight lanes x 16 bytes cover the slice of one partial, so a load instruction covers eight
// partials and NB of them are in flight together.  Lane group g adds the partials g, g + 8, ... in order,
// the eight groups are added in a fixed butterfly.
//
// PG > 1 (rows in many pieces): a workgroup per slice too, of PG waves that merge a contiguous run of the row's
// partials each; the PG results meet in LDS.  All slices of a row in one workgroup of 1024 threads send its 66 KB (129 pieces)
// through one CU's address unit, a chain that four CUs share here: one sequence of 33000 keys at 8q/1kv, decode and merge
// 11.2 -> 9.8 us, and 9.6 with six load instructions a wave instead of eight where they cover the row (half of those eight asked for the last
// partial again).  Eight waves of four instructions: 10.0.  Rows of up to 64 pieces gain nothing by the same (8.6 us either way).
template <int D, int NB, int PG, bool MQ>
__global__ __launch_bounds__(PG > 1 ? 64 * PG : 2 * D) void combine_rows_kernel(DecodeArgs a) {
  const int tc = blockIdx.x, row = blockIdx.y;
  const int pg = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 3;  // pg: PG > 1
  const int ch = (PG > 1 ? (int)blockIdx.z : (int)(threadIdx.x >> 6)) * 32 + (lane & 7) * 4;
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
    __shared__ f32x4 x_acc[PG][8];
    __shared__ f32x2 x_ml[PG];
    if (g == 0) x_acc[pg][lane] = acc;
    if (lane == 0) x_ml[pg] = (f32x2){M, den};
    __syncthreads();
    if (threadIdx.x >= 8) return;
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
  const float inv = M == -INFINITY ? 0.f : 1.0f / den;  // no keys at all: zeros
  *reinterpret_cast<bf16x4 *>(a.out + (orow * D + ch) * 2) = __builtin_convertvector(acc * inv, bf16x4);
}

template <int D, bool MQ>
static void launch_rows_combine(const DecodeArgs &a, int max_pieces, hipStream_t stream) {
  const dim3 grid((unsigned)a.cols, (unsigned)(a.batch * a.n_hgroups)), block(2 * D);
  if (max_pieces <= 16) hipLaunchKernelGGL((combine_rows_kernel<D, 2, 1, MQ>), grid, block, 0, stream, a);
  else if (max_pieces <= 64) hipLaunchKernelGGL((combine_rows_kernel<D, 8, 1, MQ>), grid, block, 0, stream, a);
  else {
    // 192 pieces: six instructions of eight pieces in each of four waves; beyond, eight have fewer rows in a second batch (one sequence
    // of 60000 keys, 235 pieces, 10.3 us, with six 10.8).
    const dim3 slices(grid.x, grid.y, D / 32);
    if (max_pieces <= 192) hipLaunchKernelGGL((combine_rows_kernel<D, 6, 4, MQ>), slices, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((combine_rows_kernel<D, 8, 4, MQ>), slices, dim3(256), 0, stream, a);
  }
}

void launch_decode_combine(const DecodeArgs &a, int max_pieces, int head_dim, hipStream_t stream) {
  if (head_dim == 128) launch_rows_combine<128, true>(a, max_pieces, stream);
  else launch_rows_combine<64, true>(a, max_pieces, stream);
}

template <int D, bool APPEND, bool MQ, int NT>
static int launch_stream(const DecodeArgs &a, dim3 wgs, int max_pieces, hipStream_t stream) {
  static bool attr_set = false;  // benign if two threads race
  constexpr int smem = kDecodeShareSmem<D, MQ>;
  auto fn = decode_stream_kernel<D, APPEND, MQ, NT>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return fail(SP_ERR_HIP, "decode smem attribute: %s", hipGetErrorString(e));
    attr_set = true;
  }
  hipLaunchKernelGGL(fn, wgs, dim3(64 * kWaves), smem, stream, a);
  if (a.row_splits != 1) launch_rows_combine<D, MQ>(a, max_pieces, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SP_ERR_HIP, "decode launch: %s", hipGetErrorString(e));
  return SP_OK;
}

int plan_decode_stream(DecodeArgs &a, int batch, int max_q, int tiles, int max_len, int head_dim, void *workspace,
                       size_t workspace_bytes, int form, bool alone, dim3 *grid, int *pieces) {
  const long rows = (long)batch * a.n_hgroups;
  const bool mq = a.cu_q != nullptr;
  if (rows > 65535) return 1;
  a.batch = batch;
  a.hg_per_kv = a.group / a.geff;
  a.q_max = max_q;
  a.cols = max_q * a.geff;
  // Workgroups that are resident at once: one per CU at head_dim 128 and two at 64 (LDS; one with two
  // column tiles, or next to prefill workgroups: registers).
  const long resident = head_dim == 128 || tiles == 2 || !alone ? 256 : 512;
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
  if (form == 0 && !mq && one_wave_pays(rows, a.geff, max_len, head_dim, splits, resident)) return 1;
  // Equal shares: a partial slot per (workgroup, row) pair along the concatenated rows, and the table of rows.
  const size_t tab = (size_t)(rows * 8 + 15) / 16 * 16;
  const long least = kMinShare + kRowCost;
  const long useful = (rows * ((max_len + 31) / 32 + kRowCost) + least - 1) / least;
  long want = resident < useful ? resident : useful;
  // Where the room is short, up to a quarter of the workgroups less: what sp_attn_decode_workspace_size returns follows the
  // one-wave splits and is a few slots short of the full number at 16 heads per KV head of 64 (29 sequences of up to 18214
  // keys at 16q/1kv: 492 of 512 fit).
  const long fit = ws < tab ? 0 : (long)((ws - tab) / slot_bytes) - rows;
  if (fit < want && 4 * fit >= 3 * want) want = fit;
  if (splits == 0 && (batch > kMaxSeqs || fit < want)) {
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
    a.inv_wgs = share_inverse(want);
    a.row_tab = (int32_t *)workspace;
    a.part_o = (float *)((char *)workspace + tab);
    a.part_ml = a.part_o + (size_t)(rows + want) * a.cols * head_dim;
  }
  *grid = wgs;
  *pieces = max_pieces;
  return 0;
}

int launch_decode_stream(DecodeArgs &a, int batch, int max_q, int tiles, int max_len, int head_dim, void *workspace,
                         size_t workspace_bytes, int form, hipStream_t stream) {
  const bool mq = a.cu_q != nullptr;
  dim3 wgs;
  int max_pieces;
  if (int rc = plan_decode_stream(a, batch, max_q, tiles, max_len, head_dim, workspace, workspace_bytes, form, true, &wgs, &max_pieces)) return rc;
#define SP_STREAM(D_)                                                                                                    \
  (!mq ? (a.k_new ? launch_stream<D_, true, false, 1>(a, wgs, max_pieces, stream) : launch_stream<D_, false, false, 1>(a, wgs, max_pieces, stream)) \
   : tiles == 1                                                                                                          \
       ? (a.k_new ? launch_stream<D_, true, true, 1>(a, wgs, max_pieces, stream) : launch_stream<D_, false, true, 1>(a, wgs, max_pieces, stream))   \
       : (a.k_new ? launch_stream<D_, true, true, 2>(a, wgs, max_pieces, stream) : launch_stream<D_, false, true, 2>(a, wgs, max_pieces, stream)))
  return head_dim == 128 ? SP_STREAM(128) : SP_STREAM(64);
#undef SP_STREAM
}

}  // namespace sp
