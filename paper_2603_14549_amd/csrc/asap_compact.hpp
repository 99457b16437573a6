// Gather of the K/V rows of one block of rows, shared by the compaction kernels and by the merge, whose
// launch takes the compaction along when both run on one stream.
#pragma once
#include "asap_device.hpp"
#include "asap_launch.hpp"

namespace asap {

constexpr int KV_ROWS_PER_THREAD = 4;          // ... except where the launch says otherwise (launch_compact_kv)
constexpr int KV_ROWS_PER_THREAD_PAGED = 2;
constexpr int KV_THREADS = 256;
// rows one workgroup moves, `rows` of them per thread
inline int kv_rows_per_block(int row_bytes, int rows = KV_ROWS_PER_THREAD) { return KV_THREADS / (row_bytes / 16) * rows; }

// Where the source rows come from: the position list of asap_merge / asap_positions, or the kept list
// and text_len directly (the output order of Fig. 3 written out: prefix | kept | valid text).
// idx = pos_out [B,Nout] and len = new_len (BY_POS); idx = kept list [B,k] and len = text_len (FROM_KEPT,
// KEPT_ONLY); FIXED_ONLY reads no index list and takes len = text_len.
template <int MODE, int ROWS = KV_ROWS_PER_THREAD>
__device__ __forceinline__ void compact_block(const KvPointers& ptrs, const int32_t* __restrict__ idx,
                                              const int32_t* __restrict__ len, int Hkv, int N, int Nout,
                                              int row_bytes, int P, int V, int k, int bx, int bg, int bz) {
  // 16-byte pieces of a row, a power of two: 8, 16 or 32
  const int lpr_log2 = 31 - __clz(row_bytes >> 4), rpi = 256 >> lpr_log2;
  const int tid = threadIdx.x, piece = tid & ((1 << lpr_log2) - 1), r0 = tid >> lpr_log2;
  const int b = bg / Hkv;
  const int n_rows = MODE == KV_BY_POS      ? min(len[b], Nout)
                     : MODE == KV_KEPT_ONLY ? k
                     : MODE == KV_FIXED_ONLY ? P + min(max(len[b], 0), Nout - P - k)
                                             : P + k + min(len[b], Nout - P - k);
  const char* src = ptrs.src[bz] + (int64_t)bg * N * row_bytes + piece * 16;
  char* dst = ptrs.dst[bz] + (int64_t)bg * Nout * row_bytes + piece * 16;
  const int32_t* ix = idx + (int64_t)b * (MODE == KV_BY_POS ? Nout : k);
  const int base = bx * rpi * ROWS + r0;
  uint4 v[ROWS];
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int r = base + i * rpi;
    if (r < n_rows) {
      const int srow = MODE == KV_BY_POS       ? ix[r]
                       : MODE == KV_KEPT_ONLY  ? P + ix[r]
                       : MODE == KV_FIXED_ONLY ? (r < P ? r : r + V)
                       : r < P                 ? r
                       : r < P + k             ? P + ix[r - P]
                                               : r - k + V;
      v[i] = ldg16_stream(src + (int64_t)srow * row_bytes);
    }
  }
#pragma unroll
  for (int i = 0; i < ROWS; ++i) {
    const int r = base + i * rpi;
    // kept slot r is output row P + r; the r-th row that no selection changes is output row r (prefix) or
    // r + k (text)
    const int drow = MODE == KV_KEPT_ONLY ? P + r : MODE == KV_FIXED_ONLY ? (r < P ? r : r + k) : r;
    if (r < n_rows) stg16_stream(dst + (int64_t)drow * row_bytes, v[i]);
  }
}

}  // namespace asap
