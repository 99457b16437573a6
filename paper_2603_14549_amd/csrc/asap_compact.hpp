// Gather of the K/V rows of one block of rows, shared by the compaction kernels and by the merge, whose
// launch takes the compaction along when both run on one stream.
#pragma once
#include "asap_device.hpp"
#include "asap_launch.hpp"

namespace asap {

constexpr int KV_ROWS_PER_THREAD = 4;
constexpr int KV_THREADS = 256;
// rows one workgroup moves
inline int kv_rows_per_block(int row_bytes) { return KV_THREADS / (row_bytes / 16) * KV_ROWS_PER_THREAD; }

// Where the source rows come from: the position list of asap_merge / asap_positions, or the kept list
// and text_len directly (the output order of Fig. 3 written out: prefix | kept | valid text).
// idx = pos_out [B,Nout] and len = new_len (BY_POS); idx = kept list [B,k] and len = text_len (FROM_KEPT,
// KEPT_ONLY); FIXED_ONLY reads no index list and takes len = text_len.
template <int MODE>
__device__ __forceinline__ void compact_block(const KvPointers& ptrs, const int32_t* __restrict__ idx,
                                              const int32_t* __restrict__ len, int Hkv, int N, int Nout,
                                              int row_bytes, int P, int V, int k, int bx, int bg, int bz) {
  const int lpr = row_bytes >> 4, rpi = 256 / lpr;
  const int tid = threadIdx.x, piece = tid % lpr, r0 = tid / lpr;
  const int b = bg / Hkv;
  const int n_rows = MODE == KV_BY_POS      ? min(len[b], Nout)
                     : MODE == KV_KEPT_ONLY ? k
                     : MODE == KV_FIXED_ONLY ? P + min(max(len[b], 0), Nout - P - k)
                                             : P + k + min(len[b], Nout - P - k);
  const char* src = ptrs.src[bz] + (int64_t)bg * N * row_bytes + piece * 16;
  char* dst = ptrs.dst[bz] + (int64_t)bg * Nout * row_bytes + piece * 16;
  const int32_t* ix = idx + (int64_t)b * (MODE == KV_BY_POS ? Nout : k);
  const int base = bx * rpi * KV_ROWS_PER_THREAD + r0;
  uint4 v[KV_ROWS_PER_THREAD];
#pragma unroll
  for (int i = 0; i < KV_ROWS_PER_THREAD; ++i) {
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
  for (int i = 0; i < KV_ROWS_PER_THREAD; ++i) {
    const int r = base + i * rpi;
    // kept slot r is output row P + r; the r-th row that no selection changes is output row r (prefix) or
    // r + k (text)
    const int drow = MODE == KV_KEPT_ONLY ? P + r : MODE == KV_FIXED_ONLY ? (r < P ? r : r + k) : r;
    if (r < n_rows) stg16_stream(dst + (int64_t)drow * row_bytes, v[i]);
  }
}

}  // namespace asap
