// asap_compact_kv: gathers the K/V rows of the surviving positions of every cached layer
// (KV-cache compatibility of the pruning stage).  Pure data movement, bit-exact.
//
// k_positions: grid (ceil(Nout / 256), B): the positions the compaction gathers, from the kept set alone.
// k_compact<MODE, ROWS>: grid (ceil(rows / kv_rows_per_block), B * Hkv, 2 * layers_in_launch), 256 threads, rows = Nout
// or, for the kept tokens' rows alone, k; the source rows come from the position list or straight from the
// kept list (then nothing of asap_merge is needed).
// k_compact_paged: the same grid for caches kept as pools of pages with one block table per sequence.
// A row is d elements = LPR 16-byte pieces; LPR consecutive lanes move one row.
#include "asap_compact.hpp"
#include "asap_device.hpp"
#include "asap_launch.hpp"

namespace asap {

void fill_kv_pointers(KvPointers* ptrs, int n_layers, const void* const* k_src, const void* const* v_src,
                      void* const* k_dst, void* const* v_dst) {
  for (int l = 0; l < n_layers; ++l) {
    ptrs->src[2 * l] = static_cast<const char*>(k_src[l]);
    ptrs->src[2 * l + 1] = static_cast<const char*>(v_src[l]);
    ptrs->dst[2 * l] = static_cast<char*>(k_dst[l]);
    ptrs->dst[2 * l + 1] = static_cast<char*>(v_dst[l]);
  }
  for (int l = 2 * n_layers; l < 2 * KV_LAYERS_PER_LAUNCH; ++l) { ptrs->src[l] = nullptr; ptrs->dst[l] = nullptr; }
}

template <int MODE, int ROWS>
__global__ __launch_bounds__(256) void k_compact(KvPointers ptrs, const int32_t* __restrict__ idx,
                                                  const int32_t* __restrict__ len, int Hkv, int N, int Nout,
                                                  int row_bytes, int P, int V, int k) {
  compact_block<MODE, ROWS>(ptrs, idx, len, Hkv, N, Nout, row_bytes, P, V, k, blockIdx.x, blockIdx.y, blockIdx.z);
}

// The rows that no selection changes, for the launch that runs beside the score kernels: a grid of
// at most two workgroups per compute unit walks the (gx, gy, gz) blocks of k_compact, so that the
// kernels of the other stream still find room on every compute unit.
__global__ __launch_bounds__(256) void k_compact_fixed(KvPointers ptrs, const int32_t* __restrict__ len, int Hkv,
                                                        int N, int Nout, int row_bytes, int P, int V, int k, int gx,
                                                        int gy, int gz) {
  const int total = gx * gy * gz;
  for (int id = blockIdx.x; id < total; id += gridDim.x) {
    const int bx = id % gx, bg = (id / gx) % gy, bz = id / (gx * gy);
    compact_block<KV_FIXED_ONLY>(ptrs, len, len, Hkv, N, Nout, row_bytes, P, V, k, bx, bg, bz);
  }
}

// Pools are [n_pages, Hkv, page_size, d]; token n of sequence b is in page table[b, n / page_size],
// slot n % page_size.
// Two rows per thread: a row is found through three loads in a row, of which one row per thread keeps too few in flight
// where the copy is all there is to do, and four crowd the search that runs beside it (us per call of the stage, four / two /
// one: 16 x 2304 tokens on 500, 28 heads on 4, 16 layers 436 / 396 / 396; 4 x 1024 on 200, 4 layers 125.7 / 122.7 / 121.8; 8 x 576 on 160,
// 40 heads, 16 layers 366 / 367 / 383).  Pages of a power of two, which is what serving engines use, are found by a
// shift (the latter in four rows: 365, now 360).
__global__ __launch_bounds__(256) void k_compact_paged(KvPointers ptrs, const int32_t* __restrict__ pos_out,
                                                        const int32_t* __restrict__ new_len,
                                                        const int32_t* __restrict__ src_table, int src_stride,
                                                        const int32_t* __restrict__ dst_table, int dst_stride,
                                                        int page_size, int page_log2, int Hkv, int Nout, int row_bytes) {
  const int lpr_log2 = 31 - __clz(row_bytes >> 4), rpi = 256 >> lpr_log2;
  const int tid = threadIdx.x, piece = tid & ((1 << lpr_log2) - 1), r0 = tid >> lpr_log2;
  const int bg = blockIdx.y, b = bg / Hkv, g = bg - b * Hkv;
  // row of token n of a sequence in its pool
  auto pool_row = [&](const int32_t* tab, int n) {
    const int page = page_log2 >= 0 ? n >> page_log2 : n / page_size;
    return ((int64_t)tab[page] * Hkv + g) * page_size + (n - page * page_size);
  };
  const int nl = new_len[b];
  const char* src = ptrs.src[blockIdx.z] + piece * 16;
  char* dst = ptrs.dst[blockIdx.z] + piece * 16;
  const int32_t* pos = pos_out + (int64_t)b * Nout;
  const int32_t* stab = src_table + (int64_t)b * src_stride;
  const int32_t* dtab = dst_table + (int64_t)b * dst_stride;
  const int base = blockIdx.x * rpi * KV_ROWS_PER_THREAD_PAGED + r0;
  uint4 v[KV_ROWS_PER_THREAD_PAGED];
#pragma unroll
  for (int i = 0; i < KV_ROWS_PER_THREAD_PAGED; ++i) {
    const int nrow = base + i * rpi;
    if (nrow < nl) v[i] = ldg16_stream(src + pool_row(stab, pos[nrow]) * row_bytes);
  }
#pragma unroll
  for (int i = 0; i < KV_ROWS_PER_THREAD_PAGED; ++i) {
    const int nrow = base + i * rpi;
    if (nrow < nl) stg16_stream(dst + pool_row(dtab, nrow) * row_bytes, v[i]);
  }
}

// Output order of the stage (Fig. 3, Sec. 4.2): prefix | kept tokens in original order | valid text.
__global__ __launch_bounds__(256) void k_positions(const int32_t* __restrict__ kept, const int32_t* __restrict__ text_len,
                                                    int P, int V, int k, int Nout, int32_t* __restrict__ pos_out,
                                                    int32_t* __restrict__ new_len) {
  const int b = blockIdx.y, n = blockIdx.x * 256 + threadIdx.x;
  const int len = text_len[b];
  if (n == 0) new_len[b] = P + k + len;
  if (n >= Nout) return;
  int pos;
  if (n < P) pos = n;
  else if (n < P + k) pos = P + kept[(int64_t)b * k + (n - P)];
  else pos = (n - P - k < len) ? P + V + (n - P - k) : -1;
  pos_out[(int64_t)b * Nout + n] = pos;
}

hipError_t launch_positions(const asap_params& p, const int32_t* kept, const int32_t* text_len, int32_t* pos_out,
                            int32_t* new_len, hipStream_t st, Timer* tm) {
  const int Nout = p.P + p.k + p.Tmax;
  ASAP_LAUNCH(tm, "k_positions", k_positions, dim3((Nout + 255) / 256, p.B), dim3(256), 0, st, kept, text_len, p.P,
              p.V, p.k, Nout, pos_out, new_len);
  return hipGetLastError();
}

// mode: KV_BY_POS (idx = pos_out, len = new_len) or KV_FROM_KEPT (idx = kept list, len = text_len)
// What bounds it: HBM.  With one row per thread in as many workgroups as that takes, which all ask at once, the copy runs at 6.2
// TB/s (5.6 with four rows; a plain copy 6.5 and 6.0): 16 x 2304 tokens, 440 MB on a stream of its own 78 -> 71 us; us per
// stage on one stream, 8 x 576 on 160, 16 layers 323 -> 290, 12 x 448 on 72, 16 layers 205 -> 187.  Four rows stay where
// few workgroups have to keep enough in flight: beside the search with two of them per compute unit (lds) or of f32 states, which
// outlasts the copy (3 x 2304 tokens of 40 heads on 500, 2 layers: 345 with one, 341 with four), and in k_compact_fixed's walk (8
// x 576, 16 layers, two streams: 282 with one row in that walk, 266 with four).
hipError_t launch_compact_kv(const asap_params& p, int mode, int n_layers, const void* const* k_src,
                             const void* const* v_src, void* const* k_dst, void* const* v_dst,
                             const int32_t* idx, const int32_t* len, hipStream_t st, Timer* tm, bool beside_search, size_t lds) {
  const int row_bytes = p.d * (p.kv_dtype == ASAP_BF16 ? 2 : 4);
  const int N = p.P + p.V + p.Tmax, Nout = p.P + p.k + p.Tmax;
  const bool few = lds != 0 || (beside_search && p.h_dtype == ASAP_F32);
  const int per_thread = mode == KV_FIXED_ONLY || few ? KV_ROWS_PER_THREAD : 1;
  const int rows_per_block = kv_rows_per_block(row_bytes, per_thread);
  const int rows = mode == KV_KEPT_ONLY ? p.k : mode == KV_FIXED_ONLY ? p.P + p.Tmax : Nout;
  for (int l0 = 0; l0 < n_layers; l0 += KV_LAYERS_PER_LAUNCH) {
    const int nl = n_layers - l0 < KV_LAYERS_PER_LAUNCH ? n_layers - l0 : KV_LAYERS_PER_LAUNCH;
    KvPointers ptrs;
    fill_kv_pointers(&ptrs, nl, k_src + l0, v_src + l0, k_dst + l0, v_dst + l0);
    dim3 grid((rows + rows_per_block - 1) / rows_per_block, p.B * p.Hkv, 2 * nl);
#define ASAP_COMPACT(MODE, ROWS)                                                                                  \
  ASAP_LAUNCH(tm, "k_compact", (k_compact<MODE, ROWS>), grid, dim3(256), lds, st, ptrs, idx, len, p.Hkv, N, Nout, \
              row_bytes, p.P, p.V, p.k)
    if (mode == KV_FIXED_ONLY) {
      const long total = (long)grid.x * grid.y * grid.z;
      ASAP_LAUNCH(tm, "k_compact_fixed", k_compact_fixed, dim3((unsigned)(total < 512 ? total : 512)), dim3(256), lds, st,
                  ptrs, len, p.Hkv, N, Nout, row_bytes, p.P, p.V, p.k, (int)grid.x, (int)grid.y, (int)grid.z);
    } else if (mode == KV_BY_POS) {
      ASAP_COMPACT(KV_BY_POS, 1);
    } else if (mode == KV_FROM_KEPT) {
      if (few) ASAP_COMPACT(KV_FROM_KEPT, KV_ROWS_PER_THREAD);
      else ASAP_COMPACT(KV_FROM_KEPT, 1);
    } else {
      if (few) ASAP_COMPACT(KV_KEPT_ONLY, KV_ROWS_PER_THREAD);
      else ASAP_COMPACT(KV_KEPT_ONLY, 1);
    }
#undef ASAP_COMPACT
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_compact_kv_paged(const asap_params& p, int n_layers, const void* const* k_src,
                                   const void* const* v_src, void* const* k_dst, void* const* v_dst, int page_size,
                                   const int32_t* src_table, int src_stride, const int32_t* dst_table,
                                   int dst_stride, const int32_t* pos_out, const int32_t* new_len, hipStream_t st,
                                   Timer* tm) {
  const int row_bytes = p.d * (p.kv_dtype == ASAP_BF16 ? 2 : 4);
  const int Nout = p.P + p.k + p.Tmax;
  const int rows_per_block = kv_rows_per_block(row_bytes, KV_ROWS_PER_THREAD_PAGED);
  const int page_log2 = (page_size & (page_size - 1)) == 0 ? __builtin_ctz(page_size) : -1;
  for (int l0 = 0; l0 < n_layers; l0 += KV_LAYERS_PER_LAUNCH) {
    const int nl = n_layers - l0 < KV_LAYERS_PER_LAUNCH ? n_layers - l0 : KV_LAYERS_PER_LAUNCH;
    KvPointers ptrs;
    fill_kv_pointers(&ptrs, nl, k_src + l0, v_src + l0, k_dst + l0, v_dst + l0);
    dim3 grid((Nout + rows_per_block - 1) / rows_per_block, p.B * p.Hkv, 2 * nl);
    ASAP_LAUNCH(tm, "k_compact_paged", k_compact_paged, grid, dim3(256), 0, st, ptrs, pos_out, new_len, src_table,
                src_stride, dst_table, dst_stride, page_size, page_log2, p.Hkv, Nout, row_bytes);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace asap
