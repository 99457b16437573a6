// asap_merge: the salience-weighted convex merge of Eq. 6 and the output sequence
// [prefix | merged kept | text], after the cosine routing of asap_sim.hip (and, for the paper's
// routing inside the kept set, the plan of asap_paper.hip).
//
//   k_merge<T>    one workgroup per output row: copies prefix / text rows, and for a final
//                 slot gathers its sources in ascending order and applies Eq. 6.  The sources are
//                 M candidate tokens with assign[] = the slot that absorbs each (or -1): the
//                 pruned tokens with ABSORB routing, the kept tokens with the paper's.
#include "asap_compact.hpp"
#include "asap_device.hpp"
#include "asap_launch.hpp"

namespace asap {

// ------------------------------------------------------------------------------------------
// k_merge: grid (B (P + k + Tmax) parts + KV blocks), 256 threads.  The first B (P + k + Tmax) parts workgroups
// take one output row each, or one of its `parts` pieces of 4 KB; the others, if the launch carries the K/V compaction along, one block of cache rows
// each (asap_compact.hpp): it needs the same list of survivors and nothing of the merge, the copies run
// under the latency of the gathers, and a launch is saved (8 us of a single image's stage).
//   What bounds it: HBM where the batch is large (every visual row of the hidden states once); a chain of
//   dependent loads -- lists, weights, rows -- where it is not.  So the lists are read with whole
//   coalesced loads before anything is known about them, and AHEAD source rows are in flight at a time: a slot's sources (V / k - 1 on
//   average, 30 to 70 for the most similar) mostly come in one turn.
// ------------------------------------------------------------------------------------------
constexpr int MERGE_SEG = 2048;   // entries of assign[] scanned per round
constexpr long MERGE_SPLIT_ROWS = 1024;

template <typename T, int CPT, int AHEAD>    // CPT = 16-byte chunks of a row (or of a part) per thread
__global__ __launch_bounds__(256) void k_merge(const T* __restrict__ hidden, int64_t sb, int64_t sr, int D,
                                                int P, int V, int k, int M, int Tmax, float mu,
                                                const float* __restrict__ s_hat, const int32_t* __restrict__ text_len,
                                                const int32_t* kept /* may be final_idx */,
                                                const int32_t* __restrict__ pruned,
                                                const int32_t* __restrict__ assign, T* __restrict__ out,
                                                int32_t* __restrict__ pos_out, int32_t* __restrict__ new_len,
                                                float* __restrict__ wsum, int32_t* final_idx, int B, int parts, MergeKv kv) {
  constexpr int E = elem<T>::per16;
  __shared__ int list[MERGE_SEG];
  // Weights of the sources: whole rows ask for them with the row, one scalar load each, which takes a load out of the chain in
  // front of the first row (k_merge of 16 x 2304 tokens 69.8 -> 66.0 us, 5 x 2083 23.5 -> 22.1); pieces, whose threads
  // have 16 rows in flight, find them in LDS (2 x 904 with the scalar loads 9.4 -> 9.9).
  constexpr bool LATE = CPT > 1;
  __shared__ float weight[LATE ? 1 : MERGE_SEG];
  __shared__ int wave_cnt[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Nout = P + k + Tmax;
  const uint32_t block = linear_block();
  const uint32_t unit = block / parts;
  const int part = block - unit * parts;
  const int b = unit / Nout, nrow = unit - (uint32_t)b * Nout;
  if (b >= B) {
    int id = block - (uint32_t)B * Nout * parts;
    if (id >= kv.blocks) return;
    const int bx = id % kv.gx;
    id /= kv.gx;
    compact_block<KV_FROM_KEPT>(kv.ptrs, kept, text_len, kv.Hkv, P + V + Tmax, Nout, kv.row_bytes, P, V, k, bx,
                                id % (B * kv.Hkv), id / (B * kv.Hkv));
    return;
  }
  const int len = text_len[b];
  // the columns of this part
  const int c0 = part * (CPT * 256), nchunks = min(D / E - c0, CPT * 256);
  const char* hb = reinterpret_cast<const char*>(hidden + b * sb) + c0 * 16;
  const int64_t rowb = sr * (int64_t)sizeof(T);
  char* orow = reinterpret_cast<char*>(out + ((int64_t)b * Nout + nrow) * D) + c0 * 16;
  if (nrow == 0 && part == 0 && tid == 0) new_len[b] = P + k + len;

  if (nrow < P || nrow >= P + k) {                       // prefix or text row: plain copy
    int src;
    if (nrow < P) src = nrow;
    else {
      int t = nrow - P - k;
      src = (t < len) ? P + V + t : -1;
    }
    if (part == 0 && tid == 0) pos_out[(int64_t)b * Nout + nrow] = src;
    if (src < 0) return;
    const char* s = hb + (int64_t)src * rowb;
    for (int c = tid; c < nchunks; c += 256) stg16_stream(orow + c * 16, ldg16_stream(s + c * 16));
    return;
  }

  const int slot = nrow - P;
  const float* sh = s_hat + (int64_t)b * V;
  const int32_t* asg = assign + (int64_t)b * M;
  const int32_t* pr = pruned + (int64_t)b * M;
  const int i_tok = kept[(int64_t)b * k + slot];
  constexpr int PER = MERGE_SEG / 256;
  // entry e of this thread in a segment: wave w takes 64 PER entries in a row, 64 at a time
  const int first = wave * (64 * PER) + lane;
  int to[PER], tok[PER];
  auto load_lists = [&](int seg) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int a = seg + first + 64 * e;
      to[e] = a < M ? asg[a] : -1;
      tok[e] = a < M ? pr[a] : 0;
    }
  };
  load_lists(0);
  const char* xrow = hb + (int64_t)(P + i_tok) * rowb;
  uint4 own[CPT];
#pragma unroll
  for (int q = 0; q < CPT; ++q)
    if (tid + q * 256 < nchunks) own[q] = ldg16_stream(xrow + (tid + q * 256) * 16);
  const float w_i = sh[i_tok];
  float acc[CPT][E];
  float den = w_i, absorbed = 0.0f;
  for (int seg = 0; seg < M; seg += MERGE_SEG) {
    if (seg) load_lists(seg);
    // ordered compaction of the sources of this slot among entries [seg, seg + MERGE_SEG)
    int before[PER], cnt = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const unsigned long long found = __ballot(to[e] == slot);
      before[e] = cnt + __popcll(found & ((1ull << lane) - 1));
      cnt += __popcll(found);
    }
    float w[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) w[e] = !LATE && to[e] == slot ? mu * sh[tok[e]] : 0.0f;
    if (seg) __syncthreads();                  // the previous round's lists have been used
    if (lane == 0) wave_cnt[wave] = cnt;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (v < wave) base += wave_cnt[v];
      total += wave_cnt[v];
    }
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (to[e] == slot) {
        list[base + before[e]] = tok[e];
        if (!LATE) weight[base + before[e]] = w[e];
      }
    __syncthreads();
    total = __builtin_amdgcn_readfirstlane(total);
    if (seg == 0) {
#pragma unroll
      for (int q = 0; q < CPT; ++q) {
        float f[E];
        unpack16<T>(own[q], f);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[q][e] = w_i * f[e];
      }
    }
    for (int s0 = 0; s0 < total; s0 += AHEAD) {
      uint4 ch[AHEAD][CPT];
      float wt[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if (s0 + u < total) {
          const int j = __builtin_amdgcn_readfirstlane(list[s0 + u]);
          const char* srow = hb + (int64_t)(P + j) * rowb;
          if (LATE) wt[u] = mu * sh[j];
#pragma unroll
          for (int q = 0; q < CPT; ++q)
            if (tid + q * 256 < nchunks) ch[u][q] = ldg16_stream(srow + (tid + q * 256) * 16);
        }
      }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if (s0 + u < total) {
          const float wu = LATE ? wt[u] : weight[s0 + u];
          den += wu;
          absorbed += wu;
#pragma unroll
          for (int q = 0; q < CPT; ++q) {
            float f[E];
            unpack16<T>(ch[u][q], f);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[q][e] = fmaf(wu, f[e], acc[q][e]);
          }
        }
      }
    }
  }
  if (part == 0 && tid == 0) {
    wsum[(int64_t)b * k + slot] = den;
    final_idx[(int64_t)b * k + slot] = i_tok;
    pos_out[(int64_t)b * Nout + nrow] = P + i_tok;
  }
  const float inv = 1.0f / den;
#pragma unroll
  for (int q = 0; q < CPT; ++q) {
    const int c = tid + q * 256;
    if (c >= nchunks) continue;
    uint4 y = own[q];                          // nothing absorbed: Eq. 6 is the identity
    if (absorbed > 0.0f) {
      float f[E];
#pragma unroll
      for (int e = 0; e < E; ++e) f[e] = acc[q][e] * inv;
      y = pack16<T>(f);
    }
    stg16_stream(orow + c * 16, y);
  }
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
template <typename T>
static hipError_t merge_typed(const asap_params& p, const void* hidden, int64_t hsb, int64_t hsr,
                              const float* s_hat, const int32_t* text_len, const int32_t* kept,
                              const int32_t* cand, int M, void* out_hidden, int32_t* pos_out, int32_t* new_len,
                              int32_t* assign, float* wsum, int32_t* final_idx, const MergeKv* kv, hipStream_t st,
                              Timer* tm) {
  const T* h = static_cast<const T*>(hidden);
  constexpr int E = elem<T>::per16;
  const int nchunks = p.D / E;
  const int cpt = (nchunks + 255) / 256;
  MergeKv mk{};
  if (kv) {
    mk = *kv;
    mk.gx = (p.P + p.k + p.Tmax + kv_rows_per_block(mk.row_bytes) - 1) / kv_rows_per_block(mk.row_bytes);
    mk.blocks = mk.gx * p.B * mk.Hkv * mk.n_bufs;
  }
  // Few rows (at most about four workgroups per compute unit): pieces of 4 KB with workgroups of their own,
  // whose threads then have registers for 16 source rows in flight (one image, 2304 tokens: 15 -> 13 us,
  // 576 tokens in f32: 16 -> 12).  Many rows: whole rows, so that the lists are scanned once per row (16 x 2304:
  // 71 us, 78 in pieces).
  const int64_t rows = (int64_t)p.B * (p.P + p.k + p.Tmax);
  const int parts = rows <= MERGE_SPLIT_ROWS ? cpt : 1;
  const dim3 grid = grid_of(rows * parts + mk.blocks);
#define ASAP_MERGE(CPT, AHEAD)                                                                                 \
  ASAP_LAUNCH(tm, "k_merge", (k_merge<T, CPT, AHEAD>), grid, dim3(256), 0, st, h, hsb, hsr, p.D, p.P, p.V, p.k, \
              M, p.Tmax, p.merge_weight, s_hat, text_len, kept, cand, assign, static_cast<T*>(out_hidden),     \
              pos_out, new_len, wsum, final_idx, p.B, parts, mk)
  if (cpt <= 1 || parts > 1) ASAP_MERGE(1, 16);
  else if (cpt <= 2) ASAP_MERGE(2, 8);
  else if (cpt <= 4) ASAP_MERGE(4, 6);
  else if (cpt <= 8) ASAP_MERGE(8, 4);
  else return hipErrorInvalidValue;
#undef ASAP_MERGE
  return hipGetLastError();
}

hipError_t launch_merge(const asap_params& p, const void* hidden, int64_t hsb, int64_t hsr, const float* s_raw,
                        const float* s_hat, const int32_t* text_len, const int32_t* kept, const int32_t* pruned,
                        void* out_hidden, int32_t* pos_out, int32_t* new_len, int32_t* assign, float* best_sim,
                        float* wsum, int32_t* final_idx, const MergeKv* kv, char* ws, hipStream_t st, Timer* tm) {
  const bool bf = p.h_dtype == ASAP_BF16;
  if (p.route == ASAP_ROUTE_PAPER) {
    // kept x kept search (destinations into the workspace) -> roots, refills, final list -> merge
    // with the kept tokens as candidates and the final list in the place of the kept list
    int32_t* dest = reinterpret_cast<int32_t*>(ws);
    hipError_t e = launch_similarity(p, hidden, hsb, hsr, kept, kept, p.k, true, s_hat, dest, best_sim,
                                     ws + paper_workspace_bytes(p), st, tm);
    if (e != hipSuccess) return e;
    e = launch_paper_plan(p, dest, kept, s_raw, final_idx, assign, st, tm);
    if (e != hipSuccess) return e;
    return bf ? merge_typed<bf16_t>(p, hidden, hsb, hsr, s_hat, text_len, final_idx, kept, p.k, out_hidden, pos_out,
                                    new_len, assign, wsum, final_idx, kv, st, tm)
              : merge_typed<float>(p, hidden, hsb, hsr, s_hat, text_len, final_idx, kept, p.k, out_hidden, pos_out,
                                   new_len, assign, wsum, final_idx, kv, st, tm);
  }
  const int M = p.V - p.k;
  if (M > 0) {
    hipError_t e = launch_similarity(p, hidden, hsb, hsr, kept, pruned, M, false, s_hat, assign, best_sim, ws, st, tm);
    if (e != hipSuccess) return e;
  }
  return bf ? merge_typed<bf16_t>(p, hidden, hsb, hsr, s_hat, text_len, kept, pruned, M, out_hidden, pos_out, new_len,
                                  assign, wsum, final_idx, kv, st, tm)
            : merge_typed<float>(p, hidden, hsb, hsr, s_hat, text_len, kept, pruned, M, out_hidden, pos_out, new_len,
                                 assign, wsum, final_idx, kv, st, tm);
}

}  // namespace asap
