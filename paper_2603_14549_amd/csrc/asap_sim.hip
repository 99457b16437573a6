// Cosine routing of pruned tokens to kept tokens (Sec. 4.2): the one dense contraction of the
// stage, (pruned rows) x (kept rows)^T over the hidden dimension, on the matrix cores, with the
// row arg-max fused into the epilogue.
//
//   k_sim<T, NT>  (bf16 hidden states)
//                 workgroup tile BM = 128 source rows x BN = 64*NT destination rows, 256 threads =
//                 4 waves (2 x 2 over the tile, each 64 x 32*NT = 2 x NT MFMA tiles of 32 x 32), one
//                 wave per SIMD so that a wave may use the whole 512-entry register file.  The
//                 hidden dimension is walked in steps of 128 bytes per row, one barrier per step.
//                 Operands reach LDS by direct global -> LDS loads (no registers in between) that
//                 every wave issues between its MFMAs; the squared norms of the rows are added up
//                 from the operands a wave holds, also in the shadow of the MFMAs (waves that hold
//                 the same rows take half of the contraction slices each).
//                 The source rows are read once, from HBM, the destination rows, which all tiles of an
//                 image share, come from L2; slices of either go through a ring of LDS slots, asked for
//                 one step (destination rows of the widest tile) to five ahead (sim_na, sim_nb).
//                 LDS rows are unpadded; the 16-byte piece p of row r is stored in slot
//                 p ^ ((r >> 1) & 7): any 16 consecutive rows then cover all 64 banks once, for the
//                 1 KiB-contiguous loads as well as for the strided 16-byte operand reads.
//                 The grid is one-dimensional and XCD-aware: consecutive workgroup ids go to the 8
//                 XCDs round-robin, so id % 8 picks the XCD, and each XCD is given one contiguous
//                 eighth of the tiles (image-major) -- the tiles of an image then share the L2 of one
//                 XCD, or of the few that an image spans, for the kept panel (see sim_work).
//                 A workgroup takes one destination tile.  When the destination rows need several
//                 (k > 64*NT), the tiles of a source tile are workgroups of their own: each leaves
//                 its row winner as a 64-bit key (order-preserving value bits, then the inverted
//                 column so that equal values keep the smaller column) in a slot of its own.
//                 Launches of at most 128 workgroups also cut the hidden dimension into slices
//                 with workgroups of their own, which leave raw partial products and partial
//                 squared norms instead of a row winner.
//   k_sim_f32<NT> (f32 hidden states) the same tile, grid and epilogue; every value is cut into three
//                 bf16 pieces once per workgroup on its way global memory -> registers -> LDS, and the
//                 waves multiply finished pieces (six piece products per pair of values)
//   k_sim_finish  largest key of a row -> assign, best_sim (threshold and source norm applied here)
//   k_sim_reduce  sums the slices of a split launch, then the same scaling, predicate and arg-max
#include "asap_device.hpp"
#include "asap_launch.hpp"
#include "asap_select.hpp"

namespace asap {

constexpr int SIM_BM = 128;
constexpr int SIM_ROWB = 128;      // bytes of a row held in LDS per step
// LDS ring slots for the source rows (NA) and the destination rows (NB) by tile width, NA >= NB >= 2, in 160 KiB.
// Narrow tiles belong to launches with few workgroups (small batches, the search inside the kept set), whose steps last as
// long as a load takes to arrive divided by how many steps ahead it was asked for.  Loads return in the order they were
// asked for, on the whole compute unit: destination rows that come from L2 arrive behind the source rows from HBM that were
// asked for before them, so that what is needed first and asked for last sets the pace.  256 columns with three slots of each
// (all loads two steps ahead) instead of four and two: search and merge of 4 x 4096 tokens on 512 98.3 -> 94.1 us, 3 x 3072 on
// 769 89.2 -> 83.5, 8 x 1024 on 256 56.9 -> 54.7.  (320 columns have no room for that.)  For the same reason source slots beyond
// NB + 1, of which 64, 128 and 320 columns have one, are without effect: the wait for the destination rows of the next step
// has the source rows of NA - NB - 1 further steps arrive too.
constexpr int sim_na(int nt) { return nt == 1 ? 6 : nt == 2 ? 5 : nt == 4 ? 3 : 4; }
constexpr int sim_nb(int nt) { return nt == 1 ? 4 : nt <= 4 ? 3 : 2; }
// Loads of a wave that may be on their way at the end of a step, all after those that the next step needs: steps s
// ask for the destination rows of step s + NB - 1, then for the source rows of step s + NA - 1.
constexpr int sim_open(int nt) { return (sim_na(nt) > sim_nb(nt) ? SIM_BM / 32 : 0) + (sim_nb(nt) - 2) * (SIM_BM / 32 + 2 * nt); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// Sum of squares of the elements of a 16-byte chunk, kept in four independent partial sums so that
// consecutive operations never wait for each other.
struct SumSq4 {
  float p[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  __device__ __forceinline__ float total() const { return (p[0] + p[1]) + (p[2] + p[3]); }
};
template <typename T> __device__ __forceinline__ void sumsq16(const uint4& c, SumSq4& acc);
template <> __device__ __forceinline__ void sumsq16<bf16_t>(const uint4& c, SumSq4& acc) {
  bf16x2_t p;
  __builtin_memcpy(&p, &c.x, 4); acc.p[0] = __builtin_amdgcn_fdot2_f32_bf16(p, p, acc.p[0], false);
  __builtin_memcpy(&p, &c.y, 4); acc.p[1] = __builtin_amdgcn_fdot2_f32_bf16(p, p, acc.p[1], false);
  __builtin_memcpy(&p, &c.z, 4); acc.p[2] = __builtin_amdgcn_fdot2_f32_bf16(p, p, acc.p[2], false);
  __builtin_memcpy(&p, &c.w, 4); acc.p[3] = __builtin_amdgcn_fdot2_f32_bf16(p, p, acc.p[3], false);
}
template <> __device__ __forceinline__ void sumsq16<float>(const uint4& c, SumSq4& acc) {
  float f[4];
  unpack16<float>(c, f);
  acc.p[0] = fmaf(f[0], f[0], acc.p[0]); acc.p[1] = fmaf(f[1], f[1], acc.p[1]);
  acc.p[2] = fmaf(f[2], f[2], acc.p[2]); acc.p[3] = fmaf(f[3], f[3], acc.p[3]);
}

// Sum over the two lane halves of a wave, in every lane (v_permlane32_swap).
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// What a workgroup knows about its tile once the products are done, and where the results go.
struct SimTile {
  int b, B, M, k, V;
  int m0, n0;                 // first source row, first destination column
  int pass, ptiles, mt;       // destination tile, their count, source tile
  int ks, ksplit;             // slice of the hidden dimension
  float threshold;
  const int32_t* kept;
  const float* s_hat;
  int32_t* assign;
  float* best_sim;
  unsigned long long* best_key;
  float* src_norm2;
  float* dots;
  float* kept_norm2;
};

// Epilogue of a 128 x 64 NT tile held as 2 x NT accumulators per wave (waves 2 x 2 over the tile):
// norm2 [HALVES][128] / normk [HALVES][64 NT] hold the squared norms of its rows / columns (this slice's share, in one
// or two parts), part [2][128] and best [4][64][BEST_ROW] are LDS scratch, srow [128] the salience of the source rows
// (ANCHORED).  The caller has put a barrier after the writes of norm2, normk and srow and the last use of best's place.
// The 32 lanes that share a row meet through LDS: each leaves the best of its NT columns, and then a lane takes a whole
// row (butterflies over 32 rows one by one, value and column each, took 6.6 of the 103 us of 16 x 2304 tokens, now
// 4.6; 5 x 2083 on 301: 4.5, now 3.1).
constexpr int BEST_ROW = 34;                   // pairs per row: 32 lanes, and rows that start on 16 bytes
constexpr size_t BEST_BYTES = (size_t)4 * 64 * BEST_ROW * sizeof(uint2);
template <int NT, bool ANCHORED, int HALVES>
__device__ __forceinline__ void sim_tile_epilogue(f32x16_t (&acc)[2][NT], const float* norm2, const float* normk,
                                                  uint2* part, const float* srow, uint2* best, const SimTile& T_) {
  constexpr int BN = 64 * NT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31;
  const int wm = wave >> 1, wn = wave & 1;
  const int b = T_.b, B = T_.B, M = T_.M, k = T_.k, V = T_.V, m0 = T_.m0, n0 = T_.n0, pass = T_.pass;
  const int ptiles = T_.ptiles, mt = T_.mt, ks = T_.ks, ksplit = T_.ksplit;
  const float threshold = T_.threshold;
  const int32_t* __restrict__ kept = T_.kept;
  const float* __restrict__ s_hat = T_.s_hat;
  auto row_norm2 = [&](int r) { return HALVES == 2 ? norm2[r] + norm2[SIM_BM + r] : norm2[r]; };
  auto col_norm2 = [&](int c) { return HALVES == 2 ? normk[c] + normk[BN + c] : normk[c]; };
  float run_v = -INFINITY;   // best of this workgroup's destination tile (threads < BM)
  int run_c = 0;
  {
    if (ksplit > 1) {
      // this slice's share of the products and of the squared norms; k_sim_reduce adds the slices up
      const int64_t img = (int64_t)ks * B + b;
      if (pass == 0 && tid < SIM_BM && m0 + tid < M) T_.src_norm2[img * M + m0 + tid] = row_norm2(tid);
      if (mt == 0)
        for (int c = tid; c < BN; c += 256)        // BN may exceed the workgroup size
          if (n0 + c < k) T_.kept_norm2[img * k + n0 + c] = col_norm2(c);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = m0 + wm * 64 + i * 32 + mma32_row(v, lane);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const int col = n0 + wn * (BN / 2) + t * 32 + n;
            if (row < M && col < k) T_.dots[(img * M + row) * k + col] = acc[i][t][v];
          }
        }
      return;
    }

    // Row arg-max of dot / |x_j| over this pass's destinations (|x_i| > 0 does not move it).
    // A lane first takes the best of its NT columns of a row (columns past k get -inf).
    float invk[NT], bias[NT];
    int colv[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int cl = wn * (BN / 2) + t * 32 + n;
      colv[t] = n0 + cl;
      const bool valid = colv[t] < k;
      invk[t] = valid ? 1.0f / fmaxf(sqrtf(col_norm2(cl)), 1e-8f) : 0.0f;
      bias[t] = valid ? 0.0f : -INFINITY;
    }
    float scol[NT];            // ANCHORED: salience of this lane's destination columns
#pragma unroll
    for (int t = 0; t < NT; ++t)
      scol[t] = (ANCHORED && colv[t] < k) ? s_hat[(int64_t)b * V + kept[(int64_t)b * k + colv[t]]] : 0.0f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      uint2* rows = best + (wave * 64 + i * 32) * BEST_ROW + n;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float c[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) c[t] = fmaf(acc[i][t][v], invk[t], bias[t]);
        if (ANCHORED) {
          const int rloc = wm * 64 + i * 32 + mma32_row(v, lane);
          const float sr_ = srow[rloc];
          const int rslot = m0 + rloc;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const bool stronger = (scol[t] > sr_) | ((scol[t] == sr_) & (colv[t] < rslot));
            c[t] = stronger ? c[t] : -INFINITY;
          }
        }
        float bv = c[0];
#pragma unroll
        for (int t = 1; t < NT; ++t) bv = fmaxf(bv, c[t]);
        int bc = 0x7fffffff;
#pragma unroll
        for (int t = NT - 1; t >= 0; --t) bc = (c[t] == bv) ? colv[t] : bc;       // columns ascend with t
        rows[mma32_row(v, lane) * BEST_ROW] = make_uint2(__float_as_uint(bv), (uint32_t)bc);
      }
    }
    wave_lds_order();
    // lane l: row l of the wave's 64; the largest value and its smallest column
    {
      const uint4* row = reinterpret_cast<const uint4*>(best + (wave * 64 + lane) * BEST_ROW);
      float mv = -INFINITY;
      int mc = 0x7fffffff;
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const uint4 q = row[x];
        auto take = [&](float v, int c) {
          const float nv = fmaxf(mv, v);
          mc = (v == nv && (mv != nv || c < mc)) ? c : mc;
          mv = nv;
        };
        if (x == 0) {
          mv = __uint_as_float(q.x);
          mc = (int)q.y;
        } else {
          take(__uint_as_float(q.x), (int)q.y);
        }
        take(__uint_as_float(q.z), (int)q.w);
      }
      part[wn * SIM_BM + wm * 64 + lane] = make_uint2(__float_as_uint(mv), (uint32_t)mc);
    }
    __syncthreads();
    if (tid < SIM_BM) {
      uint2 p0 = part[tid], p1 = part[SIM_BM + tid];
      float v0 = __uint_as_float(p0.x), v1 = __uint_as_float(p1.x);
      int c0 = (int)p0.y, c1 = (int)p1.y;
      if (v1 > v0 || (v1 == v0 && c1 < c0)) { v0 = v1; c0 = c1; }
      run_v = v0;
      run_c = c0;
    }
  }
  if (tid < SIM_BM && m0 + tid < M) {
    const int64_t o = (int64_t)b * M + m0 + tid;
    if (ptiles == 1) {
      float c = run_v / fmaxf(sqrtf(row_norm2(tid)), 1e-8f);
      T_.best_sim[o] = c;
      T_.assign[o] = (c > threshold) ? run_c : -1;
    } else {
      // several destination tiles per source row: every tile leaves its best as a 64-bit key (value,
      // then the inverted column so that equal values keep the smaller column); k_sim_finish takes the
      // largest key of a row and turns it into assign / best_sim
      const unsigned long long key = ((unsigned long long)float_key(run_v) << 32) | (0xFFFFFFFFu - (uint32_t)run_c);
      T_.best_key[(int64_t)pass * ((int64_t)B * M) + o] = key;
      if (pass == 0) T_.src_norm2[o] = row_norm2(tid);
    }
  }
}

// The unit of work of a workgroup: destination tile `pass` of slice `ks` of source tile mt of image b.
// The units are numbered image by image, source tile by source tile, the destination tiles of a slice
// next to each other, and XCD x (= the workgroup ids with id % 8 == x) takes the x-th eighth of them:
// every XCD has the same number to do whatever the batch (a whole image per XCD left three of the
// eight idle at 5 images: the last-token stage of 5 x 2083 tokens took 158 us, now 125), and an image's
// kept panel is fetched by the one or few XCDs that work on it.
// `turn` is the number of the source tile, whichever XCD its units go to: the walk over the hidden dimension
// starts from it, and all destination tiles of a source tile (and slice) must add up in the same order, so
// that the similarities of equal kept rows are equal and the smallest slot wins.
struct SimWork { int b, mt, pass, ks, turn; };
__device__ __forceinline__ bool sim_work(int B, int mtiles, int ptiles, int ksplit, SimWork& w) {
  const int units = B * mtiles * ptiles * ksplit, per_xcd = (units + NUM_XCD - 1) / NUM_XCD;
  const int slot = blockIdx.x / NUM_XCD, u = (blockIdx.x % NUM_XCD) * per_xcd + slot;
  if (u >= units) return false;                // slot < per_xcd by the size of the grid
  w.pass = u % ptiles;
  w.ks = (u / ptiles) % ksplit;
  const int tile = u / (ptiles * ksplit);
  w.b = tile / mtiles;
  w.mt = tile % mtiles;
  w.turn = tile;
  return true;
}

// ANCHORED (the routing inside the kept set, Sec. 4.2): the source rows are the kept tokens too
// (pruned == kept, M == k), and a destination counts for a source only if it is the stronger of the
// two: larger salience s_hat, ties to the smaller index -- which is the smaller slot, both lists
// being ascending.  A token is never its own destination.
template <typename T, int NT, bool ANCHORED>
__global__ __launch_bounds__(256) void k_sim(const T* __restrict__ xv, int64_t sb, int64_t sr, int D,
                                              const int32_t* __restrict__ pruned, const int32_t* __restrict__ kept,
                                              const float* __restrict__ s_hat, int V, int B, int M, int k,
                                              int mtiles, int ptiles, float threshold,
                                              int32_t* __restrict__ assign,
                                              float* __restrict__ best_sim, unsigned long long* __restrict__ best_key,
                                              float* __restrict__ src_norm2, int ksplit, float* __restrict__ dots,
                                              float* __restrict__ kept_norm2) {
  constexpr int BN = 64 * NT;
  constexpr int PA = SIM_BM / 32;                // source-row loads a thread issues per step
  constexpr int PB = BN / 32;                    // destination-row loads
  constexpr int ASTAGE = SIM_BM * SIM_ROWB, BSTAGE = BN * SIM_ROWB;
  constexpr int NA = sim_na(NT), NB = sim_nb(NT);
  static_assert(NA >= NB && NB >= 2, "ring depths");
  static_assert(PA + PB <= 8 * NT, "one load per MFMA slot");
  extern __shared__ __align__(16) char lds[];
  char* ldsB = lds + NA * ASTAGE;
  const uint32_t lds_addr = lds_address(lds), ldsB_addr = lds_addr + NA * ASTAGE;
  float* norm2 = reinterpret_cast<float*>(ldsB + NB * BSTAGE);   // [2][BM] squared norms of the source rows
  float* normk = norm2 + 2 * SIM_BM;                             // [2][BN] squared norms of this pass's kept rows
  uint2* part = reinterpret_cast<uint2*>(normk + 2 * BN);        // [2][BM] (value, column) per column half
  float* srow = reinterpret_cast<float*>(part + 2 * SIM_BM);     // [BM] salience of the source rows (ANCHORED)

  // With ksplit > 1 (launches that would leave most of the chip idle) the hidden dimension is cut into
  // ksplit slices, each with workgroups of its own, which leave raw partial products and partial
  // squared norms for k_sim_reduce instead of taking the arg-max themselves.
  SimWork w;
  if (!sim_work(B, mtiles, ptiles, ksplit, w)) return;
  const int b = w.b, mt = w.mt, pass = w.pass, ks = w.ks;
  const int m0 = mt * SIM_BM;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hf = lane >> 5;
  const int wm = wave >> 1, wn = wave & 1;
  const char* xb = reinterpret_cast<const char*>(xv + b * sb);
  const int64_t rowb = sr * (int64_t)sizeof(T);
  const int steps = (D * (int)sizeof(T)) / SIM_ROWB / ksplit;     // ksplit divides the step count
  const int step_lo = ks * steps;
  // Every workgroup walks its part of the hidden dimension from its own starting step: rows are a
  // power-of-two number of bytes apart, so workgroups in lockstep would all hit the same memory channel.
  const int rot = w.turn % steps;
  auto step_base = [&](int s) {
    int sr_ = s + rot;
    if (sr_ >= steps) sr_ -= steps;
    return xb + (int64_t)(step_lo + sr_) * SIM_ROWB;
  };

  // Loads: thread (rr, q) fetches, for rows rr + 32 i, the piece that belongs in slot q of the row;
  // one load instruction of wave w fills rows 8 w .. 8 w + 7 of a 32-row block, 1 KiB contiguous.
  const int rr = tid >> 3, q = tid & 7;
  const uint32_t piece_off = (uint32_t)((q ^ ((rr >> 1) & 7)) * 16);
  uint32_t offa[PA], offb[PB];      // byte offsets from the image base (an image spans < 4 GiB)
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    int r = min(m0 + rr + 32 * i, M - 1);
    offa[i] = (uint32_t)(pruned[(int64_t)b * M + r] * rowb) + piece_off;
  }
  // Operand reads: byte offset, inside its row, of the chunk this lane reads at position kk of a step.
  // Wave w walks the four contraction slices of a step in the order kk ^ w.  The products do not care,
  // and the sums for the norms can then be shared without a branch: every wave adds up the destination
  // chunks at positions 0 and 1 and the source chunks at positions 0 and 2; the wave below (w ^ 2, same
  // destination rows) covers the other two slices of the former, the wave beside (w ^ 1, same source
  // rows) those of the latter, and the halves meet in LDS after the last step.
  int sw[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) sw[kk] = ((hf * 4 + (kk ^ wave)) ^ ((n >> 1) & 7)) * 16;

  if (ANCHORED) {            // the barriers of the fill below make these visible
    if (tid < SIM_BM) srow[tid] = s_hat[(int64_t)b * V + pruned[(int64_t)b * M + min(m0 + tid, M - 1)]];
  }
  {
    const int n0 = pass * BN;
#pragma unroll
    for (int j = 0; j < PB; ++j) {
      int c = min(n0 + rr + 32 * j, k - 1);
      offb[j] = (uint32_t)(kept[(int64_t)b * k + c] * rowb) + piece_off;
    }
    f32x16_t acc[2][NT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][t][v] = 0.0f;
    SumSq4 ss_a[2], ss_b[NT];

    // fill: destination slices 0 .. NB-2, source slices 0 .. NA-2, as the steps before the first would ask for them (a short
    // walk asks for its last slices again), until the first have landed
    {
#pragma unroll
      for (int x = 1 - NA; x < 0; ++x) {
        const int xb_ = x + NB - 1, xa = x + NA - 1;
        if (xb_ >= 0) {
          const char* g = step_base(min(xb_, steps - 1));
#pragma unroll
          for (int j = 0; j < PB; ++j) load_to_lds16(g, offb[j], ldsB_addr + xb_ * BSTAGE + (8 * wave + 32 * j) * SIM_ROWB);
        }
        const char* ga = step_base(min(xa, steps - 1));
#pragma unroll
        for (int i = 0; i < PA; ++i) load_to_lds16(ga, offa[i], lds_addr + xa * ASTAGE + (8 * wave + 32 * i) * SIM_ROWB);
      }
      wait_vmem_but<sim_open(NT)>();
      barrier_lds();
    }

    int sa = 0, sb_ = 0;       // ring slots of the current step: s % NA, s % NB
    for (int s = 0; s < steps; ++s) {
      // During step s the waves read source slot s % NA and destination slot s % NB.  Meanwhile the
      // destination rows of step s+NB-1 are asked for first, then the source rows of step s+NA-1, each
      // into the slot the previous step has just left.  Loads retire in order, so what step s+1 needs
      // has landed once only the newest sim_open are outstanding.
      const char* A = lds + sa * ASTAGE + (wm * 64 + n) * SIM_ROWB;
      const char* Bp = ldsB + sb_ * BSTAGE + (wn * (BN / 2) + n) * SIM_ROWB;
      // Past the last step the loads repeat the current step into a slot nobody reads any more:
      // cheaper than branches around every load, which would also split the schedule below.
      const char* gb = step_base(s + NB - 1 < steps ? s + NB - 1 : s);
      const char* ga = step_base(s + NA - 1 < steps ? s + NA - 1 : s);
      const uint32_t db = ldsB_addr + (sb_ == 0 ? NB - 1 : sb_ - 1) * BSTAGE + (8 * wave) * SIM_ROWB;
      const uint32_t da = lds_addr + (sa == 0 ? NA - 1 : sa - 1) * ASTAGE + (8 * wave) * SIM_ROWB;
      sa = sa + 1 == NA ? 0 : sa + 1;
      sb_ = sb_ + 1 == NB ? 0 : sb_ + 1;
      auto load_unit = [&](int u) {      // the u-th load of this step, if there is one
        if (u < PB) load_to_lds16(gb, offb[u < PB ? u : 0], db + u * 32 * SIM_ROWB);
        else if (u < PB + PA) load_to_lds16(ga, offa[u < PB + PA ? u - PB : 0], da + (u - PB) * 32 * SIM_ROWB);
      };
      // LDS operand reads run one contraction slice ahead of the MFMAs that use them
      uint4 a[2][2], bq[2][NT];
      auto load_op = [&](int set, int kk, int u) {      // in the order the MFMAs need them
        if (u == 0) a[set][0] = *reinterpret_cast<const uint4*>(A + sw[kk]);
        else if (u == 2) a[set][1] = *reinterpret_cast<const uint4*>(A + 32 * SIM_ROWB + sw[kk]);
        else {
          const int t = u == 1 ? 0 : u - 2;
          if (t < NT) bq[set][t] = *reinterpret_cast<const uint4*>(Bp + t * 32 * SIM_ROWB + sw[kk]);
        }
      };
#pragma unroll
      for (int u = 0; u < NT + 2; ++u) load_op(0, 0, u);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        // After each MFMA: one LDS read for the next contraction slice, one global -> LDS load and a
        // few dot products for the norms, all in the MFMA's shadow.
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          __builtin_amdgcn_sched_barrier(0);
          mma32<T>(acc[0][t], a[kk & 1][0], bq[kk & 1][t]);
          if (kk < 3) load_op((kk + 1) & 1, kk + 1, 2 * t);
          if (kk < 2) sumsq16<T>(bq[kk & 1][t], ss_b[t]);
          load_unit(kk * 2 * NT + 2 * t);
          __builtin_amdgcn_sched_barrier(0);
          mma32<T>(acc[1][t], a[kk & 1][1], bq[kk & 1][t]);
          if (kk < 3) load_op((kk + 1) & 1, kk + 1, 2 * t + 1);
          if ((kk & 1) == 0) {
            if (t == 0) sumsq16<T>(a[kk & 1][0], ss_a[0]);
            if (t == 1 || NT == 1) sumsq16<T>(a[kk & 1][1], ss_a[1]);
          }
          load_unit(kk * 2 * NT + 2 * t + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (kk < 3) {
#pragma unroll
          for (int u = 2 * NT; u < NT + 2; ++u) load_op((kk + 1) & 1, kk + 1, u);     // NT == 1 only
        }
      }
      wait_vmem_but<sim_open(NT)>();
      barrier_keep_loads();
    }

    // The two lane halves hold the two halves of every 128-byte slice, and the wave beside (source
    // rows) or below (destination rows) the other two contraction slices of every step.
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float v = sum_halves(ss_a[i].total());
      if (hf == 0) norm2[wn * SIM_BM + wm * 64 + i * 32 + n] = v;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float v = sum_halves(ss_b[t].total());
      if (hf == 0) normk[wm * BN + wn * (BN / 2) + t * 32 + n] = v;
    }
    wait_all_vmem();   // the repeated loads of the last steps: the rings become the epilogue's scratch
    __syncthreads();

    SimTile tile;
    tile.b = b; tile.B = B; tile.M = M; tile.k = k; tile.V = V; tile.m0 = m0; tile.n0 = n0; tile.pass = pass;
    tile.ptiles = ptiles; tile.mt = mt; tile.ks = ks; tile.ksplit = ksplit; tile.threshold = threshold;
    tile.kept = kept; tile.s_hat = s_hat; tile.assign = assign; tile.best_sim = best_sim; tile.best_key = best_key;
    tile.src_norm2 = src_norm2; tile.dots = dots; tile.kept_norm2 = kept_norm2;
    static_assert(NA * ASTAGE + NB * BSTAGE >= BEST_BYTES, "the epilogue's scratch");
    sim_tile_epilogue<NT, ANCHORED, 2>(acc, norm2, normk, part, srow, reinterpret_cast<uint2*>(lds), tile);
  }
}

// f32 hidden states.  The bf16 matrix instructions take three bf16 pieces per value (hi + mid + lo =
// the value to 2^-27) and a product is the sum of the six piece products that matter -- a third of
// the matrix time of the f32 instruction.  Cutting a value into its pieces costs about five vector
// instructions, and a wave that issues those for every operand it multiplies (its 64 source and 32 NT
// destination rows, which the wave beside or below cuts again) is bound by its own instruction stream,
// not by the matrix cores.  So here every value is cut exactly once per workgroup: the rows travel
// global memory -> registers (asked for two steps ahead) -> pieces -> LDS, each thread cutting 8
// consecutive values of 2 + NT rows per step, and the waves read finished pieces as operands.  LDS
// holds the pieces of two steps (one being multiplied, one being written); one barrier per step.
//   LDS row of a step: 208 bytes = hi | mid | lo planes of 64 bytes (32 values x 2 bytes) + 16 bytes
//   of padding: 16 consecutive rows then start in 16 different groups of 4 banks.
// Tile, waves, grid order, slices of the hidden dimension and epilogue are those of k_sim.
constexpr int SIMF_ROWP = 208;
constexpr int SIMF_MAX_NT = 4;      // 2 x (128 + 256) rows x 208 bytes = 156 KiB
template <int NT, bool ANCHORED>
__global__ __launch_bounds__(256) void k_sim_f32(const float* __restrict__ xv, int64_t sb, int64_t sr, int D,
                                                  const int32_t* __restrict__ pruned,
                                                  const int32_t* __restrict__ kept, const float* __restrict__ s_hat,
                                                  int V, int B, int M, int k, int mtiles, int ptiles, float threshold, int32_t* __restrict__ assign,
                                                  float* __restrict__ best_sim,
                                                  unsigned long long* __restrict__ best_key,
                                                  float* __restrict__ src_norm2, int ksplit,
                                                  float* __restrict__ dots, float* __restrict__ kept_norm2) {
  constexpr int BN = 64 * NT;
  constexpr int ROWS = SIM_BM + BN;              // rows of a step in LDS: sources, then destinations
  constexpr int NJ = ROWS / 64;                  // rows a thread cuts per step (8 values of each)
  constexpr int STAGE = ROWS * SIMF_ROWP;
  extern __shared__ __align__(16) char lds[];
  // the epilogue's arrays take the place of the pieces once the last step is through
  float* norm2 = reinterpret_cast<float*>(lds);                  // [BM]
  float* normk = norm2 + SIM_BM;                                 // [BN]
  uint2* part = reinterpret_cast<uint2*>(normk + BN);            // [2][BM]
  float* srow = reinterpret_cast<float*>(part + 2 * SIM_BM);     // [BM]

  SimWork w;
  if (!sim_work(B, mtiles, ptiles, ksplit, w)) return;
  const int b = w.b, mt = w.mt, pass = w.pass, ks = w.ks;
  const int m0 = mt * SIM_BM, n0 = pass * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hf = lane >> 5;
  const int wm = wave >> 1, wn = wave & 1;
  const char* xb = reinterpret_cast<const char*>(xv + b * sb);
  const int64_t rowb = sr * (int64_t)sizeof(float);
  const int steps = (D * (int)sizeof(float)) / SIM_ROWB / ksplit;     // ksplit divides the step count
  const int step_lo = ks * steps;
  const int rot = w.turn % steps;                                     // see k_sim
  auto step_base = [&](int s) __attribute__((always_inline)) {
    int sr_ = s + rot;
    if (sr_ >= steps) sr_ -= steps;
    return xb + (int64_t)(step_lo + sr_) * SIM_ROWB;
  };

  // Cutting: thread (lr, g4) takes the values 8 g4 .. 8 g4 + 7 of the step for rows lr + 64 j.
  const int lr = tid >> 2, g4 = tid & 3;
  uint32_t off[NJ];           // byte offsets from the image base (an image spans < 4 GiB)
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int row = lr + 64 * j;
    const int idx = row < SIM_BM ? pruned[(int64_t)b * M + min(m0 + row, M - 1)]
                                 : kept[(int64_t)b * k + min(n0 + row - SIM_BM, k - 1)];
    off[j] = (uint32_t)(idx * rowb) + g4 * 32;
  }
  const int wr = lr * SIMF_ROWP + g4 * 16;        // where the thread's pieces of row lr go (+ 64 j rows)
  // Operands: lane (n, hf) reads the values 16 kb + 8 hf .. + 7 of its rows for contraction block kb.
  const int rd_a = (wm * 64 + n) * SIMF_ROWP + hf * 16;
  const int rd_b = (SIM_BM + wn * (BN / 2) + n) * SIMF_ROWP + hf * 16;

  f32x16_t acc[2][NT];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][t][v] = 0.0f;
  SumSq4 ss[NJ];              // squared norms of the thread's share of its rows

  uint4 raw[2][NJ][2];        // the values of two steps on their way
  auto fetch = [&](uint4 (&r)[NJ][2], int s) __attribute__((always_inline)) {
    const char* g = step_base(s);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      r[j][0] = ldg16(g + off[j]);
      r[j][1] = ldg16(g + off[j] + 16);
    }
  };
  auto cut = [&](const uint4 (&r)[NJ][2], char* stage) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const Split3 p3 = split_f32x8(r[j][0], r[j][1]);
      sumsq16<float>(r[j][0], ss[j]);
      sumsq16<float>(r[j][1], ss[j]);
      char* dst = stage + wr + j * 64 * SIMF_ROWP;
      *reinterpret_cast<uint4*>(dst) = p3.hi;
      *reinterpret_cast<uint4*>(dst + 64) = p3.mid;
      *reinterpret_cast<uint4*>(dst + 128) = p3.lo;
    }
  };
  // The same cut in NJ x 11 units, for a schedule written out by hand: per row of the thread, 8 units
  // that take one value pair through one of the two phases of split_pair, 2 units of squared norms,
  // and the unit that stores the three pieces and asks for the row's values two steps on (gnext: where
  // that step starts), so that every load has almost two steps to arrive.  The pieces under way live
  // in p3, r0, r1.
  constexpr int CUT_UNITS = NJ * 11;
  Split3 p3;
  float r0 = 0.0f, r1 = 0.0f;
  auto cut_unit = [&](auto uc, uint4 (&r)[NJ][2], char* stage, const char* gnext) __attribute__((always_inline)) {
    constexpr int U = decltype(uc)::value;
    constexpr int J = U / 11, R = U % 11;
    if constexpr (R < 8) {
      constexpr int Q = R / 2;
      auto put = [](uint4& v, uint32_t x) __attribute__((always_inline)) {
        if constexpr (Q == 0) v.x = x;
        else if constexpr (Q == 1) v.y = x;
        else if constexpr (Q == 2) v.z = x;
        else v.w = x;
      };
      if constexpr (R % 2 == 0) {
        const uint4& c = r[J][Q / 2];
        const float a = __uint_as_float(Q % 2 == 0 ? c.x : c.z), b = __uint_as_float(Q % 2 == 0 ? c.y : c.w);
        const uint32_t hi = pk_bf16(a, b);
        r0 = a - __uint_as_float(hi << 16);
        r1 = b - __uint_as_float(hi & 0xffff0000u);
        put(p3.hi, hi);
      } else {
        const uint32_t mid = pk_bf16(r0, r1);
        put(p3.mid, mid);
        put(p3.lo, pk_bf16(r0 - __uint_as_float(mid << 16), r1 - __uint_as_float(mid & 0xffff0000u)));
      }
    } else if constexpr (R < 10) {
      sumsq16<float>(r[J][R - 8], ss[J]);
    } else {
      char* dst = stage + wr + J * 64 * SIMF_ROWP;
      *reinterpret_cast<uint4*>(dst) = p3.hi;
      *reinterpret_cast<uint4*>(dst + 64) = p3.mid;
      *reinterpret_cast<uint4*>(dst + 128) = p3.lo;
      r[J][0] = ldg16(gnext + off[J]);
      r[J][1] = ldg16(gnext + off[J] + 16);
    }
  };
  // Operand pieces of contraction block kb (16 values) of the stage
  Split3 a3[2], b3[NT];
  auto operands = [&](const char* stage, int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const char* p = stage + rd_a + i * 32 * SIMF_ROWP + kb * 32;
      a3[i].hi = *reinterpret_cast<const uint4*>(p);
      a3[i].mid = *reinterpret_cast<const uint4*>(p + 64);
      a3[i].lo = *reinterpret_cast<const uint4*>(p + 128);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const char* p = stage + rd_b + t * 32 * SIMF_ROWP + kb * 32;
      b3[t].hi = *reinterpret_cast<const uint4*>(p);
      b3[t].mid = *reinterpret_cast<const uint4*>(p + 64);
      b3[t].lo = *reinterpret_cast<const uint4*>(p + 128);
    }
  };
  // A step, slot by slot and in this order (the compiler moves nothing across a slot's end): one piece
  // product -- product by product over the 2 NT accumulators, so that neighbouring matrix instructions
  // never wait for one another -- and that slot's share of the cut of the next step's values, a few
  // vector instructions that run in the matrix instruction's shadow.  CUT = false: the last step.
  constexpr int SLOTS = 24 * NT;
  auto multiply = [&](auto do_cut, const char* stage, uint4 (&r)[NJ][2], char* next_stage, const char* gnext) __attribute__((always_inline)) {
    constexpr bool CUT = decltype(do_cut)::value;
    static_for<SLOTS>([&](auto sc) __attribute__((always_inline)) {
      constexpr int S = decltype(sc)::value;
      constexpr int KB = S / (12 * NT), P = (S % (12 * NT)) / (2 * NT), t = (S % (2 * NT)) / 2, i = S % 2;
      if constexpr (S % (12 * NT) == 0) operands(stage, KB);
      mma_split_term<P>(acc[i][t], a3[i], b3[t]);
      if constexpr (CUT) {
        constexpr int U0 = S * CUT_UNITS / SLOTS, U1 = (S + 1) * CUT_UNITS / SLOTS;
        static_for<U1 - U0>([&](auto k) __attribute__((always_inline)) {
          cut_unit(std::integral_constant<int, U0 + decltype(k)::value>{}, r, next_stage, gnext);
        });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Step s multiplies the pieces in stage s % 2 while the values of step s + 1 (asked for during step
  // s - 1) are cut into the other stage, row by row; each row's registers then ask for step s + 3.
  // Nothing in a step
  // is conditional (past the end the registers ask for the last step again, and the last step, which
  // has nothing to cut, stands alone after the loop): the waits the compiler places before the first
  // use of a value then leave the younger set of loads in flight.  Two steps per turn, so that each
  // register set keeps its role.
  const int last = steps - 1;
  fetch(raw[0], 0);
  fetch(raw[1], min(1, last));
  cut(raw[0], lds);
  fetch(raw[0], min(2, last));
  __syncthreads();
  auto step = [&](auto parity, int s) __attribute__((always_inline)) {
    constexpr int CUR = decltype(parity)::value;
    multiply(std::true_type{}, lds + CUR * STAGE, raw[CUR ^ 1], lds + (CUR ^ 1) * STAGE,
             step_base(min(s + 3, last)));
    __syncthreads();
  };
  int s = 0;
  for (; s + 2 < steps; s += 2) {
    step(std::integral_constant<int, 0>{}, s);
    step(std::integral_constant<int, 1>{}, s + 1);
  }
  if (s + 2 == steps) {
    step(std::integral_constant<int, 0>{}, s);
    multiply(std::false_type{}, lds + STAGE, raw[0], lds, xb);
  } else {
    multiply(std::false_type{}, lds, raw[1], lds + STAGE, xb);
  }
  __syncthreads();

  // squared norms: the four threads of a row add up their shares
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    float v = ss[j].total();
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    const int row = lr + 64 * j;
    if (g4 == 0) {
      if (row < SIM_BM) norm2[row] = v;
      else normk[row - SIM_BM] = v;
    }
  }
  if (ANCHORED) {
    if (tid < SIM_BM) srow[tid] = s_hat[(int64_t)b * V + pruned[(int64_t)b * M + min(m0 + tid, M - 1)]];
  }
  __syncthreads();

  SimTile tile;
  tile.b = b; tile.B = B; tile.M = M; tile.k = k; tile.V = V; tile.m0 = m0; tile.n0 = n0; tile.pass = pass;
  tile.ptiles = ptiles; tile.mt = mt; tile.ks = ks; tile.ksplit = ksplit; tile.threshold = threshold;
  tile.kept = kept; tile.s_hat = s_hat; tile.assign = assign; tile.best_sim = best_sim; tile.best_key = best_key;
  tile.src_norm2 = src_norm2; tile.dots = dots; tile.kept_norm2 = kept_norm2;
  constexpr int BEST_AT = (4 * (2 * SIM_BM + BN) + 2 * SIM_BM * 8 + 15) / 16 * 16;      // behind those arrays
  static_assert(2 * STAGE >= BEST_AT + BEST_BYTES, "the epilogue's scratch");
  sim_tile_epilogue<NT, ANCHORED, 1>(acc, norm2, normk, part, srow, reinterpret_cast<uint2*>(lds + BEST_AT), tile);
}

// grid (ceil(n / 256)): the largest key over the destination tiles of a row -> assign, best_sim
__global__ __launch_bounds__(256) void k_sim_finish(const unsigned long long* __restrict__ best_key,
                                                     const float* __restrict__ src_norm2, int n, int ptiles,
                                                     float threshold, int32_t* __restrict__ assign,
                                                     float* __restrict__ best_sim) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  unsigned long long key = best_key[i];
  for (int t = 1; t < ptiles; ++t) {
    const unsigned long long other = best_key[(int64_t)t * n + i];
    key = other > key ? other : key;
  }
  const float v = float_unkey((uint32_t)(key >> 32));
  const int col = (int)(0xFFFFFFFFu - (uint32_t)key);
  const float c = v / fmaxf(sqrtf(src_norm2[i]), 1e-8f);
  best_sim[i] = c;
  assign[i] = (c > threshold) ? col : -1;
}

// grid (ceil(M WPR / 4), B), 256 threads: WPR waves per source row, each with every WPR-th 64 columns.  Adds the ksplit partial
// products of every destination column in slice order, scales by the destination's norm, applies the predicate
// of the anchored search, takes the row's arg-max (ties to the smaller column) and divides by the
// source norm -- the arithmetic of k_sim's own epilogue.
//   What bounds it: the chain of loads of a wave, one turn per 64 columns and four slices.  So several waves share a row where the
// chip holds them (sim_reduce_waves), and the source norm's slices are asked for at once and first: one after the other at
// the end they were a chain of their own, 1.2 us of search and merge (1 x 2304 tokens on 320 35.0 -> 33.8, 8 x 576 on 160 47.0 -> 45.6).
template <bool ANCHORED, int WPR>
__global__ __launch_bounds__(256) void k_sim_reduce(const float* __restrict__ dots, const float* __restrict__ src_norm2,
                                                     const float* __restrict__ kept_norm2, int B, int M, int k,
                                                     int ksplit, const int32_t* __restrict__ srcs,
                                                     const int32_t* __restrict__ kept, const float* __restrict__ s_hat,
                                                     int V, float threshold, int32_t* __restrict__ assign,
                                                     float* __restrict__ best_sim) {
  __shared__ float best_v[4];
  __shared__ int best_c[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, part = wave % WPR, b = blockIdx.y;
  const int row_ = blockIdx.x * (4 / WPR) + wave / WPR, row = min(row_, M - 1);       // past the end: the last row, not written
  auto norm_slice = [&](int q) { return q < ksplit ? src_norm2[((int64_t)q * B + b) * M + row] : 0.0f; };
  float sn_slice = norm_slice(lane);
  const float sr_ = ANCHORED ? s_hat[(int64_t)b * V + srcs[(int64_t)b * M + row]] : 0.0f;
  float bv = -INFINITY;
  int bc = 0x7fffffff;
  for (int col = part * 64 + lane; col < k; col += 64 * WPR) {
    // four running sums (slices q, q+1, q+2, q+3 of every four), so that the loads do not wait for
    // one another; the order of the additions is fixed all the same
    float d4[4] = {0.0f, 0.0f, 0.0f, 0.0f}, n4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const int64_t dstride = (int64_t)B * M * k, nstride = (int64_t)B * k;
    const float* dp = dots + ((int64_t)b * M + row) * k + col;
    const float* np = kept_norm2 + (int64_t)b * k + col;
    int q = 0;
    for (; q + 3 < ksplit; q += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        d4[u] += dp[(q + u) * dstride];
        n4[u] += np[(q + u) * nstride];
      }
    }
    for (; q < ksplit; ++q) {
      d4[0] += dp[q * dstride];
      n4[0] += np[q * nstride];
    }
    const float dot = (d4[0] + d4[1]) + (d4[2] + d4[3]), kn = (n4[0] + n4[1]) + (n4[2] + n4[3]);
    float c = dot * (1.0f / fmaxf(sqrtf(kn), 1e-8f));
    if (ANCHORED) {
      const float sc = s_hat[(int64_t)b * V + kept[(int64_t)b * k + col]];
      const bool stronger = (sc > sr_) | ((sc == sr_) & (col < row));
      c = stronger ? c : -INFINITY;
    }
    if (c > bv) { bv = c; bc = col; }             // a lane's columns ascend: the first maximum stays
  }
  auto take = [&](float ov, int oc) {
    if (ov > bv || (ov == bv && oc < bc)) { bv = ov; bc = oc; }
  };
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) take(__shfl_xor(bv, off), __shfl_xor(bc, off));
  if (WPR > 1) {
    if (lane == 0) { best_v[wave] = bv; best_c[wave] = bc; }
    __syncthreads();
    if (part != 0) return;
#pragma unroll
    for (int w = 1; w < WPR; ++w) take(best_v[wave + w], best_c[wave + w]);
  }
  float sn = 0.0f;
  for (int q0 = 0; q0 < ksplit; q0 += 64) {
    if (q0) sn_slice = norm_slice(q0 + lane);
    for (int q = 0; q < min(64, ksplit - q0); ++q) sn += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sn_slice), q));
  }
  if (lane == 0 && row_ < M) {
    const float c = bv / fmaxf(sqrtf(sn), 1e-8f);
    best_sim[(int64_t)b * M + row] = c;
    assign[(int64_t)b * M + row] = (c > threshold) ? bc : -1;
  }
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
static int pick_nt(const asap_params& p, int M);

// Slices of the hidden dimension: 1 unless the launch has at most 128 workgroups; then as many as
// bring it to about one workgroup per compute unit, with at least 8 steps per slice and a count that
// divides the steps, while the partial products stay under 64 MB.
static int pick_ksplit(const asap_params& p, int M, int nt) {
  const int bn = 64 * nt, ptiles = (p.k + bn - 1) / bn, mtiles = (M + SIM_BM - 1) / SIM_BM;
  const long wgs = (long)p.B * mtiles * ptiles;
  const int steps = p.D * (p.h_dtype == ASAP_BF16 ? 2 : 4) / SIM_ROWB;
  if (wgs > 128 || steps < 16) return 1;
  int ks = (int)(256 / wgs);
  if (ks > steps / 8) ks = steps / 8;
  while (ks > 1 && (steps % ks != 0 || (size_t)ks * p.B * M * p.k * sizeof(float) > ((size_t)64 << 20))) --ks;
  return ks < 1 ? 1 : ks;
}

// One key per destination tile and source row, and the source norms, for either kind of search
// (pruned -> kept: V-k source rows; inside the kept set: k), when the destination rows are split
// over several workgroups.
static size_t sim_workspace_for(const asap_params& p, int M) {
  if (M <= 0) return 0;
  const int nt = pick_nt(p, M), bn = 64 * nt, ptiles = (p.k + bn - 1) / bn, ks = pick_ksplit(p, M, nt);
  const size_t rows = (size_t)p.B * M;
  if (ks > 1)      // partial products, source norms, destination norms per slice
    return align256(sizeof(float) * ks * rows * p.k) + align256(sizeof(float) * ks * rows) +
           align256(sizeof(float) * ks * (size_t)p.B * p.k);
  return align256(sizeof(unsigned long long) * rows * ptiles) + align256(sizeof(float) * rows);
}
size_t sim_workspace_bytes(const asap_params& p) {
  const size_t a = sim_workspace_for(p, p.V - p.k), b = sim_workspace_for(p, p.k);
  return a > b ? a : b;
}

static constexpr size_t sim_lds_bytes(bool f32, int nt) {
  const int bn = 64 * nt;
  return f32 ? (size_t)2 * (SIM_BM + bn) * SIMF_ROWP
             : (size_t)(sim_na(nt) * SIM_BM + sim_nb(nt) * bn) * SIM_ROWB + sizeof(float) * (7 * SIM_BM + 2 * bn);
}

static dim3 sim_grid(int units) { return dim3(NUM_XCD * ((units + NUM_XCD - 1) / NUM_XCD)); }

// Waves per row of k_sim_reduce: as many as have columns, while the chip holds them about at once (8192).  Search and merge, us with
// 1 / 2 / 4:  1 x 1600 tokens on 488 43.1 / 37.4 / 35.4;  2 x 904 on 297 29.8 / 28.1 / 28.0;  5 x 492 on 148 30.3 / 29.8 / 29.6;  1 x 2304 on
// 320 33.8 / 32.7 / 32.8;  1 x 3776 on 880 59.7 / 55.0 / 56.5;  8 x 576 on 160 45.6 / 45.9 / 46.7;  4 x 350 on 103 23.2 / 22.7 / 23.0.
static int sim_reduce_waves(const asap_params& p, int M) {
  const long rows = (long)p.B * M;
  return p.k > 128 && rows <= 1800 ? 4 : p.k > 64 && rows <= 3000 ? 2 : 1;
}

template <typename T, int NT, bool ANCHORED>
static hipError_t launch_sim_nt(const asap_params& p, const T* xv, int64_t sb, int64_t sr, const int32_t* srcs,
                                int M, const int32_t* kept, const float* s_hat, int32_t* assign, float* best_sim,
                                char* ws, hipStream_t st, Timer* tm) {
  constexpr int BN = 64 * NT;
  constexpr bool F32 = sizeof(T) == 4;
  static_assert(!F32 || NT <= SIMF_MAX_NT, "two steps of f32 pieces must fit LDS");
  const size_t lds = sim_lds_bytes(F32, NT);
  auto kern = [] {
    if constexpr (F32) return k_sim_f32<NT, ANCHORED>;
    else return k_sim<T, NT, ANCHORED>;
  }();
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const int mtiles = (M + SIM_BM - 1) / SIM_BM;
  const int ptiles = (p.k + BN - 1) / BN;
  const int n = p.B * M;
  const int ksplit = pick_ksplit(p, M, NT);
  const char* label = F32 ? "k_sim_f32" : "k_sim";
  if (ksplit > 1) {
    float* dots = reinterpret_cast<float*>(ws);                                       // [ksplit][B][M][k]
    float* nsrc = reinterpret_cast<float*>(ws + align256(sizeof(float) * ksplit * (size_t)n * p.k));
    float* nkept = reinterpret_cast<float*>(reinterpret_cast<char*>(nsrc) + align256(sizeof(float) * ksplit * (size_t)n));
    ASAP_LAUNCH(tm, label, kern, sim_grid(p.B * mtiles * ptiles * ksplit), dim3(256), lds, st, xv, sb, sr, p.D,
                srcs, kept, s_hat, p.V, p.B, M, p.k, mtiles, ptiles, p.sim_threshold, assign, best_sim,
                static_cast<unsigned long long*>(nullptr), nsrc, ksplit, dots, nkept);
    const int wpr = sim_reduce_waves(p, M);
    auto reduce = wpr == 4 ? k_sim_reduce<ANCHORED, 4> : wpr == 2 ? k_sim_reduce<ANCHORED, 2> : k_sim_reduce<ANCHORED, 1>;
    ASAP_LAUNCH(tm, "k_sim_reduce", reduce, dim3((M * wpr + 3) / 4, p.B), dim3(256), 0, st, dots, nsrc, nkept,
                p.B, M, p.k, ksplit, srcs, kept, s_hat, p.V, p.sim_threshold, assign, best_sim);
    return hipGetLastError();
  }
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(ws);               // [ptiles][B*M]
  float* norms = reinterpret_cast<float*>(ws + align256(sizeof(unsigned long long) * (size_t)n * ptiles));
  ASAP_LAUNCH(tm, label, kern, sim_grid(p.B * mtiles * ptiles), dim3(256), lds, st, xv, sb, sr, p.D, srcs,
              kept, s_hat, p.V, p.B, M, p.k, mtiles, ptiles, p.sim_threshold, assign, best_sim, keys,
              norms, 1, static_cast<float*>(nullptr), static_cast<float*>(nullptr));
  if (ptiles > 1)
    ASAP_LAUNCH(tm, "k_sim_finish", k_sim_finish, dim3((n + 255) / 256), dim3(256), 0, st, keys, norms, n, ptiles,
                p.sim_threshold, assign, best_sim);
  return hipGetLastError();
}

// The kernel is bound by what a workgroup loads (or, for fp32, by what it multiplies): (128 + 64 nt) rows per
// step, over the steps of its slice of the hidden dimension, and the workgroups run in rounds of one per
// compute unit: rounds x steps x rows.
struct SimCost { long wgs, row_steps; };
static SimCost sim_cost(const asap_params& p, int M, int nt) {
  const long bn = 64 * nt, passes = (p.k + bn - 1) / bn, ks = pick_ksplit(p, M, nt);
  const long steps = p.D * (p.h_dtype == ASAP_BF16 ? 2 : 4) / SIM_ROWB;
  const long wgs = (long)p.B * ((M + SIM_BM - 1) / SIM_BM) * passes * ks, rounds = (wgs + 255) / 256;
  // a split launch also pays for the partial products' round trip and for k_sim_reduce: about as
  // much as 6000 row-steps, from measurements on the small configurations
  return {wgs, rounds * (steps / ks) * (SIM_BM + bn) + (ks > 1 ? 6000 : 0)};
}

// Destination tile width 64 * nt: the cheapest (the slicing of pick_ksplit taken into account), then the wider tile.
static int pick_nt(const asap_params& p, int M) {
  const int nt_max = p.h_dtype == ASAP_BF16 ? 5 : SIMF_MAX_NT;
  int best_nt = nt_max;
  long best_cost = -1;
  for (int nt = nt_max; nt >= 1; --nt) {
    const long cost = sim_cost(p, M, nt).row_steps;
    if (best_cost < 0 || cost < best_cost) { best_cost = cost; best_nt = nt; }
  }
  return best_nt;
}

int64_t sim_row_steps(const asap_params& p) {
  const int M = p.V - p.k;
  return M > 0 ? sim_cost(p, M, pick_nt(p, M)).row_steps : 0;
}

// The K/V compaction beside the search, on another stream.  LDS that a workgroup of the copy claims decides how many of
// them share a compute unit with one of the search: as many as registers let in (five), or two, half each of what
// the search's tile leaves.  Two bring both to their end together where the search has one round of workgroups and the copy
// is over before it (us per stage, five / two):
//   5 columns of tiles wide:  16 x 2304 tokens on 320, 440 MB 404 / 399;  8 x 2304 on 576, 354 MB 290 / 285
//   3:  10 x 1500 on 180, 182 MB 218 / 209;  16 x 576 on 144, 127 MB 155 / 151;  8 x 2304 on 184, 148 MB 232 / 228, 593 MB 291 / 284
//   2 and 1:  8 x 2304 on 256, 185 MB 234 / 228;  4 x 1510 on 345, 217 MB 156 / 148;  16 x 1024 on 120, 230 MB 210 / 206
// A copy that takes longer is only held up (16 x 2304 on 320, 3.5 GB 944 / 957; 8 x 2304 on 576, 1.4 GB 438 / 447; 10 x
// 1500 on 500, 392 MB 246 / 249), all the more where further rounds of the search find their compute units taken
// (8 x 2304 on 900, 440 workgroups: 523 MB 337 / 363, 2.1 GB 564 / 641).  The line: 17 KB per row-step of sim_cost,
// more where the search leaves compute units free, and twice that where it is split and the sum of the slices follows (9 x
// 1088 on 237, 4 layers, 1.5 times the line: 214 / 210;  11 x 751 on 175, 40 heads, 1.1 times: 212 / 204), which passes what gained 2 % and more but the last (210 / 206).
// With f32 hidden states, whose tiles leave no registers to share or are over late, no amount was faster (16 x 576 on 144:
// 303 / 308, 12 x 2304 on 691: 1331 / 1335).
size_t compact_lds_beside_sim(const asap_params& p, int64_t bytes) {
  const int M = p.V - p.k;
  if (M <= 0 || p.h_dtype != ASAP_BF16) return 0;
  const int nt = pick_nt(p, M);
  const SimCost c = sim_cost(p, M, nt);
  const int64_t line = 17408 * (pick_ksplit(p, M, nt) > 1 ? 2 : 1);
  if (c.wgs > 256 || bytes * c.wgs > line * c.row_steps * 256) return 0;
  constexpr size_t CU_LDS = 160 * 1024, GRANULE = 1280;        // LDS is given out in multiples of 1280 bytes
  const size_t tile = (sim_lds_bytes(false, nt) + GRANULE - 1) / GRANULE * GRANULE;
  return (CU_LDS - tile) / 2 / GRANULE * GRANULE;
}

template <typename T, bool ANCHORED>
static hipError_t sim_typed(const asap_params& p, const void* hidden, int64_t hsb, int64_t hsr,
                            const int32_t* kept, const int32_t* srcs, int M, const float* s_hat, int32_t* assign,
                            float* best_sim, char* ws, hipStream_t st, Timer* tm) {
  const T* xv = static_cast<const T*>(hidden) + (int64_t)p.P * hsr;
  switch (pick_nt(p, M)) {
    case 1: return launch_sim_nt<T, 1, ANCHORED>(p, xv, hsb, hsr, srcs, M, kept, s_hat, assign, best_sim, ws, st, tm);
    case 2: return launch_sim_nt<T, 2, ANCHORED>(p, xv, hsb, hsr, srcs, M, kept, s_hat, assign, best_sim, ws, st, tm);
    case 3: return launch_sim_nt<T, 3, ANCHORED>(p, xv, hsb, hsr, srcs, M, kept, s_hat, assign, best_sim, ws, st, tm);
    case 4: return launch_sim_nt<T, 4, ANCHORED>(p, xv, hsb, hsr, srcs, M, kept, s_hat, assign, best_sim, ws, st, tm);
    default:
      if constexpr (sizeof(T) == 2)
        return launch_sim_nt<T, 5, ANCHORED>(p, xv, hsb, hsr, srcs, M, kept, s_hat, assign, best_sim, ws, st, tm);
      else
        return hipErrorInvalidValue;        // pick_nt stays below for f32
  }
}

hipError_t launch_similarity(const asap_params& p, const void* hidden, int64_t hsb, int64_t hsr,
                             const int32_t* kept, const int32_t* srcs, int M, bool anchored, const float* s_hat,
                             int32_t* assign, float* best_sim, char* ws, hipStream_t st, Timer* tm) {
  const bool bf = p.h_dtype == ASAP_BF16;
  if (anchored)
    return bf ? sim_typed<bf16_t, true>(p, hidden, hsb, hsr, kept, srcs, M, s_hat, assign, best_sim, ws, st, tm)
              : sim_typed<float, true>(p, hidden, hsb, hsr, kept, srcs, M, s_hat, assign, best_sim, ws, st, tm);
  return bf ? sim_typed<bf16_t, false>(p, hidden, hsb, hsr, kept, srcs, M, s_hat, assign, best_sim, ws, st, tm)
            : sim_typed<float, false>(p, hidden, hsb, hsr, kept, srcs, M, s_hat, assign, best_sim, ws, st, tm);
}

}  // namespace asap
