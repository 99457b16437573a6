// asap_score: Eq. 2 (raw attention mass), Eq. 3 (salience), Eq. 4 (discount) and the text-row
// softmax of Eq. 5 reduced to one selection score per visual token.
//
// Kernels, in launch order:
//   k_qsum        column sums of the visual queries per (image, head[, row chunk]) in fp64
//   k_qsplit      fixed-order sum of those partials per kv head (fp64), also split into four bf16
//                 pieces per component (32 significant bits) for the matrix cores
//   k_mass_mfma   s_j = sum_g qbar_g . k_{g,j} / (H sqrt d)  (Eq. 2 by linearity) and the min / max of
//                 s per key tile.  The four pieces of
//                 qbar are four query rows of an MFMA tile; bf16 keys enter as they are, f32 keys
//                 as three bf16 pieces each (hi + mid + lo = the key to 2^-27), so every product is
//                 exact; one head's 128 products per piece pair are added in fp32 by the matrix
//                 instruction, everything above that in fp64.
//                 When the text rows that rank the tokens are few (rows of a kv head's query heads
//                 <= 28, bf16), they ride in the free rows of that tile: the sweep then also leaves
//                 their raw logits in the workspace, and no further sweep over the keys is needed.
//   k_mass_small, k_mass_small_ride   the same for small batches: a wave per kv head (up to 16), which takes
//                 the place of k_qsplit as well
//   k_mass_finish the (min, max) of a whole image, where those of its key tiles have no room
//   then, bf16 and up to 4096 keys (but see two_sweeps_faster),
//   k_attn_rows   the softmax of the text rows in one sweep over the keys: terms stay in registers until
//                 their row's denominator is known
//   or two sweeps over the keys
//   k_attn_stats  per (image, head, key split): key x text-query logits on the matrix cores (keys as
//                 tile rows, so a lane owns one text row), online (max, sum) of lambda'_j 2^z per row
//   k_attn_colsum the sweep again with queries as tile rows and the merged row statistics:
//                 normalised column sums per key
//   or, from stored logits,
//   k_rowstats_logits / k_colsum_logits   the same two reductions over the [rows, V] logits
//   k_score       fixed-order head reduction, times lambda' (Eq. 4) in fp64, mean over heads and
//                 text rows; also writes s_hat (Eq. 3)
//   k_score_select  the same followed by the top-k selection of asap_select in one launch (one
//                 workgroup per image), when the stage runs as one call; k_score_select_kv has further
//                 workgroups that copy the K/V rows of prefix and text meanwhile
// f32 queries and keys reach the bf16 matrix instructions as three bf16 pieces each; a logit is the
// sum of the six piece products that matter (hi.hi, hi.mid, mid.hi, mid.mid, hi.lo, lo.hi: what is
// left out is below 2^-25 of sum |q_c k_c|, half a unit of the fp32 accumulation itself).
// Logits stay in accumulator units; the factor log2(e)/sqrt(d) is applied to differences from the
// row maximum only, so its rounding error scales with the distance from the maximum.
#include "asap_device.hpp"
#include "asap_launch.hpp"
#include "asap_select.hpp"

#include <algorithm>

namespace asap {

// Minimum and maximum of masses, NaN if one of them is (as the salience of the whole image then is).
__device__ __forceinline__ double nan_min(double a, double b) { return (b < a || b != b) ? b : a; }
__device__ __forceinline__ double nan_max(double a, double b) { return (b > a || b != b) ? b : a; }

// Smallest and largest raw mass of image b (Eq. 3).  The mass kernel leaves one (min, max) pair per key
// tile, n of them in mm [B, n, 2]; every wave that needs the range takes it over those (at most 512) pairs
// itself.  Device-wide atomics on one pair per image were measured at about 13 us for 512 workgroups: they
// queue up at the memory side, one after the other.
// Asked for in two halves, so that the loads can be issued ahead of whatever else the caller waits for.
struct MassRange {
  const double2* p;
  int n;
  double2 first;
  __device__ __forceinline__ void load(const double* __restrict__ mm, int n_, int b) {
    n = n_;
    p = reinterpret_cast<const double2*>(mm) + (int64_t)b * n;
    first = p[min((int)(threadIdx.x & 63), n - 1)];
  }
  __device__ __forceinline__ void reduce(double& lo, double& hi) const {
    lo = first.x;
    hi = first.y;
    if (n == 1) return;
    for (int i = (threadIdx.x & 63) + 64; i < n; i += 64) {
      const double2 x = p[i];
      lo = nan_min(lo, x.x);
      hi = nan_max(hi, x.y);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      lo = nan_min(lo, shfl_xor_f64(lo, off));
      hi = nan_max(hi, shfl_xor_f64(hi, off));
    }
  }
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// successive bf16 roundings of what is left of x: x = p0 + p1 + p2 + p3 to 32 significant bits
__device__ __forceinline__ void split_bf16x4(double x, uint16_t* out, int stride) {
  double rest = x;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    uint32_t bits = f32_to_bf16_bits((float)rest);
    out[p * stride] = (uint16_t)bits;
    rest -= (double)bf16_bits_to_f32(bits);
  }
}

// ------------------------------------------------------------------------------------------
// k_qsum: grid (chunks, H, B), 1024 threads.  A row is d elements = LPR 16-byte pieces; thread t
// keeps piece t % LPR of rows t / LPR + RPI * i.
// With one chunk and one query head per kv head the block's sums are final (`direct`): it writes
// their bf16 split itself and k_qsplit is not needed.
// What bounds it: HBM.  Every row is added in fp64, so that the split of the rows does not decide the precision; eight rows of a
// thread added in fp32 first were no faster (us of asap_score, fp32 / fp64: 16 x 32 heads x 2304 tokens 167.5 / 167.7; 5 x 28 on 4 x
// 2083 38.3 / 36.1; f32, 16 x 32 x 576 188.0 / 187.4; 4 x 32 x 4096 180.8 / 181.7).
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(1024) void k_qsum(const T* __restrict__ q, Strides3 sq, int V, int d, int R,
                                                double* __restrict__ qpart, uint16_t* __restrict__ qsplit, int direct) {
  constexpr int E = elem<T>::per16;
  const int LPR = d / E, RPI = 1024 / LPR;
  const int tid = threadIdx.x, piece = tid % LPR, r0 = tid / LPR;
  const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int lo = c * R, hi = min(V, lo + R);
  const char* base = reinterpret_cast<const char*>(q + b * sq.b + h * sq.h + piece * E);
  const int64_t rowb = sq.r * (int64_t)sizeof(T);
  double acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.0;
  int row = lo + r0;
  for (; row + 7 * RPI < hi; row += 8 * RPI) {       // eight rows in flight
    uint4 ch[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) ch[u] = ldg16_stream(base + (int64_t)(row + u * RPI) * rowb);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      float f[E];
      unpack16<T>(ch[u], f);
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] += (double)f[e];
    }
  }
  for (; row < hi; row += RPI) {
    float f[E];
    unpack16<T>(ldg16(base + (int64_t)row * rowb), f);
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] += (double)f[e];
  }
  // fixed-order reduction: row groups inside a wave by butterfly, then the 16 waves through LDS
  __shared__ double red[16 * 128];
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    double a = acc[e];
    for (int off = LPR; off < 64; off <<= 1) a += shfl_xor_f64(a, off);
    if (lane < LPR) red[wave * d + piece * E + e] = a;
  }
  __syncthreads();
  if (tid < d) {
    double s = 0.0;
    for (int w = 0; w < 16; ++w) s += red[w * d + tid];
    qpart[(((int64_t)b * gridDim.y + h) * gridDim.x + c) * d + tid] = s;
    if (direct) split_bf16x4(s, qsplit + ((int64_t)b * gridDim.y + h) * 4 * d + tid, d);
  }
}

// k_qsplit: grid (Hkv, B), d threads.  qbar_g = sum over the heads of group g and the chunks;
// qsplit[b,g,p,:] (p = 0..3) = successive bf16 roundings of what is left of it.
__global__ void k_qsplit(const double* __restrict__ qpart, uint16_t* __restrict__ qsplit, int H,
                         int Hkv, int nchunk, int d) {
  const int g = blockIdx.x, b = blockIdx.y, c = threadIdx.x;
  const int G = H / Hkv;
  // the partials of the group's heads and chunks lie one after the other (head-major): added in that
  // order, eight loads in flight
  const double* src = qpart + ((int64_t)b * H + g * G) * nchunk * d + c;
  const int n = G * nchunk;
  double s = 0.0;
  for (int i0 = 0; i0 < n; i0 += 8) {
    double part[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) part[u] = i0 + u < n ? src[(int64_t)(i0 + u) * d] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) s += part[u];
  }
  split_bf16x4(s, qsplit + ((int64_t)b * Hkv + g) * 4 * d + c, d);
}

// A lane's share of one contraction group (8 elements): one 16-byte chunk of bf16, two of f32.
template <typename T> struct group_bytes;
template <> struct group_bytes<bf16_t> { static constexpr int value = 16; };
template <> struct group_bytes<float> { static constexpr int value = 32; };

// Text rows that ride in the mass sweep (bf16 only).  Rows 4 .. 4 + R - 1 of the A tile of kv head g
// hold text row t = r % T_eff of query head g G + r / T_eff; their logits against every key go to
// zlog [B, H, T_eff, V].
struct RideArgs {
  const void* qt; Strides3 sq;      // [B,H,Tmax,d]
  const int32_t* text_len;          // [B]
  float* zlog;
  int H, G, T_eff, Tmax, last_only;
};

// ------------------------------------------------------------------------------------------
// k_mass_mfma: grid (ceil(V/32), B), 256 threads = 4 waves.  A workgroup owns one 32-key tile; wave w walks
// the kv heads w, w + 4, ...
// The four bf16 pieces of qbar_g are rows 0..3 of the MFMA A tile (rows 4..31 are zero, or text
// rows that ride along), the keys are the B tile, so lane n (< 32) finds the four partial dot
// products of key n in its first four accumulator registers.
// The tile of a head is an isolated piece of memory (8 KiB for bf16, d = 128), and reading such
// pieces in the operand pattern (32 rows x 32 bytes per instruction) was measured at 4.2 TB/s against
// 6.0 TB/s for whole rows.  So a wave reads whole rows (LPR consecutive lanes per row) and turns the
// tile into the operand layout through an LDS buffer of its own -- written and read by the same
// wave, in order, so no barrier is involved.  NG = contraction groups of 8 elements (d = 16 NG).
// Writes s64, s_raw and, with mm, the (min, max) of its keys to mm [B, ktiles, 2].
// ------------------------------------------------------------------------------------------
template <typename T, int NG, bool RIDE>
__global__ __launch_bounds__(256, (sizeof(T) == 4 ? 2 : RIDE ? 3 : 1)) void k_mass_mfma(const T* __restrict__ kv, Strides3 sk,
                                                    const uint16_t* __restrict__ qsplit, int Hkv, int V,
                                                    double scale, double* __restrict__ s64, float* __restrict__ s_raw,
                                                    double* __restrict__ mm, RideArgs ra) {
  constexpr int GB = group_bytes<T>::value;
  constexpr int RBY = NG * 2 * GB;                    // row bytes
  constexpr int LPR = RBY / 16, RPI = 64 / LPR;       // lanes per row, rows per load instruction
  constexpr int NL = 32 / RPI;                        // load instructions per tile
  constexpr int NC = GB / 16;                         // 16-byte chunks per group and lane
  constexpr bool F32 = GB == 32;
  static_assert(!RIDE || !F32, "text rows ride with bf16 keys only");
  // one register set for the key rows (reloaded as soon as it is staged) where a second would cost a
  // workgroup per compute unit: f32 rows, and the kernel that also carries text rows
  constexpr bool REUSE = F32 || RIDE;
  __shared__ __align__(16) char stage[4][32 * RBY];
  __shared__ double part[4][32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hf = lane >> 5;
  const int piece = lane % LPR, r0 = lane / LPR;
  const int b = blockIdx.y, j0 = blockIdx.x * 32, g_hi = Hkv;
  const int64_t headb = sk.h * (int64_t)sizeof(T);
  // LDS: the 16-byte piece p of row r sits in slot p ^ x(r): whole-row writes and operand reads of 16
  // consecutive rows both cover all banks
  auto swz = [](int row) { return LPR == 8 ? (row >> 1) & 7 : row & (LPR - 1); };
  char* st = stage[wave];
  uint32_t roff[NL];          // byte offsets inside one head of one image (< 2 GiB, checked on the host)
  int wr[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int row = r0 + RPI * i;
    roff[i] = (uint32_t)(min(j0 + row, V - 1) * (int)sk.r * (int)sizeof(T) + piece * 16);
    wr[i] = row * RBY + ((piece ^ swz(row)) << 4);
  }
  // operand read (c, u): piece NC (2c + hf) + u of row n
  int rd[NG][NC];
#pragma unroll
  for (int c = 0; c < NG; ++c)
#pragma unroll
    for (int u = 0; u < NC; ++u) rd[c][u] = n * RBY + (((NC * (2 * c + hf) + u) ^ swz(n)) << 4);
  const char* kbase = reinterpret_cast<const char*>(kv + b * sk.b);
  // lane (m, hf) with m < 4 supplies piece m of qbar_g, half hf of each group's components
  const char* qbase = reinterpret_cast<const char*>(qsplit + ((int64_t)b * Hkv * 4 + (n & 3)) * (NG * 16)) + hf * 16;
  const int64_t qheadb = (int64_t)4 * NG * 16 * 2;
  // text rows that ride: lane n in [4, 4 + R) supplies text row (n - 4) % T_eff of query head g G + (n - 4) / T_eff
  int ride_rows = 0, ride_head = 0;
  const char* tbase = nullptr;
  bool ride_src = false;
  if (RIDE) {
    ride_rows = ra.G * ra.T_eff;
    const int r = n - 4;
    if (r >= 0 && r < ride_rows) {
      const int len = min(max(ra.text_len[b], 0), ra.Tmax);
      const int t = r % ra.T_eff;
      ride_head = r / ra.T_eff;
      const int src = ra.last_only ? len - 1 : t;
      ride_src = ra.last_only ? len >= 1 : t < len;         // padding rows stay zero operands
      tbase = reinterpret_cast<const char*>(static_cast<const bf16_t*>(ra.qt) + b * ra.sq.b +
                                            (int64_t)max(src, 0) * ra.sq.r) + hf * 16;
    }
  }
  const int64_t theadb = RIDE ? ra.sq.h * 2 : 0;
  const bool has_q = n < 4;
  auto load_a = [&](uint4 (&qa)[NG], int g) {
    if (has_q) {
#pragma unroll
      for (int c = 0; c < NG; ++c) qa[c] = ldg16(qbase + g * qheadb + c * 32);
    } else if (RIDE && ride_src) {
      const char* tp = tbase + (int64_t)(g * ra.G + ride_head) * theadb;
#pragma unroll
      for (int c = 0; c < NG; ++c) qa[c] = ldg16(tp + c * 32);
    }
  };
  uint4 qa[NG], kb[NL], kn[NL];
#pragma unroll
  for (int c = 0; c < NG; ++c) qa[c] = make_uint4(0, 0, 0, 0);
  int g = wave;
  if (g < g_hi) {
#pragma unroll
    for (int i = 0; i < NL; ++i) kb[i] = ldg16(kbase + g * headb + roff[i]);
    load_a(qa, g);
  }
  double sum = 0.0;
  for (; g < g_hi; g += 4) {
    const int gn = g + 4;
    if (!REUSE && gn < g_hi) {
#pragma unroll
      for (int i = 0; i < NL; ++i) kn[i] = ldg16(kbase + gn * headb + roff[i]);
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<uint4*>(st + wr[i]) = kb[i];
    wave_lds_order();
    if (REUSE && gn < g_hi) {    // the next head's rows reuse this head's registers once those are staged
#pragma unroll
      for (int i = 0; i < NL; ++i) kb[i] = ldg16(kbase + gn * headb + roff[i]);
    }
    if constexpr (!F32) {
      f32x16_t acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
      for (int c = 0; c < NG; ++c) mma32<bf16_t>(acc, qa[c], *reinterpret_cast<const uint4*>(st + rd[c][0]));
      sum += ((double)acc[0] + (double)acc[1]) + ((double)acc[2] + (double)acc[3]);   // rows 0..3 (lanes < 32)
      if (RIDE) {
        // wave-uniform base + 32-bit lane offset: row r of this head group's [G T_eff, V] block, key j0 + n
        float* zl = ra.zlog + ((int64_t)(b * ra.H + g * ra.G) * ra.T_eff) * V;
        const uint32_t lane_off = (uint32_t)((4 * hf - 4) * V + j0 + n);      // wraps for hf = 0; the sums below do not
        if (j0 + n < V) {
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int r = 8 * (v >> 2) + 4 * hf + (v & 3) - 4;
            if (r >= 0 && r < ride_rows) zl[lane_off + (uint32_t)((8 * (v >> 2) + (v & 3)) * V)] = acc[v];
          }
        }
      }
    } else {
      // key pieces as three B tiles; the accumulators of the three are added in fp64
      f32x16_t ah, am, al;
#pragma unroll
      for (int v = 0; v < 16; ++v) { ah[v] = 0.0f; am[v] = 0.0f; al[v] = 0.0f; }
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        const Split3 k3 = split_f32x8(*reinterpret_cast<const uint4*>(st + rd[c][0]),
                                      *reinterpret_cast<const uint4*>(st + rd[c][NC - 1]));
        mma32<bf16_t>(al, qa[c], k3.lo);
        mma32<bf16_t>(am, qa[c], k3.mid);
        mma32<bf16_t>(ah, qa[c], k3.hi);
      }
      const double l = ((double)al[0] + (double)al[1]) + ((double)al[2] + (double)al[3]);
      const double m = ((double)am[0] + (double)am[1]) + ((double)am[2] + (double)am[3]);
      const double h = ((double)ah[0] + (double)ah[1]) + ((double)ah[2] + (double)ah[3]);
      sum += (l + m) + h;
    }
    if (gn < g_hi) {
      load_a(qa, gn);      // small, cached: not worth registers of its own
      if (!REUSE) {
#pragma unroll
        for (int i = 0; i < NL; ++i) kb[i] = kn[i];
      }
    }
    wave_lds_order();
  }
  if (hf == 0) part[wave][n] = sum;
  __syncthreads();
  if (tid >= 32) return;
  double smin = INFINITY, smax = -INFINITY;
  const int j = j0 + n;
  if (j < V) {
    const double s = (((part[0][n] + part[1][n]) + part[2][n]) + part[3][n]) * scale;
    s64[(int64_t)b * V + j] = s;
    s_raw[(int64_t)b * V + j] = (float)s;
    smin = smax = s;
  }
  if (mm != nullptr) {
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) {
      smin = nan_min(smin, shfl_xor_f64(smin, off));
      smax = nan_max(smax, shfl_xor_f64(smax, off));
    }
    if (tid == 0) reinterpret_cast<double2*>(mm)[(int64_t)b * gridDim.x + blockIdx.x] = make_double2(smin, smax);
  }
}

// ------------------------------------------------------------------------------------------
// The mass sweep of a small batch (fewer than 256 tiles of 32 keys), where not bytes count but the length of the
// chain from the first load to the last sum: workgroups of a wave per kv head (up to 16), wave w with the heads w,
// w + NW, ..., and qbar added up by every wave for its heads from the partial sums of k_qsum, in k_qsplit's order.
//   1 x 32 heads x 2304 tokens: k_qsplit 3.3 us, heads cut into 8 groups of workgroups 6.1, their sums and (min, max) in
//   a launch of one workgroup 5.4: 14.8 us; now 8.1.  1 x 32 x 576 in f32: 2.7 + 6.0 + 3.9, now 6.9.
// ------------------------------------------------------------------------------------------
constexpr int MASS_SMALL_NW = 16;

// qbar of kv head bg = b Hkv + g: lane l gets components PL l .. PL l + PL - 1 (PL = D / 64) of the sum of the np partial
// sums of its query heads, which lie one after the other (head-major); FLY loads in flight: as many as leave a kernel of
// 16 waves at 112 registers, beside which two workgroups of k_compact_fixed still fit a compute unit.  (At 114 and 124 the
// sweep waited for the copy: 7 x 16 heads x 448 tokens in f32, 16 layers, 154 us per stage, now 137;  8 x 32 x 576 319, now
// 300;  15 x 32 x 512 in bf16 with 2 rows that ride 226, now 215.)
template <int D, int FLY> struct FoldedQuery {
  static constexpr int PL = D / 64;
  double q[PL];
  __device__ __forceinline__ FoldedQuery(const double* __restrict__ qpart, int bg, int np, int lane) {
    const double* src = qpart + (int64_t)bg * np * D + lane * PL;
#pragma unroll
    for (int e = 0; e < PL; ++e) q[e] = 0.0;
    for (int i0 = 0; i0 < np; i0 += FLY) {
      double x[FLY][PL];
#pragma unroll
      for (int u = 0; u < FLY; ++u)
#pragma unroll
        for (int e = 0; e < PL; ++e) x[u][e] = i0 + u < np ? src[(int64_t)(i0 + u) * D + e] : 0.0;
#pragma unroll
      for (int u = 0; u < FLY; ++u)
#pragma unroll
        for (int e = 0; e < PL; ++e) q[e] += x[u][e];
    }
  }
};

// The end of both kernels: part[w][i] = wave w's sum for key i of the tile of KT keys; adds them in wave order and
// leaves s64, s_raw and, with mm, the tile's (min, max).
template <int KT>
__device__ __forceinline__ void mass_tile_end(const double (*part)[KT], int NW, int b, int V, double scale,
                                              double* __restrict__ s64, float* __restrict__ s_raw,
                                              double* __restrict__ mm) {
  __syncthreads();
  const int n = threadIdx.x, j = blockIdx.x * KT + n;
  if (n >= KT) return;
  double smin = INFINITY, smax = -INFINITY;
  if (j < V) {
    double s = part[0][n];
    for (int w = 1; w < NW; ++w) s += part[w][n];
    s *= scale;
    s64[(int64_t)b * V + j] = s;
    s_raw[(int64_t)b * V + j] = (float)s;
    smin = smax = s;
  }
#pragma unroll
  for (int off = KT / 2; off >= 1; off >>= 1) {
    smin = nan_min(smin, shfl_xor_f64(smin, off));
    smax = nan_max(smax, shfl_xor_f64(smax, off));
  }
  if (n == 0 && mm != nullptr) reinterpret_cast<double2*>(mm)[(int64_t)b * gridDim.x + blockIdx.x] = make_double2(smin, smax);
}

// k_mass_small: grid (ceil(V/KT), B), 64 NW threads.  Products and sums in fp64 on the vector ALUs: a lane keeps the 16-byte
// piece l % LPR of its head's qbar and of RPI rows per load instruction, and the lanes of a row meet once, after
// the last head.  (As bf16 pieces on the matrix cores the cutting alone took 8 us for 576 keys in f32, on 36 CUs.)
template <typename T, int D, int KT>
__global__ __launch_bounds__(64 * MASS_SMALL_NW) void k_mass_small(const T* __restrict__ kv, Strides3 sk,
                                                                    const double* __restrict__ qpart, int Hkv, int np,
                                                                    int V, double scale, double* __restrict__ s64,
                                                                    float* __restrict__ s_raw, double* __restrict__ mm) {
  constexpr int E = elem<T>::per16, LPR = D / E, RPI = 64 / LPR, NI = KT / RPI;
  static_assert(NI >= 1, "at least one load instruction");
  __shared__ __align__(16) double qs[MASS_SMALL_NW][D];        // each row written and read by one wave, in order
  __shared__ double part[MASS_SMALL_NW][KT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, NW = blockDim.x >> 6;
  const int piece = lane % LPR, r0 = lane / LPR, b = blockIdx.y, j0 = blockIdx.x * KT;
  const char* base = reinterpret_cast<const char*>(kv + b * sk.b) + piece * 16;
  const int64_t headb = sk.h * (int64_t)sizeof(T);
  uint32_t roff[NI];          // byte offsets inside one head of one image (< 2 GiB, checked on the host)
  double acc[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    roff[i] = (uint32_t)(min(j0 + r0 + RPI * i, V - 1) * (int)sk.r * (int)sizeof(T));
    acc[i] = 0.0;
  }
  for (int g = wave; g < Hkv; g += NW) {
    uint4 kb[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) kb[i] = ldg16(base + g * headb + roff[i]);
    const FoldedQuery<D, sizeof(T) == 4 && KT == 16 ? 7 : 8> f(qpart, b * Hkv + g, np, lane);
#pragma unroll
    for (int e = 0; e < f.PL; ++e) qs[wave][lane * f.PL + e] = f.q[e];
    wave_lds_order();
    double q[E];
#pragma unroll
    for (int e = 0; e < E; ++e) q[e] = qs[wave][piece * E + e];
    wave_lds_order();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float x[E];
      unpack16<T>(kb[i], x);
#pragma unroll
      for (int e = 0; e < E; ++e) acc[i] = fma(q[e], (double)x[e], acc[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
#pragma unroll
    for (int off = LPR / 2; off >= 1; off >>= 1) acc[i] += shfl_xor_f64(acc[i], off);
    if (piece == 0) part[wave][r0 + RPI * i] = acc[i];
  }
  mass_tile_end<KT>(part, NW, b, V, scale, s64, s_raw, mm);
}

// k_mass_small_ride (bf16): the same with text rows that ride along (see k_mass_mfma), on the matrix cores.  Tiles of
// 16 x 16: the four pieces of qbar are rows 0 .. 3 of two tiles of query rows, rows 4 .. 31 text rows; the operands come
// straight from memory, two sectors of 64 bytes of 16 rows per instruction.
// (FLY: see FoldedQuery; 5 for workgroups of many waves.  Up to 8 heads fit beside the copy as they are, and have more
// partial sums each: 8 heads on 2, 1 x 4096 tokens, 73.9 us per stage with 5, 72.6 with 8.)
template <int NG, int FLY>
__global__ __launch_bounds__(64 * MASS_SMALL_NW) void k_mass_small_ride(const bf16_t* __restrict__ kv, Strides3 sk,
                                                                         const double* __restrict__ qpart, int Hkv,
                                                                         int np, int V, double scale,
                                                                         double* __restrict__ s64,
                                                                         float* __restrict__ s_raw,
                                                                         double* __restrict__ mm, RideArgs ra) {
  constexpr int D = 16 * NG, NC = D / 32, KT = 16;   // contraction steps of 32 components, keys of a tile
  __shared__ __align__(16) uint16_t pieces[MASS_SMALL_NW][4 * D];
  __shared__ double part[MASS_SMALL_NW][KT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, NW = blockDim.x >> 6;
  const int n = lane & 15, q4 = lane >> 4;
  const int b = blockIdx.y, j0 = blockIdx.x * KT;
  const char* krow = reinterpret_cast<const char*>(kv + b * sk.b) + (int64_t)min(j0 + n, V - 1) * sk.r * 2 + q4 * 16;
  const int64_t headb = sk.h * 2;
  // lane n supplies row 16 a + n of tile a: row 4 + r is text row r (t = r % T_eff of query head g G + r / T_eff)
  const char* tbase[2];
  const int ride_rows = ra.G * ra.T_eff, len = min(max(ra.text_len[b], 0), ra.Tmax);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int r = 16 * a + n - 4, t = r % ra.T_eff, src = ra.last_only ? len - 1 : t;
    const bool here = r >= 0 && r < ride_rows && (ra.last_only ? len >= 1 : t < len);   // padding rows: zero operands
    tbase[a] = here ? reinterpret_cast<const char*>(static_cast<const bf16_t*>(ra.qt) + b * ra.sq.b +
                                                    (int64_t)(r / ra.T_eff) * ra.sq.h + (int64_t)src * ra.sq.r) + q4 * 16
                    : nullptr;
  }
  double sum = 0.0;
  for (int g = wave; g < Hkv; g += NW) {
    uint4 kb[NC], qa[2][NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) kb[c] = ldg16(krow + g * headb + c * 64);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        qa[a][c] = tbase[a] != nullptr ? ldg16(tbase[a] + (int64_t)g * ra.G * ra.sq.h * 2 + c * 64) : make_uint4(0, 0, 0, 0);
    const FoldedQuery<D, FLY> f(qpart, b * Hkv + g, np, lane);
    uint16_t* pw = pieces[wave];                // written and read by this wave alone, in order
#pragma unroll
    for (int e = 0; e < f.PL; ++e) split_bf16x4(f.q[e], pw + lane * f.PL + e, D);
    wave_lds_order();
    if (n < 4) {
#pragma unroll
      for (int c = 0; c < NC; ++c) qa[0][c] = *reinterpret_cast<const uint4*>(pw + n * D + c * 32 + q4 * 8);
    }
    wave_lds_order();
    f32x4_t acc[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      acc[a] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c = 0; c < NC; ++c) mma16(acc[a], qa[a][c], kb[c]);
    }
    // rows 0 .. 3 of a tile lie in the first 16 lanes
    sum += ((double)acc[0][0] + (double)acc[0][1]) + ((double)acc[0][2] + (double)acc[0][3]);
    if (j0 + n < V) {
      float* zl = ra.zlog + ((int64_t)(b * ra.H + g * ra.G) * ra.T_eff) * V + j0 + n;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * a + 4 * q4 + v - 4;
          if (r >= 0 && r < ride_rows) zl[(int64_t)r * V] = acc[a][v];
        }
    }
  }
  if (q4 == 0) part[wave][n] = sum;
  mass_tile_end<KT>(part, NW, b, V, scale, s64, s_raw, mm);
}

// k_mass_finish: grid (B), 1024 threads: the image's (min, max) to mm [B, 1, 2].
__global__ __launch_bounds__(1024) void k_mass_finish(const double* __restrict__ s64, int V, double* __restrict__ mm) {
  __shared__ double wave_mm[16][2];
  const int b = blockIdx.x, tid = threadIdx.x;
  double smin = INFINITY, smax = -INFINITY;
  for (int j = tid; j < V; j += 1024) {
    const double s = s64[(int64_t)b * V + j];
    smin = nan_min(smin, s);
    smax = nan_max(smax, s);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    smin = nan_min(smin, shfl_xor_f64(smin, off));
    smax = nan_max(smax, shfl_xor_f64(smax, off));
  }
  if ((tid & 63) == 0) { wave_mm[tid >> 6][0] = smin; wave_mm[tid >> 6][1] = smax; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 16; ++w) { smin = nan_min(smin, wave_mm[w][0]); smax = nan_max(smax, wave_mm[w][1]); }
    reinterpret_cast<double2*>(mm)[b] = make_double2(smin, smax);
  }
}

// ------------------------------------------------------------------------------------------
// Text-row attention sweeps.  grid (H * RP * S, B), 256 threads = 4 waves; blockIdx.x = h + H (rp + RP sp).
//   A workgroup takes one (image, head), one pair rp of 32-row blocks of text queries (64 rows; RP
//   pairs cover Tmax) and one key-range split sp.  Two row blocks per workgroup keep its registers and
//   LDS small enough for two workgroups per compute unit, whose waves fill each other's gaps (one
//   wave's exponentials and operand splitting under the other's matrix instructions); longer text
//   costs another workgroup per 64 rows, which reads the keys again -- the pairs of one head are
//   32 ids apart in the launch order, so they run close in time on the same XCD and the second finds
//   the keys in its L2 -- and an image whose own text ends before a pair starts pays nothing for it
//   (the workgroup leaves at once).  The body is compiled for one and for two row blocks and picked by
//   the image's own text length.
//   NG = contraction groups of 8 elements (d = 16 NG).  bf16 queries stay in registers as MFMA
//   operands; f32 queries are split into bf16 pieces once and read from LDS.
// Every wave streams its own 32-key tiles of the split's key range straight from global memory:
// lane (n, hf) of a tile reads, for group c, the bytes [GB (2c + hf), + GB) of key n (GB = 16 for
// bf16, 32 for f32) -- the two lanes of a key take contiguous bytes, which halves the cache lines a
// load instruction touches -- and the query side holds the same elements of its row.
// ------------------------------------------------------------------------------------------
struct AttnArgs {
  const void* qt; Strides3 sq;          // [B,H,Tmax,d]
  const void* kv; Strides3 sk;          // [B,Hkv,V,d]
  const double* s64;                    // [B,V]
  const double* mm; int mm_n;           // [B,mm_n,2] (min, max) pairs of s (MassRange)
  const int32_t* text_len;              // [B]
  const float* lse_extra;               // [B,H,Tmax] or null
  float* pstat;                         // [B,H,S,2,NR]   partial (max, sum) per text row, NR = 64 RP
  float* upart;                         // [B,H,RP,V]     column sums per head and row pair
  float* zlog;                          // [B,H,T_eff,V]  stored logits (k_rowstats_logits / k_colsum_logits / k_colsum_rows)
  int H, Hkv, V, Tmax, S, RP, tiles_per_split;
  int T_eff, last_only;                 // rows that rank: all valid text rows, or the last one alone
  float c2;                             // log2(e) / sqrt(d): accumulator units -> log2 units
  double lambda_max, eps;
  int mask_on;
};

// first text row that ranks and how many do, for image b
__device__ __forceinline__ void ranking_rows(const AttnArgs& a, int b, int& row0, int& nrows) {
  const int len = min(max(a.text_len[b], 0), a.Tmax);
  row0 = a.last_only ? max(len - 1, 0) : 0;
  nrows = a.last_only ? min(len, 1) : len;
}

// Query operands: registers (bf16) or LDS (f32, as pieces).  Operand row m is text row row0 + m; rows
// at or past nrows (padding of a ragged batch, whatever it holds) are zero operands.
template <typename T, int NRB, int NG> struct QueryOps;
template <int NRB, int NG> struct QueryOps<bf16_t, NRB, NG> {
  uint4 qa[NRB][NG];
  __device__ __forceinline__ void init(const AttnArgs& a, int b, int h, int lane, char*, int row0, int nrows) {
    const int m = lane & 31, hf = lane >> 5;
    const char* qbase = reinterpret_cast<const char*>(static_cast<const bf16_t*>(a.qt) + b * a.sq.b + h * a.sq.h +
                                                      (int64_t)row0 * a.sq.r) + hf * 16;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      const int row = rb * 32 + m;
#pragma unroll
      for (int c = 0; c < NG; ++c)
        qa[rb][c] = row < nrows ? ldg16(qbase + (int64_t)row * a.sq.r * 2 + c * 32) : make_uint4(0, 0, 0, 0);
    }
  }
  __device__ __forceinline__ uint4 get(int rb, int c) const { return qa[rb][c]; }
};
// f32 queries: three bf16 planes in LDS, split once per workgroup
template <int NRB, int NG> struct QueryOps<float, NRB, NG> {
  static constexpr int ROWB = NG * 32, LDSROW = ROWB + 16, PLANE = NRB * 32 * LDSROW;
  const char* base;     // the workgroup's LDS
  int qoff;             // this lane's operand row and half, as a byte offset
  __device__ __forceinline__ void init(const AttnArgs& a, int b, int h, int lane, char* lds, int row0, int nrows) {
    const char* qbase = reinterpret_cast<const char*>(static_cast<const float*>(a.qt) + b * a.sq.b + h * a.sq.h +
                                                      (int64_t)row0 * a.sq.r);
    constexpr int PPR = ROWB / 16;         // groups of 8 elements per row
#pragma unroll
    for (int i = threadIdx.x; i < NRB * 32 * PPR; i += 256) {
      int row = i / PPR, pc = i % PPR;
      Split3 s;
      s.hi = s.mid = s.lo = make_uint4(0, 0, 0, 0);
      if (row < nrows) {
        const char* p = qbase + (int64_t)row * a.sq.r * 4 + pc * 32;
        s = split_f32x8(ldg16(p), ldg16(p + 16));
      }
      char* dst = lds + row * LDSROW + pc * 16;
      *reinterpret_cast<uint4*>(dst) = s.hi;
      *reinterpret_cast<uint4*>(dst + PLANE) = s.mid;
      *reinterpret_cast<uint4*>(dst + 2 * PLANE) = s.lo;
    }
    __syncthreads();
    base = lds;
    qoff = (lane & 31) * LDSROW + (lane >> 5) * 16;
  }
  // Called once per key tile: the operands are the same for every tile, and a compiler that knew it
  // would keep all of them (12 NG NRB registers) alive across the sweep.  Only the offset is hidden
  // from it, so that the reads stay LDS reads.
  __device__ __forceinline__ void per_tile() { asm volatile("" : "+v"(qoff)); }
  __device__ __forceinline__ Split3 get3(int rb, int c) const {
    const char* p = base + qoff + rb * 32 * LDSROW + c * 32;
    Split3 s;
    s.hi = *reinterpret_cast<const uint4*>(p);
    s.mid = *reinterpret_cast<const uint4*>(p + PLANE);
    s.lo = *reinterpret_cast<const uint4*>(p + 2 * PLANE);
    return s;
  }
};
// LDS of a sweep workgroup: the f32 query pieces (two row blocks at most), then 8 x 64 floats of statistics
template <typename T, int NG> constexpr size_t query_lds_bytes() {
  return sizeof(T) == 4 ? (size_t)64 * (NG * 32 + 16) * 3 : 0;
}
constexpr int ATT_ROWS = 64;       // text rows per workgroup

// A lane's share of a 32-key tile.  bf16: the chunks are the operands.  f32: the raw chunks are split
// into pieces group by group, and a group's registers take the next tile's chunks as soon as it is split.
template <typename T, int NG> struct KeyTile;
template <int NG> struct KeyTile<bf16_t, NG> {
  uint4 op[NG];
  __device__ __forceinline__ void load(const char* krow) {
#pragma unroll
    for (int c = 0; c < NG; ++c) op[c] = ldg16(krow + c * 32);
  }
};
template <int NG> struct KeyTile<float, NG> {
  uint4 raw[2 * NG];
  __device__ __forceinline__ void load(const char* krow) {
#pragma unroll
    for (int c = 0; c < NG; ++c) load_group(krow, c);
  }
  __device__ __forceinline__ void load_group(const char* krow, int c) {
    raw[2 * c] = ldg16(krow + c * 64);
    raw[2 * c + 1] = ldg16(krow + c * 64 + 16);
  }
};

__device__ __forceinline__ float discount_of(const AttnArgs& a, double s, double lo, double inv) {
  if (!a.mask_on) return 1.0f;
  return (float)fmax(a.lambda_max * ((s - lo) * inv), a.eps);
}
__device__ __forceinline__ float discount(const AttnArgs& a, int b, int j, double lo, double inv) {
  return discount_of(a, a.mask_on ? a.s64[(int64_t)b * a.V + j] : 0.0, lo, inv);
}

// merge of two (max, sum) pairs kept in accumulator units with scale c2
__device__ __forceinline__ void merge_stat(float& m, float& s, float m2, float s2, float c2) {
  float M = fmaxf(m, m2);
  s = s * fast_exp2((m - M) * c2) + s2 * fast_exp2((m2 - M) * c2);
  m = M;
}

constexpr float ATT_NEG = -1e30f;

// the value of another lane of the row of 16 lanes (rotations inside the row)
template <int CTRL> __device__ __forceinline__ float dpp_f32(float x) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}

// Sums of c[0..3] over the four groups of 16 lanes: group q gets that of c[q] (v_permlane32_swap exchanges the
// upper half of the first operand with the lower half of the second, v_permlane16_swap the odd groups of
// the first with the even groups of the second).
__device__ __forceinline__ float sum_groups_of_16(const float (&c)[4]) {
  auto swap32 = [](float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  const float lo = swap32(c[0], c[2]), hi = swap32(c[1], c[3]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// online (max, sum) update of one row block from the 16 logits a lane holds
__device__ __forceinline__ void stats_update(f32x16_t& acc, const float (&lam)[16], bool ragged, int tile, int hf, int V,
                                             float c2, float& m_run, float& s_run) {
  if (ragged) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (tile * 32 + 8 * (v >> 2) + 4 * hf + (v & 3) >= V) acc[v] = ATT_NEG;
  }
  float mx = acc[0];
#pragma unroll
  for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc[v]);
  mx = fmaxf(mx, __shfl_xor(mx, 32));                  // both halves of the row's 32 keys
  const float m_new = fmaxf(m_run, mx);
  float s = s_run * fast_exp2((m_run - m_new) * c2);
  const float off = -m_new * c2;
#pragma unroll
  for (int v = 0; v < 16; ++v) s = fmaf(lam[v], fast_exp2(fmaf(acc[v], c2, off)), s);
  s_run = s;
  m_run = m_new;
}

// (head, row pair, key split) of a sweep workgroup
struct SweepId { int h, rp, sp, b; };
__device__ __forceinline__ SweepId sweep_id(const AttnArgs& a) {
  SweepId w;
  w.h = blockIdx.x % a.H;
  const int rest = blockIdx.x / a.H;
  w.rp = rest % a.RP;
  w.sp = rest / a.RP;
  w.b = blockIdx.y;
  return w;
}

// Keys are the tile rows here: lane (n, hf) owns text row row0 + rb*32 + n and finds, in accumulator
// register v, its logit against key 8*(v/4) + 4*hf + v%4 of the tile.
// STORE: the logits of the ranking rows are also left in zlog (row t of an image's ranking rows,
// accumulator units), so that the column sums need no second sweep over the keys.
template <typename T, int NRB, int NG, bool STORE>
__device__ __forceinline__ void attn_stats_body(const AttnArgs& a, char* lds, const SweepId& w, int row0, int nrows) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int GB = group_bytes<T>::value;
  using Q = QueryOps<T, NRB, NG>;
  float* st_m = reinterpret_cast<float*>(lds + query_lds_bytes<T, NG>());   // [4][64]
  float* st_s = st_m + 4 * ATT_ROWS;                                         // [4][64]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, hf = lane >> 5;
  const int sp = w.sp, h = w.h, b = w.b;
  const int g = (h * a.Hkv) / a.H;
  const char* kbase = reinterpret_cast<const char*>(static_cast<const T*>(a.kv) + b * a.sk.b + g * a.sk.h) +
                      hf * GB;
  const int64_t krow_bytes = a.sk.r * (int64_t)sizeof(T);
  const int ntiles = (a.V + 31) >> 5;
  const int t_end = min(ntiles, (sp + 1) * a.tiles_per_split);
  const float c2 = a.c2;
  // the first key tile and its masses are asked for before the queries, so that the waits overlap
  MassRange range;
  range.load(a.mm, a.mm_n, b);
  KeyTile<T, NG> kb;
  int tile = sp * a.tiles_per_split + wave;
  if (tile < t_end) kb.load(kbase + (int64_t)min(tile * 32 + n, a.V - 1) * krow_bytes);
  const double* s64 = a.s64 + (int64_t)b * a.V;
  double sj = (a.mask_on && tile < t_end) ? s64[min(tile * 32 + n, a.V - 1)] : 0.0;
  Q q;
  q.init(a, b, h, lane, lds, row0, nrows);
  double mlo, mhi;
  range.reduce(mlo, mhi);
  const double minv = 1.0 / (mhi - mlo + a.eps);

  float m_run[NRB], s_run[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) { m_run[rb] = ATT_NEG; s_run[rb] = 0.0f; }
  // where this lane's text rows start in zlog, at the lane's first key of a tile
  float* zrow[NRB];
  const bool zvec = (a.V & 3) == 0;            // rows of zlog start on 16-byte boundaries
  if constexpr (STORE) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
      zrow[rb] = rb * 32 + n < nrows
                     ? a.zlog + (((int64_t)b * a.H + h) * a.T_eff + w.rp * ATT_ROWS + rb * 32 + n) * a.V + 4 * hf
                     : nullptr;
  }
  auto store_logits = [&](const f32x16_t& acc, int rb, int tile, bool ragged) {
    if (zrow[rb] == nullptr) return;
    float* z = zrow[rb] + tile * 32;
    if (zvec && !ragged) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(z + 8 * q) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int o = 8 * (v >> 2) + (v & 3);
        if (tile * 32 + 4 * hf + o < a.V) z[o] = acc[v];
      }
    }
  };

  for (; tile < t_end; tile += 4) {
    const int j = tile * 32 + n;
    const int tnext = tile + 4;
    const char* knext = kbase + (int64_t)min(tnext * 32 + n, a.V - 1) * krow_bytes;
    KeyTile<T, F32 ? 1 : NG> kn;      // bf16: next key tile prefetched into a second register set, first thing
    if constexpr (!F32) {
      if (tnext < t_end) kn.load(knext);
    }
    // discount of key n of the tile (its mass was asked for a tile ago), then handed to the lanes in
    // accumulator order
    const float lj = j < a.V ? discount_of(a, sj, mlo, minv) : 0.0f;
    if (a.mask_on && tnext < t_end) sj = s64[min(tnext * 32 + n, a.V - 1)];
    float lam[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) lam[v] = __shfl(lj, 8 * (v >> 2) + 4 * hf + (v & 3));
    const bool ragged = tile * 32 + 32 > a.V;
    if constexpr (!F32) {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        f32x16_t acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
        for (int c = 0; c < NG; ++c) mma32<bf16_t>(acc, kb.op[c], q.get(rb, c));
        if constexpr (STORE) store_logits(acc, rb, tile, ragged);
        stats_update(acc, lam, ragged, tile, hf, a.V, c2, m_run[rb], s_run[rb]);
      }
      if (tnext < t_end) {
#pragma unroll
        for (int c = 0; c < NG; ++c) kb.op[c] = kn.op[c];
      }
    } else {
      // group by group: a key group is split once and meets both row blocks, whose accumulators stay
      // alive across the groups; its registers then take the same group of the next tile
      q.per_tile();
      f32x16_t acc[NRB];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[rb][v] = 0.0f;
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        const Split3 ks = split_f32x8(kb.raw[2 * c], kb.raw[2 * c + 1]);
        if (tnext < t_end) kb.load_group(knext, c);
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) mma_split(acc[rb], ks, q.get3(rb, c));
      }
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        if constexpr (STORE) store_logits(acc[rb], rb, tile, ragged);
        stats_update(acc[rb], lam, ragged, tile, hf, a.V, c2, m_run[rb], s_run[rb]);
      }
    }
  }
  // the two halves of a wave share the row maximum: their sums just add; then the 4 waves
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    float s = s_run[rb] + __shfl_xor(s_run[rb], 32);
    if (hf == 0) {
      st_m[wave * ATT_ROWS + rb * 32 + n] = m_run[rb];
      st_s[wave * ATT_ROWS + rb * 32 + n] = s;
    }
  }
  __syncthreads();
  if (tid < NRB * 32) {
    float m = st_m[tid], s = st_s[tid];
    for (int wv = 1; wv < 4; ++wv) merge_stat(m, s, st_m[wv * ATT_ROWS + tid], st_s[wv * ATT_ROWS + tid], c2);
    const int NR = ATT_ROWS * a.RP;
    float* out = a.pstat + ((((int64_t)b * a.H + h) * a.S + sp) * 2) * NR + w.rp * ATT_ROWS;
    out[tid] = m;
    out[NR + tid] = s;
  }
}

template <typename T, int NG, bool STORE>
__global__ __launch_bounds__(256, 2) void k_attn_stats(AttnArgs a) {
  extern __shared__ __align__(16) char lds[];
  const SweepId w = sweep_id(a);
  int row0, nrows;
  ranking_rows(a, w.b, row0, nrows);
  row0 += w.rp * ATT_ROWS;
  nrows = min(nrows - w.rp * ATT_ROWS, ATT_ROWS);
  if (nrows <= 0) return;                      // the image's text ends before this pair of row blocks
  if (nrows <= 32) attn_stats_body<T, 1, NG, STORE>(a, lds, w, row0, nrows);
  else attn_stats_body<T, 2, NG, STORE>(a, lds, w, row0, nrows);
}

// Row statistics merged over the splits, with the rest of the row (lse_extra) folded in: per text
// row -max (log2 units) and 1 / denominator; rows that do not rank get (-inf, 0) so that they add
// nothing.  Threads tid < n_local of the workgroup handle rows first + tid of the NR-row layout;
// row0 = the text row of local row 0; fin_o / fin_i in LDS.
__device__ __forceinline__ void final_row_stats(const AttnArgs& a, int b, int h, int NR, int first, int n_local,
                                                int row0, int nrows, float* fin_o, float* fin_i) {
  const int tid = threadIdx.x;
  if (tid < n_local) {
    const bool row_ok = tid < nrows;
    float o = -INFINITY, iv = 0.0f;        // 2^(z - inf) = 0: rows that do not rank add nothing
    if (row_ok) {
      const float* ps = a.pstat + (((int64_t)b * a.H + h) * a.S * 2) * NR + first;
      float m = ps[tid], s = ps[NR + tid];
      for (int w0 = 1; w0 < a.S; w0 += 4) {     // four splits' loads in flight
        float mw[4], sw[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float* pw = ps + min(w0 + u, a.S - 1) * 2 * NR + tid;
          mw[u] = pw[0];
          sw[u] = pw[NR];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (w0 + u < a.S) merge_stat(m, s, mw[u], sw[u], a.c2);
      }
      float m2 = m * a.c2;                                           // log2 units from here on
      if (a.lse_extra != nullptr) {
        float l2 = a.lse_extra[((int64_t)b * a.H + h) * a.Tmax + row0 + tid] * 1.4426950408889634f;
        float M = fmaxf(m2, l2);
        s = s * fast_exp2(m2 - M) + fast_exp2(l2 - M);
        m2 = M;
      }
      o = -m2;
      iv = 1.0f / s;
    }
    fin_o[tid] = o;
    fin_i[tid] = iv;
  }
}

// Queries are the tile rows here: lane (n, hf) owns key n of the tile and finds, in accumulator
// register v of row block rb, its logit against text row row0 + rb*32 + 8*(v/4) + 4*hf + v%4.
template <typename T, int NRB, int NG>
__device__ __forceinline__ void attn_colsum_body(const AttnArgs& a, char* lds, const SweepId& w, int row0, int nrows) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int GB = group_bytes<T>::value;
  using Q = QueryOps<T, NRB, NG>;
  float* fin_o = reinterpret_cast<float*>(lds + query_lds_bytes<T, NG>());   // [64]  -max * c2
  float* fin_i = fin_o + ATT_ROWS;                                            // [64]  1 / denominator
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, hf = lane >> 5;
  const int sp = w.sp, h = w.h, b = w.b;
  const int g = (h * a.Hkv) / a.H;
  const float c2 = a.c2;
  const char* kbase = reinterpret_cast<const char*>(static_cast<const T*>(a.kv) + b * a.sk.b + g * a.sk.h) +
                      hf * GB;
  const int64_t krow_bytes = a.sk.r * (int64_t)sizeof(T);
  const int ntiles = (a.V + 31) >> 5;
  const int t_end = min(ntiles, (sp + 1) * a.tiles_per_split);
  // the first key tile is asked for before the statistics and the queries, so that the waits overlap
  KeyTile<T, NG> kb;
  int tile = sp * a.tiles_per_split + wave;
  if (tile < t_end) kb.load(kbase + (int64_t)min(tile * 32 + n, a.V - 1) * krow_bytes);
  final_row_stats(a, b, h, ATT_ROWS * a.RP, w.rp * ATT_ROWS, NRB * 32, row0, nrows, fin_o, fin_i);
  Q q;
  q.init(a, b, h, lane, lds, row0, nrows);
  __syncthreads();
  // bf16: the row statistics of the 16 rows a lane meets stay in registers; f32 (whose registers go to
  // the key pieces and to the accumulators) reads them from LDS after the products
  constexpr int NST = F32 ? 1 : NRB;
  float off[NST][16], inv[NST][16];
  if constexpr (!F32) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        int row = rb * 32 + mma32_row(v, lane);
        off[rb][v] = fin_o[row];
        inv[rb][v] = fin_i[row];
      }
  }
  float* out = a.upart + (((int64_t)b * a.H + h) * a.RP + w.rp) * a.V;
  for (; tile < t_end; tile += 4) {
    const int j = tile * 32 + n;
    const int tnext = tile + 4;
    const char* knext = kbase + (int64_t)min(tnext * 32 + n, a.V - 1) * krow_bytes;
    float u = 0.0f;
    if constexpr (!F32) {
      KeyTile<T, NG> kn;
      if (tnext < t_end) kn.load(knext);
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        f32x16_t acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
        for (int c = 0; c < NG; ++c) mma32<bf16_t>(acc, q.get(rb, c), kb.op[c]);
#pragma unroll
        for (int v = 0; v < 16; ++v) u = fmaf(fast_exp2(fmaf(acc[v], c2, off[rb][v])), inv[rb][v], u);
      }
      if (tnext < t_end) {
#pragma unroll
        for (int c = 0; c < NG; ++c) kb.op[c] = kn.op[c];
      }
    } else {
      q.per_tile();
      f32x16_t acc[NRB];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[rb][v] = 0.0f;
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        const Split3 ks = split_f32x8(kb.raw[2 * c], kb.raw[2 * c + 1]);
        if (tnext < t_end) kb.load_group(knext, c);
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) mma_split(acc[rb], q.get3(rb, c), ks);
      }
      int fz = 0;
      asm volatile("" : "+v"(fz));       // re-read per tile rather than kept in 32 NRB registers
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = fz + rb * 32 + mma32_row(v, lane);
          u = fmaf(fast_exp2(fmaf(acc[rb][v], c2, fin_o[row])), fin_i[row], u);
        }
    }
    u += __shfl_xor(u, 32);
    if (hf == 0 && j < a.V) out[j] = u;
  }
}

template <typename T, int NG>
__global__ __launch_bounds__(256, 2) void k_attn_colsum(AttnArgs a) {
  extern __shared__ __align__(16) char lds[];
  const SweepId w = sweep_id(a);
  int row0, nrows;
  ranking_rows(a, w.b, row0, nrows);
  row0 += w.rp * ATT_ROWS;
  nrows = min(nrows - w.rp * ATT_ROWS, ATT_ROWS);
  if (nrows <= 0) {
    // the image's text ends before this pair of row blocks: its column sums are zero
    const int ntiles = (a.V + 31) >> 5;
    const int j_lo = w.sp * a.tiles_per_split * 32, j_hi = min(a.V, min(ntiles, (w.sp + 1) * a.tiles_per_split) * 32);
    float* out = a.upart + (((int64_t)w.b * a.H + w.h) * a.RP + w.rp) * a.V;
    for (int j = j_lo + threadIdx.x; j < j_hi; j += 256) out[j] = 0.0f;
    return;
  }
  if (nrows <= 32) attn_colsum_body<T, 1, NG>(a, lds, w, row0, nrows);
  else attn_colsum_body<T, 2, NG>(a, lds, w, row0, nrows);
}

// ------------------------------------------------------------------------------------------
// k_attn_rows (bf16): both reductions of the text-row attention in one sweep over the keys, for images whose
// softmax terms fit a workgroup's registers: 512 threads = 8 waves hold 16 RG text rows x V keys, wave w the
// 32-key tiles w, w + 8, ... (TPW of them, 8 RG registers each), so V <= 256 TPW.
//   What bounds it: the keys, 256 bytes each (d = 128).  k_attn_stats + k_attn_colsum read them from HBM
//   twice; here they come once, and the further workgroups of a kv head (its G query heads and T text rows
//   give ceil(G T / 16 RG) blocks of rows) find them in the L2 of the XCD they are all dealt to.
//   Rows are packed: row r of kv head g is text row r % len of query head g G + r / len, so a group of
//   query heads or a short text fills whole blocks, and only blocks that exist get workgroups (every
//   wave counts the blocks of the images in front of it from text_len).
//   A workgroup walks GPW kv heads of an image, one after the other, and leaves the sum of their column
//   sums: with every compute unit busy, further workgroups would only add rows for k_score to read, and
//   the next head's first tiles are on their way while this head's statistics are exchanged.
//   16 images x 32 heads x 2304 keys, 64 rows: 113 us for the two sweeps, 67 us here (each key read by two
//   workgroups, 628 MB of L2 requests, 313 MB from HBM); 4 x 28 heads (4 kv heads) x 4096 keys, 48 rows: 49 -> 33 us;
//   1 x 32 heads x 2304 keys, 64 rows: 20 -> 14 us.
//   Key tiles go to LDS by direct loads (whole rows, no registers), a ring of its own per wave.
// Exponents: the logits stay in the registers until the row's largest one is known to all waves (one exchange
// through LDS), so every term is 2^(z - max) as in the two sweeps, whatever the spread of the logits; the terms
// then take the logits' registers until a second exchange gives the denominator.  (A lane's own first logit as
// the baseline of its terms saves the first exchange, but its correction underflows where logits lie 2^126 apart
// and the smaller one has the larger discount, and the rounding grows with the distance from that baseline.)
// The next head's first tiles are on their way during both exchanges.
// Matrix tiles are 16 x 16 (queries x keys), 32 components of the contraction each: lane l supplies row /
// key l % 16, components 8 (l / 16) .. + 7, and owns key l % 16 of a group of 16 and the rows 4 (l / 16) + v of
// one: 4 rows per row group to keep statistics for and to exchange over 16 lanes.  (With 32 x 32 tiles, 16
// rows per lane over 32 lanes, the exchange alone took 15 of 80 us for 16 x 2304 keys, 64 rows, 32 heads.)
// ------------------------------------------------------------------------------------------
constexpr int ROWS_NW = 8;
constexpr int ROWS_V2 = 9 * 32 * ROWS_NW;      // most keys with two row groups per workgroup (9 tiles per wave) ...
constexpr int ROWS_V1 = 16 * 32 * ROWS_NW;     // ... and with one (16)

// blocks of `block` ranking rows of one kv head of an image
__device__ __forceinline__ int row_blocks(const int32_t* text_len, int b, int Tmax, int last_only, int G, int block) {
  const int len = min(max(text_len[b], 0), Tmax);
  return (G * (last_only ? min(len, 1) : len) + block - 1) / block;
}

// Unit u of all images' units (image by image, group of GPW kv heads by group, row block by row block):
// b = -1 past the last one.
struct RowUnit { int b, grp, rb, nb; };
__device__ __forceinline__ RowUnit find_row_unit(const AttnArgs& a, int B, int groups, int block, int lane) {
  const int G = a.H / a.Hkv;
  int total = 0;
  for (int b0 = 0; b0 < B; b0 += 64)
    total += b0 + lane < B ? row_blocks(a.text_len, b0 + lane, a.Tmax, a.last_only, G, block) * groups : 0;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) total += __shfl_xor(total, off);
  // each XCD (id % 8) takes a contiguous eighth, so that the blocks of a kv head share an L2
  const int per_xcd = (total + 7) >> 3, slot = blockIdx.x >> 3;
  int u = (blockIdx.x & 7) * per_xcd + slot;
  RowUnit r{-1, 0, 0, 0};
  if (slot >= per_xcd || u >= total) return r;
  for (int b0 = 0; b0 < B; b0 += 64) {
    const int nb = b0 + lane < B ? row_blocks(a.text_len, b0 + lane, a.Tmax, a.last_only, G, block) : 0;
    int upto = nb * groups;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(upto, off);
      if (lane >= off) upto += y;
    }
    const int at = __popcll(__ballot(upto <= u));      // images of this chunk that lie wholly before u
    if (at < 64) {
      r.b = b0 + at;
      r.nb = __shfl(nb, at);
      u -= __shfl(upto, at) - r.nb * groups;
      r.grp = u / r.nb;
      r.rb = u % r.nb;
      return r;
    }
    u -= __shfl(upto, 63);
  }
  return r;
}

// Ring slots per wave: two tiles, or one where two workgroups then fit a compute unit.
constexpr int rows_slots(int rg, int tpw) { return rg * tpw <= 6 ? 1 : 2; }
template <int NG, int RG, int TPW> constexpr size_t rows_lds_bytes() {
  return (size_t)rows_slots(RG, TPW) * ROWS_NW * 32 * NG * 32 + (size_t)16 * RG * (NG * 32 + 16) +
         sizeof(float) * (2 * ROWS_NW * 16 * RG + 2 * 16 * RG + TPW * ROWS_NW * 32);
}

template <int NG, int RG, int TPW>
__global__ __launch_bounds__(64 * ROWS_NW, (rows_slots(RG, TPW) == 1 ? 4 : 2)) void k_attn_rows(AttnArgs a, int B, int GPW) {
  constexpr int RB = 16 * RG;                                  // rows of the block
  constexpr int NC = NG / 2;                                   // contraction steps of 32 components
  constexpr int KROW = NG * 32, KTILE = 32 * KROW, KLD = KTILE / 1024, QROW = KROW + 16;
  constexpr int NS = rows_slots(RG, TPW);
  constexpr int AHEAD = RG == 2 && NS == 1 ? 1 : 2;            // contraction steps whose operands are read ahead
  extern __shared__ __align__(16) char lds[];
  char* qlds = lds + NS * ROWS_NW * KTILE;
  float* st_m = reinterpret_cast<float*>(qlds + RB * QROW);                 // [8][RB]
  float* st_s = st_m + ROWS_NW * RB;                                         // [8][RB]
  float* fin_l = st_s + ROWS_NW * RB;                                        // [2][RB]  rest of the row (log2 units)
  float* lam = fin_l + 2 * RB;                                                   // [256 TPW]  discounts of the keys
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, q4 = lane >> 4;
  const int groups = (a.Hkv + GPW - 1) / GPW;
  const RowUnit unit = find_row_unit(a, B, groups, RB, lane);
  const int b = __builtin_amdgcn_readfirstlane(unit.b), grp = __builtin_amdgcn_readfirstlane(unit.grp);
  const int rb = __builtin_amdgcn_readfirstlane(unit.rb), nb = __builtin_amdgcn_readfirstlane(unit.nb);
  if (b < 0) return;                           // the same for the whole workgroup
  const int G = a.H / a.Hkv;
  int row0, nrows;
  ranking_rows(a, b, row0, nrows);
  const int live = G * nrows;                  // rows of a kv head
  const int ntiles = (a.V + 31) >> 5;
  const float c2 = a.c2;
  // Tiles of this wave, and whether tile i is one: a scalar comparison where it stands (kept across the
  // heads, the results would fill the scalar registers and spill).
  const int my_tiles = max(0, (ntiles - wave + ROWS_NW - 1) / ROWS_NW);
  auto active = [&](int i) { int x = my_tiles; asm volatile("" : "+s"(x)); return i < x; };
  int g = grp * GPW;
  const int g_end = min(g + GPW, a.Hkv);
  // Addresses that follow from the lane: hidden from the compiler behind a copy of it, they are computed
  // where they are used instead of being kept across the heads.
  auto hidden = [](int x) { asm volatile("" : "+v"(x)); return x; };

  // 1 KiB of whole rows per load instruction; the 16-byte piece p of row r lands in slot p ^ x(r), so that the
  // operand reads of 16 consecutive rows cover all banks.  x repeats after 16 rows.
  auto kswz = [](int row) { return KROW == 128 ? (row >> 1) & 7 : row & 15; };
  constexpr int NV = 16 * KROW / 1024, LPR = KROW / 16;        // load instructions per 16 rows, lanes per row
  const uint32_t krow_bytes = (uint32_t)(a.sk.r * 2);          // a head of an image spans < 2 GiB
  const uint32_t ring = lds_address(lds) + (uint32_t)wave * (NS * KTILE);
  auto issue = [&](int g_, int i, int slot) {
    const uint32_t dst = ring + (uint32_t)slot * KTILE;
    const int j0 = (wave + ROWS_NW * i) * 32, ol = hidden(lane);
    const char* base = reinterpret_cast<const char*>(static_cast<const bf16_t*>(a.kv) + b * a.sk.b + g_ * a.sk.h);
    if (j0 + 32 <= a.V) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int row = v * (16 / NV) + ol / LPR;
        const uint32_t voff = (uint32_t)row * krow_bytes + (((ol % LPR) ^ kswz(row)) << 4);
#pragma unroll
        for (int u = v; u < KLD; u += NV)
          load_to_lds16(base + (uint32_t)(j0 + 16 * (u / NV)) * krow_bytes, voff, dst + u * 1024);
      }
    } else {                                   // the last tile: keys past the end repeat the last one
#pragma unroll 1
      for (int u = 0; u < KLD; ++u) {
        const int row = u * (16 / NV) + ol / LPR;
        load_to_lds16(base, (uint32_t)min(j0 + row, a.V - 1) * krow_bytes + (((ol % LPR) ^ kswz(row)) << 4), dst + u * 1024);
      }
    }
  };
  auto start = [&](int g_) {                   // a head's first tiles
    if (active(0)) issue(g_, 0, 0);
    if (NS == 2 && TPW > 1 && active(1)) issue(g_, 1, 1);
  };
  // thread tid brings 8 components of one row of the block (rows past the end: zeros); through registers, so
  // that they can be asked for while the previous head's still stand in LDS
  static_assert(RB * 2 * NG <= 64 * ROWS_NW, "one piece per thread");
  const int qm = tid / (2 * NG), qpc = tid % (2 * NG), qr = rb * RB + qm;
  const bool q_here = qm < RB, q_row = q_here && qr < live;
  const char* qsrc = reinterpret_cast<const char*>(static_cast<const bf16_t*>(a.qt) + b * a.sq.b +
                                                   (q_row ? qr / nrows : 0) * a.sq.h +
                                                   (int64_t)(row0 + (q_row ? qr % nrows : 0)) * a.sq.r) + qpc * 16;
  // thread tid < RB also brings the rest of row tid (lse_extra, in log2 units; nothing: 2^-inf)
  const int lr = rb * RB + tid;
  const bool l_row = a.lse_extra != nullptr && tid < RB && lr < live;
  const float* lsrc = a.lse_extra + (l_row ? ((int64_t)b * a.H + lr / nrows) * a.Tmax + row0 + lr % nrows : 0);
  uint4 qx;
  float lx;
  auto load_q = [&](int g_) {
    qx = q_row ? ldg16(qsrc + (int64_t)g_ * G * a.sq.h * 2) : make_uint4(0, 0, 0, 0);
    lx = l_row ? lsrc[(int64_t)g_ * G * a.Tmax] * 1.4426950408889634f : -INFINITY;
  };
  start(g);
  load_q(g);
  {
    MassRange range;
    range.load(a.mm, a.mm_n, b);
    const double* s64 = a.s64 + (int64_t)b * a.V;
    constexpr int PER = TPW * ROWS_NW * 32 / (64 * ROWS_NW) + (TPW & 1);
    double sj[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) sj[i] = a.mask_on ? s64[min(tid + 512 * i, a.V - 1)] : 0.0;
    double mlo, mhi;
    range.reduce(mlo, mhi);
    const double minv = 1.0 / (mhi - mlo + a.eps);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int j = tid + 512 * i;
      if (j < TPW * ROWS_NW * 32) lam[j] = j < a.V ? discount_of(a, sj[i], mlo, minv) : 0.0f;
    }
  }
  const int q_off = n * QROW + q4 * 16, k_off = n * KROW + ((q4 ^ kswz(n)) << 4);

  // Column sums over the heads, in fp64: entry t holds the sums 4 t + q4 of the 2 TPW (key n of half x of tile i has
  // index 2 i + x), so that they take a quarter of the registers.
  constexpr int NU = (2 * TPW + 3) / 4;
  double u[NU];
#pragma unroll
  for (int t = 0; t < NU; ++t) u[t] = 0.0;
  // Exchange of a row value between the waves: wave w leaves its 4 RG values per 16 lanes in st[w][row], and lane n
  // picks up those of 2 RG waves of row `mine`, so that a row's eight values lie in 4 / RG neighbouring lanes.
  constexpr int LPW = 4 / RG, PICK = ROWS_NW / LPW;
  const int mine = 16 * (n / LPW / 4) + 4 * q4 + (n / LPW) % 4;
  auto leave = [&](float* st, const float (&x)[RG][4]) {
    const int at = hidden(wave * RB + 4 * q4);
    if (n == 0) {
#pragma unroll
      for (int r = 0; r < RG; ++r)
        *reinterpret_cast<float4*>(st + at + r * 16) = make_float4(x[r][0], x[r][1], x[r][2], x[r][3]);
    }
  };
  auto pick = [&](const float* st, float (&x)[PICK]) {
    const int at = hidden((n % LPW) * PICK * RB + mine);
#pragma unroll
    for (int w = 0; w < PICK; ++w) x[w] = st[at + w * RB];
  };
  // f over the lanes of a row (one after the other: a step alone waits for itself)
  auto over_row = [](float x, auto f) {
    x = f(x, dpp_f32<0xB1>(x));                // quad_perm: the lane beside
    if (LPW == 4) x = f(x, dpp_f32<0x4E>(x));  // ... and the pair beside
    return x;
  };
  // the value of the lanes of row (r, v) in every lane of the 16 (row_newbcast)
  auto spread = [&](float (&x)[RG][4], float y) {
    static_for<4 * RG>([&](auto k) { x[decltype(k)::value / 4][decltype(k)::value % 4] = dpp_f32<0x150 + decltype(k)::value * LPW>(y); });
  };
  auto each = [](auto f) {
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int v = 0; v < 4; ++v) f(r, v);
    __builtin_amdgcn_sched_barrier(0);
  };

  int par = 0;
  auto park_q = [&](int to) {
    if (q_here) *reinterpret_cast<uint4*>(qlds + qm * QROW + qpc * 16) = qx;
    if (tid < RB) fin_l[to * RB + hidden(tid)] = lx;
  };
  park_q(0);
  barrier_lds();
#pragma unroll 1
  for (;; ++g) {
    f32x4_t e[TPW][RG][2];
    float m[RG][4];
    // logits of the tile in ring slot `slot`
    auto logits = [&](f32x4_t (&z)[RG][2], int slot) {
      const int ko = hidden(k_off);
      const char* kt = lds + wave * (NS * KTILE) + slot * KTILE;
      uint4 kop[AHEAD][2], qo[AHEAD][RG];
      auto read = [&](int c) {
#pragma unroll
        for (int x = 0; x < 2; ++x) kop[c % AHEAD][x] = *reinterpret_cast<const uint4*>(kt + (ko ^ (c << 6)) + x * 16 * KROW);
#pragma unroll
        for (int r = 0; r < RG; ++r) qo[c % AHEAD][r] = *reinterpret_cast<const uint4*>(qlds + q_off + c * 64 + r * 16 * QROW);
      };
#pragma unroll
      for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int x = 0; x < 2; ++x) z[r][x] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c = 0; c < AHEAD; ++c) read(c);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
          for (int x = 0; x < 2; ++x) mma16(z[r][x], qo[c % AHEAD][r], kop[c % AHEAD][x]);
        if (c + AHEAD < NC) read(c + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto ring_read = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };    // a slot may be filled again

    each([&](int r, int v) { m[r][v] = ATT_NEG; });
    static_for<TPW>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      if (active(i)) {
        if (NS == 2 && i + 1 < TPW && active(i + 1)) wait_vmem_but<KLD>();
        else wait_all_vmem();
        logits(e[i], NS == 2 ? i & 1 : 0);
        if (i + NS < TPW && active(i + NS)) {
          ring_read();
          issue(g, i + NS, NS == 2 ? i & 1 : 0);
        }
        // (keys past the end repeat the last one: no larger logit)
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
          for (int v = 0; v < 4; ++v) m[r][v] = fmaxf(m[r][v], fmaxf(e[i][r][0][v], e[i][r][1][v]));
      }
    });
    const bool last = g + 1 >= g_end;
    if (!last) {
      load_q(g + 1);
      ring_read();
      start(g + 1);
    }

    // largest logit of every row, over the 16 lanes and then the waves; -M in log2 units, with the rest of the row
    // (lse_extra, already in log2 units) in the comparison
    each([&](int r, int v) { m[r][v] = fmaxf(m[r][v], dpp_f32<0x128>(m[r][v])); });     // row_ror:8, 4, 2, 1
    each([&](int r, int v) { m[r][v] = fmaxf(m[r][v], dpp_f32<0x124>(m[r][v])); });
    each([&](int r, int v) { m[r][v] = fmaxf(m[r][v], dpp_f32<0x122>(m[r][v])); });
    each([&](int r, int v) { m[r][v] = fmaxf(m[r][v], dpp_f32<0x121>(m[r][v])); });
    leave(st_m, m);
    barrier_lds();
    float rest;                                // the rest of the row in units of 2^M
    {
      float x[PICK];
      pick(st_m, x);
      const float l = fin_l[par * RB + hidden(mine)];
#pragma unroll
      for (int w = 1; w < PICK; ++w) x[0] = fmaxf(x[0], x[w]);
      const float big = fmaxf(over_row(x[0], [](float p, float q) { return fmaxf(p, q); }) * c2, l);
      rest = fast_exp2(l - big);
      spread(m, -big);
    }
    float s[RG][4];
    each([&](int r, int v) { s[r][v] = 0.0f; });
    static_for<TPW>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      if (active(i)) {
        const int lt = hidden(wave * 32 + n);
        const float l[2] = {lam[lt + ROWS_NW * 32 * i], lam[lt + ROWS_NW * 32 * i + 16]};
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              e[i][r][x][v] = fast_exp2(fmaf(e[i][r][x][v], c2, m[r][v]));
              s[r][v] = fmaf(l[x], e[i][r][x][v], s[r][v]);
            }
      }
    });
    each([&](int r, int v) { s[r][v] += dpp_f32<0x128>(s[r][v]); });
    each([&](int r, int v) { s[r][v] += dpp_f32<0x124>(s[r][v]); });
    each([&](int r, int v) { s[r][v] += dpp_f32<0x122>(s[r][v]); });
    each([&](int r, int v) { s[r][v] += dpp_f32<0x121>(s[r][v]); });
    leave(st_s, s);
    // the next head's queries: every wave is past the products with this head's (first exchange), and the barrier of
    // this exchange is the one they need; fin_l has two places, as slower waves may still read this head's
    if (!last) {
      par ^= 1;
      park_q(par);
    }
    barrier_lds();
    {
      float x[PICK];
      pick(st_s, x);
#pragma unroll
      for (int w = 1; w < PICK; ++w) x[0] += x[w];
      const float all = over_row(x[0], [](float p, float q) { return p + q; }) + rest;
      spread(s, rb * RB + hidden(mine) < live ? 1.0f / all : 0.0f);       // rows past the end add nothing
    }
    // this head's column sums, first over a lane's 4 RG rows, then over the four groups of 16 lanes
#pragma unroll
    for (int t = 0; t < NU; ++t) {
      if (active(2 * t)) {
        float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 2 * t; i < min(2 * t + 2, TPW); ++i)
          if (i == 2 * t || active(i)) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
              for (int r = 0; r < RG; ++r)
#pragma unroll
                for (int v = 0; v < 4; ++v) c[2 * (i & 1) + x] = fmaf(e[i][r][x][v], s[r][v], c[2 * (i & 1) + x]);
          }
        u[t] += (double)sum_groups_of_16(c);
      }
    }
    if (last) break;
  }
  float* out = a.upart + ((int64_t)b * groups * a.RP + (grp * nb + rb)) * a.V;
#pragma unroll
  for (int t = 0; t < NU; ++t) {
    const int j = (wave + ROWS_NW * (2 * t + (q4 >> 1))) * 32 + 16 * (q4 & 1) + n;
    if (j < a.V) out[j] = (float)u[t];
  }
}

// ------------------------------------------------------------------------------------------
// The same two reductions from stored logits zlog [B, H, T_eff, V] (accumulator units), for the
// text rows that rode in the mass sweep.
// k_rowstats_logits: grid (T_eff, H, B), 256 threads: (max, sum of lambda'_j 2^z) of one row, in the
// layout k_attn_stats leaves (one split, 32 rows per block).
// k_colsum_logits: grid (ceil(V / 256), H, B), 256 threads: normalised column sums per key.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_rowstats_logits(AttnArgs a) {
  __shared__ float red_m[4], red_s[4];
  const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int row0, nrows;
  ranking_rows(a, b, row0, nrows);
  if (t >= nrows) return;                                   // uniform for the workgroup
  MassRange range;
  range.load(a.mm, a.mm_n, b);
  double mlo, mhi;
  range.reduce(mlo, mhi);
  const double minv = 1.0 / (mhi - mlo + a.eps);
  const float* z = a.zlog + (((int64_t)b * a.H + h) * a.T_eff + t) * a.V;
  // Eight keys of a thread in flight: a load after the other took most of the kernel (5 x 28 heads on 4 x 2083 tokens by the
  // last row: stage 108.5 -> 105.1 us).
  float m = ATT_NEG;
  for (int j0 = tid; j0 < a.V; j0 += 8 * 256) {
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = z[min(j0 + 256 * u, a.V - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) m = fmaxf(m, x[u]);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if (lane == 0) red_m[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red_m[0], red_m[1]), fmaxf(red_m[2], red_m[3]));
  const float offv = -m * a.c2;
  float s = 0.0f;
  const double* s64 = a.s64 + (int64_t)b * a.V;
  for (int j0 = tid; j0 < a.V; j0 += 8 * 256) {
    float x[8];
    double sj[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = min(j0 + 256 * u, a.V - 1);
      x[u] = z[j];
      sj[u] = a.mask_on ? s64[j] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + 256 * u < a.V) s = fmaf(discount_of(a, sj[u], mlo, minv), fast_exp2(fmaf(x[u], a.c2, offv)), s);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) red_s[wave] = s;
  __syncthreads();
  if (tid == 0) {
    const int NR = ((a.T_eff + 31) >> 5) * 32;
    float* out = a.pstat + (((int64_t)b * a.H + h) * 2) * NR;     // one split
    out[t] = m;
    out[NR + t] = (red_s[0] + red_s[1]) + (red_s[2] + red_s[3]);
  }
}

__global__ __launch_bounds__(256) void k_colsum_logits(AttnArgs a) {
  __shared__ float fin_o[32], fin_i[32];
  const int h = blockIdx.y, b = blockIdx.z;
  const int j = blockIdx.x * 256 + threadIdx.x;
  int row0, nrows;
  ranking_rows(a, b, row0, nrows);
  final_row_stats(a, b, h, 32, 0, 32, row0, nrows, fin_o, fin_i);
  __syncthreads();
  if (j >= a.V) return;
  const float* z = a.zlog + (((int64_t)b * a.H + h) * a.T_eff) * a.V + j;
  float u = 0.0f;
  for (int t = 0; t < nrows; ++t) u = fmaf(fast_exp2(fmaf(z[(int64_t)t * a.V], a.c2, fin_o[t])), fin_i[t], u);
  a.upart[((int64_t)b * a.H + h) * a.V + j] = u;
}

// Column sums from the logits k_attn_stats<.., true> left: grid (ceil(V / 256), H, B), 256 threads.
// A lane takes four neighbouring keys, the four waves take the ranking rows t = wave, wave + 4, ...
// (256 at a time: their statistics sit in LDS), and the waves' partial sums are added in wave order.
// upart then has one row per head.
__global__ __launch_bounds__(256) void k_colsum_rows(AttnArgs a) {
  __shared__ float fin_o[256], fin_i[256];
  __shared__ float4 part[4][64];
  const int h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j0 = blockIdx.x * 256 + lane * 4;
  int row0, nrows;
  ranking_rows(a, b, row0, nrows);
  const int NR = ATT_ROWS * a.RP;
  const bool vec = (a.V & 3) == 0;
  const float* z = a.zlog + (((int64_t)b * a.H + h) * a.T_eff) * a.V + j0;
  const float c2 = a.c2;
  float4 u = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  for (int first = 0; first < nrows; first += 256) {
    if (first) __syncthreads();
    final_row_stats(a, b, h, NR, first, min(256, NR - first), row0 + first, nrows - first, fin_o, fin_i);
    __syncthreads();
    const int nl = min(256, nrows - first);
    if (j0 < a.V) {
#pragma unroll 4
      for (int t = wave; t < nl; t += 4) {
        const float* zr = z + (int64_t)(first + t) * a.V;
        float4 x;
        if (vec) {
          x = *reinterpret_cast<const float4*>(zr);
        } else {
          x.x = zr[0];
          x.y = j0 + 1 < a.V ? zr[1] : 0.0f;
          x.z = j0 + 2 < a.V ? zr[2] : 0.0f;
          x.w = j0 + 3 < a.V ? zr[3] : 0.0f;
        }
        const float o = fin_o[t], iv = fin_i[t];
        u.x = fmaf(fast_exp2(fmaf(x.x, c2, o)), iv, u.x);
        u.y = fmaf(fast_exp2(fmaf(x.y, c2, o)), iv, u.y);
        u.z = fmaf(fast_exp2(fmaf(x.z, c2, o)), iv, u.z);
        u.w = fmaf(fast_exp2(fmaf(x.w, c2, o)), iv, u.w);
      }
    }
  }
  part[wave][lane] = u;
  __syncthreads();
  if (wave == 0 && j0 < a.V) {
    float4 r = part[0][lane];
#pragma unroll
    for (int wv = 1; wv < 4; ++wv) {
      const float4 q = part[wv][lane];
      r.x += q.x; r.y += q.y; r.z += q.z; r.w += q.w;
    }
    float* out = a.upart + ((int64_t)b * a.H + h) * a.V + j0;
    if (vec) {
      *reinterpret_cast<float4*>(out) = r;
    } else {
      out[0] = r.x;
      if (j0 + 1 < a.V) out[1] = r.y;
      if (j0 + 2 < a.V) out[2] = r.z;
      if (j0 + 3 < a.V) out[3] = r.w;
    }
  }
}

// ------------------------------------------------------------------------------------------
// k_score: grid (ceil(V/64), B), 256 threads: 64 keys x 4 head groups.  rows[b] = text rows that
// ranked (the divisor of the mean).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ double rank_count(const int32_t* text_len, int b, int Tmax, int last_only) {
  const int len = min(max(text_len[b], 0), Tmax);
  return (double)(last_only ? min(len, 1) : len);
}

// Rows of upart that image b has filled, out of the HV it has room for: all of them (one per head and pair
// of text-row blocks), or with packed > 0 one per group of kv heads (packed of them) and block of rows
// (the G query heads of a kv head together, k_attn_rows).
__device__ __forceinline__ int upart_rows(const int32_t* text_len, int b, int Tmax, int last_only, int HV,
                                          int packed, int G, int block) {
  return packed > 0 ? packed * row_blocks(text_len, b, Tmax, last_only, G, block) : HV;
}

__global__ __launch_bounds__(256) void k_score(const float* __restrict__ upart, const double* __restrict__ s64,
                                                const double* __restrict__ mm, int mm_n,
                                                const int32_t* __restrict__ text_len, int H, int HV, int packed, int G, int block,
                                                int V, int Tmax, int last_only, double lambda_max, double eps,
                                                int mask_on, float* __restrict__ s_hat, float* __restrict__ score) {
  __shared__ double part[4][64];
  const int b = blockIdx.y, jl = threadIdx.x & 63, hq = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + jl;
  MassRange range;
  if (hq == 0) range.load(mm, mm_n, b);       // the wave that finishes
  const int hv = upart_rows(text_len, b, Tmax, last_only, HV, packed, G, block);
  double u = 0.0;
  if (j < V) {
    const float* up = upart + (int64_t)b * HV * V + j;
    int h = hq;
    for (; h + 12 < hv; h += 16) {
      float u0 = up[(int64_t)h * V], u1 = up[(int64_t)(h + 4) * V], u2 = up[(int64_t)(h + 8) * V],
            u3 = up[(int64_t)(h + 12) * V];
      u += (double)u0;
      u += (double)u1;
      u += (double)u2;
      u += (double)u3;
    }
    for (; h < hv; h += 4) u += (double)up[(int64_t)h * V];
  }
  part[hq][jl] = u;
  __syncthreads();
  if (hq != 0) return;
  double lo, hi;
  range.reduce(lo, hi);
  if (j < V) {
    u = ((part[0][jl] + part[1][jl]) + part[2][jl]) + part[3][jl];
    const double sh = (s64[(int64_t)b * V + j] - lo) * (1.0 / (hi - lo + eps));
    const double lam = mask_on ? fmax(lambda_max * sh, eps) : 1.0;
    s_hat[(int64_t)b * V + j] = (float)sh;
    score[(int64_t)b * V + j] = (float)(lam * u / ((double)H * rank_count(text_len, b, Tmax, last_only)));
  }
}

// ------------------------------------------------------------------------------------------
// k_score_select: grid (B), 1024 threads, dynamic LDS = V floats when V > 1024.  The threads reduce the
// per-head column sums of the keys tid, tid + 1024, ... (coalesced) in the order k_score uses (four
// interleaved head groups in fp64, then ((0+1)+2)+3), so that score and s_hat come out bit-identical to
// k_score's; the scores change hands through LDS to the blocked layout of the selection (thread t owns
// keys t*ipt .. t*ipt+ipt-1), and the workgroup then selects exactly as k_select does.
// ------------------------------------------------------------------------------------------
template <int IPT>
__device__ __forceinline__ void score_select_image(const int b, const float* __restrict__ upart,
                                                   const double* __restrict__ s64,
                                                   const double* __restrict__ mm, int mm_n,
                                                   const int32_t* __restrict__ text_len, int H, int HV, int packed, int G, int block,
                                                   int V, int k, int Tmax, int last_only, double lambda_max, double eps, int mask_on,
                                                   float* __restrict__ s_hat, float* __restrict__ score,
                                                   int32_t* __restrict__ kept, int32_t* __restrict__ pruned) {
  __shared__ SelectShared sh;
  extern __shared__ float sc_lds[];
  const int tid = threadIdx.x;
  const int ipt = (V + SEL_THREADS - 1) / SEL_THREADS;
  const int i0 = tid * ipt;
  MassRange range;
  range.load(mm, mm_n, b);
  double lo, hi;
  range.reduce(lo, hi);
  const double inv = 1.0 / (hi - lo + eps);
  const double norm = (double)H * rank_count(text_len, b, Tmax, last_only);
  const int hv = upart_rows(text_len, b, Tmax, last_only, HV, packed, G, block);
  const float* up = upart + (int64_t)b * HV * V;
  float mine = 0.0f;
  for (int j = tid; j < V; j += SEL_THREADS) {
    double part[4] = {0.0, 0.0, 0.0, 0.0};
    int h = 0;
    for (; h + 16 <= hv; h += 16) {         // 16 loads in flight; row h adds to group h % 4, in order
      float u[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) u[q] = up[(int64_t)(h + q) * V + j];
#pragma unroll
      for (int q = 0; q < 16; ++q) part[q & 3] += (double)u[q];
    }
    for (; h < hv; ++h) part[h & 3] += (double)up[(int64_t)h * V + j];
    const double usum = ((part[0] + part[1]) + part[2]) + part[3];
    const double shat = (s64[(int64_t)b * V + j] - lo) * inv;
    const double lam = mask_on ? fmax(lambda_max * shat, eps) : 1.0;
    const float sc = (float)(lam * usum / norm);
    s_hat[(int64_t)b * V + j] = (float)shat;
    score[(int64_t)b * V + j] = sc;
    if (ipt > 1) sc_lds[j] = sc;
    else mine = sc;
  }
  if (ipt > 1) __syncthreads();
  uint32_t key[IPT];
#pragma unroll
  for (int e = 0; e < IPT; ++e) {
    const int i = i0 + e;
    key[e] = (e < ipt && i < V) ? float_key(ipt > 1 ? sc_lds[i] : mine) : 0u;
  }
  int n_keep;
  const uint32_t keep_bits = topk(key, ipt, i0, V, k, sh, &n_keep);
  int tot;
  int kept_before = block_scan_excl(n_keep, sh.wave_sums, &tot);
  int32_t* kout = kept + (int64_t)b * k;
  int32_t* pout = pruned + (int64_t)b * (V - k);
#pragma unroll
  for (int e = 0; e < IPT; ++e) {
    const int i = i0 + e;
    if (e < ipt && i < V) {
      if (keep_bits & (1u << e)) kout[kept_before++] = i;
      else pout[i - kept_before] = i;
    }
  }
}

template <int IPT>
__global__ __launch_bounds__(SEL_THREADS) void k_score_select(const float* __restrict__ upart,
                                                               const double* __restrict__ s64,
                                                               const double* __restrict__ mm, int mm_n,
                                                               const int32_t* __restrict__ text_len, int H, int HV,
                                                               int packed, int G, int block, int V, int k, int Tmax, int last_only, double lambda_max,
                                                               double eps, int mask_on, float* __restrict__ s_hat,
                                                               float* __restrict__ score, int32_t* __restrict__ kept,
                                                               int32_t* __restrict__ pruned) {
  score_select_image<IPT>(blockIdx.x, upart, s64, mm, mm_n, text_len, H, HV, packed, G, block, V, k, Tmax, last_only, lambda_max, eps, mask_on,
                     s_hat, score, kept, pruned);
}

// k_score_select_kv: grid (B + n_bufs * B * Hkv).  The first B workgroups are k_score_select's.  Each of the
// others copies, for one (cache buffer, image, kv head), the rows that survive whatever is selected
// (Fig. 3: prefix rows stay where they are, valid text row t moves from P + V + t to P + k + t): they
// depend on no result of the stage, and the B selecting workgroups leave the memory system idle.
// A row is row_bytes / 16 pieces of 16 bytes; two rows per thread are in flight.
template <int IPT>
__global__ __launch_bounds__(SEL_THREADS) void k_score_select_kv(
    const float* __restrict__ upart, const double* __restrict__ s64, const double* __restrict__ mm, int mm_n,
    const int32_t* __restrict__ text_len, int H, int HV, int packed, int G, int block, int V, int k, int Tmax, int last_only,
    double lambda_max, double eps, int mask_on, float* __restrict__ s_hat, float* __restrict__ score, int32_t* __restrict__ kept,
    int32_t* __restrict__ pruned, int B, KvFixedRows fx) {
  if ((int)blockIdx.x < B) {
    score_select_image<IPT>(blockIdx.x, upart, s64, mm, mm_n, text_len, H, HV, packed, G, block, V, k, Tmax, last_only, lambda_max, eps,
                       mask_on, s_hat, score, kept, pruned);
    return;
  }
  const int gid = blockIdx.x - B, groups = B * fx.Hkv;
  const int buf = gid / groups, bg = gid % groups, b = bg / fx.Hkv;
  const int lpr = fx.row_bytes >> 4, rpi = SEL_THREADS / lpr;
  const int tid = threadIdx.x, piece = tid % lpr, r0 = tid / lpr;
  const int n_fixed = fx.P + min(max(text_len[b], 0), fx.Tmax);
  const char* src = fx.ptrs.src[buf] + (int64_t)bg * fx.N * fx.row_bytes + piece * 16;
  char* dst = fx.ptrs.dst[buf] + (int64_t)bg * fx.Nout * fx.row_bytes + piece * 16;
  for (int r = r0; r < n_fixed; r += 2 * rpi) {
    const int r2 = r + rpi;
    const int sa = r < fx.P ? r : r + fx.V, da = r < fx.P ? r : r + fx.k;
    const int sb = r2 < fx.P ? r2 : r2 + fx.V, db = r2 < fx.P ? r2 : r2 + fx.k;
    const uint4 va = ldg16_stream(src + (int64_t)sa * fx.row_bytes);
    uint4 vb = va;
    if (r2 < n_fixed) vb = ldg16_stream(src + (int64_t)sb * fx.row_bytes);
    stg16_stream(dst + (int64_t)da * fx.row_bytes, va);
    if (r2 < n_fixed) stg16_stream(dst + (int64_t)db * fx.row_bytes, vb);
  }
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
static int ranking_rows_max(const asap_params& p) { return p.score_rows == ASAP_ROWS_LAST ? 1 : p.Tmax; }

// Key-range splits of the two text-row sweeps.  Their workgroups run in rounds of as many as fit
// on the chip at once (1 to 4 per compute unit, by the registers of the instantiation); a round
// costs the tiles of one split plus a fixed part (start-up, the text queries, the last tiles' tail:
// about 8 tile times, fitted to measurements), and more than one workgroup per compute unit at a
// time slows each of them (about 1.4x).  The count with the least modelled time wins, fewer splits
// on ties; a split has at least 4 tiles (one per wave).
static int attn_splits(const asap_params& p) {
  const int ntiles = (p.V + 31) / 32;
  const int rows = ranking_rows_max(p);
  const int rb = rows > 32 ? 2 : 1, ch = p.d / 16, rp = (rows + 63) / 64;
  int per_cu = rb * ch <= 4 ? 4 : (rb * ch <= 8 && ch == 8) ? 3 : 2;
  if (p.qk_dtype != ASAP_BF16) per_cu = 2;
  const long slots = 256L * per_cu, groups = (long)p.H * p.B * rp;
  int smax = ntiles / 4;
  if (smax > 16) smax = 16;
  if (smax < 1) smax = 1;
  int best = 1;
  double best_cost = -1.0;
  for (int s = 1; s <= smax; ++s) {
    const int tps = (ntiles + s - 1) / s;
    if ((ntiles + tps - 1) / tps != s) continue;           // the same split length with fewer splits exists
    const long wgs = groups * s, rounds = (wgs + slots - 1) / slots;
    const double crowd = (wgs < slots ? wgs : slots) <= 256 ? 1.0 : 1.4;
    const double cost = (double)rounds * (tps + 8) * crowd;
    if (best_cost < 0.0 || cost < best_cost) { best_cost = cost; best = s; }
  }
  return best;
}

// key tiles per wave of k_attn_rows
static int rows_tpw(const asap_params& p) { return ((p.V + 31) / 32 + ROWS_NW - 1) / ROWS_NW; }

// kv heads a workgroup of k_attn_rows walks: workgroups run in rounds of as many as the registers let
// onto the chip (two per compute unit where a wave holds few tiles, see rows_slots), and a workgroup costs
// its heads plus about half a head for its start.  Least rounds x cost; ties go to fewer workgroups, which
// leave fewer rows of column sums.
static int rows_heads_per_wg(const asap_params& p, int row_blocks, int rg) {
  const long slots = rows_slots(rg, rows_tpw(p)) == 1 ? 512 : 256;
  int best = 1;
  double best_cost = -1.0;
  for (int n = 1; n <= p.Hkv; ++n) {
    const long wgs = (long)p.B * ((p.Hkv + n - 1) / n) * row_blocks;
    const double cost = (double)((wgs + slots - 1) / slots) * (n + 0.5);
    if (best_cost < 0.0 || cost <= best_cost) { best_cost = cost; best = n; }
  }
  return best;
}

// Above ROWS_V2 keys a block of the one sweep has 16 rows, half of what the two sweeps take per pass over a
// key tile, and a wave walks up to 16 tiles in a row.  Both forms of asap_score, timed over 780 shapes of 2305
// to 4096 keys: the one sweep is 1.13 times as fast on average, 1.00 times in full launches of 113 to 128 rows with a
// kv head per query head (0.93 to 1.12 for sizes close to each other: 16 x 32 heads x 2560 keys 309 us, two sweeps 300;
// 16 x 40 heads 385 and 402).  The two sweeps are taken where they are clearly ahead:
//  * 16 or more query heads of 64 components on one kv head, more than four rounds of 256 workgroups and text rows
//    that fill the two sweeps' blocks of 64: the partial column sums of 16 rows each then outweigh the keys
//    (16 x 16 heads on 1 x 4096 keys, 128 rows: 145 and 117 us; 16 x 32 on 2 x 2560, 64 rows: 104 and 94; with 80 rows
//    6 x 64 on 4 x 2305 the one sweep, 86 and 108);
//  * at most 32 workgroups that walk more than 12 tiles of 256 bytes a row (1 x 8 heads x 3617 keys, 32 rows: 38 and 34 us;
//    with seven query heads per kv head the one sweep is not behind, 48.4 and 48.6 us).
static bool two_sweeps_faster(const asap_params& p, int t_eff) {
  const int G = p.H / p.Hkv;
  const long wgs = (long)p.B * p.Hkv * ((G * t_eff + 15) / 16);
  const bool full = (t_eff + 63) / 64 * 64 - t_eff < 16;
  if (p.d == 64 && G >= 16 && full && wgs > 1024) return true;
  return p.d == 128 && p.V > 12 * 256 && wgs <= 32 && G <= 4;
}

static long mass_tiles(const asap_params& p) { return (long)((p.V + 31) / 32) * p.B; }

// Text rows may ride in the mass sweep when the rows of one kv head's query heads fit the free rows of
// its tile and their logits -- written once, read twice, 12 bytes per row and key -- weigh less than
// the two sweeps over the keys they replace.
static bool text_rows_fit(const asap_params& p) {
  const int rows = p.H / p.Hkv * ranking_rows_max(p), row_bytes = p.d * 2;
  return p.qk_dtype == ASAP_BF16 && rows <= 28 && 12 * rows < 2 * row_bytes;
}

// Small batches: every workgroup of the mass sweep reads all text rows of its image for 16 keys, so that a sweep of its
// own over the keys is faster unless the rows are few for the keys that an image (k_attn_rows' chain gets longer) and
// the batch (more workgroups that read them again) have.  The line follows measurements at 18 to 252 tiles of 32 keys (us
// per stage, riding / swept / as text rows rode before k_mass_small_ride):  1 x 32 heads x 576 tokens, 1 row 55 / 52 / 59, 28 rows
// 66 / 54 / 64;  8 x 40 x 576, 28 rows 138 / 108 / 123;  15 x 32 x 512, 1 row 94 / 99 / 101, 16 rows 119 / 104 / 117;  1 x 32 x
// 4096, 4 rows 100 / 104 / 111;  1 x 40 x 8000, 8 rows 212 / 228 / 214.
// With up to 4 kv heads the rows cost a tile of 16 keys little, and k_attn_rows has few workgroups for an image: the keys decide
// (28 heads on 4, 7 or 14 rows:  8 x 576 tokens 73 / 69,  7 x 1152 92 / 91,  1 x 2304 73 / 75,  1 x 4096 91 / 95;  8 on 2, 16 rows:
// 2 x 2488 67 / 71).
static bool sweep_faster_than_riding(const asap_params& p) {
  if (mass_tiles(p) >= 256) return false;
  if (p.Hkv <= 4) return p.V < 2000;
  const int rows = p.H / p.Hkv * ranking_rows_max(p);
  return 2000l * (rows + 1) > 3l * p.V + 40 * mass_tiles(p);
}

// The plan with text rows riding along or not, which keeps to the budget where it can.
static ScoreWorkspace plan_score(const asap_params& p, size_t budget, bool ride) {
  ScoreWorkspace w{};
  // The mass sweep of few keys: smaller tiles, a wave per head.  8 keys per workgroup where 16 would leave more than half
  // of the chip idle (1 x 32 heads x 576 tokens in f32: 76.0 us per stage, 78.3 with 16; 1 x 2304: 87.6, 89.8 with 8).
  const long tiles = mass_tiles(p);
  w.mass_small = tiles < 256 ? 1 : 0;
  // rows per k_qsum block: whole image span unless that leaves the chip short of blocks.  Small batches, whose
  // workgroups all read every partial sum, take no more than 128 blocks (6 x 28 heads x 1225 tokens: 123.4 us per
  // stage, 125.0 with 256 blocks, 128.5 with 512; 1 x 32 x 2304: 87.6, 87.2, 90.4).  The others take up to 256, one per compute
  // unit: more come in a second round that is nearly empty, and a block per head and no group needs no k_qsplit (us of
  // asap_score with 512 blocks or more / up to 256: 4 x 28 heads on 4 x 4096 69.5 / 65.4;  2 x 28 on 4 x 4096 44.2 / 42.4;  5 x 28 on 4 x 2083
  // 38.4 / 36.1;  6 x 32 x 2304 72.2 / 67.9;  8 x 32 x 1536 63.6 / 62.0).  Two blocks per compute unit are ahead only where both rounds are
  // full and long:
  //  * 86 to 128 heads of all images, 4 or 5 blocks each of 160 KB or more (4 x 32 x 4096 79.9, two blocks 81.2;  3 x 40 x 4096 76.9 / 78.2;
  //    3 x 32 x 4096 66.5 / 67.2;  3 x 40 x 2800 62.9 both;  4 x 32 x 2048 49.4 / 49.3), unless k_qsplit has many of their sums to
  //    add (4 x 28 on 4 x 2304 41.6 / 40.7);
  //  * 257 to 384 heads, two blocks of 192 KB or more (9 x 32 x 2304 98.9, one block 101.6;  11 x 32 x 2304 114.2 / 116.7;  12 x 32 x
  //    2304 121.0 / 122.2;  f32 12 x 28 on 4 x 1200 107.5 / 110.6;  9 x 40 x 1536 82.8 both;  11 x 32 x 800 56.8 / 54.4;  10 x 40 x 1800 108.2 / 102.9).
  const int heads = p.B * p.H, G = p.H / p.Hkv;
  const int64_t head_bytes = (int64_t)p.V * p.d * (p.qk_dtype == ASAP_BF16 ? 2 : 4);
  auto most_chunks = [&](int want) {
    const int chunks = std::min((want + heads - 1) / heads, (p.V + 255) / 256);
    return chunks < 1 ? 1 : chunks;
  };
  auto per_head = [&] {
    if (heads > 256) return heads <= 384 && head_bytes >= 384 * 1000 ? 2 : 1;
    const bool two_rounds = heads > 85 && heads <= 128 && head_bytes >= 4 * 160 * 1000 && G * (512 / heads) <= 16;
    return (two_rounds ? 512 : 256) / heads;
  };
  const int room = most_chunks(w.mass_small ? 128 : 512);      // partial sums that the workspace has room for
  const int chunks = w.mass_small ? room : std::min(room, per_head());
  w.q_rows = (p.V + chunks - 1) / chunks;
  w.q_chunks = (p.V + w.q_rows - 1) / w.q_rows;
  const int q_room = (p.V + (p.V + room - 1) / room - 1) / ((p.V + room - 1) / room);
  w.attn_splits = attn_splits(p);
  w.t_eff = ranking_rows_max(p);
  w.ride = ride ? 1 : 0;
  w.mass_keys = 2 * tiles >= 128 || w.ride ? 16 : 8;
  w.row_pairs = w.ride ? 1 : (w.t_eff + 63) / 64;
  // f32 keys: the first text-row sweep leaves its logits (4 bytes per ranking row and key, never more
  // than the key sweeps they replace at 512 bytes per key and 64 rows) and the column sums read them
  // back instead of sweeping the keys and forming the products again, as long as the workspace stays
  // moderate.
  const size_t zlog_bytes = sizeof(float) * (size_t)p.B * p.H * w.t_eff * p.V;
  w.store_logits = (!w.ride && p.qk_dtype != ASAP_BF16 && zlog_bytes <= STORED_LOGITS_MAX_BYTES) ? 1 : 0;
  const int NR = w.ride ? 32 : 64 * w.row_pairs;
  const int splits = w.ride ? 1 : w.attn_splits;
  // One sweep over the keys where the softmax terms of 32 text rows fit a workgroup's registers.
  // Two row groups per workgroup read the keys half as often; one leaves twice the workgroups and half the
  // work in each, which is what a launch that leaves half the chip idle needs, and holds more keys.
  if (!w.ride && p.qk_dtype == ASAP_BF16) {
    const long units2 = (long)p.B * p.Hkv * ((G * w.t_eff + 31) / 32);
    w.one_sweep = p.V <= ROWS_V2 ? (units2 > 128 ? 2 : 1) : p.V <= ROWS_V1 && !two_sweeps_faster(p, w.t_eff) ? 1 : 0;
  }
  size_t off = 0;
  w.off_qpart = off;
  off = align256(off + sizeof(double) * p.B * p.H * q_room * p.d);
  off = align256(off + sizeof(double) * p.B * p.Hkv * p.d);
  w.off_qsplit = off; off = align256(off + sizeof(uint16_t) * p.B * p.Hkv * 4 * p.d);
  w.off_s64 = off;    off = align256(off + sizeof(double) * p.B * p.V);
  // The (min, max) pairs of the key tiles lie where nothing is read any more when the masses are formed: in the place
  // of the partial sums of the queries (k_qsplit is through with them), or of the pieces of their sums (which
  // a small batch does not use).  Where they do not fit (few heads, thousands of tokens), k_mass_finish takes one pair per image.
  const int ktiles = w.mass_small ? (p.V + w.mass_keys - 1) / w.mass_keys : (p.V + 31) / 32;
  w.finish = sizeof(double) * 2 * (size_t)p.B * ktiles > (w.mass_small ? w.off_s64 - w.off_qsplit : w.off_qsplit);
  w.mm_n = w.finish ? 1 : ktiles;
  w.off_mm = w.finish ? off : w.mass_small ? w.off_qsplit : w.off_qpart;
  off = align256(off + sizeof(double) * 2 * p.B);
  // The one sweep has no row statistics.  Many query heads on few kv heads leave more of those sums than the two sweeps do
  // (one row for 16 or 32 text rows instead of 64): where the caller's scratch does not hold them, the two sweeps run.
  if (w.one_sweep) {
    const int blocks = (G * w.t_eff + 16 * w.one_sweep - 1) / (16 * w.one_sweep);
    const int heads = rows_heads_per_wg(p, blocks, w.one_sweep);
    const size_t rows = (size_t)((p.Hkv + heads - 1) / heads) * blocks;
    const size_t total = off + align256(sizeof(float) * p.B * rows * p.V);
    if (total <= budget) {
      w.row_pairs = blocks;
      w.heads_per_wg = heads;
      w.off_upart = w.off_pstat = off;
      w.off_zlog = w.total = total;
      return w;
    }
    w.one_sweep = 0;
  }
  w.off_pstat = off;  off = align256(off + sizeof(float) * (size_t)p.B * p.H * splits * 2 * NR);
  w.off_upart = off;  off = align256(off + sizeof(float) * (size_t)p.B * p.H * w.row_pairs * p.V);
  w.off_zlog = off;
  if (w.store_logits && align256(off + zlog_bytes) > budget) w.store_logits = 0;
  if (w.ride || w.store_logits) off = align256(off + zlog_bytes);
  w.total = off;
  return w;
}

ScoreWorkspace score_workspace(const asap_params& p, size_t budget) {
  if (!text_rows_fit(p)) return plan_score(p, budget, false);
  if (sweep_faster_than_riding(p)) {
    const ScoreWorkspace w = plan_score(p, budget, false);
    if (w.total <= budget) return w;           // else: the logits of few rows and keys may take less
  }
  return plan_score(p, budget, true);
}

size_t score_workspace_least(const asap_params& p) {
  return score_workspace(p, p.qk_dtype == ASAP_BF16 ? 0 : ~size_t(0)).total;
}

template <typename T, int NG>
static hipError_t launch_attn(const asap_params& p, const AttnArgs& a, bool store_logits, hipStream_t st,
                              Timer* tm) {
  const size_t lds = query_lds_bytes<T, NG>() + sizeof(float) * 8 * ATT_ROWS;
  const dim3 grid(p.H * a.RP * a.S, p.B);
  if constexpr (sizeof(T) == 4) {
    if (store_logits) {
      auto ks = k_attn_stats<T, NG, true>;
      if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(ks),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
      }
      ASAP_LAUNCH(tm, "k_attn_stats", ks, grid, dim3(256), lds, st, a);
      ASAP_LAUNCH(tm, "k_colsum_rows", k_colsum_rows, dim3((p.V + 255) / 256, p.H, p.B), dim3(256), 0, st, a);
      return hipGetLastError();
    }
  }
  auto k1 = k_attn_stats<T, NG, false>;
  auto k2 = k_attn_colsum<T, NG>;
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k1),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(k2), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    if (e != hipSuccess) return e;
  }
  ASAP_LAUNCH(tm, "k_attn_stats", k1, grid, dim3(256), lds, st, a);
  ASAP_LAUNCH(tm, "k_attn_colsum", k2, grid, dim3(256), lds, st, a);
  return hipGetLastError();
}

template <int NG, int RG, int TPW>
static hipError_t launch_attn_rows_as(const asap_params& p, const ScoreWorkspace& w, const AttnArgs& a, hipStream_t st,
                                      Timer* tm) {
  const int units = p.B * ((p.Hkv + w.heads_per_wg - 1) / w.heads_per_wg) * w.row_pairs;
  auto kern = k_attn_rows<NG, RG, TPW>;
  constexpr size_t lds = rows_lds_bytes<NG, RG, TPW>();
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
  }
  ASAP_LAUNCH(tm, "k_attn_rows", kern, dim3(8 * ((units + 7) / 8)), dim3(64 * ROWS_NW), lds, st, a, p.B, w.heads_per_wg);
  return hipGetLastError();
}

template <int NG>
static hipError_t launch_attn_rows(const asap_params& p, const ScoreWorkspace& w, const AttnArgs& a, hipStream_t st,
                                   Timer* tm) {
  const int tpw = rows_tpw(p);
  if (w.one_sweep == 2) {
    if (tpw <= 3) return launch_attn_rows_as<NG, 2, 3>(p, w, a, st, tm);
    if (tpw <= 5) return launch_attn_rows_as<NG, 2, 5>(p, w, a, st, tm);
    if (tpw <= 7) return launch_attn_rows_as<NG, 2, 7>(p, w, a, st, tm);
    return launch_attn_rows_as<NG, 2, 9>(p, w, a, st, tm);
  }
  if (tpw <= 3) return launch_attn_rows_as<NG, 1, 3>(p, w, a, st, tm);
  if (tpw <= 6) return launch_attn_rows_as<NG, 1, 6>(p, w, a, st, tm);
  if (tpw <= 9) return launch_attn_rows_as<NG, 1, 9>(p, w, a, st, tm);
  return launch_attn_rows_as<NG, 1, 16>(p, w, a, st, tm);
}

template <typename T, int NG>
static hipError_t launch_mass(const asap_params& p, const ScoreWorkspace& w, const void* k_vis, Strides3 kv,
                              const uint16_t* qsplit, const double* qpart, int q_chunks, double scale, double* s64,
                              float* s_raw, double* mm, const RideArgs& ra, hipStream_t st, Timer* tm) {
  const T* kp = static_cast<const T*>(k_vis);
  if (w.mass_small) {
    const dim3 grid((p.V + w.mass_keys - 1) / w.mass_keys, p.B), block(64 * std::min(p.Hkv, MASS_SMALL_NW));
    const int np = p.H / p.Hkv * q_chunks;
    if constexpr (sizeof(T) == 2) {
      if (w.ride) {
        auto kern = p.Hkv <= 8 ? k_mass_small_ride<NG, 8> : k_mass_small_ride<NG, 5>;
        ASAP_LAUNCH(tm, "k_mass_small_ride", kern, grid, block, 0, st, kp, kv, qpart, p.Hkv, np, p.V, scale, s64, s_raw,
                    mm, ra);
        return hipGetLastError();
      }
    }
    if (w.mass_keys == 16)
      ASAP_LAUNCH(tm, "k_mass_small", (k_mass_small<T, 16 * NG, 16>), grid, block, 0, st, kp, kv, qpart, p.Hkv, np, p.V, scale,
                  s64, s_raw, mm);
    else
      ASAP_LAUNCH(tm, "k_mass_small", (k_mass_small<T, 16 * NG, 8>), grid, block, 0, st, kp, kv, qpart, p.Hkv, np, p.V, scale,
                  s64, s_raw, mm);
    return hipGetLastError();
  }
  const dim3 grid((p.V + 31) / 32, p.B);
  if constexpr (sizeof(T) == 2) {
    if (w.ride) {
      ASAP_LAUNCH(tm, "k_mass_mfma", (k_mass_mfma<T, NG, true>), grid, dim3(256), 0, st, kp, kv, qsplit, p.Hkv, p.V, scale,
                  s64, s_raw, mm, ra);
      return hipGetLastError();
    }
  }
  ASAP_LAUNCH(tm, "k_mass_mfma", (k_mass_mfma<T, NG, false>), grid, dim3(256), 0, st, kp, kv, qsplit, p.Hkv, p.V, scale, s64,
              s_raw, mm, ra);
  return hipGetLastError();
}

template <typename T>
static hipError_t score_typed(const asap_params& p, const void* q_vis, Strides3 qv, const void* q_txt,
                              Strides3 qt, const void* k_vis, Strides3 kv, const int32_t* text_len,
                              const float* lse_extra, float* s_raw, float* s_hat, float* score, int32_t* kept,
                              int32_t* pruned, const FrontArgs* fe, const KvFixedRows* fixed, char* ws,
                              size_t ws_budget, hipStream_t st, Timer* tm) {
  const ScoreWorkspace w = score_workspace(p, ws_budget);
  double* qpart = reinterpret_cast<double*>(ws + w.off_qpart);
  uint16_t* qsplit = reinterpret_cast<uint16_t*>(ws + w.off_qsplit);
  double* s64 = reinterpret_cast<double*>(ws + w.off_s64);
  double* mm = reinterpret_cast<double*>(ws + w.off_mm);
  float* pstat = reinterpret_cast<float*>(ws + w.off_pstat);
  float* upart = reinterpret_cast<float*>(ws + w.off_upart);
  float* zlog = reinterpret_cast<float*>(ws + w.off_zlog);
  const int mask_on = p.mask_mode == ASAP_MASK_KEYBIAS;
  const int last_only = p.score_rows == ASAP_ROWS_LAST;
  const int ng = p.d / 16;      // contraction groups of 8 elements per lane half
  const int ktiles = (p.V + 31) / 32;
  const int q_chunks = fe != nullptr ? 1 : w.q_chunks;

  if (fe != nullptr) {
    // the summed visual queries come from the hidden states (asap_front.hip), one chunk per head
    hipError_t e0 = launch_front_end(p, fe->hidden, fe->hsb, fe->hsr, fe->wq, fe->rope_theta, fe->vis_positions,
                                     qpart, fe->ws, st, tm);
    if (e0 != hipSuccess) return e0;
    if (!w.mass_small)
      ASAP_LAUNCH(tm, "k_qsplit", k_qsplit, dim3(p.Hkv, p.B), dim3(p.d), 0, st, qpart, qsplit, p.H, p.Hkv, 1, p.d);
  } else {
    const int direct = (!w.mass_small && w.q_chunks == 1 && p.H == p.Hkv) ? 1 : 0;
    ASAP_LAUNCH(tm, "k_qsum", k_qsum<T>, dim3(w.q_chunks, p.H, p.B), dim3(1024), 0, st, static_cast<const T*>(q_vis),
                qv, p.V, p.d, w.q_rows, qpart, qsplit, direct);
    if (!direct && !w.mass_small)
      ASAP_LAUNCH(tm, "k_qsplit", k_qsplit, dim3(p.Hkv, p.B), dim3(p.d), 0, st, qpart, qsplit, p.H, p.Hkv,
                  w.q_chunks, p.d);
  }
  const double scale = 1.0 / ((double)p.H * sqrt((double)p.d));
  RideArgs ra;
  ra.qt = q_txt; ra.sq = qt; ra.text_len = text_len; ra.zlog = zlog;
  ra.H = p.H; ra.G = p.H / p.Hkv; ra.T_eff = w.t_eff; ra.Tmax = p.Tmax; ra.last_only = last_only;
  double* tile_mm = w.finish ? nullptr : mm;
  hipError_t e = ng == 8
                     ? launch_mass<T, 8>(p, w, k_vis, kv, qsplit, qpart, q_chunks, scale, s64, s_raw, tile_mm, ra, st, tm)
                     : launch_mass<T, 4>(p, w, k_vis, kv, qsplit, qpart, q_chunks, scale, s64, s_raw, tile_mm, ra, st, tm);
  if (e != hipSuccess) return e;
  if (w.finish)
    ASAP_LAUNCH(tm, "k_mass_finish", k_mass_finish, dim3(p.B), dim3(1024), 0, st, s64, p.V, mm);

  AttnArgs a;
  a.qt = q_txt; a.sq = qt; a.kv = k_vis; a.sk = kv; a.s64 = s64; a.mm = mm; a.mm_n = w.mm_n; a.text_len = text_len;
  a.lse_extra = lse_extra; a.pstat = pstat; a.upart = upart; a.zlog = zlog;
  a.H = p.H; a.Hkv = p.Hkv; a.V = p.V; a.Tmax = p.Tmax; a.S = w.ride ? 1 : w.attn_splits; a.RP = w.row_pairs;
  a.tiles_per_split = (ktiles + a.S - 1) / a.S;
  a.T_eff = w.t_eff; a.last_only = last_only;
  a.c2 = (float)(1.4426950408889634 / sqrt((double)p.d));
  a.lambda_max = (double)p.lambda_max; a.eps = (double)p.eps; a.mask_on = mask_on;
  if (w.ride) {
    ASAP_LAUNCH(tm, "k_rowstats_logits", k_rowstats_logits, dim3(w.t_eff, p.H, p.B), dim3(256), 0, st, a);
    ASAP_LAUNCH(tm, "k_colsum_logits", k_colsum_logits, dim3((p.V + 255) / 256, p.H, p.B), dim3(256), 0, st, a);
    e = hipGetLastError();
  } else if (w.one_sweep) {
    e = ng == 8 ? launch_attn_rows<8>(p, w, a, st, tm) : launch_attn_rows<4>(p, w, a, st, tm);
  } else if (ng == 8) {
    e = launch_attn<T, 8>(p, a, w.store_logits != 0, st, tm);
  } else {
    e = launch_attn<T, 4>(p, a, w.store_logits != 0, st, tm);
  }
  if (e != hipSuccess) return e;
  const int packed = w.one_sweep ? (p.Hkv + w.heads_per_wg - 1) / w.heads_per_wg : 0;
  const int u_rows = w.one_sweep ? packed * w.row_pairs : p.H * (w.store_logits ? 1 : w.row_pairs);  // rows of upart per image
  // One workgroup per image fetches the column sums slowly, so in small batches the selection rides along only where they
  // are few: up to 96 KB saves about a microsecond (1 x 16 x 576: 50.0 -> 49.1 us per stage, 1 x 32 x 576 in f32: 72.4 ->
  // 71.5), 2 x 8 heads of 2000 tokens with as many bytes cost four (64.6 -> 68.8), 5 x 28 x 2083 with 230 KB eight.
  const bool fuse = score_fuses_selection(p) || (p.V <= SEL_THREADS && sizeof(float) * u_rows * p.V <= 96 * 1024);
  if (kept != nullptr && !fuse) {
    ASAP_LAUNCH(tm, "k_score", k_score, dim3((p.V + 63) / 64, p.B), dim3(256), 0, st, upart, s64, mm, w.mm_n, text_len,
                p.H, u_rows, packed, p.H / p.Hkv, 16 * w.one_sweep, p.V, p.Tmax, last_only, (double)p.lambda_max, (double)p.eps, mask_on, s_hat, score);
    hipError_t e2 = hipGetLastError();
    return e2 != hipSuccess ? e2 : launch_select(p, score, kept, pruned, st, tm);
  }
  if (kept != nullptr) {
    const size_t lds = p.V > SEL_THREADS ? sizeof(float) * (size_t)p.V : 0;
    return with_ipt(p.V, [&](auto ipt) {
      constexpr int IPT = decltype(ipt)::value;
      const void* fn = fixed ? reinterpret_cast<const void*>(k_score_select_kv<IPT>)
                             : reinterpret_cast<const void*>(k_score_select<IPT>);
      if (lds > 32 * 1024) {
        hipError_t e2 = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e2 != hipSuccess) return e2;
      }
      if (fixed)
        ASAP_LAUNCH(tm, "k_score_select_kv", k_score_select_kv<IPT>, dim3(p.B + fixed->n_bufs * p.B * p.Hkv),
                    dim3(SEL_THREADS), lds, st, upart, s64, mm, w.mm_n, text_len, p.H, u_rows, packed, p.H / p.Hkv, 16 * w.one_sweep, p.V, p.k, p.Tmax,
                    last_only, (double)p.lambda_max, (double)p.eps, mask_on, s_hat, score, kept, pruned, p.B, *fixed);
      else
        ASAP_LAUNCH(tm, "k_score_select", k_score_select<IPT>, dim3(p.B), dim3(SEL_THREADS), lds, st, upart, s64, mm, w.mm_n,
                    text_len, p.H, u_rows, packed, p.H / p.Hkv, 16 * w.one_sweep, p.V, p.k, p.Tmax, last_only, (double)p.lambda_max, (double)p.eps,
                    mask_on, s_hat, score, kept, pruned);
      return hipGetLastError();
    });
  } else {
    ASAP_LAUNCH(tm, "k_score", k_score, dim3((p.V + 63) / 64, p.B), dim3(256), 0, st, upart, s64, mm, w.mm_n, text_len,
                p.H, u_rows, packed, p.H / p.Hkv, 16 * w.one_sweep, p.V, p.Tmax, last_only, (double)p.lambda_max, (double)p.eps, mask_on, s_hat, score);
  }
  return hipGetLastError();
}

hipError_t launch_score(const asap_params& p, const void* q_vis, Strides3 qv, const void* q_txt, Strides3 qt,
                        const void* k_vis, Strides3 kv, const int32_t* text_len, const float* lse_extra,
                        float* s_raw, float* s_hat, float* score, int32_t* kept, int32_t* pruned,
                        const FrontArgs* fe, const KvFixedRows* fixed, char* ws, size_t ws_budget, hipStream_t st,
                        Timer* tm) {
  if (fixed && (kept == nullptr || !score_fuses_selection(p))) return hipErrorInvalidValue;
  if (p.qk_dtype == ASAP_BF16)
    return score_typed<bf16_t>(p, q_vis, qv, q_txt, qt, k_vis, kv, text_len, lse_extra, s_raw, s_hat, score,
                               kept, pruned, fe, fixed, ws, ws_budget, st, tm);
  return score_typed<float>(p, q_vis, qv, q_txt, qt, k_vis, kv, text_len, lse_extra, s_raw, s_hat, score, kept,
                            pruned, fe, fixed, ws, ws_budget, st, tm);
}

}  // namespace asap
