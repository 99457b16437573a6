// asap_attention: the attention forward of one decoder layer in front of the pruning layer under the
// salience-guided bidirectional mask (Eq. 4-5 on the whole sequence; Eq. 1 with the mask off):
//   out[b,h,i,:] = sum_j A_ij v[b,g(h),j,:],  A_i. = softmax_j( q_i.k_j / sqrt(d) + M_ij ),
//   M_ij = 0 (j <= i);  ln(max(lambda_max s_hat_j, eps)) (j > i, both inside the image span);  -inf otherwise.
// Flash-style: one pass over the keys with running row maxima and sums, both contractions on the
// matrix cores, nothing of size N x N ever stored.
//
//   k_att_bias      log2 of the per-key discount by sequence position, [B,Npad] (-inf off the image span,
//                   and everywhere with the mask off), for sequences whose discounts have no room in LDS; else
//                   every workgroup forms its image's itself, with its first loads on their way (att_own_bias)
//   k_vtranspose    values transposed per (image, kv head) to [d, Npad]: the second contraction wants
//                   its A operand (a row of values^T) contiguous along the keys, in the key order in
//                   which the first contraction leaves P^T in the accumulators.  Not needed for bf16
//                   with d = 128: there the values go to LDS row-major and the operand is fetched
//                   with the chip's transposing LDS read (ds_read_b64_tr_b16), two per operand.
//   k_attention     B H ceil(N/256) workgroups of 512 threads = 8 waves (two per SIMD) of 32 queries, or, where the chip holds
//                   them all, B H ceil(N/128) of four waves.  Per
//                   sub-tile of 32 keys a wave computes S^T = K Q^T (keys are the tile rows, so lane l owns
//                   query l % 32 and holds 16 of the keys: the softmax bookkeeping is per lane),
//                   then O^T += V^T P^T, where the P^T operand is taken straight from the
//                   accumulator registers: the contraction slice a lane half supplies is defined as
//                   the keys that lane half already holds, and the V^T operand is stored to match.
//                   A turn is 64 keys (32 with 4-byte elements) and one barrier; a step, one look at the maxima and
//                   one change of the baseline, is a whole turn, or half of one (bf16, d = 64).  A turn's keys, values and discounts go to LDS by direct
//                   global -> LDS loads, once for all waves, into rings of four slots; the waits
//                   for those loads are placed by hand and no other vector-memory instruction is left
//                   in the loop, because any wait the compiler adds for one would drain the ring.
//                   The products of a turn stand in a row, each with the LDS read of the operand five
//                   products on, the turn's loads spread between them.
//   What bounds it (16 x 32 heads x 2403 positions, d = 128, bf16): issue first, power next.  A turn takes 3700
//   cycles for the two waves of a SIMD, 2100 of them matrix instructions, 2200 the softmax when alone, and the
//   clock falls from 2.4 to 2.0 GHz on random data (the same instructions on zeros: 1.35 ms; the products and
//   loads alone 1.24 ms at 1.7 GHz).  Turns of 32 keys with a barrier each, offsets and operand addresses formed anew
//   and the halves' maxima exchanged through LDS took 1.74 ms, now 1.63 (28 heads on 4, 6 x 1337 positions: 201, now
//   191 us; f32, 2 x 28 x 2352: 1.80, now 1.72 ms; 16 x 32 x 180 with the mask, where a few turns are all: 33.5, then 34.8 us).  The discounts formed in the
//   workgroup instead of a launch before it, and no wait for the queries in front of the ring's first loads: 16 x 32 x 180 34.9 -> 32.7
//   us, 1 x 16 x 137 14.0 -> 10.8, 3 x 40 x 1095 100.8 -> 96.9, 16 x 32 x 2403 the same (1659 / 1664).  Two groups of waves half a turn apart with a barrier per phase,
//   one group's products beside the other's softmax, measured the same as one barrier and no order between them.
#include "asap_device.hpp"
#include "asap_launch.hpp"

namespace asap {

// log2 discount of sequence position j: that of an image key (s_hat of its image), -inf for every other one
__device__ __forceinline__ float att_bias(const float* __restrict__ s_hat, int j, int P, int V, float lambda_max, float eps) {
  return j >= P && j < P + V ? log2f(fmaxf(lambda_max * s_hat[j - P], eps)) : -INFINITY;
}

// grid (ceil(Npad/256), B): bias2[b,j] by sequence position j (prefix, image, text, padding), where a workgroup of
// k_attention has no room for an image's
__global__ __launch_bounds__(256) void k_att_bias(const float* __restrict__ s_hat, int P, int V, int Npad,
                                                   float lambda_max, float eps, float* __restrict__ bias2) {
  const int j = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (j >= Npad) return;
  const float x = s_hat != nullptr ? att_bias(s_hat + (int64_t)b * V, j, P, V, lambda_max, eps) : -INFINITY;
  bias2[(int64_t)b * Npad + j] = x;
}

// grid (ceil(Npad/32), Hkv, B), 256 threads; vt[b,g,c,p] = v[b,g,att_vt_key(p),c] for keys < N, 0 for the
// keys N .. Npad-1.
// 16-byte loads along d into LDS, 16-byte stores along the keys out of it.
// Key stored at position p of a values^T row.  The second product takes its P^T operand straight from
// the accumulators of the first, where a lane half holds keys 4 hf .. 4 hf + 3 and 8 + 4 hf .. 8 + 4 hf + 3 of
// every 16; with 2-byte elements (8 keys per 16-byte operand) the row is therefore stored in the order
// 0-3, 8-11, 4-7, 12-15 within every 16 keys, so that a lane half's operand is one contiguous piece.
__device__ __forceinline__ int att_vt_key(int p, int elems_per_16) {
  if (elems_per_16 != 8) return p;
  const int g = p & 15;
  return (p & ~15) | (g & 3) | ((g & 4) << 1) | ((g & 8) >> 1);
}

template <typename T>
__global__ __launch_bounds__(256) void k_vtranspose(const T* __restrict__ v, Strides3 sv, int N, int Npad, int d,
                                                     T* __restrict__ vt) {
  constexpr int E = elem<T>::per16;
  __shared__ T tile[32][128 + E];
  const int n0 = blockIdx.x * 32, g = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  const T* src = v + b * sv.b + g * sv.h;
  const int cpr = d / E;                                   // 16-byte chunks per row
  for (int idx = tid; idx < 32 * cpr; idx += 256) {
    const int r = idx / cpr, c = idx - r * cpr;
    uint4 x = make_uint4(0, 0, 0, 0);
    if (n0 + r < N) x = ldg16_stream(src + (int64_t)(n0 + r) * sv.r + c * E);
    *reinterpret_cast<uint4*>(&tile[r][c * E]) = x;
  }
  __syncthreads();
  T* dst = vt + ((int64_t)b * gridDim.y + g) * d * Npad;
  const int gpr = 32 / E;                                  // 16-byte groups of keys per output row
  for (int idx = tid; idx < d * gpr; idx += 256) {
    const int c = idx / gpr, r0 = (idx - c * gpr) * E;
    T x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = tile[att_vt_key(r0 + e, E)][c];
    uint4 y;
    __builtin_memcpy(&y, x, 16);
    *reinterpret_cast<uint4*>(dst + (int64_t)c * Npad + n0 + r0) = y;
  }
}

__device__ __forceinline__ float fast_exp2_att(float x) { return __builtin_amdgcn_exp2f(x); }

// Floats to the storage type with the hardware's packed conversion (round to nearest even): the
// probabilities are converted once per key tile, which makes the integer version too expensive here.
typedef __bf16 att_bf16x2 __attribute__((ext_vector_type(2)));
typedef float att_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
  att_f32x2 x = {a, b};
  att_bf16x2 y = __builtin_convertvector(x, att_bf16x2);
  uint32_t u;
  __builtin_memcpy(&u, &y, 4);
  return u;
}
template <typename T> __device__ __forceinline__ uint4 att_pack16(const float* in);
template <> __device__ __forceinline__ uint4 att_pack16<float>(const float* in) { return pack16<float>(in); }
template <> __device__ __forceinline__ uint4 att_pack16<bf16_t>(const float* in) {
  return make_uint4(cvt_pk_bf16(in[0], in[1]), cvt_pk_bf16(in[2], in[3]), cvt_pk_bf16(in[4], in[5]),
                    cvt_pk_bf16(in[6], in[7]));
}

// four consecutive output elements from floats (one rounding to the storage type)
template <typename T> __device__ __forceinline__ void store4(T* dst, const float* f);
template <> __device__ __forceinline__ void store4<float>(float* dst, const float* f) {
  *reinterpret_cast<uint4*>(dst) = pack16<float>(f);
}
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t* dst, const float* f) {
  *reinterpret_cast<uint2*>(dst) =
      make_uint2(cvt_pk_bf16(f[0], f[1]), cvt_pk_bf16(f[2], f[3]));
}

// The transposing LDS read of gfx950 for 16-bit elements (ds_read_b64_tr_b16): every lane names 8
// bytes; in each group of 16 lanes, lane 4 a + c receives the c-th 16-bit element of the pieces named
// by lanes a, 4 + a, 8 + a and 12 + a, in that order.
typedef short att_i16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 att_tr_read(uint32_t lds_addr) {
  const att_i16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) att_i16x4*)(uintptr_t)lds_addr);
  uint2 u;
  __builtin_memcpy(&u, &r, 8);
  return u;
}

// key held in accumulator register v of a lane of half hf, relative to the tile
__device__ __forceinline__ int att_key_of(int v, int hf) { return 8 * (v >> 2) + 4 * hf + (v & 3); }

constexpr int ATT_NW = 8;                      // waves per workgroup (two per SIMD), 32 queries each
constexpr float ATT_LAZY = 8.0f;               // growth of a row maximum (log2 units) that moves the baseline

// LDS swizzles: the 16-byte piece p of row r is stored in slot p ^ x(r), so that 16 consecutive rows
// spread over all banks for the strided operand reads while the loads still write 1 KiB at a time
__device__ __forceinline__ int att_kswz(int row, int row_bytes) { return row_bytes <= 128 ? (row >> 1) & 7 : row & 15; }
__device__ __forceinline__ int att_vswz(int row) { return (row >> 1) & 7; }      // rows of 128 bytes

// how the mask acts on one (32 keys x 32 queries) tile
enum { ATT_PLAIN = 0,     // every key precedes every query: no mask
       ATT_AHEAD = 1,     // every key follows every query and all queries are image rows: the key's discount
       ATT_GENERAL = 2 }; // anything else: decided per element

// Sub-tiles of 32 keys that a wave takes per step, steps per turn (per barrier), and the LDS ring: four turns of keys,
// values and discounts.  bf16 with d = 64 takes its turn in two steps: with one sub-tile's scores and terms at a time a
// wave needs 121 registers (160 with two), and 67 KB of LDS then leave room for a second workgroup on a compute unit.
// 64 x 16 heads x 300 positions: 112 us in one step per turn, 92 in turns of 32 keys with a barrier each, now 81;
// 12 x 16 x 2400: 423, 403, 374; 1 x 8 x 2400, where no compute unit has two to do: 64.5, 71.9, 60.8.  (One step is
// faster just above a workgroup per compute unit where the keys are many: 272 workgroups of 4200 positions 145, 172, 155.)
template <typename T> constexpr int att_sub(int d) { return sizeof(T) == 2 && d == 128 ? 2 : 1; }
template <typename T> constexpr int att_steps(int d) { return sizeof(T) == 2 && d == 64 ? 2 : 1; }
constexpr int ATT_NS = 4;
// LDS: the rings of keys and values, then that of the discounts (npad = 0) or an image's, by position
template <typename T> constexpr size_t att_lds_bytes(int d, int npad) {
  constexpr int NS = ATT_NS;
  const size_t keys = 32 * att_sub<T>(d) * att_steps<T>(d);
  return NS * keys * 2 * d * sizeof(T) + sizeof(float) * (npad ? npad : NS * keys);
}
// The workgroup forms the discounts itself, and k_att_bias is not launched, where an image's fit beside the rings: up to 8160
// positions with d = 128, 24544 in f32 with d = 64 (whose rings take 64 KiB), 4064 in bf16 with d = 64, where two workgroups share a compute unit.
template <typename T> constexpr bool att_own_bias(int d, int npad) {
  return att_lds_bytes<T>(d, npad) <= (att_steps<T>(d) == 2 ? 80 : 160) * 1024;
}

// CH = 16-byte chunks of a row per lane half (row bytes = 32 * CH)
// The bound on registers is that of the eight waves for four waves too, which need no more of them.  Left twice as many, the compiler
// puts accumulators into AGPRs, and softmax and rescaling move them to and fro (us with them / without: 1 x 40 heads x 643 positions
// 24.4 / 21.0, 1 x 16 x 2048 59.5 / 50.5, 1 x 8 on 2 x 3900 107.2 / 88.8; f32 1 x 32 x 643 106.4 / 101.2, d = 64 60.3 / 56.3).
template <typename T, int CH, bool OWN_BIAS, int NW>
__global__ __launch_bounds__(64 * NW, att_steps<T>(32 * CH / (int)sizeof(T)) == 2 ? 4 : 2) void k_attention(const T* __restrict__ q, Strides3 sq,
                                                            const T* __restrict__ k, Strides3 sk,
                                                            const T* __restrict__ vt, int Npad,
                                                            const T* __restrict__ vrm, Strides3 sv,
                                                            const float* __restrict__ bias2,
                                                            const float* __restrict__ s_hat, float lambda_max, float eps, int bidir,
                                                            T* __restrict__ out, int B, int H, int Hkv, int N, int P,
                                                            int V, float c2) {
  constexpr int QWG = 32 * NW;                 // queries per workgroup
  constexpr int E = elem<T>::per16;            // elements per 16-byte chunk
  constexpr int D = CH * 2 * E;                // head dimension
  constexpr int DT = D / 32;                   // 32-row tiles of O^T
  constexpr int SUB = att_sub<T>(D), STEPS = att_steps<T>(D), KEYS = 32 * SUB * STEPS;      // keys per turn
  constexpr int NPS = 32 * SUB / (2 * E);      // contraction steps of the second product per step of a turn
  constexpr int RB = 32 * CH;                  // bytes of a key row
  constexpr int VB = KEYS * (int)sizeof(T);    // bytes of a values^T row per turn
  static_assert(VB == 128, "att_vswz");
  constexpr int KTILE = KEYS * RB, VTILE = D * VB, BTILE = KEYS * (int)sizeof(float);
  constexpr int KLD = KTILE / 1024 / NW, VLD = VTILE / 1024 / NW;    // 1 KiB load instructions per wave and turn
  static_assert(KLD >= 1 && VLD >= 1, "every wave loads");
  constexpr int NS = ATT_NS;                   // slots of the three rings
  constexpr int VRING = NS * KTILE, BRING = VRING + NS * VTILE;
  static_assert((size_t)(BRING + NS * BTILE) == att_lds_bytes<T>(D, 0), "LDS");
  // 2-byte elements with d = 128: the values stay row-major, as the caller has them, and the second
  // product's operand is fetched with the transposing LDS read of this chip (see att_tr_read)
  constexpr bool TR = (E == 8 && CH == 8);
  extern __shared__ __align__(16) char lds[];
  const uint32_t lds_addr = lds_address(lds);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hf = lane >> 5;
  // Consecutive workgroup ids go to the 8 XCDs in turn; each XCD takes a contiguous eighth of the units
  // (image by image, head by head, 256 queries by 256 queries), so that the workgroups that read the same keys
  // and values share its L2 (with an image's blocks dealt to all eight, every L2 held the keys and values of
  // some 26 heads at a time, 31 MB at 16 x 32 heads x 2403 positions: 1.94 ms, now 1.80).
  const int qblocks = (N + QWG - 1) / QWG, units = B * H * qblocks, per_xcd = (units + NUM_XCD - 1) / NUM_XCD;
  const int block = linear_block(), slot = block / NUM_XCD;
  const int unit = (block % NUM_XCD) * per_xcd + slot;
  if (slot >= per_xcd || unit >= units) return; // the same for the whole workgroup
  const int bh = unit / qblocks, b = bh / H, h = bh - b * H, g = (h * Hkv) / H;
  const int iw = (unit - bh * qblocks) * QWG;       // first query of the workgroup
  const int i0 = iw + wave * 32;                // first query of the wave
  const float inv_c2 = 1.0f / c2;
  const float lazy_raw = ATT_LAZY * inv_c2;     // ATT_LAZY log2 units, in units of the raw products
  const int img_lo = P, img_hi = P + V;         // image span [img_lo, img_hi)

  // keys to visit: up to the last query, or to the end of the image span if image rows are held
  // (their future image keys count, discounted)
  auto last_key = [&](int first, int count) {
    const int hi = min(first + count - 1, N - 1);
    int jl = hi;
    if (bidir && hi >= img_lo && first < img_hi) jl = max(jl, img_hi - 1);
    return first < N ? jl : -1;
  };
  const int jl_wg = last_key(iw, QWG), jl_w = last_key(i0, 32);
  const int turns = jl_wg / KEYS + 1;           // the same for every wave of the workgroup
  // This wave's turns are 0 .. my_turns - 1 (none if its queries are past N).  Where the second sub-tile of another one lies
  // behind the wave's last key, it takes no part at all in that turn: a term of zero would still make NaN of a value
  // that is none, and what lies behind a short prompt may be anything.
  const int my_turns = jl_w < 0 ? 0 : (jl_w + (KEYS == 64 ? 32 : KEYS)) / KEYS;
  const bool half_turn = KEYS == 64 && jl_w >= 0 && jl_w % KEYS < 32;

  // queries: B operand of S^T, pieces 2c + hf of the row
  uint4 qa[CH];
  const int qi = i0 + n;
  {
    const char* qrow =
        reinterpret_cast<const char*>(q + b * sq.b + h * sq.h + (int64_t)min(qi, N - 1) * sq.r) + hf * 16;
#pragma unroll
    for (int c = 0; c < CH; ++c) qa[c] = ldg16(qrow + c * 32);
  }

  // Loads: a turn's keys and its values are 8 KLD and 8 VLD pieces of 1 KiB, wave w takes the pieces w, w + 8, ...; one
  // wave also brings the discounts.  Offsets move on by a turn at a time and stop at the last row (keys and
  // row-major values) or turn (values^T, discounts), so that every turn issues the same number of loads.
  const char* kg = reinterpret_cast<const char*>(k + b * sk.b + g * sk.h);
  const char* vg = TR ? reinterpret_cast<const char*>(vrm + b * sv.b + g * sv.h)
                      : reinterpret_cast<const char*>(vt + ((int64_t)b * Hkv + g) * D * Npad);
  const char* bg = reinterpret_cast<const char*>(bias2 + (int64_t)b * Npad);
  const int off0 = wave * 1024 + 16 * lane;    // of the wave's first piece in a slot
  auto rows_ahead = [](int64_t bytes) { return (uint32_t)min(bytes, (int64_t)0x7fffffff); };
  const int64_t krow_bytes = sk.r * (int64_t)sizeof(T), vrow_bytes = TR ? sv.r * (int64_t)sizeof(T) : Npad * (int64_t)sizeof(T);
  constexpr int KSTEP = 1024 * NW / RB, VSTEP = 1024 * NW / (TR ? RB : VB);     // rows between two pieces of a wave
  // (KFLIP: the wave's odd pieces are eight rows on from its even ones, and the swizzle repeats after 16)
  constexpr bool KFLIP = RB > 128 && (KSTEP & 15) == 8;
  static_assert(KFLIP || (KSTEP & 15) == 0, "swizzle");
  const int krow = off0 / RB, kpiece = ((off0 % RB) >> 4) ^ att_kswz(krow, RB);
  const uint32_t kpart[2] = {(uint32_t)kpiece * 16, (uint32_t)(kpiece ^ 8) * 16};      // with KFLIP added last
  const uint32_t kmax = (uint32_t)((N - 1) * krow_bytes) + (KFLIP ? 0 : kpart[0]);
  uint32_t koff = (uint32_t)min((int64_t)krow, (int64_t)N - 1) * (uint32_t)krow_bytes + (KFLIP ? 0 : kpart[0]);
  const uint32_t kturn = rows_ahead(KEYS * krow_bytes), kstep = rows_ahead(KSTEP * krow_bytes);
  uint32_t voff, vmax, vturn, vstep;
  if constexpr (TR) {
    // row-major values: piece p of row r in slot p ^ 4 (r & 3)
    const int row = off0 / RB, piece = ((off0 % RB) >> 4) ^ ((row & 3) << 2);
    vmax = (uint32_t)((N - 1) * vrow_bytes) + piece * 16;
    voff = (uint32_t)min(row, N - 1) * (uint32_t)vrow_bytes + piece * 16;
    vturn = rows_ahead(KEYS * vrow_bytes);
    vstep = rows_ahead(VSTEP * vrow_bytes);
  } else {
    const int row = off0 / VB, piece = ((off0 % VB) >> 4) ^ att_vswz(row);
    voff = (uint32_t)(row * vrow_bytes) + piece * 16;
    vmax = voff + (uint32_t)(turns - 1) * VB;
    vturn = VB;
    vstep = (uint32_t)(VSTEP * vrow_bytes);
  }
  // (pieces past the second follow from the one before, as u * step may pass 2^32)
  uint32_t kpast = 0, vpast = 0;
  auto issue_keys = [&](uint32_t slot, int u) {       // piece u of the next turn's, u = 0, 1, ... in this order
    const uint32_t off = u ? min((u > 1 ? kpast : koff) + kstep, kmax) : koff;
    if (KLD > 2) kpast = off;
    load_to_lds16(kg, KFLIP ? off + kpart[u & 1] : off, lds_addr + slot * KTILE + wave * 1024 + u * NW * 1024);
    if (u == KLD - 1) koff = min(koff + kturn, kmax);
  };
  auto issue_values = [&](uint32_t slot, int u) {
    const uint32_t next = (u > 1 ? vpast : voff) + vstep, off = u ? (TR ? min(next, vmax) : next) : voff;
    if (VLD > 2) vpast = off;
    load_to_lds16(vg, off, lds_addr + VRING + slot * VTILE + wave * 1024 + u * NW * 1024);
    if (u == VLD - 1) voff = min(voff + vturn, vmax);
  };
  const bool bias_wave = !OWN_BIAS && wave == 0;          // the one that brings the discounts
  auto issue_bias = [&](uint32_t slot, int t) {
    if (!OWN_BIAS && bias_wave && lane < BTILE / 16)
      load_to_lds16(bg, (uint32_t)(min(t, turns - 1) * BTILE + 16 * lane), lds_addr + BRING + slot * BTILE);
  };
  // all but the loads of the newest two turns, or of the newest one
  constexpr int OPEN = STEPS == 1 ? 2 : 1;
  auto wait_turn = [&] {
    if (bias_wave) wait_vmem_but<OPEN * (KLD + VLD + 1)>();
    else wait_vmem_but<OPEN * (KLD + VLD)>();
  };

  f32x16_t o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[t][v] = 0.0f;
  float m_run = -INFINITY, l_run = 0.0f;

  // Operand addresses of slot 0, one register each: hidden from the compiler, which would otherwise form them
  // anew for every turn; a turn's slot is then an immediate offset.
  auto hidden = [](uint32_t x) { asm volatile("" : "+v"(x)); return x; };
  auto lds_read16 = [](uint32_t addr) {
    const auto x = *(const __attribute__((address_space(3))) u32x4_nt*)(uintptr_t)addr;
    return make_uint4(x.x, x.y, x.z, x.w);
  };
  uint32_t k_at[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) k_at[c] = hidden(lds_addr + n * RB + (((2 * c + hf) ^ att_kswz(n, RB)) << 4));
  // Transposing read (TR): a lane is both a source -- it names 8 bytes, four consecutive columns of one key
  // row -- and a receiver.  Inside a group of 16 lanes, source 4 i + a names key i of four consecutive
  // keys and column block a, and lane 4 a + c receives column 4 a + c of those four keys: the 16 lanes
  // cover 16 consecutive columns (rows of values^T) with four keys each, which is half of the
  // operand.  The key of slot e of contraction step c for lane half hf is 16 c + 8 (e / 4) + 4 hf + e % 4,
  // the order in which the first product leaves P^T in the accumulators.
  // Row tile tt of values^T = columns 32 tt .. 32 tt + 31 = 16-byte pieces 4 tt .. 4 tt + 3 of a key row, stored in
  // slots (4 tt + x) ^ 4 (key & 3).
  // (Otherwise: the values^T swizzle of row tt * 32 + n looks at row bits below 5 only, so one address per
  // contraction step serves all DT row tiles.)
  uint32_t v_at[TR ? DT : NPS * STEPS];
  if constexpr (TR) {
    const int src16 = lane & 15, src_key = src16 >> 2;
    const int base = (4 * hf + src_key) * RB + ((2 * ((lane >> 4) & 1) + ((src16 & 3) >> 1)) << 4) + 8 * (src16 & 1);
#pragma unroll
    for (int tt = 0; tt < DT; ++tt) v_at[tt] = hidden(lds_addr + VRING + base + ((tt ^ src_key) << 6));
  } else {
#pragma unroll
    for (int c = 0; c < NPS * STEPS; ++c) v_at[c] = hidden(lds_addr + VRING + n * VB + (((2 * c + hf) ^ att_vswz(n)) << 4));
  }

  // The matrix phase in front of the next step: S^T of the wave's queries against that step's keys (raw, unscaled
  // products), then O^T += V^T P^T of this one: piece 2c + hf of a values^T row holds the keys this lane half has in
  // P^T.  Item by item, in this order: one product, and the LDS read of the operand AHEAD products on -- the first ones
  // in front of the barrier, so that no product waits for LDS (left to itself the compiler reads an operand right in
  // front of its product).
  constexpr int SI = CH * SUB, ITEMS = SI + NPS * DT, AHEAD = STEPS == 2 ? 3 : 5, RING = AHEAD + 1;
  f32x16_t s[SUB];
  uint4 pb[NPS], op[RING];
  auto read_value = [&](uint32_t slot, auto y_c, auto i_c) __attribute__((always_inline)) {
    constexpr int c = decltype(y_c)::value * NPS + decltype(i_c)::value / DT, tt = decltype(i_c)::value % DT;
    if constexpr (TR) {
      const uint32_t src = v_at[tt] + slot * VTILE + 16 * c * RB;
      const uint2 lo = att_tr_read(src), hi = att_tr_read(src + 8 * RB);
      return make_uint4(lo.x, lo.y, hi.x, hi.y);
    } else {
      return lds_read16(v_at[c] + slot * VTILE + tt * 32 * VB);
    }
  };
  // (at_c: where the keys of the next step lie in their ring, cur_c and y_c: turn's slot and step of the values)
  auto read_item = [&](auto i_c, auto at_c, auto cur_c, auto y_c) {
    constexpr int I = decltype(i_c)::value;
    if constexpr (I < SI) {
      op[I % RING] = lds_read16(k_at[I / SUB] + decltype(at_c)::value + (I % SUB) * 32 * RB);
    } else if constexpr (I < ITEMS) {
      op[I % RING] = read_value(decltype(cur_c)::value, y_c, std::integral_constant<int, I - SI>{});
    }
  };
  auto first_items = [&](auto at_c, auto cur_c, auto y_c) {
    static_for<AHEAD>([&](auto i_c) { read_item(i_c, at_c, cur_c, y_c); });
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](auto at_c, auto cur_c, auto y_c, auto count_c, auto loads) {
#pragma unroll
    for (int x = 0; x < SUB; ++x)
#pragma unroll
      for (int v = 0; v < 16; ++v) s[x][v] = 0.0f;
    static_for<decltype(count_c)::value>([&](auto i_c) {
      constexpr int I = decltype(i_c)::value;
      if constexpr (I < SI) mma32<T>(s[I % SUB], op[I % RING], qa[I / SUB]);
      else mma32<T>(o[(I - SI) % DT], op[I % RING], pb[(I - SI) / DT]);
      if constexpr (I + AHEAD < decltype(count_c)::value) read_item(std::integral_constant<int, I + AHEAD>{}, at_c, cur_c, y_c);
      loads(i_c);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // The second product of a turn's first sub-tile alone.
  auto first_values = [&](uint32_t slot) __attribute__((always_inline)) {
    static_for<NPS / SUB * DT>([&](auto i_c) {
      mma32<T>(o[decltype(i_c)::value % DT], read_value(slot, std::integral_constant<int, 0>{}, i_c), pb[decltype(i_c)::value / DT]);
    });
  };
  // The vector phase of step y of turn t, of its first or of all sub-tiles: the mask on the raw scores, the baseline, the softmax terms.
  // The exponent's baseline m_run of a query follows the running maximum lazily: it moves only when the
  // maximum has grown by more than ATT_LAZY (in log2 units), so that the accumulated columns are rescaled
  // a few times per query instead of at most turns; terms are then at most 2^ATT_LAZY, and the quotient
  // O / l does not depend on the baseline.
  const bool wave_img = bidir && i0 >= img_lo && i0 + 31 < img_hi;
  auto softmax = [&](uint32_t slot, int t, int y, auto subs_c) __attribute__((always_inline)) {
    constexpr int SUBS = decltype(subs_c)::value;
#pragma unroll
    for (int x = 0; x < SUBS; ++x) {
      // the mask, by the kind of sub-tile (a wave-uniform choice; ATT_PLAIN: raw, the scale goes into the exponent)
      const int j0 = t * KEYS + 32 * (y * SUB + x);
      const int mode = (j0 + 31 <= i0) ? ATT_PLAIN : (j0 > i0 + 31 && wave_img) ? ATT_AHEAD : ATT_GENERAL;
      if (mode == ATT_PLAIN) continue;
      // discounts of this lane's 16 keys
      const char* Bt = lds + BRING + (OWN_BIAS ? 4 * j0 : slot * BTILE + 128 * (y * SUB + x));
      float kbias[16];
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const float4 y = *reinterpret_cast<const float4*>(Bt + (8 * gq + 4 * hf) * 4);
        kbias[4 * gq] = y.x; kbias[4 * gq + 1] = y.y; kbias[4 * gq + 2] = y.z; kbias[4 * gq + 3] = y.w;
      }
      if (mode == ATT_AHEAD) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s[x][v] = fmaf(kbias[v], inv_c2, s[x][v]);
      } else {
        const bool q_img = bidir && qi >= img_lo && qi < img_hi;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int j = j0 + att_key_of(v, hf);
          const float ahead = q_img ? kbias[v] : -INFINITY;      // a key after the query
          s[x][v] += (j <= qi ? 0.0f : ahead) * inv_c2;
        }
      }
    }
    float mx = s[0][0];
#pragma unroll
    for (int x = 0; x < SUBS; ++x)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[x][v]);
    {
      const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(y[0]), __uint_as_float(y[1]));      // both lane halves of a query see the same maximum
    }
    // maxima are kept in units of the raw products (finite from the first turn on: key 0 precedes
    // every query)
    const bool moved = mx > m_run + lazy_raw;
    if (__any(moved)) {
      const float m_new = moved ? mx : m_run;
      float alpha = fast_exp2_att((m_run - m_new) * c2);
      // The products below are assembly, for which the compiler keeps none of the distances that a use of an exponential's
      // result, or of a matrix product's, needs.
      asm volatile("s_nop 15\n\ts_nop 15" : "+v"(alpha));
      m_run = m_new;
      l_run *= alpha;
      // in place, as assembly: a plain product is hoisted above the branch and the untouched
      // accumulators are then copied register by register on the path that skips it
#pragma unroll
      for (int tt = 0; tt < DT; ++tt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float x = o[tt][v];
          asm volatile("v_mul_f32 %0, %0, %1" : "+v"(x) : "v"(alpha));
          o[tt][v] = x;
        }
    }
    const float m_c = m_run * c2;
    float psum[SUBS];
#pragma unroll
    for (int x = 0; x < SUBS; ++x) {
      float p[16];
      psum[x] = 0.0f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        p[v] = fast_exp2_att(fmaf(s[x][v], c2, -m_c));
        psum[x] += p[v];
      }
#pragma unroll
      for (int c = 0; c < NPS / SUB; ++c) pb[x * (NPS / SUB) + c] = att_pack16<T>(&p[c * E]);
    }
    l_run += SUBS == 2 ? psum[0] + psum[SUBS - 1] : psum[0];
    asm volatile("" : "+v"(l_run));            // here, not between the products and the barrier (2 % of the whole)
  };

  // Turn t of a wave: the softmax of a step, then the products in front of the next, then the turn's one barrier.
  // Under the products the wave asks for its share of the keys of turn t + 4, of the values of turn t + 3 and of the
  // discounts of turn t + 3, into slots that were last read before the previous barrier (keys of turn t, values and
  // discounts of turn t - 1).  At the barrier everything but the newest two turns' loads has landed: the keys of
  // turn t + 2, the values and discounts of turn t + 1, i.e. what turn t + 1 reads.
  // In two steps, turn t reads keys of its own as well as of turn t + 1: the keys asked for are those of turn t + 3 too, and
  // at the barrier everything but the newest turn's loads has landed, the keys of turn t + 2 among them.
  static_for<3>([&](auto t_c) {
    constexpr int U = decltype(t_c)::value;
#pragma unroll
    for (int u = 0; u < KLD; ++u) issue_keys(U, u);
    issue_bias(U, U);
    if constexpr (U > 0 || STEPS == 2) {
#pragma unroll
      for (int u = 0; u < VLD; ++u) issue_values(STEPS == 2 ? U : U - 1, u);
    }
  });
  // The discounts, with all of these loads on their way; and the queries are touched here so that the compiler's wait for
  // their loads stands in front of the loop, not inside it, where it would also wait for the ring.  (In front
  // of the ring's first loads that wait was a round trip to memory of its own.)
  if (OWN_BIAS && bidir) {
    const float* sh = s_hat + (int64_t)b * V;
    for (int j = tid; j < turns * KEYS; j += 64 * NW)
      *reinterpret_cast<float*>(lds + BRING + 4 * j) = att_bias(sh, j, P, V, lambda_max, eps);
  }
#pragma unroll
  for (int c = 0; c < CH; ++c) asm volatile("" ::"v"(qa[c].x), "v"(qa[c].y), "v"(qa[c].z), "v"(qa[c].w));
  auto end_turn = [&] {
    wait_turn();
    __builtin_amdgcn_sched_barrier(0);
    barrier_keep_loads();
    __builtin_amdgcn_sched_barrier(0);
  };
  wait_turn();
  barrier_lds();
  __builtin_amdgcn_sched_barrier(0);
  {
    constexpr std::integral_constant<int, 0> zero{};
    first_items(zero, zero, zero);
    multiply(zero, zero, zero, std::integral_constant<int, SI>{}, [&](auto i_c) {
      constexpr int I = decltype(i_c)::value;
      if constexpr (STEPS == 2) return;
      else if constexpr (I < KLD) issue_keys(3, I);
      else if constexpr (I < KLD + VLD) issue_values(2, I - KLD);
      else if constexpr (I == KLD + VLD) issue_bias(2, 2);
    });
    if constexpr (STEPS == 1) end_turn();
  }
  auto loads = [&](auto i_c, uint32_t slot, int t) {        // turn t's, spread over the products
    constexpr int I = decltype(i_c)::value, EVERY = STEPS * ITEMS / (KLD + VLD), J = I / EVERY;
    if constexpr (I % EVERY == 2) {
      if constexpr (J < KLD) issue_keys((slot + (STEPS == 2 ? 3 : 0)) % NS, J);
      else if constexpr (J < KLD + VLD) issue_values((slot + 3) % NS, J - KLD);
    }
    if constexpr (I == 4) issue_bias((slot + 3) % NS, t + 3);
  };
  for (int t0 = 0; t0 < my_turns; t0 += NS) {
    static_for<NS>([&](auto u_c) {
      constexpr int U = decltype(u_c)::value;
      const int t = t0 + U;
      if (t < my_turns) {
        static_for<STEPS>([&](auto y_c) {
          constexpr int Y = decltype(y_c)::value;
          softmax(U, t, Y, std::integral_constant<int, SUB>{});
          constexpr std::integral_constant<int, Y + 1 < STEPS ? U * KTILE + (Y + 1) * 32 * SUB * RB : (U + 1) % NS * KTILE> at{};
          first_items(at, u_c, y_c);
          __builtin_amdgcn_s_setprio(1);
          multiply(at, u_c, y_c, std::integral_constant<int, ITEMS>{},
                   [&](auto i_c) { loads(std::integral_constant<int, Y * ITEMS + decltype(i_c)::value>{}, U, t); });
          __builtin_amdgcn_s_setprio(0);
        });
        end_turn();
      }
    });
  }
  // The workgroup's turns that this wave takes half a part in, or none: its loads and barriers stay.
  for (int t = my_turns; t < turns; ++t) {
    const uint32_t slot = t % NS;
    if (t == my_turns && half_turn) {
      softmax(slot, t, 0, std::integral_constant<int, 1>{});
      first_values(slot);
    }
    static_for<STEPS * ITEMS>([&](auto i_c) { loads(i_c, slot, t); });
    end_turn();
  }
  wait_all_vmem();                             // the surplus requests of the last iterations

  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const float inv = 1.0f / l_tot;
  if (qi < N) {
    T* orow = out + (((int64_t)b * H + h) * N + qi) * D;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        float f[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = o[t][4 * gq + e] * inv;
        store4<T>(orow + t * 32 + 8 * gq + 4 * hf, f);
      }
  }
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
static int att_npad(const asap_params& p) { return ((p.P + p.V + p.Tmax + 31) / 32) * 32 + 32; }

// bf16 values with d = 128 are read as they are; every other case goes through a transposed copy
static bool att_row_major_values(const asap_params& p) { return p.qk_dtype == ASAP_BF16 && p.d == 128; }

size_t attention_workspace_bytes(const asap_params& p) {
  const size_t es = p.qk_dtype == ASAP_BF16 ? 2 : 4;
  const size_t vt = att_row_major_values(p) ? 0 : align256(es * (size_t)p.B * p.Hkv * p.d * att_npad(p));
  return vt + align256(sizeof(float) * (size_t)p.B * att_npad(p));
}

template <typename T>
static hipError_t attention_typed(const asap_params& p, const void* q, Strides3 sq, const void* k, Strides3 sk,
                                  const void* v, Strides3 sv, const float* s_hat, void* out, char* ws,
                                  hipStream_t st, Timer* tm) {
  constexpr int E = elem<T>::per16;
  const int N = p.P + p.V + p.Tmax, Npad = att_npad(p);
  const bool row_major_values = att_row_major_values(p);    // the kernel transposes while it reads LDS
  T* vt = reinterpret_cast<T*>(ws);                         // (not used then)
  float* bias2 = reinterpret_cast<float*>(
      ws + (row_major_values ? 0 : align256(sizeof(T) * (size_t)p.B * p.Hkv * p.d * Npad)));
  const bool bidir = p.mask_mode == ASAP_MASK_KEYBIAS;
  // (with the mask off the table is -inf everywhere and s_hat is not read)
  const bool own_bias = att_own_bias<T>(p.d, Npad);
  if (!own_bias)
    ASAP_LAUNCH(tm, "k_att_bias", k_att_bias, dim3((Npad + 255) / 256, p.B), dim3(256), 0, st, bidir ? s_hat : nullptr,
              p.P, p.V, Npad, p.lambda_max, p.eps, bias2);
  if (!row_major_values)
    ASAP_LAUNCH(tm, "k_vtranspose", k_vtranspose<T>, dim3(Npad / 32, p.Hkv, p.B), dim3(256), 0, st,
                static_cast<const T*>(v), sv, N, Npad, p.d, vt);
  const float c2 = 1.4426950408889634f / sqrtf((float)p.d);
  // Four waves per workgroup, one per SIMD, where the chip then still holds all of them at a time: a turn takes a wave that has a
  // SIMD to itself little more than half as long (1 x 40 heads x 643 positions 27.5 -> 20.9 us; d = 64, 16 heads 21.8 -> 18.8; f32, 32
  // heads 175 -> 101; 2 x 32 x 643, in two rounds then, 30.0 -> 37.5, f32 176 -> 187).
  auto units_of = [&](int queries) { return p.B * p.H * ((N + queries - 1) / queries); };
  const bool four = own_bias && units_of(128) <= 256;
  const int units = units_of(four ? 128 : 32 * ATT_NW);
  const dim3 grid = grid_of(NUM_XCD * (int64_t)((units + NUM_XCD - 1) / NUM_XCD));
  const size_t lds = att_lds_bytes<T>(p.d, own_bias ? Npad : 0);
#define ASAP_ATT(CHV, OWN, NWV)                                                                                    \
  do {                                                                                                         \
    auto kern = k_attention<T, CHV, OWN, NWV>;                                                                 \
    if (lds > 48 * 1024) {                                                                                     \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                  \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                \
      if (e != hipSuccess) return e;                                                                           \
    }                                                                                                          \
    ASAP_LAUNCH(tm, "k_attention", kern, grid, dim3(64 * NWV), lds, st, static_cast<const T*>(q), sq,          \
                static_cast<const T*>(k), sk, vt, Npad, static_cast<const T*>(v), sv, bias2, s_hat,            \
                p.lambda_max, p.eps, bidir ? 1 : 0, static_cast<T*>(out), p.B, p.H, p.Hkv, N, p.P, p.V, c2);   \
  } while (0)
  if (p.d != 64 && p.d != 128) return hipErrorInvalidValue;
  if (four) {
    if (p.d == 64) ASAP_ATT(32 / E, true, 4);
    else ASAP_ATT(64 / E, true, 4);
  } else if (own_bias) {
    if (p.d == 64) ASAP_ATT(32 / E, true, ATT_NW);
    else ASAP_ATT(64 / E, true, ATT_NW);
  } else {
    if (p.d == 64) ASAP_ATT(32 / E, false, ATT_NW);
    else ASAP_ATT(64 / E, false, ATT_NW);
  }
#undef ASAP_ATT
  return hipGetLastError();
}

hipError_t launch_attention(const asap_params& p, const void* q, Strides3 sq, const void* k, Strides3 sk,
                            const void* v, Strides3 sv, const float* s_hat, void* out, char* ws, hipStream_t st,
                            Timer* tm) {
  if (p.qk_dtype == ASAP_BF16) return attention_typed<bf16_t>(p, q, sq, k, sk, v, sv, s_hat, out, ws, st, tm);
  return attention_typed<float>(p, q, sq, k, sk, v, sv, s_hat, out, ws, st, tm);
}

}  // namespace asap
