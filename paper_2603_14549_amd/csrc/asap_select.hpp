// Exact top-k selection inside one 1024-thread workgroup, shared by the selection kernels and by the
// budget reallocation of the paper's routing.  Integer work throughout.
//   What bounds it: the chain of barriers and LDS round trips of one workgroup.  So the keys are dealt to 256 bins of equal
//   width between the smallest and the largest, the bin of the k-th largest is found by every wave for itself, and the
//   bin's keys are dealt again until at most 64 are left, which one wave ranks against each other.  (A radix search over
//   the 32 bits takes four such passes with a wave that the others wait for in each, and its first digit, sign and
//   exponent, puts nearly every score into two or three bins, whose atomics queue up.)
//   k_select, 1 x 2304 tokens: 10.9 -> 5.9 us; 4 x 4096: 13.5 -> 9; the plan of the paper's routing 16 x 2304: stage 348 ->
//   337 us.
#pragma once
#include "asap_device.hpp"

namespace asap {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_IPT = 16;   // V <= 16384
// Items per thread that a kernel is compiled for (1, 4 or 16): one workgroup runs its code once, and fetching unrolled
// steps that it skips is a good part of its time (1 x 576 tokens: 9.8 us compiled for 16 items, 8.1 for one; 1 x 2304: 7.6 and, for four, 5.9).
template <typename F> static auto with_ipt(int V, F&& f) {
  if (V <= SEL_THREADS) return f(std::integral_constant<int, 1>{});
  if (V <= 4 * SEL_THREADS) return f(std::integral_constant<int, 4>{});
  return f(std::integral_constant<int, SEL_IPT>{});
}

// order-preserving map float -> uint32 (larger float, larger key); every float maps above 0, the NaN of all ones too
__device__ __forceinline__ uint32_t float_key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? max(~u, 1u) : (u | 0x80000000u);
}

__device__ __forceinline__ float float_unkey(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// inclusive sums over the lanes of a wave
__device__ __forceinline__ int wave_scan_incl(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);      // row_bcast:15 to rows 1 and 3, row_bcast:31 to
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);      // rows 2 and 3
  return x;
}

// exclusive block scan of one int per thread; returns the exclusive prefix, total via *total.
__device__ __forceinline__ int block_scan_excl(int x, int* wave_sums /*[17]*/, int* total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int incl = wave_scan_incl(x);
  __syncthreads();                       // protects wave_sums against the previous use
  if (lane == 63) wave_sums[wave] = incl;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < SEL_THREADS / 64; ++w) {
    int s = wave_sums[w];
    if (w < wave) base += s;
    tot += s;
  }
  *total = tot;
  return base + incl - x;
}

// LDS the selection needs
constexpr int SEL_LIST = 64;
struct SelectShared {
  uint4 hist[2][64];      // two histograms of 256 bins used alternately
  uint2 list[SEL_LIST];   // (key, item) of the bin that holds the take-th largest
  uint2 wave_range[SEL_THREADS / 64];      // (smallest, largest) key
  int wave_sums[17];
  int listed;
  uint2 last;             // the take-th largest (key, item)
};

// Thread tid holds the keys of items i0 .. i0+ipt-1 (blocked layout, so index order = thread order);
// items past V or not taking part carry key 0 and `take` must not exceed the number of keys > 0.
// Returns the bit mask of this thread's items among the `take` largest (ties: smaller index) and
// their count.  All threads of the workgroup must call it; take is the same for all.
template <int IPT>
__device__ __forceinline__ uint32_t topk(const uint32_t (&key)[IPT], int ipt, int i0, int V, int take, SelectShared& sh,
                                         int* n_mine) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  *n_mine = 0;
  if (take <= 0) return 0u;
  // smallest and largest key (of those that take part), first of the wave, then of all
  uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int e = 0; e < IPT; ++e)
    if (e < ipt && i0 + e < V && key[e] != 0u) { lo = min(lo, key[e]); hi = max(hi, key[e]); }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
  }
  __syncthreads();                       // the arrays may still be read from an earlier call
  if (lane == 0) sh.wave_range[wave] = make_uint2(lo, hi);
  if (tid < 128) (&sh.hist[0][0])[tid] = make_uint4(0, 0, 0, 0);
  if (tid == 0) sh.listed = 0;
  __syncthreads();
  {
    const uint2 r = sh.wave_range[lane & (SEL_THREADS / 64 - 1)];
    lo = r.x;
    hi = r.y;
#pragma unroll
    for (int off = SEL_THREADS / 128; off >= 1; off >>= 1) {
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
    }
  }
  // The window [lo, lo + bins 2^shift); the first holds every key, the next one bin of the one before and no key above it
  // (those are counted already), so it has fewer than 256 bins where that bin is narrower.  (Keys 0 lie below the first
  // window and count with its first bin: they are never taken while others are left.)
  const uint32_t width = hi > lo ? hi - lo : 0u;
  int shift = width < 256u ? 0 : 24 - __clz((int)width), left = take, size, pass = 0;
  uint32_t at, bins = 256u;
  auto bin = [&](uint32_t k) { return k < lo ? (pass == 0 ? 0u : 256u) : (k - lo) >> shift; };
  for (;; ++pass) {
    int* h = reinterpret_cast<int*>(sh.hist[pass & 1]);
#pragma unroll
    for (int e = 0; e < IPT; ++e) {
      if (e < ipt && i0 + e < V) {
        const uint32_t x = bin(key[e]);
        if (x < bins) atomicAdd(&h[x], 1);
      }
    }
    __syncthreads();
    // every wave walks the bins from 255 down: lane l holds bins 255 - 4l .. 252 - 4l
    const uint4 q4 = sh.hist[pass & 1][63 - lane];
    const int c[4] = {(int)q4.w, (int)q4.z, (int)q4.y, (int)q4.x};
    const int all = c[0] + c[1] + c[2] + c[3];
    int above = wave_scan_incl(all) - all, b = -1, l = 0, n = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (above < left && above + c[q] >= left) { b = 255 - (4 * lane + q); l = left - above; n = c[q]; }
      above += c[q];
    }
    const int who = __ffsll((unsigned long long)__ballot(b >= 0)) - 1;
    at = (uint32_t)__builtin_amdgcn_readlane(b, who);
    left = __builtin_amdgcn_readlane(l, who);
    size = __builtin_amdgcn_readlane(n, who);
    if (size <= SEL_LIST || shift == 0) break;                  // the same for all
    if (pass > 0) {                                             // both histograms have been used
      __syncthreads();
      if (tid < 64) sh.hist[(pass + 1) & 1][tid] = make_uint4(0, 0, 0, 0);
      __syncthreads();
    }
    lo += at << shift;
    bins = 1u << min(shift, 8);
    shift = max(shift - 8, 0);
  }
  uint32_t bits = 0;
  int n = 0;
  if (size <= SEL_LIST) {
    // the keys of that bin, ranked against each other: the one with left - 1 in front of it is the last taken
#pragma unroll
    for (int e = 0; e < IPT; ++e) {
      if (e < ipt && i0 + e < V) {
        if (bin(key[e]) == at) sh.list[atomicAdd(&sh.listed, 1)] = make_uint2(key[e], (uint32_t)(i0 + e));
      }
    }
    __syncthreads();
    if (wave == 0) {
      const uint2 mine = sh.list[lane];
      int rank = lane < size ? 0 : SEL_LIST;
      for (int x = 0; x < size; ++x) {
        const uint32_t ok = (uint32_t)__builtin_amdgcn_readlane((int)mine.x, x), oi = (uint32_t)__builtin_amdgcn_readlane((int)mine.y, x);
        rank += (ok > mine.x || (ok == mine.x && oi < mine.y)) ? 1 : 0;
      }
      if (rank == left - 1) sh.last = mine;
    }
    __syncthreads();
    const uint2 last = sh.last;
#pragma unroll
    for (int e = 0; e < IPT; ++e) {
      const int i = i0 + e;
      if (e < ipt && i < V && (key[e] > last.x || (key[e] == last.x && (uint32_t)i <= last.y))) { bits |= 1u << e; ++n; }
    }
  } else {
    // a bin of one key value (shift is 0), more than SEL_LIST times: `left` of them are taken, smallest index first.  (In
    // the first window the keys 0 count with the smallest key; they come after it.)
    const uint32_t thr = lo + at;
    int n_eq = 0;
#pragma unroll
    for (int e = 0; e < IPT; ++e)
      if (e < ipt && i0 + e < V && key[e] == thr) ++n_eq;
    int tot;
    int eq_before = block_scan_excl(n_eq, sh.wave_sums, &tot);
#pragma unroll
    for (int e = 0; e < IPT; ++e) {
      const int i = i0 + e;
      if (e < ipt && i < V) {
        bool keep = key[e] > thr;
        if (key[e] == thr) { keep = eq_before < left; ++eq_before; }
        if (keep) { bits |= 1u << e; ++n; }
      }
    }
  }
  *n_mine = n;
  return bits;
}

}  // namespace asap
