// tail.h -- the ends of short launches.
//
// Short calls are bound by launches: a block of 10007 samples at one SNR point
// took 5.8 us in its first tier and 2.0 + 2.8 + 4.8 us in the three kernels
// after it, which had almost nothing to do. There the second tier reads the
// first tier's lists itself, and the last block of a call's last demapping
// kernel reduces the sums: two kernels, 20.6 -> 13.0 us per call. (The gathering
// in the first tier's last block instead cost that kernel 4 % on full sweeps.)
#pragma once
#include "tier2_list.h"

namespace air {

// Whether this block is the last of the launch to get here; every block of the
// launch calls it once, after its last write for other blocks. Those writes
// and the last block's reads (BlockSums, which has no other access) go past the
// caches that the blocks do not share, and a thread waits for its own before
// it gets here. No fence: one at device scope writes back the whole L2, with
// the LLRs in it (1e5 samples: +30 us). The ticket is zero again afterwards.
__device__ __forceinline__ bool last_block(unsigned int* ticket) {
  __shared__ int last;
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned int n = gridDim.x * gridDim.y;
    const unsigned int t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = t == n - 1u;
    if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return last != 0;
}

// Statistics of SNR point s by one block of 256 threads: wave q sums quantity
// q over the blocks of both tiers in a fixed order (lane l takes blocks l,
// l + 64, ...; then a fixed butterfly), so the result does not depend on
// timing. stats[4 s + q] = MI, GMI, SE_MI, SE_GMI; NaN if a tx index was
// invalid. SUM: how lane l's share of one list is read.
template <typename SUM>
__device__ __forceinline__ void finish_point(int s, int64_t N, int M, int m, bool bad, int no_mi,
                                             double* stats, SUM&& sum) {
  __shared__ double sums[4];
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double t = wave_sum(sum(s, q, lane));
  if (lane == 0) sums[q] = t;
  __syncthreads();
  if (threadIdx.x == 0 && stats) {
    const double n = (double)N;
    const double su = sums[0], sv = sums[1], suu = sums[2], svv = sums[3];
    double mi = log2((double)M) - su / n;
    double gmi = (double)m - sv / n;
    double se_mi = __builtin_nan(""), se_gmi = __builtin_nan("");
    if (N > 1) {
      const double vu = (suu - su * su / n) / (n - 1.0);
      const double vv = (svv - sv * sv / n) / (n - 1.0);
      se_mi = sqrt((vu > 0.0 ? vu : 0.0) / n);
      se_gmi = sqrt((vv > 0.0 ? vv : 0.0) / n);
    }
    if (no_mi) mi = se_mi = __builtin_nan("");       // max-log: no symbol-wise MI
    if (bad) mi = gmi = se_mi = se_gmi = __builtin_nan("");
    stats[4 * s + 0] = mi;
    stats[4 * s + 1] = gmi;
    stats[4 * s + 2] = se_mi;
    stats[4 * s + 3] = se_gmi;
  }
  __syncthreads();
}

// The end of a call in the last block of its last demapping kernel. nblocks:
// blocks of the first tier's partials.
__device__ __forceinline__ void finish_in_last_block(const DemapArgs& a, int nblocks) {
  if (!a.fin.in_last_block || !last_block(a.fin.ticket)) return;
  const bool bad = from_other_block(&a.fin.call->err) != 0;
  if (a.fin.stats)
    for (int s = 0; s < a.S; ++s)
      finish_point(s, a.N, a.M, a.m, bad, a.fin.no_mi, a.fin.stats, [&](int sp, int q, int lane) {
        double t = 0.0;
#pragma unroll 4
        for (int i = lane; i < nblocks; i += 64) t += a.partials.get(4 * sp + q, i, nblocks);
#pragma unroll 4
        for (int i = lane; i < a.fin.blocks2; i += 64) t += a.t2_partials.get(4 * sp + q, i, a.fin.blocks2);
        return t;
      });
  if (threadIdx.x == 0) {
    if (bad) flag_sticky(a.fin.sticky);
    clear_call_words(a.fin.next);
  }
}

// Short lists: one SNR point and at most 256 first-tier waves (16384 samples).
// The second tier's blocks scan the waves' counts themselves and find each
// item in its wave's list, without the gathering kernel between the tiers.
constexpr int kShortWaves = 256;

// The counts' exclusive sums to pre[0 .. 255] (block-wide, 256 threads);
// returns their total.
__device__ __forceinline__ unsigned int short_scan(const DemapArgs& a, unsigned int (&pre)[kShortWaves]) {
  __shared__ unsigned int wtot[4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const unsigned int own = t < a.blocks1 * 4 ? a.t2_nitem[t] : 0u;
  unsigned int inc = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int v = __shfl_up(inc, off);
    if (lane >= off) inc += v;
  }
  if (lane == 63) wtot[wave] = inc;
  __syncthreads();
  unsigned int base = 0, all = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    base += k < wave ? wtot[k] : 0u;
    all += wtot[k];
  }
  pre[t] = base + inc - own;
  __syncthreads();
  return all;
}

// Sample index of item `pos` (below the total): in (wave, slot, lane) order,
// as the gathering kernel lists them.
__device__ __forceinline__ uint32_t short_item(const DemapArgs& a, const unsigned int (&pre)[kShortWaves],
                                               unsigned int pos) {
  int w = 0;                               // the last wave whose first item is <= pos
#pragma unroll
  for (int step = kShortWaves / 2; step >= 1; step >>= 1)
    if (pre[w + step] <= pos) w += step;
  unsigned int r = pos - pre[w];
  const unsigned long long* src = a.t2_list + (int64_t)w * a.t2_tpw;
  for (int q = 0; q < a.t2_tpw; ++q) {
    const unsigned long long ent = src[q];
    uint32_t mask = (uint32_t)(ent >> 32);
    const unsigned int c = (unsigned int)__builtin_popcount(mask);
    if (r < c) {
      for (; r > 0; --r) mask &= mask - 1u;
      return (uint32_t)(ent & 0xffffffffull) * 32u + (uint32_t)__builtin_ctz(mask);
    }
    r -= c;
  }
  return 0u;                               // (not reached: the counts match the lists)
}

}  // namespace air
