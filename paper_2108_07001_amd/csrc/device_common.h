// device_common.h -- launch arguments and device helpers shared by the demapping kernels.
//
// Metric convention on the device: for a received point y, SNR s and
// constellation point x_j (label order), the log2-likelihood up to a
// sample constant is a_j = -c_s |y - x_j|^2 with c_s = 1 / (2 sigma_s^2 ln 2)
// (sigma_s^2 = Es / (D 10^(snr_db/10)) per real dimension). The kernels
// exponentiate arg_j = a_j + K with the fixed shift K = Emax - 1 - m of the
// working type (126 - m for FP32, 1022 - m for FP64): a_j <= 0, so no term
// and no sum of M terms can overflow, and no per-sample maximum pass is
// needed. A bit side (or the total) whose sum falls below
// starve(m) = 2^(m + Emin + guard) is "starved": terms flushed below the
// normal range could then matter, and that entry is recomputed exactly with
// its own maximum as shift (slow_rel). guard = 20 bits for FP32 (the flushed
// mass is then < 2^-20 of the side), 60 for FP64.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "exact_rule.h"
#include "launch_rules.h"

namespace air {

constexpr int kMaxSnrPerLaunch = 64;
constexpr int kMaxBits = 12;        // M <= 4096
constexpr int kMaxD = 16;

// Where a demapping kernel is launched: the stream and, for a timed launch,
// two events that take the kernel's own start and end times from its
// dispatch (no marker commands between the kernels). Both null: untimed.
struct Launch {
  hipStream_t stream;
  hipEvent_t start;
  hipEvent_t stop;
};

template <typename F, typename... Args>
inline void launch_kernel(const Launch& l, F kernel, dim3 grid, dim3 block, uint32_t shmem, Args... args) {
  if (l.start || l.stop)
    hipExtLaunchKernelGGL(kernel, grid, block, shmem, l.stream, l.start, l.stop, 0u, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, shmem, l.stream, args...);
}

// Sets the context's error flag, which the host reads (host memory: a plain
// store; every writer stores the same value).
__device__ __forceinline__ void flag_sticky(int* sticky) {
  __hip_atomic_store(sticky, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Per-call device words: the tx-range error of a call and the numbers of items
// that left the first tier; zero when the call starts.
struct CallWords {
  int err;
  int pad;
  unsigned long long recomputed;   // items finished outside the first tier's sums
  unsigned long long exact;        // of those, items that needed the exact path
};

// A value from another block of the same launch, written by an atomic.
template <typename T>
__device__ __forceinline__ T from_other_block(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The per-block sums of a launch, [S][4][blocks]: sum u, sum v, sum u^2, sum v^2
// per SNR point (entry 4 s + q). The last block of a short launch reads the
// others' (tail.h), so every access goes past the caches that blocks do not
// share; there is no other way to the words.
class BlockSums {
 public:
  void set(double* words) { p_ = words; }
  __host__ __device__ explicit operator bool() const { return p_ != nullptr; }
  // this block's
  __device__ __forceinline__ void put(int entry, double v) const {
    __hip_atomic_store(p_ + ((int64_t)entry * gridDim.x + blockIdx.x), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // block b's, of `blocks`
  __device__ __forceinline__ double get(int entry, int b, int blocks) const {
    return from_other_block(p_ + ((int64_t)entry * blocks + b));
  }

 private:
  double* p_;
};

// Zeroes the words of the next call (one thread).
__device__ inline void clear_call_words(CallWords* next) {
  if (next) {
    next->err = 0;
    next->pad = 0;
    next->recomputed = 0ull;
    next->exact = 0ull;
  }
}

// Per-SNR scalars of one launch, passed by value in the kernel arguments.
struct SnrTable {
  double sigma[kMaxSnrPerLaunch];   // noise standard deviation per real dimension
  double c[kMaxSnrPerLaunch];       // 1 / (2 sigma^2 ln 2)
  float sigmaf[kMaxSnrPerLaunch];
  float cf[kMaxSnrPerLaunch];
};

// What ends a call: the reduction of the per-block sums into statistics and the
// hand-over of the call words, by finish_kernel or, for short launches, by the
// last block of the call's last demapping kernel (tail.h).
struct FinishArgs {
  double* stats;                    // [S][4] of the launch, or nullptr
  const CallWords* call;
  CallWords* next;                  // zeroed for the next call
  int* sticky;
  unsigned int* ticket;             // blocks done; zero between launches
  int blocks2;                      // blocks of the second tier's partials, 0 for none
  int no_mi;                        // max-log: no symbol-wise MI
  int in_last_block;                // 1: the last kernel's last block finishes the call
  int short_lists;                  // 1: the second tier reads the first one's lists itself
};

// Arguments of every demapping kernel.
struct DemapArgs {
  const void* in;                   // Y (N x D) or, in sweep mode, unit noise Z (N x D)
  const uint32_t* tx;               // N transmitted indices into X, or nullptr
  void* llr;                        // [S][N][m] LLRs (nats) or nullptr
  BlockSums partials;
  int* err;                         // set to 1 when a tx index >= M is seen
  unsigned long long* recomputed;   // (sample, SNR) items finished outside the fast sums
  unsigned long long* exact;        // of those, items that needed the exact path
  const void* xl;                   // M x D coordinates in label order (float or double)
  const uint32_t* lab;              // label of original point index j
  int64_t N;
  int64_t llr_stride_s;             // elements between consecutive SNR planes of llr
  int M, m, D, S;
  int s_per;                        // SNR points per block (blockIdx.y: a run of them)
  int sweep;                        // 1: y = x_t + sigma_s z from `in`
  // second tier (matrix-core forms and the FP32 vector kernel)
  unsigned long long* t2_list;      // [S][waves][tpw]: sample tile (32 bits) | lane mask (32)
  BlockSums t2_partials;            // from the second tier
  int blocks1;                      // gridDim.x of the first tier
  int t2_tpw;                       // list slots per (SNR point, wave)
  unsigned int* t2_nitem;           // [S][waves]: samples flagged in each wave's list
  // the flagged samples gathered per SNR point: point s's samples, in (wave,
  // slot, lane) order, from entry s * t2_cap of t2_items
  uint32_t* t2_items;               // sample indices
  int64_t t2_cap;                   // entries of t2_items per SNR point (waves x tpw x 32)
  unsigned int* t2_tot;             // [S]: samples flagged at each SNR point
  FinishArgs fin;
  SnrTable snr;
};

template <typename T> struct Real;

template <> struct Real<float> {
  static __device__ __forceinline__ float exp2(float x) { return __builtin_amdgcn_exp2f(x); }
  static __device__ __forceinline__ float log2(float x) { return __builtin_amdgcn_logf(x); }
  static __device__ __forceinline__ float fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
  static __device__ __forceinline__ float shift(int m) { return 126.0f - (float)m; }
  static __device__ __forceinline__ float starve(int m) { return __builtin_ldexpf(1.0f, m - 126 + 20); }
  static __device__ __forceinline__ float ln2() { return 0.693147180559945309f; }
  static __device__ __forceinline__ float nan() { return __builtin_nanf(""); }
  static __device__ __forceinline__ float inf() { return __builtin_inff(); }
  static __device__ __forceinline__ float sigma(const SnrTable& t, int s) { return t.sigmaf[s]; }
  static __device__ __forceinline__ float c(const SnrTable& t, int s) { return t.cf[s]; }
};

template <> struct Real<double> {
  static __device__ __forceinline__ double exp2(double x) { return ::exp2(x); }
  static __device__ __forceinline__ double log2(double x) { return ::log2(x); }
  static __device__ __forceinline__ double fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
  static __device__ __forceinline__ double shift(int m) { return 1022.0 - (double)m; }
  static __device__ __forceinline__ double starve(int m) { return __builtin_ldexp(1.0, m - 1022 + 60); }
  static __device__ __forceinline__ double ln2() { return 0.6931471805599453094; }
  static __device__ __forceinline__ double nan() { return __builtin_nan(""); }
  static __device__ __forceinline__ double inf() { return __builtin_inf(); }
  static __device__ __forceinline__ double sigma(const SnrTable& t, int s) { return t.sigma[s]; }
  static __device__ __forceinline__ double c(const SnrTable& t, int s) { return t.c[s]; }
};

// Received point of sample n at SNR s: read from Y, or x_t + sigma z (sweep).
template <typename T, int D>
__device__ __forceinline__ void load_point(const DemapArgs& a, int64_t n, int tl, T sigma, T (&y)[D]) {
  const T* in = static_cast<const T*>(a.in) + n * D;
  if (a.sweep) {
    const T* xt = static_cast<const T*>(a.xl) + (int64_t)tl * D;
#pragma unroll
    for (int d = 0; d < D; ++d) y[d] = Real<T>::fma(sigma, in[d], xt[d]);
  } else {
#pragma unroll
    for (int d = 0; d < D; ++d) y[d] = in[d];
  }
}

template <typename T, int D>
__device__ __forceinline__ T sqdist(const T (&y)[D], const T* __restrict__ x) {
  T d2 = 0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    T df = y[d] - x[d];
    d2 = Real<T>::fma(df, df, d2);
  }
  return d2;
}

// ---- exact recomputation (rare path) -------------------------------------
// Used for items whose fast-path sums fall below the starvation bound. All
// metrics are taken relative to a reference point r (the nearest point), and
// the difference a_j - a_r = -c (|y-x_j|^2 - |y-x_r|^2) is formed as
// -c sum_d (x_r - x_j)_d (2 y - x_r - x_j)_d, which keeps its relative
// accuracy even when y is far from every point (|a_j| huge, difference not).
// In line, with rolled loops and the sums copied to memory for them in the
// branch that needs them: a call makes the kernel keep everything that lives
// across it in every other block of eight registers (FP64, 16 points in 2-D: 185
// registers with calls, 117 without), and a loop over a run-time number of
// sums outside the branch put every item's sums into scratch memory.

template <typename T, int D>
__device__ __forceinline__ void reload_point(const T* __restrict__ in, int sweep,
                                             const T* __restrict__ xl, T sigma, int64_t n, int tl,
                                             T (&y)[D]) {
  const T* p = in + n * D;
  if (sweep) {
#pragma unroll
    for (int d = 0; d < D; ++d) y[d] = Real<T>::fma(sigma, p[d], xl[(int64_t)tl * D + d]);
  } else {
#pragma unroll
    for (int d = 0; d < D; ++d) y[d] = p[d];
  }
}

template <typename T, int D>
__device__ __forceinline__ T rel_metric(const T (&y)[D], const T* __restrict__ xr,
                                        const T* __restrict__ xj, T c) {
  T acc = 0;
#pragma unroll
  for (int d = 0; d < D; ++d) acc = Real<T>::fma(xr[d] - xj[d], (y[d] - xr[d]) + (y[d] - xj[d]), acc);
  return -c * acc;
}

// Index (label order) of the point nearest to the received point; ties to the lowest.
template <typename T, int D>
__device__ __forceinline__ int slow_nearest(const T (&y)[D], const T* __restrict__ xl, int M) {
  int best = 0;
  T bd = sqdist<T, D>(y, xl);
#pragma unroll 4
  for (int j = 1; j < M; ++j) {
    T d2 = sqdist<T, D>(y, xl + (int64_t)j * D);
    if (d2 < bd) { bd = d2; best = j; }
  }
  return best;
}

// log2 sum_{j in selection} 2^(a_j - a_r): bit side (k, b), or all points (k = -1).
template <typename T, int D>
__device__ __forceinline__ T slow_rel(const T (&y)[D], const T* __restrict__ xl, int M, T c, int r, int k, int b) {
  const T* xr = xl + (int64_t)r * D;
  // the selection's labels: all of them, or those with bit k equal to b
  // (index i with b inserted at bit k)
  const int cnt = k >= 0 ? M >> 1 : M;
  const int lowmask = k >= 0 ? (1 << k) - 1 : 0;
  auto label = [&](int i) { return k >= 0 ? (((i & ~lowmask) << 1) | (b << k) | (i & lowmask)) : i; };
  T dmax = -__builtin_huge_val();
#pragma unroll 4
  for (int i = 0; i < cnt; ++i) {
    T dj = rel_metric<T, D>(y, xr, xl + (int64_t)label(i) * D, c);
    dmax = dj > dmax ? dj : dmax;
  }
  T sum = 0;
#pragma unroll 4
  for (int i = 0; i < cnt; ++i)
    sum += Real<T>::exp2(rel_metric<T, D>(y, xr, xl + (int64_t)label(i) * D, c) - dmax);
  return dmax + Real<T>::log2(sum);
}

// What the exact path needs of one call: where the sample's point comes from
// and the constellation, with the SNR's scalars in the working type.
template <typename T>
struct ExactArgs {
  const T* in;                      // received points, or unit noise in sweep mode
  int sweep;
  const T* xl;                      // label-ordered coordinates
  int M, m;
  T sigma, c;
};

template <typename T>
__device__ __forceinline__ ExactArgs<T> exact_args(const DemapArgs& a, int s) {
  return ExactArgs<T>{static_cast<const T*>(a.in), a.sweep, static_cast<const T*>(a.xl), a.M, a.m,
                      Real<T>::sigma(a.snr, s), Real<T>::c(a.snr, s)};
}

// Outputs of one (sample, SNR) item whose fast-path sums are all above the
// starvation bound: the m LLRs (if llr_out) and u, v (when tl >= 0).
//  total:   sum_j 2^arg_j;  side[2k+b]: the same over bit side (k, b).
//  arg_t:   arg of the transmitted point.
template <typename T>
__device__ __forceinline__ void finish_fast(int m, int tl, T total, const T (&side)[2 * kMaxBits], T arg_t,
                                            T* llr_out, T& u, T& v) {
  const T lam_tot = Real<T>::log2(total);
  T acc = 0;
#pragma unroll
  for (int k = 0; k < kMaxBits; ++k) {
    if (k < m) {
      const T l0 = Real<T>::log2(side[2 * k]), l1 = Real<T>::log2(side[2 * k + 1]);
      if (llr_out) llr_out[k] = Real<T>::ln2() * (l0 - l1);
      acc += lam_tot - (((tl >> k) & 1) ? l1 : l0);
    }
  }
  if (tl >= 0) {
    // log2 of the very term that entered the sum (not arg_t itself): u >= 0
    // then holds exactly, whatever the rounding of exp2 and log2.
    u = lam_tot - Real<T>::log2(Real<T>::exp2(arg_t));
    v = acc;
  }
}

// The two outputs of an item beside its LLRs.
template <typename T>
struct ItemUV {
  T u, v;
};

// Outputs of an item with starved entries: those are recomputed relative to
// the nearest point r. If the total itself is starved, every entry is
// recomputed and all stay relative to a_r (a side need not be below the total
// bit for bit: the two are summed in different orders); otherwise the
// recomputed sides are put back in the fast path's units by adding K + a_r,
// which is then small. mem: the sums, the recomputed ones replaced by their
// logarithms.
template <typename T, int D>
__device__ __forceinline__ ItemUV<T> finish_exact(const ExactArgs<T>& a, int64_t n, int tl, T total, T* mem,
                                                  T arg_t, T* llr_out) {
  const int m = a.m;
  const T thr = Real<T>::starve(m);
  T y[D];
  reload_point<T, D>(a.in, a.sweep, a.xl, a.sigma, n, tl, y);
  const int r = slow_nearest<T, D>(y, a.xl, a.M);
  const bool total_slow = !(total >= thr);
  const T base = total_slow ? T(0) : Real<T>::shift(m) - a.c * sqdist<T, D>(y, a.xl + (int64_t)r * D);
  const uint32_t redo = exact_entries<T>(total, mem, m, thr);
  T lam_tot = total_slow ? T(0) : Real<T>::log2(total);
  // The total (entry -1) and the starved sides. Where a bit's two sides are
  // starved in different lanes, one pass takes each lane's side (its loads are
  // then per lane), and a further one side 1 of the lanes with both: 1.2e5
  // FP64 samples with LLRs, two passes with half the lanes each / this: 4-D/256 at 31
  // dB 1.76 / 0.66 ms, 8-D/512 (5.9e4 samples) at 28 dB 3.2 / 1.15 ms.
#pragma unroll 1
  for (int i = -1; i < 2 * m; ++i) {
    const int k = i < 0 ? -1 : i >> 1;
    const uint32_t own = i < 0 ? 0u : (redo >> (2 * k)) & 3u;
    const bool mixed = i >= 0 && __ballot(own & 1u) != 0ull && __ballot(own & 2u) != 0ull;
    T lam = 0;
    int at = i;
    bool take = i < 0 ? total_slow : ((own >> (i & 1)) & 1u) != 0u;
    if (!mixed) {
      if (take) lam = base + slow_rel<T, D>(y, a.xl, a.M, a.c, r, k, i & 1);
    } else {
      const int b = (i & 1) || own == 2u ? 1 : 0;
      take = (i & 1) ? own == 3u : own != 0u;
      at = 2 * k + b;
      if (take) lam = base + slow_rel<T, D>(y, a.xl, a.M, a.c, r, k, b);
    }
    if (take) {
      if (i < 0) lam_tot = lam;
      else mem[at] = lam;
    }
  }
  T acc = 0;
#pragma unroll 1
  for (int k = 0; k < m; ++k) {
    const T l0 = ((redo >> (2 * k)) & 1u) ? mem[2 * k] : Real<T>::log2(mem[2 * k]);
    const T l1 = ((redo >> (2 * k + 1)) & 1u) ? mem[2 * k + 1] : Real<T>::log2(mem[2 * k + 1]);
    if (llr_out) llr_out[k] = Real<T>::ln2() * (l0 - l1);
    acc += lam_tot - (((tl >> k) & 1) ? l1 : l0);
  }
  T u = 0;
  if (tl >= 0)
    u = total_slow ? lam_tot - rel_metric<T, D>(y, a.xl + (int64_t)r * D, a.xl + (int64_t)tl * D, a.c)
                   : lam_tot - Real<T>::log2(Real<T>::exp2(arg_t));
  return ItemUV<T>{u, acc};
}

// Outputs of one (sample, SNR) item from its fast-path sums, as finish_fast,
// with the entries below the starvation bound recomputed exactly; the return
// value says whether that happened (the caller counts such items).
template <typename T, int D>
__device__ __forceinline__ bool finish_item(const ExactArgs<T>& a, int64_t n, int tl,
                                            T total, const T (&side)[2 * kMaxBits], T arg_t,
                                            T* llr_out, T& u, T& v) {
  const int m = a.m;
  const T thr = Real<T>::starve(m);
  bool slow = !(total >= thr);
#pragma unroll
  for (int i = 0; i < 2 * kMaxBits; ++i)
    if (i < 2 * m) slow |= !(side[i] >= thr);
  if (__builtin_expect(!slow, 1)) {
    finish_fast<T>(m, tl, total, side, arg_t, llr_out, u, v);
  } else {
    T mem[2 * kMaxBits];
#pragma unroll
    for (int i = 0; i < 2 * kMaxBits; ++i) mem[i] = side[i];
    const ItemUV<T> r = finish_exact<T, D>(a, n, tl, total, mem, arg_t, llr_out);
    if (tl >= 0) {
      u = r.u;
      v = r.v;
    }
  }
  return slow;
}

// floor(x) as an integer in one instruction (v_cvt_flr_i32_f32; the compiler
// forms it from a floor and a conversion). For finite x within the int range.
// `after` is a value the compiler formed from x (the fraction of x): the
// instruction is held behind it, so when x is a matrix-core result the
// compiler's own wait states before that reader cover this one too (it does
// not place them before inline assembly).
__device__ __forceinline__ int floor_i32(float x, float after) {
  int r;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x), "v"(after));
  return r;
}

// log2 of a positive double through its binary exponent and an FP32 log2 of
// the mantissa: absolute error ~2e-7, far inside every tolerance on the
// quantities it feeds (differences of such logs), at a fraction of the cost
// of the FP64 library routine.
__device__ __forceinline__ double log2_wide(double x) {
  int e;
  const double mant = __builtin_frexp(x, &e);   // in [0.5, 1)
  return (double)e + (double)__builtin_amdgcn_logf((float)mant);
}

// ---- the second tiers' exact path ------------------------------------------
// Outputs of FP32-family items from sums in the FP64 frame 2^(a + K64) whose
// entries fall below the bound thr64 of that frame. Those entries are
// recomputed relative to the nearest point r and put back in the frame by
// adding K64 + a_r; if the total itself is below thr64 every entry is
// recomputed and all stay relative to a_r. lt_t is log2 of the transmitted
// point's own term in the frame (used when tl >= 0 and the total is not
// recomputed). The caller counts the items.
//
// Two forms: one item per lane, or one item after another by the whole wave,
// which shares each pass over the points. The bits of an item do not depend on
// the other items of its wave: sets of up to 2^NB points have both forms, which
// add a sum's terms in the same order (a tree over each run of 16 labels, then
// the runs in turn), and larger sets are always finished by the wave, whose
// lanes add their own points' terms first. (With the form chosen by the number
// of items alone, and a serial sum in one of them, an item's last bits changed
// with the company it was listed in.)

// -c times it: a_j - a_r, with its relative accuracy (rel_metric).
template <int D>
__device__ __forceinline__ float rel_dot(const float (&y)[D], const float (&xr)[D], const float* __restrict__ xj) {
  float acc = 0.0f;
#pragma unroll
  for (int d = 0; d < D; ++d) acc = __builtin_fmaf(xr[d] - xj[d], (y[d] - xr[d]) + (y[d] - xj[d]), acc);
  return acc;
}

// u, v and the LLRs from the recomputed logarithms: lam[i] where bit i of
// redo is set, the frame's own sums elsewhere. NB: the most bits of a label.
template <int NB>
__device__ __forceinline__ void finish_frame64_outputs(int m, int tl, uint32_t redo, const double (&side)[2 * kMaxBits],
                                                       const double (&lam)[2 * NB], double lam_tot, double arg_t,
                                                       float* llr_out, float& u, float& v) {
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < NB; ++k)
    if (k < m) {
      const double l0 = ((redo >> (2 * k)) & 1u) ? lam[2 * k] : log2_wide(side[2 * k]);
      const double l1 = ((redo >> (2 * k + 1)) & 1u) ? lam[2 * k + 1] : log2_wide(side[2 * k + 1]);
      if (llr_out) llr_out[k] = (float)(0.6931471805599453094 * (l0 - l1));
      acc += lam_tot - (((tl >> k) & 1) ? l1 : l0);
    }
  if (tl >= 0) {
    u = (float)(lam_tot - arg_t);
    v = (float)acc;
  }
}

// This lane's item of a set of at most 16 points (demap_vec_small): a pass per
// starved entry in rolled loops, which leaves the kernel its registers (8-QAM:
// 78 against 99 with the form below, six waves per SIMD against four).
template <int D>
__device__ __forceinline__ void finish_small_item64(const ExactArgs<float>& a, int64_t n, int tl, double total,
                                                    const double (&side)[2 * kMaxBits], double thr64, int K64,
                                                    double lt_t, float* llr_out, float& u, float& v) {
  const int m = a.m;
  float y[D];
  reload_point<float, D>(a.in, a.sweep, a.xl, a.sigma, n, tl, y);
  const int r = slow_nearest<float, D>(y, a.xl, a.M);
  const bool total_slow = !(total >= thr64);
  const double base =
      total_slow ? 0.0 : (double)K64 - (double)a.c * (double)sqdist<float, D>(y, a.xl + (int64_t)r * D);
  const uint32_t redo = exact_entries<double>(total, side, m, thr64);
  double lam_tot = log2_wide(total), arg_t = lt_t;
  double mem[2 * kMaxBits];      // logarithms of the recomputed entries; entry -1: the total
#pragma unroll 1
  for (int i = total_slow ? -1 : 0; i < 2 * m; ++i)
    if (i < 0 || ((redo >> i) & 1u)) {
      const double lam = base + (double)slow_rel<float, D>(y, a.xl, a.M, a.c, r, i < 0 ? -1 : i >> 1, i & 1);
      if (i < 0) lam_tot = lam;
      else mem[i] = lam;
    }
  if (total_slow && tl >= 0)
    arg_t = (double)rel_metric<float, D>(y, a.xl + (int64_t)r * D, a.xl + (int64_t)tl * D, a.c);
  finish_frame64_outputs<kMaxBits>(m, tl, redo, side, mem, lam_tot, arg_t, llr_out, u, v);
}

// Pairs, quads, eights, ... of e[0 .. N).
template <int N>
__device__ __forceinline__ float run_sum(float (&e)[N]) {
#pragma unroll
  for (int w = N / 2; w >= 1; w >>= 1)
#pragma unroll
    for (int i = 0; i < w; ++i) e[i] = e[2 * i] + e[2 * i + 1];
  return e[0];
}

// As slow_rel, one bit side (k, b) of a lane's item.
template <int D>
__device__ __forceinline__ float lane_rel(const float (&y)[D], const float (&xr)[D], const float* __restrict__ xl,
                                          int M, float c, int k, int b) {
  const int lowmask = (1 << k) - 1;
  auto label = [&](int i) { return ((i & ~lowmask) << 1) | (b << k) | (i & lowmask); };
  const int cnt = M >> 1;
  float dmax = -__builtin_inff(), sum = 0.0f;
#pragma unroll 4
  for (int i = 0; i < cnt; ++i) dmax = __builtin_fmaxf(dmax, -c * rel_dot<D>(y, xr, xl + (int64_t)label(i) * D));
  // eight of the side's labels are a run's (k < 4) or half of one's
  float half = 0.0f;
  for (int i0 = 0; i0 < cnt; i0 += 8) {
    float e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      e[i] = i0 + i < cnt ? Real<float>::exp2(__builtin_fmaf(
                                -c, rel_dot<D>(y, xr, xl + (int64_t)label(i0 + i < cnt ? i0 + i : 0) * D), -dmax))
                          : 0.0f;
    const float t = run_sum(e);
    if (k < 4) sum += t;
    else if (i0 & 8) sum += half + t;
    else half = t;
  }
  return dmax + Real<float>::log2(sum);
}

// This lane's item (sets of at most 2^NB points). Where the lanes' items have
// many starved sides together, one pass over the points takes the maxima of
// all sides and one the sums; with few, each side takes its own two passes over
// its half of the points.
template <int D, int NB>
__device__ __forceinline__ void finish_item_frame64(const ExactArgs<float>& a, int64_t n, int tl, double total,
                                                    const double (&side)[2 * kMaxBits], double thr64, int K64,
                                                    double lt_t, float* llr_out, float& u, float& v) {
  const int m = a.m;
  const float c = a.c;
  float y[D];
  reload_point<float, D>(a.in, a.sweep, a.xl, a.sigma, n, tl, y);
  const int r = slow_nearest<float, D>(y, a.xl, a.M);
  float xr[D];
#pragma unroll
  for (int d = 0; d < D; ++d) xr[d] = a.xl[(int64_t)r * D + d];
  const bool total_slow = !(total >= thr64);
  const double base = total_slow ? 0.0 : (double)K64 - (double)c * (double)sqdist<float, D>(y, xr);
  const uint32_t redo = exact_entries<double>(total, side, m, thr64);
  // the sides that are starved in any lane here, and whether a total is
  uint32_t sides = 0u;
#pragma unroll
  for (int i = 0; i < 2 * NB; ++i) sides |= __ballot((redo >> i) & 1u) != 0ull ? 1u << i : 0u;
  const bool totals = __ballot(total_slow) != 0ull;
  float rel[2 * NB], rel_tot = 0.0f;
  if (totals || __builtin_popcount(sides) * (3 * D + 4) > 6 * D + 8 * NB) {
    constexpr int LB = NB < 4 ? NB : 4;
    constexpr int G = 1 << LB;         // points at a time: a run
    float mx[2 * NB], sm[2 * NB], mx_tot = -__builtin_inff(), sm_tot = 0.0f;
#pragma unroll
    for (int i = 0; i < 2 * NB; ++i) {
      mx[i] = -__builtin_inff();
      sm[i] = 0.0f;
    }
#pragma unroll 1
    for (int g = 0; g < a.M; g += G) {
      float dj[G];
#pragma unroll
      for (int i = 0; i < G; ++i) dj[i] = -c * rel_dot<D>(y, xr, a.xl + (int64_t)(g + i) * D);
#pragma unroll
      for (int i = 0; i < G; ++i) mx_tot = __builtin_fmaxf(mx_tot, dj[i]);
#pragma unroll
      for (int k = 0; k < LB; ++k)
#pragma unroll
        for (int i = 0; i < G; ++i) mx[2 * k + ((i >> k) & 1)] = __builtin_fmaxf(mx[2 * k + ((i >> k) & 1)], dj[i]);
#pragma unroll
      for (int k = LB; k < NB; ++k) {
        const bool one = (g >> k) & 1;
        float cur = one ? mx[2 * k + 1] : mx[2 * k];
#pragma unroll
        for (int i = 0; i < G; ++i) cur = __builtin_fmaxf(cur, dj[i]);
        mx[2 * k] = one ? mx[2 * k] : cur;
        mx[2 * k + 1] = one ? cur : mx[2 * k + 1];
      }
    }
#pragma unroll 1
    for (int g = 0; g < a.M; g += G) {
      float dot[G];
#pragma unroll
      for (int i = 0; i < G; ++i) dot[i] = rel_dot<D>(y, xr, a.xl + (int64_t)(g + i) * D);
      auto term = [&](int i, float top) { return Real<float>::exp2(__builtin_fmaf(-c, dot[i], -top)); };
#pragma unroll
      for (int k = 0; k < LB; ++k)
        if ((sides >> (2 * k)) & 3u) {
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            float e[G / 2];
#pragma unroll
            for (int i = 0; i < G / 2; ++i)
              e[i] = term(((i >> k) << (k + 1)) | (b << k) | (i & ((1 << k) - 1)), mx[2 * k + b]);
            sm[2 * k + b] += run_sum(e);
          }
        }
#pragma unroll
      for (int k = LB; k < NB; ++k)
        if ((sides >> (2 * k + ((g >> k) & 1))) & 1u) {
          const bool one = (g >> k) & 1;
          const float top = one ? mx[2 * k + 1] : mx[2 * k];
          float e[G];
#pragma unroll
          for (int i = 0; i < G; ++i) e[i] = term(i, top);
          const float t = run_sum(e);
          sm[2 * k] += one ? 0.0f : t;
          sm[2 * k + 1] += one ? t : 0.0f;
        }
      if (totals) {
        float e[G];
#pragma unroll
        for (int i = 0; i < G; ++i) e[i] = term(i, mx_tot);
        sm_tot += run_sum(e);
      }
    }
#pragma unroll
    for (int i = 0; i < 2 * NB; ++i) rel[i] = mx[i] + Real<float>::log2(sm[i]);
    rel_tot = mx_tot + Real<float>::log2(sm_tot);
  } else {
#pragma unroll
    for (int i = 0; i < 2 * NB; ++i) rel[i] = 0.0f;
#pragma unroll 1
    for (uint32_t left = sides; left; left &= left - 1u) {
      const int i = __builtin_ctz(left);
      const float x = lane_rel<D>(y, xr, a.xl, a.M, c, i >> 1, i & 1);
#pragma unroll
      for (int q = 0; q < 2 * NB; ++q) rel[q] = q == i ? x : rel[q];
    }
  }
  double lam[2 * NB];
#pragma unroll
  for (int i = 0; i < 2 * NB; ++i) lam[i] = base + (double)rel[i];
  const double lam_tot = total_slow ? (double)rel_tot : log2_wide(total);
  double arg_t = lt_t;
  if (total_slow && tl >= 0) arg_t = (double)(-c * rel_dot<D>(y, xr, a.xl + (int64_t)tl * D));
  finish_frame64_outputs<NB>(m, tl, redo, side, lam, lam_tot, arg_t, llr_out, u, v);
}

// Sum of a double over the 64 lanes of a wave (every lane gets the result).
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Moves within a row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_of(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppXor3 = 0x1b, kDppXor7 = 0x141, kDppXor8 = 0x128;

// op (commutative) over the lanes of each row of 16 that agree in bit SKIP of
// their number (SKIP > 3: over the row), in every lane; all lanes take part. In
// each step both partners apply op to the same two values.
template <int SKIP, typename OP>
__device__ __forceinline__ uint32_t row_reduce(uint32_t x, OP&& op) {
  if (SKIP != 0) x = op(x, dpp_of<kDppXor1>(x));
  if (SKIP != 1) x = op(x, dpp_of<kDppXor2>(x));
  if (SKIP != 2) x = op(x, dpp_of<kDppXor7>(dpp_of<kDppXor3>(x)));
  if (SKIP != 3) x = op(x, dpp_of<kDppXor8>(x));
  return x;
}
// ... over the lanes of the wave that agree in bit SKIP (6: over all 64).
template <int SKIP, typename OP>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t x, OP&& op) {
  x = row_reduce<SKIP>(x, op);
  if (SKIP != 4) {
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = op(p[0], p[1]);
  }
  if (SKIP != 5) {
    const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    x = op(p[0], p[1]);
  }
  return x;
}
__device__ __forceinline__ uint32_t fadd_bits(uint32_t p, uint32_t q) {
  return __float_as_uint(__uint_as_float(p) + __uint_as_float(q));
}
template <int SKIP = 6>
__device__ __forceinline__ float wave_max_f(float x) {      // NaN only if every lane's is
  return __uint_as_float(wave_reduce<SKIP>(__float_as_uint(x), [](uint32_t p, uint32_t q) {
    return __float_as_uint(__builtin_fmaxf(__uint_as_float(p), __uint_as_float(q)));
  }));
}
template <int SKIP = 6>
__device__ __forceinline__ float wave_sum_f(float x) {
  return __uint_as_float(wave_reduce<SKIP>(__float_as_uint(x), fadd_bits));
}
template <int SKIP = 6>
__device__ __forceinline__ float row_sum_f(float x) {
  return __uint_as_float(row_reduce<SKIP>(__float_as_uint(x), fadd_bits));
}
__device__ __forceinline__ float lane_value(float x, int l) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), l));
}

// Index of the point nearest to y (uniform); ties to the lowest.
template <int D>
__device__ __forceinline__ int wave_nearest(const float (&y)[D], const float* __restrict__ xl, int M) {
  int best = 0;
  float bd = __builtin_inff();
#pragma unroll 2
  for (int j = threadIdx.x & 63; j < M; j += 64) {
    const float d2 = sqdist<float, D>(y, xl + (int64_t)j * D);
    if (d2 < bd) { bd = d2; best = j; }
  }
  const float least = -wave_max_f(-bd);
  // the lowest index among the lanes at the least distance
  const uint32_t at = wave_reduce<6>(bd == least ? (uint32_t)best : 0x7fffffffu,
                                  [](uint32_t p, uint32_t q) { return p < q ? p : q; });
  return __builtin_amdgcn_readfirstlane((int)at);
}

// As slow_rel, for uniform y, r, k, b, by the whole wave: the sums are taken
// per lane and then across the lanes.
template <int D>
__device__ __forceinline__ float wave_rel(const float (&y)[D], const float (&xr)[D], const float* __restrict__ xl,
                                          int M, float c, int k, int b) {
  const int cnt = k >= 0 ? M >> 1 : M;
  const int lowmask = k >= 0 ? (1 << k) - 1 : 0;
  auto label = [&](int i) { return k >= 0 ? (((i & ~lowmask) << 1) | (b << k) | (i & lowmask)) : i; };
  const int lane = threadIdx.x & 63;
  float dmax = -__builtin_inff();
#pragma unroll 2
  for (int i = lane; i < cnt; i += 64) dmax = __builtin_fmaxf(dmax, -c * rel_dot<D>(y, xr, xl + (int64_t)label(i) * D));
  dmax = wave_max_f(dmax);
  float sum = 0.0f;
#pragma unroll 2
  for (int i = lane; i < cnt; i += 64)
    sum += Real<float>::exp2(__builtin_fmaf(-c, rel_dot<D>(y, xr, xl + (int64_t)label(i) * D), -dmax));
  return dmax + Real<float>::log2(wave_sum_f(sum));
}

// Both sides of label bit K < 6 from the kept metrics of a wave's points
// (point lane + 64 p in lane `lane`): the lanes of a side reduce among
// themselves. RUNS: a row holds a run of 16 labels; the runs are added in turn.
template <int K, bool RUNS, int P>
__device__ __forceinline__ void kept_sides(const float (&dot)[P], int M, float c, float (&rel)[2]) {
  const int lane = threadIdx.x & 63;
  float top = -__builtin_inff();
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (lane + 64 * p < M) top = __builtin_fmaxf(top, -c * dot[p]);
  top = wave_max_f<K>(top);
  float e[P];
#pragma unroll
  for (int p = 0; p < P; ++p)
    e[p] = lane + 64 * p < M ? Real<float>::exp2(__builtin_fmaf(-c, dot[p], -top)) : 0.0f;
  float s0 = 0.0f, s1 = 0.0f;
  if constexpr (RUNS) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      if (64 * p < M) {
        const float t = row_sum_f<K>(e[p]);
#pragma unroll
        for (int l = 0; l < 64; l += 16) {
          if (K < 4) {
            s0 += lane_value(t, l);
            s1 += lane_value(t, l | (1 << (K & 3)));
          } else if ((l >> K) & 1) {
            s1 += lane_value(t, l);
          } else {
            s0 += lane_value(t, l);
          }
        }
      }
    }
  } else {
    float sum = 0.0f;
#pragma unroll
    for (int p = 0; p < P; ++p) sum += e[p];
    sum = wave_sum_f<K>(sum);
    s0 = lane_value(sum, 0);
    s1 = lane_value(sum, 1 << K);
  }
  rel[0] = lane_value(top, 0) + Real<float>::log2(s0);
  rel[1] = lane_value(top, 1 << K) + Real<float>::log2(s1);
}

// One selection of the kept metrics (k: a label bit from 6 on, or -1 for all points).
template <bool RUNS, int P>
__device__ __forceinline__ float kept_rel(const float (&dot)[P], int M, float c, int k, int b) {
  const int lane = threadIdx.x & 63;
  float top = -__builtin_inff(), sum = 0.0f;
  auto in = [&](int p) { return lane + 64 * p < M && (k < 0 || ((p >> (k - 6)) & 1) == b); };
#pragma unroll
  for (int p = 0; p < P; ++p) top = in(p) ? __builtin_fmaxf(top, -c * dot[p]) : top;
  top = wave_max_f(top);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const float e = in(p) ? Real<float>::exp2(__builtin_fmaf(-c, dot[p], -top)) : 0.0f;
    if constexpr (RUNS) {
      const float t = row_sum_f(e);
#pragma unroll
      for (int l = 0; l < 64; l += 16) sum += lane_value(t, l);
    } else {
      sum += e;
    }
  }
  if constexpr (!RUNS) sum = wave_sum_f(sum);
  return top + Real<float>::log2(sum);
}

// The items of a wave's lanes (`mine`: this lane holds one), one after another
// by the whole wave. A lane that walks a large set alone holds its wave for
// ~0.5 ms per item (8-D, M = 2048), and the few waves with such items end the
// launch alone: 8-D/2048, 1e6 samples with LLRs, 484 such items at 24 dB, 3.86 ->
// 1.00 ms; 1969 at 25 dB, 9.01 -> 1.06 ms. Up to 256 points each lane keeps its
// points' metrics for all entries.
template <typename T, T V>
struct Const {
  static constexpr T value = V;
};
template <int D, int NB, bool ALL>
__device__ __forceinline__ void finish_items_by_wave(const ExactArgs<float>& a, bool mine, int64_t n, int tl,
                                                     double total, const double (&side)[2 * kMaxBits], double thr64,
                                                     int K64, double lt_t, float* llr_out, float& u, float& v) {
  const int m = a.m;
  const float c = a.c;
  const int lane = threadIdx.x & 63;
  double mem[2 * kMaxBits];      // logarithms of the recomputed entries
  const uint32_t redo = mine ? exact_entries<double>(total, side, m, thr64) : 0u;
  const bool total_slow = !(total >= thr64);
  double lam_tot = log2_wide(total), arg_t = lt_t;
  constexpr int kKept = 4;       // points per lane whose metrics are kept
  unsigned long long todo = __ballot(mine);
  while (todo) {
    const int src = __builtin_ctzll(todo);
    todo &= todo - 1ull;
    const int64_t ns = (int64_t)(((uint64_t)__builtin_amdgcn_readlane((uint32_t)((uint64_t)n >> 32), src) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((uint32_t)n, src));
    const int ts = __builtin_amdgcn_readlane(tl, src);
    uint32_t left = __builtin_amdgcn_readlane(redo, src);
    const bool all = __builtin_amdgcn_readlane(total_slow ? 1 : 0, src) != 0;
    float y[D];
    reload_point<float, D>(a.in, a.sweep, a.xl, a.sigma, ns, ts, y);
    const int r = wave_nearest<D>(y, a.xl, a.M);
    float xr[D];
#pragma unroll
    for (int d = 0; d < D; ++d) xr[d] = a.xl[(int64_t)r * D + d];
    const double base = all ? 0.0 : (double)K64 - (double)c * (double)sqdist<float, D>(y, xr);
    if (all && ts >= 0) {
      const double dt = (double)(-c * rel_dot<D>(y, xr, a.xl + (int64_t)ts * D));
      if (lane == src) arg_t = dt;
    }
    // entry i of the item: the total (-1) or a bit side
    auto put = [&](int i, float rel) {
      const double lam = base + (double)rel;
      if (lane == src) {
        if (i < 0) lam_tot = lam;
        else mem[i] = lam;
      }
    };
    auto entries = [&](auto runs, auto points) {
      constexpr bool RUNS = decltype(runs)::value;
      constexpr int P = decltype(points)::value;
      float dot[P];
#pragma unroll
      for (int p = 0; p < P; ++p)
        dot[p] = lane + 64 * p < a.M ? rel_dot<D>(y, xr, a.xl + (int64_t)(lane + 64 * p) * D) : 0.0f;
      if (all) put(-1, kept_rel<RUNS>(dot, a.M, c, -1, 0));
      while (left) {
        const int i = __builtin_ctz(left), k = i >> 1;
        if (k < 6) {
          float rel[2];
          switch (k) {
            case 0: kept_sides<0, RUNS>(dot, a.M, c, rel); break;
            case 1: kept_sides<1, RUNS>(dot, a.M, c, rel); break;
            case 2: kept_sides<2, RUNS>(dot, a.M, c, rel); break;
            case 3: kept_sides<3, RUNS>(dot, a.M, c, rel); break;
            case 4: kept_sides<4, RUNS>(dot, a.M, c, rel); break;
            default: kept_sides<5, RUNS>(dot, a.M, c, rel); break;
          }
          put(2 * k, rel[0]);
          put(2 * k + 1, rel[1]);
          left &= ~(3u << (2 * k));
        } else {
          put(i, kept_rel<RUNS>(dot, a.M, c, k, i & 1));
          left &= left - 1u;
        }
      }
    };
    if (ALL || (NB > 0 && a.M <= (1 << NB))) {
      if constexpr (NB > 0) entries(Const<bool, true>{}, Const<int, NB <= 6 ? 1 : (1 << NB) / 64>{});
    } else if constexpr (!ALL) {
      if (a.M <= 64 * kKept) {
        entries(Const<bool, false>{}, Const<int, kKept>{});
      } else {
        if (all) put(-1, wave_rel<D>(y, xr, a.xl, a.M, c, -1, 0));
        for (; left; left &= left - 1u) {
          const int i = __builtin_ctz(left);
          put(i, wave_rel<D>(y, xr, a.xl, a.M, c, i >> 1, i & 1));
        }
      }
    }
  }
  if (mine) finish_frame64_outputs<kMaxBits>(m, tl, redo, side, mem, lam_tot, arg_t, llr_out, u, v);
}

// A pass costs the lanes' form M points however many items the wave has; the
// wave's form costs each item about as much as kItemPoints of them. 600003
// samples with LLRs on the matrix cores, each lane alone with two passes per
// starved side / this line: 4-D/64 at 28 dB (a few items in a wave) 342 / 157 us,
// at 34 dB (all of them) 749 / 316 us; 16-D/64 at 28 dB 2242 / 787 us, 16-D/128 (the
// wave's form alone) 4948 / 2364 us. With the line at 4 and 8 points per item 4-D/32
// at 28 dB 206 and 223 us, 16-D/64 at 22 dB 877 and 787 us.
constexpr int kItemPoints = 6;

// The lanes' form serves sets of up to 2^NB points: 64 in the matrix-core second
// tiers, whose waves hold at most 32 items, 128 in the vector one (64 items);
// NB = 0: none (larger sets). ALL: the kernel's sets are no larger. Called by all lanes of a wave
// together.
template <int D, int NB, bool ALL>
__device__ __forceinline__ void finish_items_frame64(const ExactArgs<float>& a, bool mine, int64_t n, int tl,
                                                     double total, const double (&side)[2 * kMaxBits],
                                                     double thr64, int K64, double lt_t, float* llr_out, float& u,
                                                     float& v) {
  const unsigned long long items = __ballot(mine);
  // (the usual case, said so: the scalars that the exact path has no room for are
  // then spilled around it and not in the kernel's point loop)
  if (__builtin_expect(items == 0ull, 1)) return;
  if constexpr (NB > 0)
    if ((ALL || a.M <= (1 << NB)) && __builtin_popcountll(items) * kItemPoints >= a.M) {
      if (mine) finish_item_frame64<D, NB>(a, n, tl, total, side, thr64, K64, lt_t, llr_out, u, v);
      return;
    }
  finish_items_by_wave<D, NB, ALL>(a, mine, n, tl, total, side, thr64, K64, lt_t, llr_out, u, v);
}

// The same out of line, for the serving kernels, which have no registers to
// spare: in line 42 of the second tier's are spilled at D = 8, out of line 17, and
// bursts of 12 to 32 jobs took 1 to 3 % longer. The sums are copied to memory for the
// call alone.
struct ItemOut {
  float u, v;
};
template <int D, int NB, bool ALL>
__device__ __noinline__ ItemOut finish_items_call(const ExactArgs<float>* a, bool mine, int64_t n, int tl, double total,
                                                  const double (*side)[2 * kMaxBits], double thr64, int K64,
                                                  double lt_t, float* llr_out) {
  ItemOut r{0.0f, 0.0f};
  finish_items_frame64<D, NB, ALL>(*a, mine, n, tl, total, *side, thr64, K64, lt_t, llr_out, r.u, r.v);
  return r;
}

}  // namespace air
