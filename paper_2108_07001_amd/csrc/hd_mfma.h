// hd_mfma.h -- hard decisions on the matrix cores, with the decisions of
// hd_kernel (the nearest point by FP32 distances, ties to the lower label).
//
// For constellations of M >= 32 points whose coordinates are of moderate
// range, the distances to all points come from the product tiles of the
// first tier, in a metric scaled per sample so that every term is bounded:
// x_j = c (2 y.x_j - |x_j|^2 - |y|^2) = -c |y - x_j|^2 with
// c = 16 / (|y|^2 + R^2), R = max |x_j|, so c (|y| + |x_j|)^2 <= 32 and the
// split operands and the FP32 sums of the products leave an absolute error
// below ~3e-4 in x_j. The FP32 procedure of hd_kernel rounds by less than
// 1e-4 in these units, so the point it would pick, and every point tied with
// it, lies within kHdTheta = 2^-9 of the largest x_j (the near points). One
// pass over the tiles keeps, per lane and 32-sample group,
//  - the largest x_j of each of the 16 row positions over all tiles,
//  - the largest tile maximum, its tile, and the second largest.
// Where exactly one row position reaches the near range and the second tile
// does not, the near point is unique: it is the row position in the best
// tile, and the decision needs no distance. Of the other samples every near point
// lies in a near row position (of 32 over both lane halves), and hd_kernel's
// procedure runs on the points of those rows alone:
//  - few such samples among the wave's 64: the wave shares the tiles of one
//    sample after another;
//  - many: each lane takes its own sample. From kHdPass2 tiles on a second pass
//    over the products first finds the tiles that hold a near point in a half.
// How many there are depends on the set: about 1 % at low SNR on 2048 points in
// 8-D, 3 % of 256-QAM, half of 4096-QAM, most of 256-PAM and all of a set whose
// points coincide in pairs. The two ways meet where a wave has about NT / 4 + 4
// of them (a pass costs ~100 cycles per tile, a sample of the first way ~400).
//
// Bound by VALU issue: 20 maxima per 16 points and group against 128 matrix
// cycles per tile and group pair at D = 8. Against a maximum pass and a second
// one that compares every product with the threshold for every sample: 8-D/2048,
// N = 4e6, 11 SNR points 17.8 -> 6.8 ms; 12-D/4096, N = 1e6, 896 -> 400 us per
// SNR point; 8-PSK^2 sweep (N = 1e6, 21 points) 420 -> 280 us; and on dense sets, N = 1e6 at
// 24 dB: 4096-QAM 605 -> 377 us, 1024-QAM 174 -> 87, 2-D/4096 650 -> 423, 8-D/2048 in
// pairs 452 -> 307 (with every such sample's full set scanned by the wave these
// four took 2222, 217, 3246 and 2683 us).
#pragma once
#include "hd_kernels.h"
#include "mfma_wide.h"

namespace air {

constexpr float kHdTheta = 0x1p-9f;

// The FP32 distance of hd_kernel: acc = fma(y_d - x_d, y_d - x_d, acc) from 0.
template <int D>
__device__ __forceinline__ float hd_dist(const float (&y)[D], const float* __restrict__ x) {
  float acc = 0.0f;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const float df = y[d] - x[d];
    acc = __builtin_fmaf(df, df, acc);
  }
  return acc;
}

// (distance, label) kept in hd_kernel's order: a smaller distance, or the same
// distance at a lower label, replaces the current one (a NaN never does).
__device__ __forceinline__ void hd_take(float d, int l, float& bd, int& bl) {
  const bool better = d < bd || (d == bd && l < bl);
  bd = better ? d : bd;
  bl = better ? l : bl;
}

// Row of a tile of row position e: 0 .. 15 in the lower lane half, 16 .. 31 in the upper.
__device__ __forceinline__ int hd_row(int e) { return 8 * ((e >> 2) & 3) + 4 * (e >> 4) + (e & 3); }

// hd_kernel's decision over the points label(0 .. cnt - 1) for the sample of
// lane src, by the whole wave.
template <int D, typename LABEL>
__device__ __forceinline__ int hd_wave(const float (&y)[D], int src, int cnt, const float* __restrict__ xl,
                                       LABEL&& label) {
  float ys[D];
#pragma unroll
  for (int d = 0; d < D; ++d) ys[d] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(y[d]), src));
  float bd = __builtin_inff();
  int bl = 0;
  for (int i = threadIdx.x & 63; i < cnt; i += 64) {
    const int l = label(i);
    hd_take(hd_dist<D>(ys, xl + (int64_t)l * D), l, bd, bl);
  }
  const float least = -wave_max_f(-bd);
  const uint32_t at = wave_reduce<6>(bd == least ? (uint32_t)bl : 0x7fffffffu,
                                     [](uint32_t p, uint32_t q) { return p < q ? p : q; });
  return __builtin_amdgcn_readfirstlane((int)at);
}

// Tiles from which on a second pass over the products pays for the samples
// without a unique near point (below: every tile's near rows).
constexpr int kHdPass2 = 8;

// Bytes of the block-local copies of the coordinates and point records.
__host__ __device__ constexpr int64_t hd_table_bytes(int M, int D) {
  return (int64_t)M * D * 4 + 16 + (int64_t)M * mfma_nk(D, false) * 32;
}

// +inf as a value the compiler does not see through.
__device__ __forceinline__ float opaque_inf() {
  float x = __builtin_inff();
  asm("" : "+s"(x));
  return x;
}

// The larger of two numbers in one instruction: the middle one of them and
// +inf (fmax of a product's element is preceded by a quieting of it, and
// with a known +inf the compiler makes this an fmax again).
__device__ __forceinline__ float max2(float a, float b, float inf) { return __builtin_amdgcn_fmed3f(a, b, inf); }

// Largest of the 16 elements of a product tile.
__device__ __forceinline__ float max16(const float16_t& v, float inf) {
  auto m3 = [](float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); };
  const float a = m3(v[0], v[1], v[2]), b = m3(v[3], v[4], v[5]), c = m3(v[6], v[7], v[8]);
  const float d = m3(v[9], v[10], v[11]), e = m3(v[12], v[13], v[14]);
  return max2(m3(m3(a, b, c), d, e), v[15], inf);
}

// Running maxima of one lane and group over the point tiles.
struct HdBest {
  float row[16];       // per row position, over all tiles
  float b1, b2;        // largest and second largest tile maximum
  int t1;              // tile of b1
  float inf;
  __device__ __forceinline__ void init() {
    inf = opaque_inf();
    const float ninf = -__builtin_inff();
#pragma unroll
    for (int e = 0; e < 16; ++e) row[e] = ninf;
    b1 = b2 = ninf;
    t1 = 0;
  }
  __device__ __forceinline__ void tile(float m, int t) {
    b2 = __builtin_amdgcn_fmed3f(b1, b2, m);     // b1 >= b2: the middle one
    t1 = m > b1 ? t : t1;
    b1 = max2(b1, m, inf);
  }
  __device__ __forceinline__ void add(const float16_t& a0, const float16_t& a1, int t) {
#pragma unroll
    for (int e = 0; e < 16; ++e) row[e] = __builtin_fmaxf(__builtin_fmaxf(row[e], a0[e]), a1[e]);
    tile(max16(a0, inf), t);
    tile(max16(a1, inf), t + 1);
  }
  __device__ __forceinline__ void add(const float16_t& a0, int t) {
#pragma unroll
    for (int e = 0; e < 16; ++e) row[e] = __builtin_fmaxf(row[e], a0[e]);
    tile(max16(a0, inf), t);
  }
  // row positions that reach `floor`
  __device__ __forceinline__ uint32_t near(float floor) const {
    uint32_t bits = 0u;
#pragma unroll
    for (int e = 0; e < 16; ++e) bits |= row[e] >= floor ? (1u << e) : 0u;
    return bits;
  }
};

// One wave takes 64 samples per round (two 32-sample tiles, as the first
// tier); lane (j, h) forms sample j of tile h, holds rows 8 (e / 4) + 4 h +
// e % 4 of column j of both tiles' products and finishes its own sample.
template <int D, bool TBL>
__global__ __launch_bounds__(256, D <= 4 ? 4 : (D <= 8 ? 3 : 2)) void hd_mfma(const HdArgs a, const MfmaOp<false>::vec* __restrict__ rec,
                                                float R2) {
  typedef MfmaOp<false>::vec V;
  typedef WideOperand<D, false> OP;
  constexpr int NK = OP::NK;
  extern __shared__ char hd_lds[];
  __shared__ unsigned long long part[4][2];
  const int lane = threadIdx.x & 63;
  const int h = lane >> 5;
  const int j = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform per wave
  const int waves = blockDim.x >> 6;
  const int M = a.M;
  const int NT = M >> 5;
  const float* __restrict__ xl = a.xl;
  const V* __restrict__ rp = rec;
  if (TBL) {
    float* l_xl = reinterpret_cast<float*>(hd_lds);
    V* l_rec = reinterpret_cast<V*>(hd_lds + ((M * D * 4 + 15) & ~15));
    for (int i = threadIdx.x; i < M * D; i += blockDim.x) l_xl[i] = a.xl[i];
    for (int i = threadIdx.x; i < M * NK * 2; i += blockDim.x) l_rec[i] = rec[i];
    __syncthreads();
    xl = l_xl;
    rp = l_rec;
  }
  const int64_t ntiles = (a.N + 31) >> 5;
  const int64_t npairs = (ntiles + 1) >> 1;
  const int64_t wstride = (int64_t)gridDim.x * waves;
  const int64_t wgid = (int64_t)blockIdx.x * waves + wave;
  const int s0 = blockIdx.y * a.s_per;
  const int s1 = s0 + a.s_per < a.S ? s0 + a.s_per : a.S;
  for (int s = s0; s < s1; ++s) {
    unsigned int se = 0, be = 0;
    for (int64_t q = wgid; q < npairs; q += wstride) {
      // the lane's own sample, formed as hd_kernel forms it
      const int64_t n = (2 * q + h) * 32 + j;
      const bool valid = n < a.N;
      const int64_t nc = valid ? n : a.N - 1;
      int tl = -1;
      if (a.tx) {
        const uint32_t t = a.tx[nc];
        if (t >= (uint32_t)M) {
          if (s == 0 && valid) atomicOr(a.err, 1);
          tl = -2;
        } else {
          tl = (int)a.lab[t];
        }
      }
      float y[D];
      const float* __restrict__ in = a.in + nc * D;
      if (a.sweep) {
        const int lt = tl >= 0 ? tl : 0;
#pragma unroll
        for (int d = 0; d < D; ++d) y[d] = __builtin_fmaf(a.sigma[s], in[d], xl[lt * D + d]);
      } else {
#pragma unroll
        for (int d = 0; d < D; ++d) y[d] = in[d];
      }
      float yy = 0.0f;
#pragma unroll
      for (int d = 0; d < D; ++d) yy = __builtin_fmaf(y[d], y[d], yy);
      // m = 126 makes the operand's shift 0: x_j = -c |y - x_j|^2. With this
      // c every operand is in range for finite |y|^2 (c |y|^2 < 16, c <= 16 / R2
      // <= 4096), so only an infinite or NaN |y|^2 counts as out of range.
      OP opA, opB;
      OP::build_pair(y, 16.0f / (yy + R2), __FLT_MAX__, 126, opA, opB);
      HdBest bA, bB;
      bA.init();
      bB.init();
      auto load = [&](V (&A)[NK], int t) {
        const V* r = rec_row<false, false, NK>(rp, t, j, h);
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) A[kk] = r[2 * kk];
      };
      if (NT > 1) {
        // two tiles at a time (M is a power of two), the next two's records
        // loaded as soon as the products have taken these
        V A0[NK], A1[NK];
        load(A0, 0);
        load(A1, 1);
        for (int t = 0; t < NT; t += 2) {
          const float16_t a0 = opA.product(A0), a1 = opA.product(A1);
          const float16_t b0 = opB.product(A0), b1 = opB.product(A1);
          const int tn = t + 2 < NT ? t + 2 : 0;     // the last pair reloads the first
          load(A0, tn);
          load(A1, tn + 1);
          // keeps these loads here (they would be merged with the first
          // pair's into loads at the top of the loop, right before their use)
          asm volatile("" ::: "memory");
          bA.add(a0, a1, t);
          bB.add(b0, b1, t);
        }
      } else {
        V A0[NK];
        load(A0, 0);
        bA.add(opA.product(A0), 0);
        bB.add(opB.product(A0), 0);
      }
      // the largest x_j of both groups' samples of this column, over both
      // lane halves, then the row positions near it in this lane's half
      float lo, hi;
      own_halves(bA.b1, bB.b1, lo, hi);
      const float own = __builtin_fmaxf(lo, hi);
      const float floor_own = own - kHdTheta;
      float fA, fB;
      own_halves(floor_own, floor_own, fA, fB);
      const uint32_t nearA = bA.near(fA), nearB = bB.near(fB);
      // the own sample's near rows, best tiles and second tiles of both halves
      const auto nr = __builtin_amdgcn_permlane32_swap(nearA, nearB, false, false);
      const auto tr = __builtin_amdgcn_permlane32_swap((uint32_t)bA.t1, (uint32_t)bB.t1, false, false);
      float s0, s1;
      own_halves(bA.b2, bB.b2, s0, s1);
      const uint32_t rows = (uint32_t)nr[0] | ((uint32_t)nr[1] << 16);
      const bool unique = (rows & (rows - 1u)) == 0u && rows != 0u && !(__builtin_fmaxf(s0, s1) >= floor_own);
      int l_own = (int)(__builtin_ctz(rows | 0x80000000u) < 16 ? tr[0] : tr[1]) * 32 +
                  hd_row(__builtin_ctz(rows | 0x80000000u));
      // the others: the near points of each lie in its near rows (operands out
      // of their range: anywhere)
      unsigned long long rest = __ballot(valid && (!unique || opA.ovf));
      if (rest) {
        unsigned long long todo = rest & __ballot(rows != 0u && !opA.ovf);
        rest &= ~todo;
        if (__builtin_popcountll(todo) * 4 > (NT < kHdPass2 ? 8 : NT + 16)) {
          // many: each lane its own sample's near rows in the tiles that hold a
          // near point in its half, found by a second pass over the products
          const bool mine = (todo >> lane) & 1ull;
          float bd = __builtin_inff();
          int bl = 0;
          for (int t0 = 0; t0 < NT; t0 += 32) {
            uint32_t w0 = NT < 32 ? (1u << NT) - 1u : ~0u, w1 = w0;
            if (NT >= kHdPass2) {
              uint32_t wA = 0u, wB = 0u;
              const float inf = bA.inf;
              const int nt = NT < 32 ? NT : 32;
              V A0[NK], A1[NK];
              load(A0, t0);
              load(A1, t0 + 1);
              for (int t = 0; t < nt; t += 2) {
                const float16_t a0 = opA.product(A0), a1 = opA.product(A1);
                const float16_t b0 = opB.product(A0), b1 = opB.product(A1);
                const int tn = t + 2 < nt ? t0 + t + 2 : 0;
                load(A0, tn);
                load(A1, tn + 1);
                asm volatile("" ::: "memory");
                wA |= max16(a0, inf) >= fA ? 1u << t : 0u;
                wA |= max16(a1, inf) >= fA ? 2u << t : 0u;
                wB |= max16(b0, inf) >= fB ? 1u << t : 0u;
                wB |= max16(b1, inf) >= fB ? 2u << t : 0u;
              }
              const auto w = __builtin_amdgcn_permlane32_swap(wA, wB, false, false);
              w0 = w[0];
              w1 = w[1];
            }
            if (mine) {
              auto half = [&](uint32_t tiles, uint32_t r16, int hh) {
                if (r16 == 0u) return;
                for (; tiles; tiles &= tiles - 1u) {
                  const int l0 = (t0 + __builtin_ctz(tiles)) * 32 + 4 * hh;
                  for (uint32_t r = r16; r; r &= r - 1u) {
                    const int l = l0 + hd_row(__builtin_ctz(r));
                    hd_take(hd_dist<D>(y, xl + (int64_t)l * D), l, bd, bl);
                  }
                }
              };
              half(w0, rows & 0xffffu, 0);
              half(w1, rows >> 16, 1);
            }
          }
          if (mine) l_own = bl;
        } else {
          // few: the wave shares the tiles of one sample's near rows
          const int lg = 31 - __builtin_clz(NT);
          while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1ull;
            const uint32_t rs = __builtin_amdgcn_readlane(rows, src);
            const int bl = hd_wave<D>(y, src, __builtin_popcount(rs) << lg, xl, [&](int i) {
              uint32_t r = rs;
              for (int q = i >> lg; q > 0; --q) r &= r - 1u;
              return (i & (NT - 1)) * 32 + hd_row(__builtin_ctz(r));
            });
            if (lane == src) l_own = bl;
          }
        }
        while (rest) {
          const int src = __builtin_ctzll(rest);
          rest &= rest - 1ull;
          const int bl = hd_wave<D>(y, src, M, xl, [](int i) { return i; });
          if (lane == src) l_own = bl;
        }
      }
      if (valid) {
        if (a.decided) a.decided[(int64_t)s * a.N + n] = a.pos[l_own];
        if (tl >= 0 && l_own != tl) {
          se += 1;
          be += (unsigned int)__builtin_popcount((unsigned)(l_own ^ tl));
        }
      }
    }
    const double ws = wave_sum((double)se), wb = wave_sum((double)be);
    if (lane == 0) {
      part[wave][0] = (unsigned long long)ws;
      part[wave][1] = (unsigned long long)wb;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
      unsigned long long tt = 0;
      for (int w = 0; w < waves; ++w) tt += part[w][threadIdx.x];
      if (a.counts && tt) atomicAdd(a.counts + 2 * s + threadIdx.x, tt);
    }
    __syncthreads();
  }
}

template <int D>
hipError_t launch_hd_mfma_d(const HdArgs& a, const void* rec, float R2, int grid, hipStream_t st) {
  typedef MfmaOp<false>::vec V;
  const V* r = static_cast<const V*>(rec);
  const dim3 g(grid, (a.S + a.s_per - 1) / a.s_per);
  const int64_t tb = hd_table_bytes(a.M, D);
  if (tb <= 40 * 1024)
    hipLaunchKernelGGL((hd_mfma<D, true>), g, dim3(256), (size_t)tb, st, a, r, R2);
  else
    hipLaunchKernelGGL((hd_mfma<D, false>), g, dim3(256), 0, st, a, r, R2);
  return hipGetLastError();
}

}  // namespace air
