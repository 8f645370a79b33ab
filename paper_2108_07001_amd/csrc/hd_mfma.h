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
// tile, and the decision needs no distance. The other samples (about 1 % at
// low SNR on 2048 points, fewer elsewhere) are decided by the whole wave, which
// runs hd_kernel's procedure over all points, one stride of 64 per step.
//
// Bound by VALU issue: 20 maxima per 16 points and group against 128 matrix
// cycles per tile and group pair at D = 8. The two-pass form before it (a
// maximum pass, then every tile formed again, compared point by point, with
// the FP32 distance of each near point) took ~50: 8-D/2048, N = 4e6, 11 SNR
// points 17.8 -> 6.8 ms; 12-D/4096, N = 1e6, 1.00 -> 0.41-0.51 ms per SNR
// point; 8-PSK^2 sweep (N = 1e6, 21 points) 0.42 -> 0.28 ms. At 4 dB, where
// the wave's scans are most frequent, a point costs 1.35x one at 24 dB.
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
__global__ __launch_bounds__(256, D <= 8 ? 3 : 2) void hd_mfma(const HdArgs a, const MfmaOp<false>::vec* __restrict__ rec,
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
      const int e = __builtin_ctz(rows | 0x80000000u);
      int l_own = (int)(e < 16 ? tr[0] : tr[1]) * 32 + 8 * ((e >> 2) & 3) + 4 * (e >> 4) + (e & 3);
      // the others (and operands out of their range): all points, by the wave
      unsigned long long todo = __ballot(valid && (!unique || opA.ovf));
      while (todo) {
        const int src = __builtin_ctzll(todo);
        todo &= todo - 1ull;
        float ys[D];
#pragma unroll
        for (int d = 0; d < D; ++d)
          ys[d] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(y[d]), src));
        float bd = __builtin_inff();
        int bl = 0;
        for (int l = lane; l < M; l += 64) hd_take(hd_dist<D>(ys, xl + (int64_t)l * D), l, bd, bl);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
          const float od = __shfl_xor(bd, off, 64);
          const int ol = __shfl_xor(bl, off, 64);
          hd_take(od, ol, bd, bl);
        }
        if (lane == src) l_own = bl;
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
