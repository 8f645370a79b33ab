// serve_kernels.h -- batched matrix-core kernels of the serving loop.
//
// A batch holds jobs of uneven M, D and N. Jobs that share a kernel class
// (D, operand type, 16-point form) are contiguous in the batch's descriptor
// array, and one launch per class walks the flattened (job, chunk) work items
// of all of them: wave w of the grid takes items w, w + waves, ... Each item
// is a fixed run of sample tiles of one job, so every sum the kernels form
// depends on the job alone -- never on which jobs share the batch or which
// wave ran the item -- and a job's result is bitwise the same alone and in
// any mix. The per-tile arithmetic is the one of the sweep kernels
// (tier1_tile / tier2_tile).
#pragma once

#include "mfma_kernels.h"

namespace air {

// Result record of one job, written by the kernels (cleared by the host).
struct JobOut {
  double stats[4];                  // MI, GMI, SE_MI, SE_GMI (bits per symbol)
  unsigned long long recomputed;    // items finished by the second tier or the exact path
  int err;                          // a transmitted index >= M was seen
  int pad;
};

// One job of a batch, as the kernels see it.
struct JobDesc {
  const float* in;                  // N x D received points, or unit noise (sweep)
  const uint32_t* tx;               // N transmitted indices, or nullptr (LLRs only)
  float* llr;                       // N x m LLRs (nats), or nullptr
  const uint32_t* lab;              // label of point index j
  const float* xl;                  // M x D coordinates in label order
  const void* rec;                  // matrix-core point records, label order
  double* partials;                 // [nitems][8]: sums u, v, u^2, v^2 of tier 1, then tier 2
  unsigned long long* list;         // [nitems][chunk]: tiles left to tier 2 (tile | lane mask << 32)
  unsigned int* count;              // [nitems]: entries of each item's list
  JobOut* out;
  int64_t N;
  int64_t item0;                    // first item of this job in its class launch
  int64_t unit0;                    // first second-tier unit of this job, likewise
  int nitems;
  int chunk;                        // sample tiles per item
  int unit;                         // items per second-tier unit
  int M, m, sweep;
  float c, sigma;                   // metric scale 1/(2 sigma^2 ln 2) and noise deviation
};

// Sample tiles per work item of a job with N samples: a function of N alone
// (at most 4096 items per job).
__host__ __device__ inline int serve_chunk(int64_t N) {
  const int64_t tiles = (N + 31) / 32;
  const int64_t c = (tiles + 4095) / 4096;
  return (int)(c < 1 ? 1 : c);
}

// Items per second-tier unit, a function of N alone. The second tier is bound
// by the vector work of its tiles, whose cost does not depend on how many of
// the 32 samples are flagged: a wave gathers a unit's flagged samples into
// dense tiles (5 % flagged over 8 tiles: 1 or 2 tiles instead of 6 or 7).
// Measured on a burst of 32 jobs of the mix: 1.48 ms with every listed tile
// run as it stands, 1.22 ms gathered. Units grow with N so that a job whose
// samples are all flagged still spreads over about 1000 waves, one per SIMD;
// jobs of up to 65504 samples keep one tile per unit.
constexpr int kUnitTiles = 8;
__host__ __device__ inline int serve_unit(int64_t N) {
  const int64_t tiles = (N + 31) / 32;
  int64_t u = tiles / 1024;
  u = u < 1 ? 1 : (u > kUnitTiles ? kUnitTiles : u);
  const int64_t items = u / serve_chunk(N);
  return (int)(items < 1 ? 1 : items);
}

// The job of work item `it`: the last job whose first item is <= it (T2: of
// second-tier unit `it`).
template <bool T2>
__device__ __forceinline__ int serve_job_of(const JobDesc* __restrict__ jobs, int njobs, int64_t it) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((T2 ? jobs[mid].unit0 : jobs[mid].item0) <= it) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ SampleParams job_params(const JobDesc& jd) {
  return SampleParams{jd.in, jd.tx, jd.N, jd.M, jd.m, jd.sweep, jd.c, jd.sigma, &jd.out->err};
}

// Flagged samples of a 32-sample tile from which a serving work item hands
// its remaining tiles to the second tier directly (three quarters, as in the
// sweep's first tier).
constexpr int kDirectTile = 24;

// Bound by vector issue (exponentials). At most 8 dimensions are held to the
// registers of three waves per SIMD; with the point loop four tiles per step
// (sets of 128 points and more) the burst took 1.48 ms against 1.60 ms before.
template <int D, bool BF, bool HALF>
__global__ __launch_bounds__(256, D <= 8 ? 3 : 2) void serve_tier1(const JobDesc* __restrict__ jobs, int njobs,
                                                   int64_t nitems) {
  typedef typename MfmaOp<BF>::vec V;
  typedef SampleTile<D, BF> ST;
  const int lane = threadIdx.x & 63;
  const int h = lane >> 5;
  const int j = lane & 31;
  const int64_t waves = blockDim.x >> 6;
  const int64_t wstride = (int64_t)gridDim.x * waves;
  for (int64_t it = (int64_t)blockIdx.x * waves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); it < nitems;
       it += wstride) {
    const JobDesc& jd = jobs[serve_job_of<false>(jobs, njobs, it)];
    const int64_t li = it - jd.item0;
    const int m = jd.m;
    const int NT = HALF ? 1 : (jd.M >> 5);
    const int ntb = HALF ? 0 : m - 5;
    const float thr = Real<float>::starve(m);
    const SampleParams sp = job_params(jd);
    const Tables<BF> tb{jd.lab, jd.xl, static_cast<const V*>(jd.rec)};
    const int64_t ntiles = (jd.N + 31) >> 5;
    const int64_t st0 = li * jd.chunk;
    const int64_t st1 = st0 + jd.chunk < ntiles ? st0 + jd.chunk : ntiles;
    unsigned long long* slots = jd.list + li * jd.chunk;
    double au = 0.0, av = 0.0, auu = 0.0, avv = 0.0;
    int nlisted = 0;
    // once a tile of the item has had at least kDirectTile of its 32 samples
    // flagged, the item's later tiles go to the second tier as they are (as
    // in the sweep's first tier; the item's tiles are a function of the job
    // alone, so the choice is too)
    bool direct = false;
    for (int64_t st = st0; st < st1; ++st) {
      TileInput<D> ti;
      ti.load(sp, tb, st, j);
      ST smp;
      smp.setup(sp, st, j, h, true, ti);
      float* lout = (jd.llr && smp.valid) ? jd.llr + smp.n * m : nullptr;
      float u = 0.f, v = 0.f;
      bool need2;
      if (!direct) {
        tier1_tile<D, BF, HALF>(smp, tb, jd.tx != nullptr, j, h, m, NT, ntb, thr, lout, u, v, need2,
                                jd.llr != nullptr || jd.tx == nullptr);
      } else {
        need2 = smp.live;
        if (smp.valid && !smp.live && lout && h == 0)
          for (int k = 0; k < m; ++k) lout[k] = Real<float>::nan();
      }
      const unsigned long long fm = __ballot(need2 && h == 0) & 0xffffffffull;
      if (!HALF && __builtin_popcountll(fm) >= kDirectTile) direct = true;
      if (fm != 0) {
        if (lane == 0) slots[nlisted] = (fm << 32) | (unsigned long long)st;
        ++nlisted;
      }
      if (h == 0 && smp.live && smp.tl >= 0 && !need2) {
        const double du = (double)u, dv = (double)v;
        au += du;
        av += dv;
        auu = __builtin_fma(du, du, auu);
        avv = __builtin_fma(dv, dv, avv);
      }
    }
    const double w0 = wave_sum(au), w1 = wave_sum(av);
    const double w2 = wave_sum(auu), w3 = wave_sum(avv);
    if (lane == 0) {
      double* p = jd.partials + li * 8;
      p[0] = w0;
      p[1] = w1;
      p[2] = w2;
      p[3] = w3;
      jd.count[li] = (unsigned int)nlisted;
    }
  }
}

// One wave per second-tier unit: the flagged samples of the unit's items,
// gathered in (item, list, lane) order, are re-formed 32 to a tile; the unit's
// sums go to its first item's record (its other items' are zero).
template <int D, bool BF, bool HALF>
__global__ __launch_bounds__(256, 2) void serve_tier2(const JobDesc* __restrict__ jobs, int njobs,
                                                   int64_t nunits) {
  typedef typename MfmaOp<BF>::vec V;
  typedef SampleTile<D, BF> ST;
  // (chunks of more than kUnitTiles tiles, jobs of over a million samples, are
  // gathered in several runs)
  __shared__ uint32_t queue[4][kUnitTiles * 32];
  const int lane = threadIdx.x & 63;
  const int h = lane >> 5;
  const int j = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t waves = blockDim.x >> 6;
  const int64_t wstride = (int64_t)gridDim.x * waves;
  for (int64_t it = (int64_t)blockIdx.x * waves + wave; it < nunits; it += wstride) {
    const JobDesc& jd = jobs[serve_job_of<true>(jobs, njobs, it)];
    const int64_t li0 = (it - jd.unit0) * jd.unit;
    const int64_t li1 = li0 + jd.unit < jd.nitems ? li0 + jd.unit : jd.nitems;
    const int64_t st0 = li0 * jd.chunk;  // the queue holds samples from this tile on
    double au = 0.0, av = 0.0, auu = 0.0, avv = 0.0;
    unsigned long long items = 0;
    const int m = jd.m;
    const int NT = HALF ? 1 : (jd.M >> 5);
    const int ntb = HALF ? 0 : m - 5;
    const SampleParams sp = job_params(jd);
    const Tables<BF> tb{jd.lab, jd.xl, static_cast<const V*>(jd.rec)};
    const ExactArgs<float> ex{jd.in, jd.sweep, jd.xl, jd.M, m, jd.sigma, jd.c};
    int qn = 0;
    auto finish = [&]() {
      for (int b = 0; b < qn; b += 32) {
        const bool flagged = b + j < qn;
        const int64_t sn = flagged ? st0 * 32 + (int64_t)queue[wave][b + j] : -1;
        TileInput<D> ti;
        ti.fetch_n(sp, sn);
        ti.resolve(sp, tb);
        ST smp;
        smp.setup_n(sp, sn, h, false, ti);
        float* lout = (jd.llr && smp.valid) ? jd.llr + smp.n * m : nullptr;
        float u, v;
        tier2_tile<D, BF, HALF, 2>(smp, tb, ex, jd.tx != nullptr, flagged, j, h, m, NT, ntb, lout, u, v);
        if (flagged && h == 0 && smp.tl >= 0) {
          const double du = (double)u, dv = (double)v;
          au += du;
          av += dv;
          auu = __builtin_fma(du, du, auu);
          avv = __builtin_fma(dv, dv, avv);
        }
      }
      items += (unsigned long long)qn;
      qn = 0;
    };
    for (int64_t li = li0; li < li1; ++li) {
      const int nlisted = (int)jd.count[li];
      const unsigned long long* slots = jd.list + li * jd.chunk;
      for (int q = 0; q < nlisted; ++q) {
        if (qn > (kUnitTiles - 1) * 32) finish();
        const unsigned long long ent = slots[q];
        const uint32_t mask = (uint32_t)(ent >> 32);
        // (one wave's queue: its own LDS operations are in order)
        if (h == 0 && ((mask >> j) & 1u))
          queue[wave][qn + __builtin_popcount(mask & ((1u << j) - 1u))] = 
              (uint32_t)((int64_t)(ent & 0xffffffffull) - st0) * 32u + (uint32_t)j;
        qn += __builtin_popcount(mask);
        __builtin_amdgcn_wave_barrier();
      }
    }
    if (qn > 0) finish();
    if (items && lane == 0) atomicAdd(&jd.out->recomputed, items);
    const double w0 = wave_sum(au), w1 = wave_sum(av);
    const double w2 = wave_sum(auu), w3 = wave_sum(avv);
    for (int64_t li = li0 + lane; li < li1; li += 64) {
      double* p = jd.partials + li * 8 + 4;
      p[0] = li == li0 ? w0 : 0.0;
      p[1] = li == li0 ? w1 : 0.0;
      p[2] = li == li0 ? w2 : 0.0;
      p[3] = li == li0 ? w3 : 0.0;
    }
  }
}

// Both tiers of one kernel class: `jobs` is the class's contiguous run of
// descriptors, `nitems` and `nunits` the sums of their items and second-tier
// units, `cap` the most blocks of a launch.
template <int D, bool BF>
hipError_t launch_serve_td(const JobDesc* jobs, int njobs, int64_t nitems, int64_t nunits, bool half, int cap,
                           hipStream_t st) {
  auto grid = [cap](int64_t n) { return dim3((unsigned)((n + 3) / 4 < cap ? (n + 3) / 4 : cap)); };
  if (half) {
    hipLaunchKernelGGL((serve_tier1<D, BF, true>), grid(nitems), dim3(256), 0, st, jobs, njobs, nitems);
    hipLaunchKernelGGL((serve_tier2<D, BF, true>), grid(nunits), dim3(256), 0, st, jobs, njobs, nunits);
  } else {
    hipLaunchKernelGGL((serve_tier1<D, BF, false>), grid(nitems), dim3(256), 0, st, jobs, njobs, nitems);
    hipLaunchKernelGGL((serve_tier2<D, BF, false>), grid(nunits), dim3(256), 0, st, jobs, njobs, nunits);
  }
  return hipGetLastError();
}

}  // namespace air
