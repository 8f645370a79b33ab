// launch_rules.h -- the grids of the demapping launches and what of the
// second tier's workspace one of them takes. Plain C++, so that host tests can
// check the rules themselves.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define AIR_RULE __host__ __device__ inline
#else
#define AIR_RULE inline
#endif

namespace air {

constexpr int kBlock = 256;         // threads per block of the vector kernels
// Blocks of a demapping launch that writes per-block sums: what the workspace
// for them, their reduction and the gathering of the lists are sized for.
constexpr int kMaxGrid = 1536;

// Grid of a matrix-core launch: 4 waves per block, one pair of 32-sample
// tiles (64 samples) per wave and round.
AIR_RULE int mfma_grid(int64_t N) {
  const int64_t pairs = (N + 63) / 64;
  const int64_t g = (pairs + 3) / 4;
  return (int)(g < kMaxGrid ? g : kMaxGrid);
}

// Grid of a vector-kernel launch: one sample per thread and round. For the sets
// of at most 16 points, whose samples are cheap, the per-block reductions weigh
// more, and 1024 blocks measured faster than 1536 (2-D QAM-4 buffers of 2^20
// symbols: 25 %); with no sums to write (`sums` false: LLR-only calls of the
// exact form) 2048. Larger sets take up to kMaxGrid blocks at one SNR point, and at
// several 1024 that the points are dealt out to (8-D/2048, 1e6 samples: 5 points
// 4.78 -> 4.48 ms with 2 x 1024, one point 0.96 -> 1.09 ms with 1024).
AIR_RULE int vec_grid(int64_t N, int M = 0, int S = 1, bool sums = true) {
  const int64_t cap = M > 16 ? (S > 1 ? 1024 : kMaxGrid) : (sums ? 1024 : 2048);
  const int64_t g = (N + kBlock - 1) / kBlock;
  return (int)(g < cap ? g : cap);
}

// Runs of SNR points a first-tier launch is cut into (gridDim.y), for a grid
// of gx blocks over the samples: few samples leave most of the chip idle while
// their waves walk all S points, so the points are dealt out until ~2048 blocks
// exist. 1e4 samples, 41 points, with and without: 8-D/2048 964 -> 253 us, 4-D/256
// 239 -> 71 us, 8-PSK^2 126 -> 46 us; 3e5 samples, 11 points: unchanged to 4 %
// faster.
AIR_RULE int snr_slices(int gx, int S) {
  const int n = 2048 / (gx > 0 ? gx : 1);
  return n < 1 ? 1 : (n < S ? n : S);
}

// Blocks of a second-tier launch over the gathered list (dealt out to the
// waves evenly). Small sets: at most 512 (2048 waves, one round of the chip at
// two waves per SIMD); their listed items are few, and more blocks cost more
// than they spread. Sets of 512 points and more: as many as the first tier
// (three rounds): of two waves that share a SIMD the older one takes most
// issue slots, finishes at about half the time and leaves the other alone, so
// further blocks have to follow (8-D/2048, 4e6 samples at 22 dB: 1.54 -> 1.78
// waves per SIMD, VALU busy 81 -> 87 % of the time, sweep 16.9 -> 16.2 ms; at M
// = 128 the items are short, and 1e6 of them took 307 us with 512 blocks, 344 us
// with 1536).
AIR_RULE int t2_grid(int grid, int M) { return M >= 512 || grid < 512 ? grid : 512; }

// The second tier's lists per SNR point of a launch of `grid` blocks: a run of
// slots per wave, one per sample tile that the wave owns (matrix cores: pairs of
// tiles dealt out to the waves; vector kernel: two tiles per wave and round,
// every slot written).
struct ListSize {
  int64_t waves, tpw;
  // list slots (8 bytes), flagged counts per wave (4) and 32 gathered sample
  // indices per slot (4 each)
  AIR_RULE int64_t bytes() const { return waves * tpw * 8 + waves * 4 + waves * tpw * 32 * 4; }
};
AIR_RULE ListSize list_size(int64_t N, int grid, bool mfma) {
  const int64_t waves = (int64_t)grid * 4;
  const int64_t npairs = ((N + 31) / 32 + 1) / 2;
  const int64_t stride = (int64_t)grid * kBlock;
  return ListSize{waves, mfma ? 2 * ((npairs + waves - 1) / waves) : 2 * ((N + stride - 1) / stride)};
}

// SNR points whose lists fit into `bytes` of scratch (three parts, each starting
// on a 256-byte boundary).
AIR_RULE int64_t lists_that_fit(const ListSize& ls, int64_t bytes) {
  const int64_t avail = bytes - 3 * 256;
  return avail > 0 ? avail / ls.bytes() : 0;
}

}  // namespace air
