// Host-side choice of the SGEMM tile configuration of a launch (no HIP types;
// a CPU test checks it).
#pragma once

#include <algorithm>
#include <cstdint>

namespace gvm {

// Time of a launch under one tile configuration, in us:
//
//   t0 + W / peak * (k / x) * e_k,   x = tiles / CUs,  k = ceil(x)
//
// with W the FLOP of the whole tiles (ragged edges padded to the tile, as the
// kernel computes them), peak the FP32 matrix rate of the CUs the launch may
// use (157.3 TFLOP/s for all 256; a masked partition has fewer), x the tiles
// per CU and k / x what the fullest CU has more than the mean.  t0 is
// the part no tile size takes away (launch, first fetch, store of C); e1, e2
// and e3 are the inverse of the rate a CU reaches with one, two and more tiles
// (one tile alone has nothing to hide its barriers and fetches behind).  t0
// and e1 .. e3 are fitted to launches of 1, 2, 3, 4, 8 and 16 requests of 46
// sizes from 64 to 2048 on an MI355X (rms 2-7 % per configuration).  Over
// those 276 launches the cheapest configuration by this formula is on average
// 0.7 % and at most 13 % (0.5 us, n = 96) slower than the fastest of all 31
// measured, where a table by size alone (the fastest for 8 requests) is 13 %
// and up to 89 % slower for 4 requests and 2 % and up to 15 % for 16.
struct GemmCost {
  int config;
  uint32_t bm, bn;
  float t0, e1, e2, e3;
};
constexpr GemmCost kGemmCosts[] = {
    {0, 32, 32, 4.1f, 0.48f, 1.12f, 1.39f},    {1, 32, 32, 3.8f, 0.81f, 1.18f, 1.36f},
    {3, 32, 64, 3.9f, 0.93f, 1.13f, 1.20f},    {5, 64, 32, 4.1f, 0.83f, 1.11f, 1.18f},
    {6, 64, 64, 3.7f, 1.04f, 1.15f, 1.14f},    {10, 64, 64, 4.7f, 1.00f, 1.13f, 1.14f},
    {11, 64, 96, 3.6f, 1.14f, 1.21f, 1.18f},   {13, 96, 96, 3.8f, 1.13f, 1.17f, 1.16f},
    {17, 64, 128, 3.8f, 1.10f, 1.13f, 1.12f},  {18, 128, 64, 3.8f, 1.10f, 1.11f, 1.10f},
    {22, 128, 128, 4.3f, 1.07f, 1.09f, 1.09f}, {24, 128, 256, 5.5f, 1.05f, 1.07f, 1.08f},
    {30, 160, 64, 3.8f, 1.15f, 1.20f, 1.17f},
};
constexpr int kGemmCus = 256;
constexpr double kGemmPeakFlopPerUs = 157.3e6 / kGemmCus;   // of one CU

inline uint64_t gemm_tiles(const GemmCost& c, uint64_t n) {
  return ((n + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn);
}

// Mixed sizes: the tiles differ in length by their n, so a CU may end on a
// long one; its share of that (half, as measured on the 32-rank uneven mix)
// is added to the mean time, or the mean to the longest tile where that is
// the longer of the two.
inline double gemm_launch_us(const GemmCost& c, uint32_t count, const uint32_t* n, int cus) {
  double flop = 0.0, tiles = 0.0;
  uint32_t nmax = 0, nmin = ~0u;
  for (uint32_t i = 0; i < count; ++i) {
    const double t = static_cast<double>(gemm_tiles(c, n[i]));
    tiles += t;
    flop += t * 2.0 * c.bm * c.bn * n[i];
    nmax = std::max(nmax, n[i]);
    nmin = std::min(nmin, n[i]);
  }
  const double x = tiles / cus;
  const double k = static_cast<double>(static_cast<uint64_t>(x) + (x > static_cast<uint64_t>(x) ? 1 : 0));
  const double e = k <= 1 ? c.e1 : k <= 2 ? c.e2 : c.e3;
  const double peak = kGemmPeakFlopPerUs * cus;
  const double mean = flop / peak * e;
  if (nmin == nmax) return c.t0 + mean * k / x;
  const double longest = 2.0 * c.bm * c.bn * nmax * cus / peak * e;
  return c.t0 + std::max(mean, longest) + 0.5 * std::min(mean, longest);
}

// The cheapest configuration for one launch of requests of sizes n[0..count)
// on `cus` CUs.
inline int gemm_cheapest(uint32_t count, const uint32_t* n, int cus = kGemmCus) {
  int best = kGemmCosts[0].config;
  double t_best = 0.0;
  for (const GemmCost& c : kGemmCosts) {
    const double t = gemm_launch_us(c, count, n, cus);
    if (&c == &kGemmCosts[0] || t < t_best) {
      t_best = t;
      best = c.config;
    }
  }
  return best;
}

}  // namespace gvm
