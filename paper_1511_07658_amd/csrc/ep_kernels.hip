// EP-like compute-intensive kernel of the GVM for gfx950: the paper's small
// compute-intensive benchmark (NPB EP, Table 3, Section 6) in the form given
// in the public header: Gaussian pairs by Marsaglia's polar method from the
// counter-based generator Philox4x64-10 (Salmon et al., SC 2011), reduced to
// two binary64 sums and ten annulus counts.
//
// A request of n pairs is cut into work units of ep_unit(n) pairs (the cut
// depends on n only).  One grouped launch computes every unit of every request
// of the group and writes a partial record per unit into the request's device
// scratch; a second launch, one workgroup per request, sums the partials in
// unit order.  A request of one unit is written out by the first launch.  Both
// sums run in a fixed order (per thread in block order, then a fixed tree), so
// a request's result is bit-identical alone and in any mix.  Counts are
// integers and order-free.
#include "common.hpp"
#include "group_device.hpp"

#include <algorithm>

namespace gvm {

namespace {

constexpr int kEpThreads = 512;
constexpr int kEpWaves = kEpThreads / 64;
constexpr uint64_t kEpGrid = 1 << 20;   // workgroups of the unit launch: one per unit up to here
static_assert(kEpUnit / kEpThreads <= 255, "per-thread 8-bit annulus counts of a unit would overflow");
static_assert(kEpUnit <= 65535 && kEpRecordBytes >= 2 * 8 + 10 * 2, "a record holds 16-bit annulus counts");

// Philox4x64 multipliers and Weyl key increments (Salmon et al., 2011).
constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull, kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull, kPhiloxW1 = 0xBB67AE8584CAA73Bull;

// 128-bit product from four 32 x 32 + 64 bit multiply-adds.  The third one's
// carry goes into the top word as a 0 / 1 register: the multiply-add gives it
// in a scalar pair, which plain C++ recomputes with a compare (13 % slower
// at 2^27 pairs).  A vector instruction may read a scalar pair written by another
// only after two wait states, and the compiler does not look into inline
// assembly, so the write, the wait and the read are one block.
__device__ __forceinline__ void mul128(uint64_t m, uint64_t a, uint64_t& hi, uint64_t& lo) {
  const uint32_t a0 = static_cast<uint32_t>(a), a1 = static_cast<uint32_t>(a >> 32);
  const uint32_t m0 = static_cast<uint32_t>(m), m1 = static_cast<uint32_t>(m >> 32);
  const uint64_t p0 = static_cast<uint64_t>(a0) * m0;
  uint64_t p2 = static_cast<uint64_t>(a1) * m0 + (p0 >> 32), mask;
  uint32_t c;
  asm("v_mad_u64_u32 %0, %1, %3, %4, %0\n\t"
      "s_nop 1\n\t"
      "v_cndmask_b32 %2, 0, 1, %1"
      : "+&v"(p2), "=&s"(mask), "=&v"(c)
      : "v"(a0), "s"(m1));
  hi = static_cast<uint64_t>(a1) * m1 + ((p2 >> 32) | (static_cast<uint64_t>(c) << 32));
  lo = (p2 << 32) | static_cast<uint32_t>(p0);
}

__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
  const uint32_t lo = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(a), static_cast<uint32_t>(b),
                                                  static_cast<uint32_t>(c), 0x96);
  const uint32_t hi = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(a >> 32), static_cast<uint32_t>(b >> 32),
                                                  static_cast<uint32_t>(c >> 32), 0x96);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Philox4x64 with 10 rounds of counter (b, 0, 0, 0) under key (k0, k1): per
// round the full 128-bit products of words 0 and 2 with the multipliers;
// the next counter is (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1,
// lo(M0 c0)); the key is bumped by the Weyl increments between rounds.  The
// first two rounds are written out: of their four products, M1 * 0 is zero
// and M0 * k0 (`h`, `l`) is the same for every block of a request.
__device__ __forceinline__ void philox_block(uint64_t b, uint64_t k0, uint64_t k1, uint64_t h, uint64_t l,
                                             uint64_t w[4]) {
  uint64_t hi0, lo0, hi1, lo1;
  mul128(kPhiloxM0, b, hi0, lo0);
  uint64_t c2 = hi0 ^ k1;                 // round 1: counter (k0, 0, c2, lo0)
  k0 += kPhiloxW0;
  k1 += kPhiloxW1;
  mul128(kPhiloxM1, c2, hi1, lo1);
  uint64_t c0 = hi1 ^ k0, c1 = lo1, c3 = l;   // round 2
  c2 = lo0 ^ (h ^ k1);
#pragma unroll
  for (int r = 2; r < 10; ++r) {
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
    mul128(kPhiloxM0, c0, hi0, lo0);
    mul128(kPhiloxM1, c2, hi1, lo1);
    c0 = xor3(hi1, c1, k0);
    c1 = lo1;
    c2 = xor3(hi0, c3, k1);
    c3 = lo0;
  }
  w[0] = c0;
  w[1] = c1;
  w[2] = c2;
  w[3] = c3;
}

// {1/c, 2 ln(1/c)} of the 256 intervals of [1/2, 1) by leading bits, c the
// middle of interval i, except that the first takes c = 1/2 and the last c = 1,
// so that ln is exact where it is zero (t = 1 as 2 * 1/2) and keeps its relative
// accuracy as t approaches 1 from below.  A table in memory: computed by the
// workgroup it was a chain of a divide and a logarithm before the first pair
// (2^15 pairs: 5.2 -> 4.8 us with the shorter sums below).
constexpr int kLogTable = 256;
constexpr double kLn2 = 0x1.62e42fefa39efp-1;
struct alignas(16) LogEntry {
  double inv, m2log;
};
__device__ const LogEntry kLogEntries[kLogTable] = {
#include "ep_log_table.inc"
};
__device__ const double kLogLow[kLogTable] = {   // what the rounded m2log lacks
#include "ep_log_low.inc"
};

// The logarithms in two parts, to which e ln 2 (|e| <= 105) is added in two
// parts: the upper ones are multiples of 2^-44, so their sum, below 2^8, is exact.
__host__ __device__ constexpr double upper44(double x) { return (x + 0x1.8p8) - 0x1.8p8; }
constexpr double kTwoLn2 = 2.0 * kLn2, kTwoLn2Low = 0x1.abc9e3b39803fp-55;
constexpr double kTwoLn2Hi = upper44(kTwoLn2), kTwoLn2Lo = (kTwoLn2 - kTwoLn2Hi) + kTwoLn2Low;
struct LogTable {
  LogEntry e[kLogTable];   // {1/c, upper part}
  double low[kLogTable];
  __device__ __forceinline__ void fill(int i) {
    const LogEntry x = kLogEntries[i];
    const double hi = upper44(x.m2log);
    e[i] = LogEntry{x.inv, hi};
    low[i] = (x.m2log - hi) + kLogLow[i];
  }
};

// A thread's annulus counts within one work unit, 8 bits each: counts 0..7
// in `lo`, 8..9 in `hi` (a thread tallies at most kEpUnit / kEpThreads = 64
// pairs of a unit, so no field overflows).
struct Tally {
  uint64_t lo = 0, hi = 0;
};

// 2^63 (2u - 1) with u = (w >> 11) 2^-53, exactly: the word's upper 53 bits
// less 2^63.  The halves stand as the low mantissa words of 2^84 and 2^52; both
// sums are exact (2^27 pairs: 448 -> 436 us against two conversions and a
// multiply-add).
__device__ __forceinline__ double centred(uint64_t w) {
#pragma clang fp contract(off)
  const double hi = __longlong_as_double(0x4530000000000000ull | (w >> 32));             // 2^84 + 2^32 (w >> 32)
  const double lo = __longlong_as_double(0x4330000000000000ull | (w & 0xFFFFF800ull));   // 2^52 + the lower bits
  return (hi - (0x1p84 + 0x1p63 + 0x1p52)) + lo;
}

// One pair from two generator words: accept it when 0 < t <= 1, add its
// Gaussian pair to the running sums and its annulus, returned, to counts 0..7
// (an annulus of 8 and more goes to the wrong count, for far_annulus to mend:
// about one pair in 10^14).
//
// x, y and t are carried as 2^63 x, 2^63 y and 2^126 t (powers of two: every
// rounding is the one of the definition).  The factor is f = sqrt(s / t) with s =
// -2 ln t, from the table above, the exponent and a polynomial (|r| <= 2^-9, or
// 2^-8 in the first interval: the term left out is below 2^-57 of s).  With y0
// near 1 / sqrt(s t), f0 = s y0 is near f, and s - f0^2 t, from the parts of s
// before they are rounded to one, corrects it: one third-order step instead of a
// division and a root, and two roundings that count (f0 t under the root, f).
// Root mean square and largest error of f in 2^-53 over 2 x 10^7 pairs, emulated:
// 0.468 and 1.86, against 0.520 and 1.89 of a correctly rounded logarithm, divide
// and root (the product of a rounded s with the reciprocal root: 0.752 and 3.24,
// and 445 -> 477 us for 2^27 pairs).
__device__ __forceinline__ int ep_pair(uint64_t wx, uint64_t wy, const LogTable& table, double& sx, double& sy,
                                       Tally& q) {
#pragma clang fp contract(off)
  const double x = centred(wx), y = centred(wy);
  const double t = x * x + y * y;  // two rounded products, one rounded sum
  const bool ok = t > 0.0 && t <= 0x1p126;
  const uint64_t tb = __double_as_longlong(t);
  const uint32_t th = static_cast<uint32_t>(tb >> 32);
  const int e = static_cast<int>(th >> 20) - (1022 + 126);
  const double m = __longlong_as_double((static_cast<uint64_t>((th & 0xFFFFFu) | 0x3FE00000u) << 32) |
                                        static_cast<uint32_t>(tb));
  const uint32_t i = (th >> 12) & (kLogTable - 1);
  const LogEntry c = table.e[i];
  const double r = __builtin_fma(m, c.inv, -1.0);
  double p = __builtin_fma(r, 1.0 / 3.0, -2.0 / 5.0);
  p = __builtin_fma(r, p, 1.0 / 2.0);
  p = __builtin_fma(r, p, -2.0 / 3.0);
  p = __builtin_fma(r, p, 1.0);
  const double ed = static_cast<double>(e);
  const double hi = __builtin_fma(ed, -kTwoLn2Hi, c.m2log);   // s = hi - 2 r + lo
  const double lo = __builtin_fma(r * r, p, __builtin_fma(ed, -kTwoLn2Lo, table.low[i]));
  const double s = __builtin_fma(-2.0, r, hi) + lo;
  const double y0 = __builtin_amdgcn_rsq(__builtin_fma(s, t, 0x1p-900));   // t = 1: s = 0
  const double f0 = s * y0, u = f0 * t;
  const double rest = __builtin_fma(-2.0, r, __builtin_fma(-u, f0, hi)) + lo;
  const double d = __builtin_fma(-u, y0, 1.0);
  const double f = ok ? __builtin_fma(rest * y0, __builtin_fma(d, 0.375, 0.5), f0) : 0.0;   // 2^-63 sqrt(-2 ln t / t)
  const double X = x * f, Y = y * f;
  sx += X;
  sy += Y;
  const int l = static_cast<int>(fmax(fabs(X), fabs(Y)));  // floor; at most 12
  q.lo += static_cast<uint64_t>(ok) << ((8 * l) & 63);
  return l;
}

__device__ __forceinline__ void far_annulus(int l, Tally& q) {
  if (l < 8) return;
  q.lo -= 1ull << ((8 * l) & 63);
  if (l < 10) q.hi += 1ull << (8 * (l - 8));
}

// Fixed-order sum over the 64 lanes, valid in lane 63: lane shifts by 1, 2, 4
// and 8 within the rows of 16, then the rows' last lanes into the rows after
// them (DPP moves instead of shuffles through LDS: with the reduction of few
// records by one wave, 4.1 -> 2.2 us for the second launch of 2^15 pairs).
template <int CTRL, int ROWS, class T>
__device__ __forceinline__ T dpp_move(T v) {
  static_assert(sizeof(T) == 8, "two registers");
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(b), CTRL, ROWS, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<uint32_t>(b >> 32), CTRL, ROWS, 0xF, false);
  return __builtin_bit_cast(T, (static_cast<uint64_t>(hi) << 32) | lo);
}
template <class T>
__device__ __forceinline__ T wave_sum(T v) {
  v += dpp_move<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8
  v += dpp_move<0x112, 0xF>(v);
  v += dpp_move<0x114, 0xF>(v);
  v += dpp_move<0x118, 0xF>(v);
  v += dpp_move<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_move<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

struct EpRecord {
  double sx, sy;
  uint16_t q[10];
  uint32_t pad;
};
static_assert(sizeof(EpRecord) == kEpRecordBytes, "record layout");

// Bound by VALU issue: with two waves or more on a SIMD a wave64 instruction
// takes 4 cycles in binary64, in 64-bit integers and for 32-bit multiplies, a
// plain 32-bit one 2 and a binary64 root 16 (measured with loops of one kind).
// The 285 of two pairs come to about 960 cycles that way; a request of 2^27
// pairs runs at 281 Gpairs/s, 1120 cycles at 2.4 GHz (307 and 1024 with 14
// instructions fewer and the larger error, see ep_pair).  8 waves per workgroup on
// small units fill the SIMDs for requests of any size (a unit of 2^15 pairs on
// 256 threads left a request of 2^15 pairs to one CU: 88 us).
template <int N>
__global__ __launch_bounds__(kEpThreads) void ep_units_kernel(EpGroupN<N> g) {
  __shared__ LogTable table;
  __shared__ double wsx[kEpWaves], wsy[kEpWaves];
  __shared__ uint64_t wq[kEpWaves][3];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint64_t u = blockIdx.x; u < g.total_units; u += g.grid) {
    const int r = find_request(g, u);
    const EpDesc& d = g.d[r];
    const uint64_t local = u - d.unit_begin;
    const uint64_t p0 = local * d.unit;                      // first pair (even)
    const uint64_t p1 = min(p0 + d.unit, d.n);               // end of pairs
    const uint64_t k0 = d.inline_key ? d.key_value[0] : d.key[0];
    const uint64_t k1 = d.inline_key ? d.key_value[1] : d.key[1];
    if (d.inline_key && local == 0 && threadIdx.x < 2) d.key[threadIdx.x] = threadIdx.x ? k1 : k0;
    if (u == blockIdx.x && threadIdx.x < kLogTable) table.fill(threadIdx.x);
    uint64_t h, l;
    mul128(kPhiloxM0, k0, h, l);
    double sx = 0.0, sy = 0.0;
    Tally q;
    __syncthreads();  // the table; wsx .. wq of the unit before
    uint64_t b = p0 / 2 + threadIdx.x;
    for (const uint64_t whole = p1 / 2; b < whole; b += kEpThreads) {
      uint64_t w[4];
      philox_block(b, k0, k1, h, l, w);
      const int la = ep_pair(w[0], w[1], table, sx, sy, q);
      const int lb = ep_pair(w[2], w[3], table, sx, sy, q);
      if (__builtin_expect(max(la, lb) >= 8, 0)) {
        far_annulus(la, q);
        far_annulus(lb, q);
      }
    }
    if (2 * b < p1) {  // the half block at the end of an odd request
      uint64_t w[4];
      philox_block(b, k0, k1, h, l, w);
      far_annulus(ep_pair(w[0], w[1], table, sx, sy, q), q);
    }
    // counts 0, 2, 4, 6 and 1, 3, 5, 7 and 8, 9 in 16-bit fields (64 lanes
    // of at most 64 pairs)
    sx = wave_sum(sx);
    sy = wave_sum(sy);
    const uint64_t q0 = wave_sum(q.lo & 0x00FF00FF00FF00FFull), q1 = wave_sum((q.lo >> 8) & 0x00FF00FF00FF00FFull);
    const uint64_t q2 = wave_sum((q.hi & 0xFF) | ((q.hi & 0xFF00) << 8));
    if (lane == 63) {
      wsx[wave] = sx;
      wsy[wave] = sy;
      wq[wave][0] = q0;
      wq[wave][1] = q1;
      wq[wave][2] = q2;
    }
    __syncthreads();
    EpRecord* rec = reinterpret_cast<EpRecord*>(d.partial) + local;
    const bool only = d.units == 1;
    if (threadIdx.x < 10) {
      const int i = threadIdx.x;
      const int word = i < 8 ? i & 1 : 2, shift = 16 * (i < 8 ? i >> 1 : i - 8);
      uint32_t c = 0;
#pragma unroll
      for (int w = 0; w < kEpWaves; ++w) c += static_cast<uint32_t>(wq[w][word] >> shift) & 0xFFFF;
      if (only) d.out[2 + i] = c;
      else rec->q[i] = static_cast<uint16_t>(c);
    } else if (threadIdx.x == 64 || threadIdx.x == 128) {
      const double* ws = threadIdx.x == 64 ? wsx : wsy;
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < kEpWaves; ++w) sum += ws[w];
      const int i = threadIdx.x == 64 ? 0 : 1;
      if (only) d.out[i] = __double_as_longlong(sum);
      else (i ? rec->sy : rec->sx) = sum;
    }
  }
}

// Sum of a request's records.  Latency: two records per thread at 2^24 pairs
// (4.5 us), and one wave where it holds the records of every request (2.2 us for
// 32 or 49; ten LDS counters added to by every thread took 6.5 us for 32 and
// 13 us for 1024).  Up to 64 records both sum in the same order: the other seven
// waves add zeros, so the choice does not show in the result.
template <int THREADS, int N>
__global__ __launch_bounds__(THREADS) void ep_reduce_kernel(EpGroupN<N> g) {
  constexpr int kWaves = THREADS / 64;
  __shared__ uint64_t ws[kWaves][kEpWords];
  const EpDesc& d = g.d[blockIdx.x];
  if (d.units == 1) return;  // written by the unit launch
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t* rec = static_cast<const uint64_t*>(d.partial);
  double sx = 0.0, sy = 0.0;
  uint64_t q[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (uint64_t i = threadIdx.x; i < d.units; i += THREADS) {
    uint64_t w[kEpRecordBytes / 8];
#pragma unroll
    for (uint64_t k = 0; k < kEpRecordBytes / 8; ++k) w[k] = rec[i * (kEpRecordBytes / 8) + k];
    sx += __longlong_as_double(w[0]);
    sy += __longlong_as_double(w[1]);
#pragma unroll
    for (int l = 0; l < 10; ++l) q[l] += (w[2 + l / 4] >> (16 * (l % 4))) & 0xFFFF;
  }
  sx = wave_sum(sx);
  sy = wave_sum(sy);
#pragma unroll
  for (int l = 0; l < 10; ++l) q[l] = wave_sum(q[l]);
  if (lane == 63) {
    ws[wave][0] = __double_as_longlong(sx);
    ws[wave][1] = __double_as_longlong(sy);
#pragma unroll
    for (int l = 0; l < 10; ++l) ws[wave][2 + l] = q[l];
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += __longlong_as_double(ws[w][threadIdx.x]);
    d.out[threadIdx.x] = __double_as_longlong(sum);
  } else if (threadIdx.x < kEpWords) {
    uint64_t c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c += ws[w][threadIdx.x];
    d.out[threadIdx.x] = c;
  }
}

}  // namespace

void finalize_ep_group(EpGroup& g) {
  uint64_t u = 0;
  for (uint32_t i = 0; i < g.count; ++i) {
    g.d[i].unit = ep_unit(g.d[i].n);
    g.d[i].unit_begin = u;
    g.d[i].units = (g.d[i].n + g.d[i].unit - 1) / g.d[i].unit;
    u += g.d[i].units;
  }
  g.total_units = u;
}

namespace {
template <int N>
hipError_t launch_ep(const EpGroupN<N>& g, hipStream_t s) {
  const hipError_t e = launch_group(ep_units_kernel<N>, g.grid, kEpThreads, s, g);
  if (e != hipSuccess || g.total_units == g.count) return e;
  uint64_t most = 0;
  for (uint32_t i = 0; i < g.count; ++i) most = std::max(most, g.d[i].units);
  return most <= 64 ? launch_group(ep_reduce_kernel<64, N>, g.count, 64, s, g)
                    : launch_group(ep_reduce_kernel<512, N>, g.count, 512, s, g);
}
}  // namespace

hipError_t launch_ep_group(const EpGroup& g0, hipStream_t s) {
  const uint32_t grid = static_cast<uint32_t>(std::min(g0.total_units, kEpGrid));
  if (g0.count == 1) return launch_ep(EpGroupN<1>{1, grid, g0.total_units, {g0.d[0]}}, s);
  EpGroup g = g0;
  g.grid = grid;
  return launch_ep(g, s);
}

}  // namespace gvm
