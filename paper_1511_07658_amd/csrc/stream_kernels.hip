// Streaming per-rank kernels of the GVM, written for gfx950 (CDNA4, wave64):
//
//  * vector add / multiply (Table 3 "VecAdd", "VecMul"): HBM-bound;
//  * Black-Scholes call + put (Table 3 "BlackScholes"): HBM-bound with a
//    transcendental-heavy body.
//
// Both are grouped launches: one grid walks the work units (vector chunks) of
// every request of the group; the unit -> request map is a search over the
// per-request first unit held in the kernel arguments.  An element is always
// computed by the same operations, whatever unit it falls into and whatever
// else is in the group, so a rank's output is bit-identical alone and in the
// mix.
#include "group_device.hpp"

#include <algorithm>
#include <cmath>
#include <cstdlib>

namespace gvm {

namespace {

// Launch shape, measured on the MI355X (float4 per thread and cache policy,
// 0.26M to 268M elements; three buffers in turn, and one read again).  One
// workgroup per work unit: the dispatcher keeps every SIMD at its
// register-limited occupancy and balances the tail.  Results are stored
// non-temporal at any size: nothing here reads them back, and the 256 MB
// memory-side cache keeps the inputs instead (vector add of 2^22 read again:
// 6.9 us, 8.4 with cached stores).  Inputs are loaded
//  * cached up to kCachedInput bytes of them, with 2 float4 per thread (8M
//    elements 15.0 us, 16.7 non-temporal);
//  * beyond it with 4 float4 per thread, the last operand (b, T) cached where
//    it alone stays within kCachedInput and the others non-temporal: that
//    operand is then read from the memory-side cache the next time (16M
//    elements 29.3 us, 31.7 all non-temporal, 34.6 all cached; 14.5M 26.0, 27.5
//    and 29.8; 16M options 52.9 and 57.8), and a wave that starts inside a line
//    finds it there (b of odd length on its first pass: 36.5 us, 40.3 all
//    non-temporal);
//  * all non-temporal beyond that (three buffers of 33.5M in turn: 61.8 us, 63.0
//    with b cached; 134M 251 and 257).
constexpr uint64_t kCachedInput = 96ull << 20;
enum Loads { kAllCached, kLastCached, kNoneCached };

// ---------------------------------------------------------------- vectors

struct AddOp { __device__ __forceinline__ float operator()(float x, float y) const { return x + y; } };
struct MulOp { __device__ __forceinline__ float operator()(float x, float y) const { return x * y; } };

template <class T, bool NT>
__device__ __forceinline__ T stream_load(const T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

template <class T>
__device__ __forceinline__ void stream_store(T v, T* p) { __builtin_nontemporal_store(v, p); }

// Four consecutive floats at any float alignment: one 16-byte access.
typedef f32x4 f32x4u __attribute__((aligned(4)));

template <class Op>
__device__ __forceinline__ f32x4 op4(Op op, f32x4 a, f32x4 b) {
  return f32x4{op(a.x, b.x), op(a.y, b.y), op(a.z, b.z), op(a.w, b.w)};
}

// Bound by memory.  The operands of a request of odd length start anywhere
// (b is a + n), so every access is 16 bytes at float alignment: 14.5M elements
// 26.0 us (6.7 TB/s, 2^24 has 6.9), 34.8 element by element.
template <class Op, int V4, Loads LOADS, int N>
__global__ __launch_bounds__(kThreads) void vec_group_kernel(VecGroupN<N> g) {
  constexpr uint64_t kUnit = V4 * 4 * kThreads;
  Op op;
  for (uint64_t u = blockIdx.x; u < g.total_units; u += g.grid) {
    const VecDesc& d = g.d[find_request(g, u)];
    const uint64_t e0 = (u - d.unit_begin) * kUnit;
    const uint64_t left = d.n - e0;
    const f32x4u* a4 = reinterpret_cast<const f32x4u*>(d.a + e0);
    const f32x4u* b4 = reinterpret_cast<const f32x4u*>(d.b + e0);
    f32x4u* c4 = reinterpret_cast<f32x4u*>(d.c + e0);
    if (left >= kUnit) {
      f32x4 va[V4], vb[V4];
#pragma unroll
      for (int j = 0; j < V4; ++j) {
        va[j] = stream_load<f32x4u, LOADS != kAllCached>(a4 + threadIdx.x + j * kThreads);
        vb[j] = stream_load<f32x4u, LOADS == kNoneCached>(b4 + threadIdx.x + j * kThreads);
      }
#pragma unroll
      for (int j = 0; j < V4; ++j) stream_store<f32x4u>(op4(op, va[j], vb[j]), c4 + threadIdx.x + j * kThreads);
    } else {
      for (uint64_t e = 4 * threadIdx.x; e < left; e += 4 * kThreads) {
        if (e + 4 <= left) {
          c4[e / 4] = op4(op, a4[e / 4], b4[e / 4]);
        } else {
          for (uint64_t k = e0 + e; k < d.n; ++k) d.c[k] = op(d.a[k], d.b[k]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------- Black-Scholes
//
// Standard normal distribution function from the polynomial approximation of
// Abramowitz and Stegun, Handbook of Mathematical Functions, formula 26.2.17
// (absolute error below 7.5e-8):
//   N(x) = 1 - phi(x) (b1 t + b2 t^2 + b3 t^3 + b4 t^4 + b5 t^5),  t = 1/(1 + p x),  x >= 0
// and N(x) = 1 - N(-x) for x < 0.  The pricing formula itself is the
// Black-Scholes (1973) one of the reference:
//   d1 = (ln(S/K) + (r + sigma^2/2) T) / (sigma sqrt T),  d2 = d1 - sigma sqrt T
//   call = S N(d1) - K e^{-rT} N(d2),  put = K e^{-rT} (1 - N(d2)) - S (1 - N(d1))

// Quotients and reciprocals: a hardware reciprocal with one Newton step and,
// for a quotient, one step on its remainder (within an ulp; the correctly
// rounded divide takes ten instructions and was 40 of the 102 per option).
__device__ __forceinline__ float recip(float a) {
  const float y = __builtin_amdgcn_rcpf(a);
  return fmaf(fmaf(-a, y, 1.0f), y, y);
}
__device__ __forceinline__ float refine(float q, float a, float b, float inv_b) {  // q near a / b
  return fmaf(fmaf(-q, b, a), inv_b, q);
}

// N(x) and 1 - N(x).  The clamp keeps the Newton step of t finite for an
// infinite x; a NaN comes through the exponential.
__device__ __forceinline__ void norm_cdf_as(float x, float& n, float& m) {
  constexpr float p = 0.2316419f;
  constexpr float kPhi = 0.39894228040143267794f;   // 1 / sqrt(2 pi)
  constexpr float b1 = 0.319381530f * kPhi, b2 = -0.356563782f * kPhi, b3 = 1.781477937f * kPhi,
                  b4 = -1.821255978f * kPhi, b5 = 1.330274429f * kPhi;
  constexpr float kHalfLog2e = -0.72134752044448170368f;   // -log2(e) / 2
  const float ax = fabsf(x);
  const float t = recip(fminf(fmaf(p, ax, 1.0f), 0x1p100f));
  const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, b5, b4), b3), b2), b1);
  const float upper = __builtin_amdgcn_exp2f(ax * ax * kHalfLog2e) * poly;   // 1 - N(|x|)
  const float lower = 1.0f - upper;
  n = x >= 0.0f ? lower : upper;
  m = x >= 0.0f ? upper : lower;
}

// Uniform parameters of a launch.  Volatilities outside the range where
// 1 / v refines a quotient take the library's divide.
struct BsParams {
  float r, v, inv_v, half_v2;
};

template <bool SAFE>
__device__ __forceinline__ void bs_price(float S, float K, float T, const BsParams& c, float& call, float& put) {
  float ratio;
  if constexpr (SAFE) {
    ratio = S / K;
  } else {
    const float inv_k = recip(K);
    ratio = refine(S * inv_k, S, K, inv_k);
  }
  const float rs = __frsqrt_rn(T);
  const float sqrt_t = T * rs;
  const float vs = c.v * sqrt_t;
  const float per_vol = SAFE ? rs / c.v : refine(rs * c.inv_v, rs, c.v, c.inv_v);
  const float d1 = (__logf(ratio) + (c.r + c.half_v2) * T) * per_vol;
  const float d2 = d1 - vs;
  const float kd = K * __expf(-c.r * T);
  float n1, m1, n2, m2;
  norm_cdf_as(d1, n1, m1);
  norm_cdf_as(d2, n2, m2);
  call = S * n1 - kd * n2;
  put = kd * m2 - S * m1;
}

// One option; operands that a bare reciprocal does not serve are priced again
// with the library's divide, whatever their neighbours are, so an option's bits
// depend on itself alone.  The step on the remainder turns a quotient beyond
// the float range, or an infinite root, into NaN where a divide keeps it
// infinite.  Between these bounds |S / K| stays below 2^120 and, with v within
// 2^-60 .. 2^60 (the launch's rule), 1 / (v sqrt T) below 2^90; a NaN operand
// gives NaN either way.
template <bool SAFE>
__device__ __forceinline__ bool bs_extreme(float S, float K, float T) {
  const float k = fabsf(K);
  return !SAFE && (fabsf(S) > 0x1p60f || __builtin_amdgcn_fmed3f(k, 0x1p-60f, 0x1p60f) != k || T < 0x1p-60f);
}

template <bool SAFE, int V4, Loads LOADS>
__device__ __forceinline__ void bs_quads(const BsDesc& d, uint64_t e, const BsParams& c) {
  const f32x4u* S4 = reinterpret_cast<const f32x4u*>(d.S + e);
  const f32x4u* K4 = reinterpret_cast<const f32x4u*>(d.K + e);
  const f32x4u* T4 = reinterpret_cast<const f32x4u*>(d.T + e);
  f32x4 S[V4], K[V4], T[V4];
#pragma unroll
  for (int j = 0; j < V4; ++j) {
    S[j] = stream_load<f32x4u, LOADS != kAllCached>(S4 + j * kThreads);
    K[j] = stream_load<f32x4u, LOADS != kAllCached>(K4 + j * kThreads);
    T[j] = stream_load<f32x4u, LOADS == kNoneCached>(T4 + j * kThreads);
  }
#pragma unroll
  for (int j = 0; j < V4; ++j) {
    f32x4 call, put;
    bool extreme = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float x, y;
      bs_price<SAFE>(S[j][k], K[j][k], T[j][k], c, x, y);
      call[k] = x;
      put[k] = y;
      extreme |= bs_extreme<SAFE>(S[j][k], K[j][k], T[j][k]);
    }
    if (__builtin_expect(extreme, 0)) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (bs_extreme<SAFE>(S[j][k], K[j][k], T[j][k])) {
          float x, y;
          bs_price<true>(S[j][k], K[j][k], T[j][k], c, x, y);
          call[k] = x;
          put[k] = y;
        }
    }
    stream_store<f32x4u>(call, reinterpret_cast<f32x4u*>(d.call + e) + j * kThreads);
    stream_store<f32x4u>(put, reinterpret_cast<f32x4u*>(d.put + e) + j * kThreads);
  }
}

// Bound by memory at millions of options: 84 MB of 4M in 14.7-14.9 us, 13.6 at
// the 6.17 TB/s of its access mix.  17.6 us with 102 instructions per option
// (76 now); 300001 options 8.3 us element by element in 74 units of 4096, now
// 3.8 in units of 2048.
template <int V4, Loads LOADS, bool SAFE, int N>
__global__ __launch_bounds__(kThreads) void bs_group_kernel(BsGroupN<N> g) {
  constexpr uint64_t kUnit = V4 * 4 * kThreads;
  const BsParams c{g.rate, g.volatility, 1.0f / g.volatility, 0.5f * g.volatility * g.volatility};
  for (uint64_t u = blockIdx.x; u < g.total_units; u += g.grid) {
    const BsDesc& d = g.d[find_request(g, u)];
    const uint64_t e0 = (u - d.unit_begin) * kUnit;
    const uint64_t left = d.n - e0;
    if (left >= kUnit) {
      bs_quads<SAFE, V4, LOADS>(d, e0 + 4 * threadIdx.x, c);
    } else {
      for (uint64_t e = 4 * threadIdx.x; e < left; e += 4 * kThreads) {
        if (e + 4 <= left) {
          bs_quads<SAFE, 1, LOADS>(d, e0 + e, c);
        } else {
          for (uint64_t k = e0 + e; k < d.n; ++k) {
            float x, y;
            if (bs_extreme<SAFE>(d.S[k], d.K[k], d.T[k])) bs_price<true>(d.S[k], d.K[k], d.T[k], c, x, y);
            else bs_price<SAFE>(d.S[k], d.K[k], d.T[k], c, x, y);
            d.call[k] = x;
            d.put[k] = y;
          }
        }
      }
    }
  }
}

}  // namespace

namespace {

constexpr uint64_t kMaxGrid = 1ull << 24;

// Cut the requests of a launch into units of V4 float4 per thread.
template <int V4, class G>
void cut_units(G& g) {
  constexpr uint64_t kUnit = V4 * 4 * kThreads;
  uint64_t u = 0;
  for (uint32_t i = 0; i < g.count; ++i) {
    g.d[i].unit_begin = u;
    u += (g.d[i].n + kUnit - 1) / kUnit;
  }
  g.total_units = u;
  g.grid = static_cast<uint32_t>(std::min(u, kMaxGrid));
}

// How a launch loads its `operands` inputs of 4 bytes an element.  Tuning
// override (read once per process): GVM_STREAM_NT = 0 (cached) / 1 (not).
template <class G>
Loads stream_loads(const G& g, uint64_t operands) {
  static const int env = [] {
    const char* e = getenv("GVM_STREAM_NT");
    return e ? atoi(e) : -1;
  }();
  if (env >= 0) return env != 0 ? kNoneCached : kAllCached;
  uint64_t n = 0;
  for (uint32_t i = 0; i < g.count; ++i) n += g.d[i].n;
  return n <= kCachedInput / 4 / operands ? kAllCached : n <= kCachedInput / 4 ? kLastCached : kNoneCached;
}

template <class Op, int V4, Loads LOADS>
hipError_t launch_vec_shape(const VecGroup& g0, hipStream_t s) {
  if (g0.count == 1) {
    VecGroupN<1> g{1, 0, 0, {g0.d[0]}};
    cut_units<V4>(g);
    return launch_group(vec_group_kernel<Op, V4, LOADS, 1>, g.grid, kThreads, s, g);
  }
  VecGroup g = g0;
  cut_units<V4>(g);
  return launch_group(vec_group_kernel<Op, V4, LOADS, kMaxGroup>, g.grid, kThreads, s, g);
}

template <class Op>
hipError_t launch_vec(const VecGroup& g, hipStream_t s) {
  switch (stream_loads(g, 2)) {
    case kAllCached: return launch_vec_shape<Op, 2, kAllCached>(g, s);
    case kLastCached: return launch_vec_shape<Op, 4, kLastCached>(g, s);
    default: return launch_vec_shape<Op, 4, kNoneCached>(g, s);
  }
}

template <int V4, Loads LOADS, bool SAFE>
hipError_t launch_bs_shape(const BsGroup& g0, hipStream_t s) {
  if (g0.count == 1) {
    BsGroupN<1> g{1, 0, 0, g0.rate, g0.volatility, {g0.d[0]}};
    cut_units<V4>(g);
    return launch_group(bs_group_kernel<V4, LOADS, SAFE, 1>, g.grid, kThreads, s, g);
  }
  BsGroup g = g0;
  cut_units<V4>(g);
  return launch_group(bs_group_kernel<V4, LOADS, SAFE, kMaxGroup>, g.grid, kThreads, s, g);
}

}  // namespace

hipError_t launch_vecadd_group(const VecGroup& g, hipStream_t s) { return launch_vec<AddOp>(g, s); }

hipError_t launch_vecmul_group(const VecGroup& g, hipStream_t s) { return launch_vec<MulOp>(g, s); }

hipError_t launch_bs_group(const BsGroup& g, hipStream_t s) {
  // 1 / sigma refines a quotient in this range; outside it (zero, NaN) the
  // kernel with the library's divide runs
  const float v = std::fabs(g.volatility);
  if (!(v >= 0x1p-60f && v <= 0x1p60f)) return launch_bs_shape<2, kAllCached, true>(g, s);
  switch (stream_loads(g, 3)) {
    case kAllCached: return launch_bs_shape<2, kAllCached, false>(g, s);
    case kLastCached: return launch_bs_shape<4, kLastCached, false>(g, s);
    default: return launch_bs_shape<4, kNoneCached, false>(g, s);
  }
}

}  // namespace gvm
