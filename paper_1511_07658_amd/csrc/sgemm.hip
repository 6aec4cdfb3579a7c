// SGEMM C = A B (Table 3 "MM", single precision) for the GVM on gfx950:
// FP32 MFMA on LDS-staged, double-buffered tiles, as one grouped launch over
// the tiles of every request of the group, one workgroup per tile.  The tile
// -> request map is a search over the per-request first tile held in the
// kernel arguments; every tile configuration sums a C element in the same
// order, so a rank's C is bit-identical alone and in any mix.
#include "gemm_balance.hpp"
#include "gemm_choice.hpp"
#include "group_device.hpp"

#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace gvm {

namespace {

// ---------------------------------------------------------------- SGEMM

// Instruction order of the first half of a k-step: MFMAs with the LDS writes
// of the next tile and then the fetches between them.
template <int M, int W, int L>
__device__ __forceinline__ void sched_mix() {
  constexpr int per = (W + L + M - 1) / M < 1 ? 1 : (W + L + M - 1) / M;
#pragma unroll
  for (int i = 0, w = 0, l = 0; i < M; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
    for (int k = 0; k < per; ++k) {
      if (w < W) {
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        ++w;
      } else if (l < L) {
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        ++l;
      }
    }
  }
}

// ... and of the second half: MFMAs with the reads of the next fragments.
template <int M, int R>
__device__ __forceinline__ void sched_reads() {
  constexpr int H = M / 2 < 1 ? 1 : M / 2;
  constexpr int per = (R + H - 1) / H;
#pragma unroll
  for (int i = 0, r = 0; i < M; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
    for (int k = 0; k < per; ++k)
      if (r < R) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        ++r;
      }
  }
}

// Four consecutive floats at any float alignment (one 16-byte load).
__device__ __forceinline__ f32x4 load4(const void* p) {
  typedef f32x4 f32x4u __attribute__((aligned(4)));
  return *static_cast<const f32x4u*>(p);
}

// Four floats of row r from column c of an n x n matrix, each index clamped
// into the matrix, and the same with zeros in the places outside it.
__device__ __forceinline__ f32x4 edge4(const float* M, int n, int r, int c) {
  const float* p = M + static_cast<size_t>(min(r, n - 1)) * n;
  return f32x4{p[min(c, n - 1)], p[min(c + 1, n - 1)], p[min(c + 2, n - 1)], p[min(c + 3, n - 1)]};
}
__device__ __forceinline__ f32x4 inside4(f32x4 x, int n, int r, int c) {
  return f32x4{r < n && c < n ? x.x : 0.0f, r < n && c + 1 < n ? x.y : 0.0f, r < n && c + 2 < n ? x.z : 0.0f,
               r < n && c + 3 < n ? x.w : 0.0f};
}

// Workgroup tile BM x BN, k-step BK, WM x WN waves; each wave owns a
// (BM/WM) x (BN/WN) block of C in accumulators of one MFMA each: 32x32x2
// (MF 32) or 16x16x4 (MF 16) FP32.
//
// Order of the sum.  Both MFMAs add their k products one after another, each a
// fused multiply-add on the running value (checked on the device bit for bit
// against fmaf), so the order of the k values an MFMA chain is given is the
// order of the sum.  Every run of 16 k is taken as 0 4 8 12, 1 5 9 13,
// 2 6 10 14, 3 7 11 15.  A lane then needs whole runs of four consecutive k
// under either MFMA: with 16x16x4, lane group g = lane / 16 supplies k = 4g + t
// in step t; with 32x32x2, lane group h = lane / 32 supplies 4h + t and
// 8 + 4h + t in the two steps of t.  So tiles lie in LDS in natural order, a
// lane's A values of 16 k are one or two 16-byte reads, and all configurations
// give the same bits.
//
// What bounds it: the matrix unit, once a CU has tiles enough (FP32 MFMA:
// 157.3 TFLOP/s).  A launch of few tiles is bound by what one wave per SIMD
// can hide by itself, which the order within a k-step is for (PIPE):
//   * first half of the k-tile's MFMAs, with the LDS writes of the next k-tile
//     (fetched DEPTH steps ago) and the fetches that take its registers placed
//     between them, one after each MFMA;
//   * the step's one barrier;
//   * second half, with the reads of the next fragments (a second register
//     set) between the MFMAs.
// So no MFMA waits for LDS, for memory or for the barrier's other waves
// longer than one MFMA, and one barrier orders both LDS hazards (buffer kt & 1
// is written in step kt - 1 and read in the same step after the barrier; its
// previous tile was read before the barrier of step kt - 2).  Left to itself
// the compiler moves the fragment reads to their uses, waits for every fetch
// in flight where fetches of the prologue may have changed places, and keeps
// part of the accumulators where it has to move them back every trip: 23.8 us
// for one 1024 x 1024 request, 18.5 us in this order (13.7 us of MFMAs), 96x96
// tiles of 1536 67 and 55.6 us; 8 x 1024 x 1024 134.0 -> 123.8 us, 8 x 2048 x
// 2048 974 -> 934 us against the previous kernel's best tiles.  The two
// largest MF 16 tiles do not have the registers for a second fragment set and
// read their fragments at the start of the step.
//
// Any n: rows of A and columns of B outside the matrix are fetched from a
// valid place (they only reach elements of C that are not stored), so every
// full k-tile runs the same branch-free step, and only the remainder of k is
// masked, once per tile.  Fetches are 16 bytes at any float alignment (a row
// of n floats starts anywhere when n is odd).  n = 517: 73.7 us with masked
// 4-byte fetches in 45 tiles of 64x128 (40 + 5 in a grid of whole rounds over
// the XCDs), 7.4 us now.
//
// Tiles in units, requests in order, tiles of a request row-major.  Workgroup
// w runs on XCD w % 8, so unit (w % 8) * (grid / 8) + w / 8 gives each XCD a
// contiguous block: tiles sharing rows of A and columns of B share an L2.
//
// Balanced grid (mixed sizes): the blocks are cut by work instead of by
// count.  The requests come largest first, so equal counts would give the
// first XCD the longest tiles and the last one the shortest.  The units are
// cut into 16 contiguous slices of equal k-step work instead, and XCD x takes
// slice x from the long end and then slice 15 - x from the short end, so every
// XCD ends on short tiles; the grid holds as many workgroups per XCD as the
// longest pair has units (the rest exit at once).
template <int BM, int BN, int BK, int WM, int WN, int MF, int DEPTH, bool PIPE, int N>
__global__ __launch_bounds__(WM * WN * 64) void sgemm_group_kernel(GemmGroupN<N> g) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / MF, FN = TN / MF;
  constexpr int LG = 64 / MF;       // lane groups of one MFMA, one k each
  constexpr int P = 4 / LG;         // float4 per lane and 16 k
  constexpr int KB = BK / 16;       // runs of 16 k
  constexpr int NK = KB * 4 * P;    // MFMA steps of a k-tile
  constexpr int AST = BK + 4, BST = BN + 4;
  constexpr int A4 = BM * BK / 4 / NT, B4 = BK * BN / 4 / NT;
  static_assert(MF == 16 || MF == 32, "MFMA shape");
  static_assert(TM % MF == 0 && TN % MF == 0 && BK % 16 == 0, "tile shape");
  static_assert(A4 >= 1 && B4 >= 1 && A4 * NT * 4 == BM * BK && B4 * NT * 4 == BK * BN, "tile/threads mismatch");
  static_assert(DEPTH % 2 == 0, "the slot and the fragment set of a step are compile-time");
  using Acc = typename std::conditional<MF == 32, f32x16, f32x4>::type;

  __shared__ __attribute__((aligned(16))) float As[2][BM * AST];
  __shared__ __attribute__((aligned(16))) float Bs[2][BK * BST];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int li = lane % MF, lg = lane / MF;

  // the workgroup's unit (tile)
  uint32_t u = (blockIdx.x % kXcds) * (g.grid / kXcds) + blockIdx.x / kXcds;
  uint32_t uend = g.total_units;
  if (N > 1 && g.balanced) {
    // the j-th workgroup of XCD x takes the j-th unit of the XCD's two
    // slices; the grid holds as many per XCD as the longest pair has units
    // (the slices of xcd_slices(): 2x and 2x + 1, or x and 15 - x when paired)
    const int x = static_cast<int>(blockIdx.x % kXcds);
    const int s0 = g.balanced == 2 ? x : 2 * x;
    const int s1 = g.balanced == 2 ? kGemmSlices - 1 - x : 2 * x + 1;
    const uint32_t j = blockIdx.x / kXcds;
    const uint32_t len0 = g.cut[s0 + 1] - g.cut[s0];
    u = j < len0 ? g.cut[s0] + j : g.cut[s1] + (j - len0);
    uend = j < len0 ? g.cut[s0 + 1] : g.cut[s1 + 1];
  }
  if (u >= uend) return;
  const GemmDesc& d = g.d[find_request(g, u)];
  const int n = static_cast<int>(d.n);
  const uint32_t local = u - d.unit_begin;
  const int row0 = static_cast<int>(local / d.tiles_n) * BM;
  const int col0 = static_cast<int>(local % d.tiles_n) * BN;
  const float* __restrict__ Ab = d.A + static_cast<size_t>(row0) * n;
  const float* __restrict__ Bb = d.B + col0;
  const int nfull = n / BK, rem = n - nfull * BK;

  // per-thread offsets inside a k-tile; rows of A and columns of B outside
  // the matrix read a valid element instead (they only reach elements of C
  // that are not stored)
  uint32_t offa[A4], offb[B4];
#pragma unroll
  for (int i = 0; i < A4; ++i) {
    const int f = tid + i * NT;
    offa[i] = 4u * (static_cast<uint32_t>(min(f / (BK / 4), n - 1 - row0)) * n + (f % (BK / 4)) * 4);
  }
#pragma unroll
  for (int i = 0; i < B4; ++i) {
    const int f = tid + i * NT;
    const int c = (f % (BN / 4)) * 4;
    offb[i] = 4u * (static_cast<uint32_t>(f / (BN / 4)) * n + (col0 + c < n ? c : 0));
  }
  f32x4 ra[DEPTH][A4], rb[DEPTH][B4];
  auto load_tile = [&](int kt, auto slot) {
    constexpr int SL = decltype(slot)::value;
    const char* pa = reinterpret_cast<const char*>(Ab + kt * BK);
    const char* pb = reinterpret_cast<const char*>(Bb + static_cast<size_t>(kt) * BK * n);
#pragma unroll
    for (int i = 0; i < A4; ++i) ra[SL][i] = load4(pa + offa[i]);
#pragma unroll
    for (int i = 0; i < B4; ++i) rb[SL][i] = load4(pb + offb[i]);
  };
  auto store_tile = [&](int buf, const f32x4* a, const f32x4* b) {
#pragma unroll
    for (int i = 0; i < A4; ++i) {
      const int f = tid + i * NT;
      *reinterpret_cast<f32x4*>(&As[buf][(f / (BK / 4)) * AST + (f % (BK / 4)) * 4]) = a[i];
    }
#pragma unroll
    for (int i = 0; i < B4; ++i) {
      const int f = tid + i * NT;
      *reinterpret_cast<f32x4*>(&Bs[buf][(f / (BN / 4)) * BST + (f % (BN / 4)) * 4]) = b[i];
    }
  };
  constexpr int SETS = PIPE ? 2 : 1;
  float af[SETS][FM][KB * P * 4], bf[SETS][FN][KB * P * 4];
  auto read_frags = [&](int buf, auto set) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int k = 16 * b + 4 * (LG * p + lg);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(&As[buf][(wm * TM + i * MF + li) * AST + k]);
          float* o = &af[S][i][(b * P + p) * 4];
          o[0] = x.x; o[1] = x.y; o[2] = x.z; o[3] = x.w;
        }
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            bf[S][j][(b * P + p) * 4 + t] = Bs[buf][(k + t) * BST + wn * TN + j * MF + li];
      }
  };
  Acc acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = Acc{0};
  auto mfma = [&](auto set, int s0, int s1) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      if (s < s0 || s >= s1) continue;
      const int b = s / (4 * P), t = (s / P) % 4, p = s % P;
      const int e = (b * P + p) * 4 + t;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          if constexpr (MF == 32)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[S][i][e], bf[S][j][e], acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[S][i][e], bf[S][j][e], acc[i][j], 0, 0, 0);
        }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  // The k-tile beyond the full ones: fetched in the prologue, or, where the
  // MFMAs of one k-tile take longer than a fetch, before those of the last
  // full tile (the registers are free until then); masked with zeros outside
  // the matrix when it is written to LDS.
  constexpr bool kLateTail = NK * FM * FN * (MF == 32 ? 64 : 32) >= 2048;
  f32x4 ta[A4], tb[B4];
  auto tail = [&](auto f) {
    const int k0 = nfull * BK;
#pragma unroll
    for (int i = 0; i < A4; ++i) {
      const int e = tid + i * NT;
      f(ta[i], d.A, row0 + e / (BK / 4), k0 + (e % (BK / 4)) * 4);
    }
#pragma unroll
    for (int i = 0; i < B4; ++i) {
      const int e = tid + i * NT;
      f(tb[i], d.B, k0 + e / (BN / 4), col0 + (e % (BN / 4)) * 4);
    }
  };
  auto tail_fetch = [&] { tail([&](f32x4& x, const float* M, int r, int c) { x = edge4(M, n, r, c); }); };
  auto tail_store = [&](int buf) {
    tail([&](f32x4& x, const float*, int r, int c) { x = inside4(x, n, r, c); });
    store_tile(buf, ta, tb);
  };
  auto tail_mfma = [&](auto set) {   // only the runs of 16 k that hold any
#pragma unroll
    for (int b = 0; b < KB; ++b)
      if (b == 0 || 16 * b < rem) mfma(set, b * NK / KB, (b + 1) * NK / KB);
  };
  if (nfull == 0) {
    tail_fetch();
    tail_store(0);
    __syncthreads();
    read_frags(0, I0{});
    tail_mfma(I0{});
  } else {
    // tile t waits in slot t % DEPTH; the slots are fetched in the order the
    // loop takes them, or it would wait for the newest one
    load_tile(0, I0{});
    __builtin_amdgcn_sched_barrier(0);
    load_tile(min(1, nfull - 1), I1{});
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (DEPTH >= 4) {
      load_tile(min(2, nfull - 1), std::integral_constant<int, 2 % DEPTH>{});
      __builtin_amdgcn_sched_barrier(0);
      load_tile(min(3, nfull - 1), std::integral_constant<int, 3 % DEPTH>{});
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!kLateTail && rem) tail_fetch();
    store_tile(0, ra[0], rb[0]);
    __builtin_amdgcn_sched_barrier(0);
    load_tile(min(DEPTH, nfull - 1), I0{});
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    if constexpr (PIPE) read_frags(0, I0{});
    auto step = [&](int kt, auto slot, auto set) {
      constexpr int SL = decltype(slot)::value;
      constexpr int S = decltype(set)::value;
      constexpr int MH = NK / 2 * FM * FN;              // MFMAs of half a step
      constexpr int MV = A4 + B4;                       // LDS writes, and fetches, of a step
      constexpr int RD = KB * P * (FM + 2 * FN);        // LDS reads of a step (pairs of 4-byte reads as one)
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (PIPE) {
        store_tile(S ^ 1, ra[SL], rb[SL]);
        load_tile(min(kt + 1 + DEPTH, nfull - 1), slot);
        mfma(set, 0, NK / 2);
        sched_mix<MH, MV, MV>();
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        read_frags(S ^ 1, std::integral_constant<int, S ^ 1>{});
        mfma(set, NK / 2, NK);
        sched_reads<MH, RD>();
      } else {
        read_frags(S, I0{});
        __builtin_amdgcn_sched_barrier(0);
        store_tile(S ^ 1, ra[SL], rb[SL]);
        load_tile(min(kt + 1 + DEPTH, nfull - 1), slot);
        mfma(I0{}, 0, NK);
        sched_mix<2 * MH, MV, MV>();
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto last = [&](auto set) {   // tile nfull - 1, then the remainder
      constexpr int S = decltype(set)::value;
      using Next = std::integral_constant<int, PIPE ? S ^ 1 : 0>;
      using This = std::integral_constant<int, PIPE ? S : 0>;
      if constexpr (!PIPE) read_frags(S, I0{});
      if (kLateTail && rem) tail_fetch();
      if (!kLateTail && rem) tail_store(S ^ 1);
      mfma(This{}, 0, NK);
      if (rem) {
        if (kLateTail) tail_store(S ^ 1);
        __syncthreads();
        read_frags(S ^ 1, Next{});
        tail_mfma(Next{});
      }
    };
    // DEPTH steps per trip, so that every slot is a compile-time tag, then the
    // 0 .. DEPTH - 1 left.  The loop has no exit inside a trip: with one, the
    // compiler takes the newest fetch of any exit as the one to wait for.
    // The parity of the last step names the fragment set of tile nfull - 1.
    const int steps = nfull - 1;
    int kt = 0;
    for (; kt + DEPTH <= steps; kt += DEPTH) {
      step(kt, std::integral_constant<int, 1 % DEPTH>{}, I0{});
      step(kt + 1, std::integral_constant<int, 2 % DEPTH>{}, I1{});
      if constexpr (DEPTH >= 4) {
        step(kt + 2, std::integral_constant<int, 3 % DEPTH>{}, I0{});
        step(kt + 3, std::integral_constant<int, 4 % DEPTH>{}, I1{});
      }
    }
    bool odd = false;
    if (kt < steps) {
      step(kt, std::integral_constant<int, 1 % DEPTH>{}, I0{});
      odd = true;
    }
    if constexpr (DEPTH >= 4) {
      if (kt + 1 < steps) {
        step(kt + 1, std::integral_constant<int, 2 % DEPTH>{}, I1{});
        odd = false;
      }
      if (kt + 2 < steps) {
        step(kt + 2, std::integral_constant<int, 3 % DEPTH>{}, I0{});
        odd = true;
      }
    }
    if (odd) last(I1{});
    else last(I0{});
  }

  float* __restrict__ C = d.C;
  const bool whole = row0 + BM <= n && col0 + BN <= n;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = col0 + wn * TN + j * MF + li;
#pragma unroll
      for (int r = 0; r < MF * MF / 64; ++r) {
        const int row = row0 + wm * TM + i * MF + (MF == 32 ? 8 * (r / 4) + 4 * lg + (r % 4) : 4 * lg + r);
        if (whole || (row < n && col < n)) C[static_cast<size_t>(row) * n + col] = acc[i][j][r];
      }
    }
}

// Tile configurations.  Index order is part of the tuner table format.
const GemmConfig kGemmConfigs[] = {
    {0, 32, 32, 32, 2, 2, false},
    {1, 32, 32, 32, 2, 2, false},
    {2, 32, 32, 64, 2, 2, false},
    {3, 32, 64, 32, 2, 2, false},
    {4, 32, 64, 64, 2, 2, false},
    {5, 64, 32, 32, 2, 2, false},
    {6, 64, 64, 32, 2, 4, false},
    {7, 64, 64, 32, 2, 2, false},
    {8, 64, 64, 32, 2, 2, false},
    {9, 64, 64, 16, 2, 2, false},
    {10, 64, 64, 64, 2, 2, false},
    {11, 64, 96, 32, 2, 2, false},
    {12, 96, 64, 32, 2, 2, false},
    {13, 96, 96, 32, 2, 2, false},
    {14, 96, 128, 32, 2, 2, false},
    {15, 128, 96, 32, 2, 2, false},
    {16, 64, 128, 16, 2, 2, false},
    {17, 64, 128, 32, 2, 2, false},
    {18, 128, 64, 32, 4, 2, false},
    {19, 128, 64, 32, 2, 2, false},
    {20, 128, 128, 16, 2, 2, false},
    {21, 128, 128, 32, 2, 2, false},
    {22, 128, 128, 16, 4, 2, false},
    {23, 128, 128, 32, 2, 4, false},
    {24, 128, 256, 16, 2, 4, false},
    {25, 256, 128, 16, 4, 2, false},
    {26, 64, 256, 16, 1, 4, false},
    {27, 256, 64, 16, 4, 1, false},
    {28, 128, 192, 32, 2, 4, false},
    {29, 192, 128, 32, 4, 2, false},
    {30, 160, 64, 32, 2, 2, false},
};
constexpr int kNumGemmConfigs = sizeof(kGemmConfigs) / sizeof(kGemmConfigs[0]);

int g_forced_config = -1;

#include "gemm_tiles.inc"   // kTileTable: (n_max, config index) rows written by the tuner
constexpr uint64_t kTileTableEnd = 1ull << 30;  // the last row's bound: every larger size

// BT (B staged transposed in LDS) is false in every configuration: the 16-byte
// fragment reads it gives B cost four times the fetch or LDS write instructions.
template <int BM, int BN, int BK, int WM, int WN, bool BT, int MF, int DEPTH, bool PIPE>
hipError_t launch_cfg(const GemmGroup& g0, hipStream_t s) {
  constexpr int NT = WM * WN * 64;
  // one workgroup per unit, in whole rounds over the 8 XCDs
  uint32_t per_xcd = (g0.total_units + kXcds - 1) / kXcds;
  if (g0.balanced) {  // as many as the longest XCD pair of slices has units
    per_xcd = 0;
    for (int x = 0; x < kXcds; ++x) {
      int s0, s1;
      xcd_slices(x, g0.balanced == 2, &s0, &s1);
      per_xcd = std::max(per_xcd, (g0.cut[s0 + 1] - g0.cut[s0]) + (g0.cut[s1 + 1] - g0.cut[s1]));
    }
  }
  const uint32_t grid = per_xcd * kXcds;
  if (g0.count == 1) {
    const GemmGroupN<1> g{1, g0.total_units, grid, 0, {g0.d[0]}, {0}};
    return launch_group(sgemm_group_kernel<BM, BN, BK, WM, WN, MF, DEPTH, PIPE, 1>, grid, NT, s, g);
  }
  GemmGroup g = g0;
  g.grid = grid;
  return launch_group(sgemm_group_kernel<BM, BN, BK, WM, WN, MF, DEPTH, PIPE, kMaxGroup>, grid, NT, s, g);
}

}  // namespace

int gemm_config_count() { return kNumGemmConfigs; }
const GemmConfig& gemm_config(int idx) { return kGemmConfigs[idx]; }
void gemm_config_force(int idx) { g_forced_config = (idx >= 0 && idx < kNumGemmConfigs) ? idx : -1; }

int gemm_config_forced() {
  if (g_forced_config >= 0) return g_forced_config;
  // tuning and tests only: force one configuration for every size
  if (const char* env = getenv("GVM_SGEMM_CONFIG")) {
    const int c = atoi(env);
    if (c >= 0 && c < kNumGemmConfigs) return c;
  }
  return -1;
}
// The tuner times launches of kTableCount requests of one size, so its rows
// hold for those; any other launch takes the cheapest configuration by the
// cost formula, which knows how many tiles the launch has for the chip (one
// 1024 x 1024 request: 18.7 us with the formula's 64x64 tiles, 119 us with the
// 256x128 tiles that are within 1 % of the best for eight of them).  For eight
// requests, over the 32 multiples of 64 up to 2048, the two name the same tiles
// at 19; at the others the table's are faster at small sizes (448: 20.8 and 22.8
// us, 512: 23.7 and 24.4), the formula's at 384 (16.7 and 15.8) and by 1-2 % at
// 768, 1152, 1280 and 1536, and 0.2 % lies between them on average.
int gemm_config_for(uint32_t count, const uint32_t* n, int cus) {
  const int forced = gemm_config_forced();
  if (forced >= 0) return forced;
  constexpr uint32_t kTableCount = 8, kTableStep = 64;
  bool table = count == kTableCount && n[0] % kTableStep == 0 && !cus;
  for (uint32_t i = 1; i < count; ++i) table &= n[i] == n[0];
  if (table)
    for (const auto& row : kTileTable)
      if (n[0] <= row[0] && row[0] < kTileTableEnd) return static_cast<int>(row[1]);
  return gemm_cheapest(count, n, cus ? cus : kGemmCus);
}
int gemm_config_for(const GemmGroup& g, int cus) {
  uint32_t n[kMaxGroup];
  for (uint32_t i = 0; i < g.count; ++i) n[i] = g.d[i].n;
  return gemm_config_for(g.count, n, cus);
}
void finalize_gemm_group(GemmGroup& g, int config_idx) {
  const GemmConfig& c = kGemmConfigs[config_idx];
  uint32_t u = 0;
  for (uint32_t i = 0; i < g.count; ++i) {
    const uint32_t n = g.d[i].n;
    const uint32_t tm = (n + c.bm - 1) / c.bm, tn = (n + c.bn - 1) / c.bn;
    g.d[i].tiles_n = tn;
    g.d[i].unit_begin = u;
    g.d[i].units = tm * tn;
    u += tm * tn;
  }
  g.total_units = u;
  uint32_t units[kMaxGroup], ksteps[kMaxGroup];
  for (uint32_t i = 0; i < g.count; ++i) {
    units[i] = g.d[i].units;
    ksteps[i] = (g.d[i].n + c.bk - 1) / c.bk;
  }
  balance_slices(g.count, units, ksteps, g.cut);
  g.balanced = 0;
}
hipError_t launch_sgemm_group(const GemmGroup& g_in, int config_idx, hipStream_t s) {
  GemmGroup g = g_in;
  bool mixed = false;
  for (uint32_t i = 1; i < g.count; ++i) mixed |= g.d[i].n != g.d[0].n;
  // GVM_SGEMM_XCD_PAIRED=0 keeps each XCD on one contiguous run (tuning)
  static const bool paired = [] {
    const char* e = getenv("GVM_SGEMM_XCD_PAIRED");
    return !(e && e[0] == '0');
  }();
  g.balanced = !mixed ? 0 : paired ? 2 : 1;
  switch (config_idx) {
    case 0: return launch_cfg<32, 32, 32, 2, 2, false, 16, 4, true>(g, s);
    case 1: return launch_cfg<32, 32, 32, 2, 2, false, 16, 2, true>(g, s);
    case 2: return launch_cfg<32, 32, 64, 2, 2, false, 16, 2, true>(g, s);
    case 3: return launch_cfg<32, 64, 32, 2, 2, false, 16, 2, true>(g, s);
    case 4: return launch_cfg<32, 64, 64, 2, 2, false, 16, 2, true>(g, s);
    case 5: return launch_cfg<64, 32, 32, 2, 2, false, 16, 2, true>(g, s);
    case 6: return launch_cfg<64, 64, 32, 2, 4, false, 16, 2, true>(g, s);
    case 7: return launch_cfg<64, 64, 32, 2, 2, false, 16, 4, true>(g, s);
    case 8: return launch_cfg<64, 64, 32, 2, 2, false, 32, 2, true>(g, s);
    case 9: return launch_cfg<64, 64, 16, 2, 2, false, 32, 4, true>(g, s);
    case 10: return launch_cfg<64, 64, 64, 2, 2, false, 32, 2, true>(g, s);
    case 11: return launch_cfg<64, 96, 32, 2, 2, false, 16, 2, true>(g, s);
    case 12: return launch_cfg<96, 64, 32, 2, 2, false, 16, 2, true>(g, s);
    case 13: return launch_cfg<96, 96, 32, 2, 2, false, 16, 2, true>(g, s);
    case 14: return launch_cfg<96, 128, 32, 2, 2, false, 16, 2, true>(g, s);
    case 15: return launch_cfg<128, 96, 32, 2, 2, false, 16, 2, true>(g, s);
    case 16: return launch_cfg<64, 128, 16, 2, 2, false, 32, 4, true>(g, s);
    case 17: return launch_cfg<64, 128, 32, 2, 2, false, 32, 2, true>(g, s);
    case 18: return launch_cfg<128, 64, 32, 4, 2, false, 32, 2, true>(g, s);
    case 19: return launch_cfg<128, 64, 32, 2, 2, false, 32, 2, true>(g, s);
    case 20: return launch_cfg<128, 128, 16, 2, 2, false, 32, 2, true>(g, s);
    case 21: return launch_cfg<128, 128, 32, 2, 2, false, 32, 2, true>(g, s);
    case 22: return launch_cfg<128, 128, 16, 4, 2, false, 32, 4, true>(g, s);
    case 23: return launch_cfg<128, 128, 32, 2, 4, false, 32, 2, true>(g, s);
    case 24: return launch_cfg<128, 256, 16, 2, 4, false, 32, 2, true>(g, s);
    case 25: return launch_cfg<256, 128, 16, 4, 2, false, 32, 2, true>(g, s);
    case 26: return launch_cfg<64, 256, 16, 1, 4, false, 32, 2, true>(g, s);
    case 27: return launch_cfg<256, 64, 16, 4, 1, false, 32, 2, true>(g, s);
    case 28: return launch_cfg<128, 192, 32, 2, 4, false, 16, 2, false>(g, s);
    case 29: return launch_cfg<192, 128, 32, 4, 2, false, 16, 2, false>(g, s);
    case 30: return launch_cfg<160, 64, 32, 2, 2, false, 16, 2, true>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gvm
