// Device kernels of the GVM for gfx950 and their host-side launchers.
//
// Every launcher takes a *group* of requests of one kernel id and covers all
// of them with one persistent launch; a single request is a group of one, so
// a rank's result does not depend on what else runs with it (each output
// element is produced by the same code with the same operation order).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gvm {

// Requests per grouped launch.  The descriptors are kernel arguments, and a
// launch costs the host by their size (2.7 us with 64 bytes, 3.3 with 256, 4.1
// with 1408), so each group type comes with a capacity N: kMaxGroup (< 2 KiB)
// for a group, 1 for a launch of one request.
constexpr int kMaxGroup = 32;

struct VecDesc {
  const float* a;
  const float* b;
  float* c;
  uint64_t n;
  uint64_t unit_begin;  // first work unit of this request in the group
};

template <int N>
struct VecGroupN {
  uint32_t count;
  uint32_t grid;         // workgroups of the launch
  uint64_t total_units;
  VecDesc d[N];
};
using VecGroup = VecGroupN<kMaxGroup>;

struct BsDesc {
  const float* S;
  const float* K;
  const float* T;
  float* call;
  float* put;
  uint64_t n;
  uint64_t unit_begin;
};

template <int N>
struct BsGroupN {
  uint32_t count;
  uint32_t grid;
  uint64_t total_units;
  float rate;
  float volatility;
  BsDesc d[N];
};
using BsGroup = BsGroupN<kMaxGroup>;

struct GemmDesc {
  const float* A;
  const float* B;
  float* C;
  uint32_t n;        // square size
  uint32_t tiles_n;  // tiles along the columns of C
  uint32_t unit_begin;
  uint32_t units;    // tiles of this request
};

constexpr int kGroupXcds = 8;  // MI355X: workgroup w is dispatched to XCD w % 8

template <int N>
struct GemmGroupN {
  uint32_t count;
  uint32_t total_units;
  uint32_t grid;
  uint32_t balanced;
  GemmDesc d[N];
  // Balanced launch (mixed sizes, one workgroup per tile): the units are cut
  // into 16 slices of equal k-step work, slice s = [cut[s], cut[s + 1]), and
  // each XCD takes two of them (csrc/gemm_balance.hpp): balanced = 1 two
  // neighbouring slices, balanced = 2 one from each end.  Filled by
  // finalize_gemm_group; set by the launcher.  One request is never mixed.
  uint32_t cut[N > 1 ? 2 * kGroupXcds + 1 : 1];
};
using GemmGroup = GemmGroupN<kMaxGroup>;

struct EpDesc {
  uint64_t* key;         // (k0, k1) on the device
  uint64_t* out;         // sx, sy (binary64 bit patterns), q[0..9]
  void* partial;         // one record (kEpRecordBytes) per work unit, 8-byte aligned
  uint64_t n;            // pairs
  uint64_t unit;         // pairs per work unit (ep_unit(n), set by finalize_ep_group)
  uint64_t unit_begin;
  uint64_t units;
  // inline_key: the key comes with the launch, and the kernel leaves it at
  // `key` for requests on the resident input
  uint64_t inline_key, key_value[2];
};

template <int N>
struct EpGroupN {
  uint32_t count;
  uint32_t grid;
  uint64_t total_units;
  EpDesc d[N];
};
using EpGroup = EpGroupN<kMaxGroup>;

// SGEMM tile configurations available to the tuner.  Every configuration sums
// a C element in the same order, so the choice changes a launch's time and
// never its bits.
struct GemmConfig {
  int id;
  int bm, bn, bk;   // macro tile of one workgroup
  int wm, wn;       // waves along M and N (wave tile = bm/wm x bn/wn)
  bool bt;          // B staged k-contiguous in LDS (transposed), else row-major (every one now)
};

int gemm_config_count();
const GemmConfig& gemm_config(int idx);
// Tile configuration of one launch of the sizes n[0 .. count), or of a group
// whose sizes are filled in, on `cus` of the chip's CUs (0: all).
int gemm_config_for(uint32_t count, const uint32_t* n, int cus = 0);
int gemm_config_for(const GemmGroup& g, int cus = 0);
// The configuration forced for every launch (by gemm_config_force or the
// environment), or -1.
int gemm_config_forced();
// Override the table (tuner only): config index for every n, or -1 to restore.
void gemm_config_force(int idx);

// Launchers of the streaming kernels: they cut the requests into work units
// for the launch (unit_begin, total_units).  Return hipSuccess or the error.
hipError_t launch_vecadd_group(const VecGroup& g, hipStream_t s);
hipError_t launch_vecmul_group(const VecGroup& g, hipStream_t s);
hipError_t launch_bs_group(const BsGroup& g, hipStream_t s);
// One workgroup per tile; for a group of mixed sizes the tiles are spread over
// the XCDs by their k-steps (GemmGroup.cut) instead of by count.
hipError_t launch_sgemm_group(const GemmGroup& g, int config_idx, hipStream_t s);
// EP-like tally: one launch over the work units of every request (partials),
// then one workgroup per request sums its partials.
hipError_t launch_ep_group(const EpGroup& g, hipStream_t s);

// Fill the unit bookkeeping of a group (unit_begin, tiles, totals).
void finalize_gemm_group(GemmGroup& g, int config_idx);
void finalize_ep_group(EpGroup& g);

}  // namespace gvm
