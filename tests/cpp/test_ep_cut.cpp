// CPU check of the EP-like kernel's cut (csrc/common.hpp): for every n the
// records of its units fit the request's scratch, a unit is even and at most
// kEpUnit pairs, and the device slot takes the arena granules that 96 bytes
// per 2^15 pairs would take.
#include <cstdio>
#include <random>

#include "common.hpp"

int main() {
  using namespace gvm;
  std::mt19937_64 rng(1);
  int failures = 0;
  auto check = [&](uint64_t n) {
    const uint64_t unit = ep_unit(n), units = (n + unit - 1) / unit;
    const uint64_t coarse = ((n + kEpUnit - 1) / kEpUnit) * 96;
    const uint64_t slot = 2 * kAlign + align_up(ep_scratch_bytes(n), kAlign);
    const uint64_t was = 2 * kAlign + align_up(coarse, kAlign);
    if (unit == 0 || unit % 2 || unit > kEpUnit || units * kEpRecordBytes > ep_scratch_bytes(n) ||
        align_up(slot, 4096) != align_up(was, 4096)) {
      ++failures;
      printf("FAIL: n %llu unit %llu units %llu\n", (unsigned long long)n, (unsigned long long)unit,
             (unsigned long long)units);
    }
  };
  for (uint64_t n = 1; n < 20000; ++n) check(n);
  for (int b = 0; b <= 40; ++b) check(1ull << b);
  for (int i = 0; i < 200000; ++i) check(1 + rng() % (1ull << (13 + i % 28)));
  check(357892096);
  check(357892097);
  printf("%s: %d failures\n", failures ? "FAILED" : "ok", failures);
  return failures != 0;
}
