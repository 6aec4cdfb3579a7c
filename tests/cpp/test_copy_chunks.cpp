// Chunks of a host copy: eight for one that finds nothing queued, 4 MiB behind
// others; every byte arrives.
#include <atomic>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "copy_pool.hpp"

namespace {
constexpr size_t kMiB = size_t(1) << 20;
int failed = 0;
void check(bool ok, const char* what) {
  if (!ok) std::printf("FAILED %s\n", what), ++failed;
}
void drain(std::atomic<int>& pending) {
  while (pending.load(std::memory_order_acquire) != 0) std::this_thread::yield();
}
}  // namespace

int main() {
  gvm::CopyEngine e;
  e.start(1);
  std::vector<char> a(128 * kMiB + 5), b(a.size());
  for (size_t i = 0; i < a.size(); ++i) a[i] = static_cast<char>(i * 2654435761u >> 24);
  std::atomic<int> first{0}, second{0}, small{0};

  const size_t sizes[] = {16385, 512 << 10, 8 * kMiB, 8 * kMiB + 5, 64 * kMiB + 1};
  const size_t chunks[] = {1, 1, 8, 8, 17};
  for (int i = 0; i < 5; ++i) {
    std::memset(b.data(), 0, b.size());
    e.reset_stats();
    e.submit(b.data(), a.data(), sizes[i], &first);
    check(e.stats().max_queue == chunks[i], "chunks of a copy alone");
    drain(first);
    check(std::memcmp(a.data(), b.data(), sizes[i]) == 0 && (sizes[i] == b.size() || b[sizes[i]] == 0), "bytes of a copy alone");
  }

  std::memset(b.data(), 0, b.size());
  e.reset_stats();
  e.submit(b.data(), a.data(), 120 * kMiB, &first);                                   // 30 chunks, one worker
  e.submit(b.data() + 120 * kMiB, a.data() + 120 * kMiB, 8 * kMiB, &second, true);    // 2 more
  check(e.stats().max_queue <= 32, "chunks behind other copies");
  e.submit(b.data() + 128 * kMiB, a.data() + 128 * kMiB, 5, &small);
  check(small.load() == 0 && std::memcmp(b.data() + 128 * kMiB, a.data() + 128 * kMiB, 5) == 0, "a few bytes at once");
  drain(first);
  drain(second);
  check(a == b, "bytes behind other copies");
  e.stop();
  if (!failed) std::printf("ok\n");
  return failed != 0;
}
