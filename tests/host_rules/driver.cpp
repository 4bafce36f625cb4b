// Checks of csrc/host_rules.hpp, built with g++ under UndefinedBehaviorSanitizer
// by tests/test_host_rules.py.
#include <atomic>
#include <climits>
#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include <stdexcept>
#include <thread>
#include <vector>

#include "host_rules.hpp"

using namespace expmv;

static int fails = 0;
static void check(bool ok, const char* what) {
  std::printf("%s %s\n", ok ? "ok  " : "FAIL", what);
  if (!ok) ++fails;
}

// the chunks of a staged tile: every entry of [b, e) once, in order, in chunks
// of at most `most`
static bool covers(int b, int e, int most) {
  int64_t at = b;
  for (int steps = 0; at < e; ++steps) {
    const int ce = chunk_end(int(at), e, most);
    if (ce <= at || ce > e || ce - at > most || steps > 100) return false;
    volatile int fetched = ce + most;   // the fetch one chunk ahead
    if (fetched < ce) return false;
    at = ce;
  }
  return at == e && chunk_end(e, e, most) == e;
}

int main() {
  bool ordinary = true, at_the_limit = true;
  for (int most : {512, 1024, 2048})
    for (int len : {0, 1, 511, 512, 513, 2047, 2048, 2049, 10000}) {
      ordinary = ordinary && covers(0, len, most) && covers(12345, 12345 + len, most);
      // up to the last operator that is staged
      for (int gap : {kStageMost, kStageMost + 1, kStageMost + 7})
        at_the_limit = at_the_limit && covers(INT_MAX - gap - len, INT_MAX - gap, most);
    }
  const int64_t n = int64_t(1) << 30;
  check(stage_entries(INT_MAX - kStageMost, n) && !stage_entries(INT_MAX - kStageMost + 1, n) &&
            stage_entries(80, 10) && !stage_entries(81, 10),
        "which operators are staged");
  check(ordinary, "chunks of ordinary runs");
  check(at_the_limit, "chunks of runs that end near INT32_MAX");

  alignas(16) static double block[8];
  check(aligned16(block, block + 2) && !aligned16(block + 1, block) && !aligned16(block, block + 3),
        "16-byte accesses only when both blocks are aligned");

  const size_t d = sizeof(double);
  check(same_or_apart(block, 4 * d, block, 4 * d) && same_or_apart(block, 4 * d, block + 4, 4 * d) &&
            same_or_apart(block + 4, 4 * d, block, 4 * d) &&
            !same_or_apart(block, 4 * d, block + 3, 4 * d) &&
            !same_or_apart(block + 1, 4 * d, block, 4 * d) &&
            !same_or_apart(block, 4 * d, block, 3 * d),
        "columns in parallel only when the blocks are apart or the same");

  // several threads, each using every kernel on two devices: one set() per
  // kernel and device, finished before any thread goes on to its launch
  const int kernels = 6, threads = 8;
  static char fn[kernels];
  std::atomic<int> sets[2][kernels] = {};
  std::atomic<bool> early{false};
  std::vector<std::thread> pool;
  for (int t = 0; t < threads; ++t)
    pool.emplace_back([&, t]() {
      for (int i = 0; i < 2000; ++i) {
        const int k = (i + t) % kernels, d = (i / kernels) % 2;
        once_per_kernel(&fn[k], d, [&]() {
          std::this_thread::yield();
          ++sets[d][k];
        });
        if (sets[d][k].load() != 1) early = true;
      }
    });
  for (auto& th : pool) th.join();
  bool once = true;
  for (auto& dev : sets)
    for (auto& s : dev) once = once && s.load() == 1;
  check(once && !early.load(), "attributes set once per kernel and device, before use");

  // a set() that fails is tried again
  static char other;
  int calls = 0;
  for (int i = 0; i < 3; ++i) {
    try {
      once_per_kernel(&other, 0, [&]() {
        if (++calls == 1) throw std::runtime_error("refused");
      });
    } catch (const std::runtime_error&) {
    }
  }
  check(calls == 2, "a failed setting is repeated, a successful one is not");
  if (!fails) std::printf("ALL OK\n");
  return fails != 0;
}
