// Checks of csrc/host_rules.hpp, built with g++ under UndefinedBehaviorSanitizer
// by tests/test_host_rules.py.
#include <climits>
#include <cstdint>
#include <cstdio>
#include <initializer_list>

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
    at = ce;
  }
  return at == e && chunk_end(e, e, most) == e;
}

int main() {
  bool ordinary = true, at_the_limit = true;
  for (int most : {512, 1024, 2048})
    for (int len : {0, 1, 511, 512, 513, 2047, 2048, 2049, 10000}) {
      ordinary = ordinary && covers(0, len, most) && covers(12345, 12345 + len, most);
      for (int gap : {0, 1, 7, 511, 2048})
        at_the_limit = at_the_limit && covers(INT_MAX - gap - len, INT_MAX - gap, most);
    }
  check(ordinary, "chunks of ordinary runs");
  check(at_the_limit, "chunks of runs that end near INT32_MAX");
  if (!fails) std::printf("ALL OK\n");
  return fails != 0;
}
