// A restart eigenproblem that is not needed any more ends early
// (tests/test_host_stop.py): the host eigensolvers under a StopToken.
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <future>
#include <random>
#include <thread>
#include <vector>

#include "eig_host.hpp"

using namespace expmv;
using Clock = std::chrono::steady_clock;

static int fails = 0;
static void check(bool ok, const char* what) {
  std::printf("%s %s\n", ok ? "ok  " : "FAIL", what);
  if (!ok) ++fails;
}
static double seconds(Clock::time_point a) {
  return std::chrono::duration<double>(Clock::now() - a).count();
}

int main() {
  const int n = 500;
  std::mt19937_64 rng(7);
  std::normal_distribution<double> g;
  std::vector<double> A(size_t(n) * n), S(A.size());
  for (auto& a : A) a = g(rng);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) S[size_t(i) * n + j] = A[size_t(i) * n + j] + A[size_t(j) * n + i];

  auto general = [&](StopToken stop) {
    std::vector<double> wr(n), wi(n), Vr(A.size()), Vi(A.size());
    HessForm hf;
    if (!general_eigvals(n, A.data(), wr.data(), wi.data(), &hf, stop)) return false;
    general_eigvecs(n, A.data(), wr.data(), wi.data(), nullptr, Vr.data(), Vi.data(), &hf, stop);
    return true;
  };
  auto symmetric = [&](StopToken stop) {
    std::vector<double> w(n), Q(S.size());
    return sym_eig(n, S.data(), w.data(), Q.data(), stop);
  };
  for (int kind = 0; kind < 2; ++kind) {
    auto solve = [&](StopToken stop) { return kind ? symmetric(stop) : general(stop); };
    const char* name = kind ? "symmetric" : "general";
    auto t0 = Clock::now();
    std::atomic<bool> flag{false};
    check(solve(StopToken{&flag}), name);   // a token that is never set changes nothing
    const double full = seconds(t0);
    for (double part : {0.0, 0.1, 0.4, 0.7}) {
      flag = false;
      auto f = std::async(std::launch::async, solve, StopToken{&flag});
      std::this_thread::sleep_for(std::chrono::duration<double>(part * full));
      flag = true;
      t0 = Clock::now();
      bool stopped = false;
      try {
        f.get();
      } catch (const Stopped&) {
        stopped = true;
      }
      const double wait = seconds(t0);
      std::printf("%s: whole %.3f s, stopped after %.1f of it, then %.4f s\n", name, full, part, wait);
      // it ends within one step of its loops (n or more of them in each)
      check(stopped && wait < 0.15 * full, "stopped early");
    }
  }
  if (!fails) std::printf("ALL OK\n");
  return fails != 0;
}
