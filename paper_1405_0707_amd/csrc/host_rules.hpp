// Index arithmetic and rules that kernels and launches share, in plain C++ so
// that it can be checked on a CPU.
#pragma once

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <set>
#include <utility>

#ifdef __HIPCC__
#define EXPMV_HOST_DEVICE __host__ __device__
#else
#define EXPMV_HOST_DEVICE
#endif

namespace expmv {

// Longest staged chunk of CSR entries (csr_rows_staged), and whether an
// operator's entries are staged: rows of at most 8 on average (longer ones would
// leave most lanes idle in each chunk), and entries that end a chunk short of
// INT32_MAX, as chunk_end and the fetch one chunk ahead add up to that to 32-bit
// indices (forming them by difference cost the 128^3 product 0.6%).
constexpr int kStageMost = 2048;
inline bool stage_entries(int64_t nnz, int64_t n) {
  return nnz <= 8 * n && nnz <= INT32_MAX - kStageMost;
}

// End of the chunk of at most `most` (<= kStageMost) entries that starts at b in
// the run [b, e), 0 <= b <= e <= INT32_MAX - kStageMost.
EXPMV_HOST_DEVICE inline int chunk_end(int b, int e, int most) {
  return b + most < e ? b + most : e;
}

// Whether kernels may read and write both blocks 16 bytes at a time.  Blocks of
// the caller need only the alignment of their values.
inline bool aligned16(const void* a, const void* b) {
  return (reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) % 16 == 0;
}

// Whether workgroups that each read some columns of one block and then write the
// same columns of the other may run side by side: the blocks (bytes na, nb) are
// apart or the same.
inline bool same_or_apart(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return (x == y && na == nb) || x + na <= y || y + nb <= x;
}

// Calls set() on the first use of `kernel` on `device` in the process, and
// returns only after a set() that did not throw.  For kernel attributes, which
// belong to the function and not to a plan: they are set once, to a value that
// serves every launch, so that plans on several threads cannot lower each
// other's.  One entry is kept per kernel and device.
template <typename Set>
void once_per_kernel(const void* kernel, int device, Set&& set) {
  static std::mutex mutex;
  static std::set<std::pair<const void*, int>> done;
  std::lock_guard<std::mutex> lock(mutex);
  if (done.count({kernel, device})) return;
  set();
  done.insert({kernel, device});
}

}  // namespace expmv
