// Index arithmetic and rules that kernels and launches share, in plain C++ so
// that it can be checked on a CPU.
#pragma once

#ifdef __HIPCC__
#define EXPMV_HOST_DEVICE __host__ __device__
#else
#define EXPMV_HOST_DEVICE
#endif

namespace expmv {

// End of the chunk of at most `most` entries that starts at b in the run
// [b, e), 0 <= b <= e.  By difference: b + most passes INT32_MAX where a run
// ends within `most` of it.
EXPMV_HOST_DEVICE inline int chunk_end(int b, int e, int most) {
  return e - b > most ? b + most : e;
}

}  // namespace expmv
