// Toeplitz products and Gohberg-Semencul inverses of short length: one
// workgroup takes one complex column (two real ones) through every transform
// and pointwise step in LDS.
//
// The streaming passes of toeplitz.hpp cost one launch each, 2 to 3 us
// whatever the length: at n = 1,000 an inverse took 32 launches and 130-154 us
// for 16 KB of data (44 us here, 26 of them in the kernel; the source-term solve
// 17.5 -> 11.5 ms).  Here a pass is a read of the column from LDS into
// registers, a barrier and a write back in place (Stockham order), with the
// roots of unity in an LDS table made once per launch.  The bound is the
// latency of the passes' barriers and of LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "toeplitz.hpp"

namespace expmv {

constexpr int kSmallFftThreads = 512;
// Longest transforms.  An inverse keeps the table and two columns (48 bytes an
// element, 54 with the padding) in 160 KB.  A product of length 4,096 took 36 us
// here and 29 in its six streaming launches, of length 2,048 15 us and 27.
constexpr int kSmallFftProduct = 2048, kSmallFftInverse = 3000;

// Place of element i of the table or a column in LDS: one element of padding
// after every eight, so that the strided writes of the first passes (stride 8:
// every lane on the same two groups of banks) spread over the banks: product of
// length 2,048 19.4 -> 14.6 us, inverse at n = 1,001 66 -> 52 us
__device__ __host__ inline int small_fft_at(int i) { return i + (i >> 3); }

// A transform length as radices 8, 4, 2, 5, 3 in pass order (at most 7 passes
// up to 3,000, reached by 3^7 = 2,187)
struct SmallRadices {
  int len, passes;
  unsigned char r[12];
};

// table[k] = exp(-2 pi i k / L)
__device__ inline void small_fft_table(int L, cplx* tw) {
  for (int k = threadIdx.x; k < L; k += kSmallFftThreads) {
    double si, co;
    sincospi(-2.0 * double(k) / double(L), &si, &co);
    tw[small_fft_at(k)] = {co, si};
  }
}

// One pass of radix R over NB columns at buf, buf + column (in place; the caller's
// data is visible to the workgroup on entry and on return).  The butterflies
// of all columns are spread over the threads.
template <int R, int NB>
__device__ inline void small_fft_pass(int L, int Ns, const cplx* tw, cplx* buf, double sign) {
  static_assert(kSmallFftProduct <= kSmallFftInverse, "longest transform");
  constexpr int M = (NB * kSmallFftInverse / R + kSmallFftThreads - 1) / kSmallFftThreads;
  const int column = small_fft_at(L) + 1;
  const int S = L / R, ts = S / Ns;   // ts: table step of w = exp(2 pi i / (Ns R))
  cplx V[M][R];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    int j = threadIdx.x + m * kSmallFftThreads;
    if (j >= NB * S) break;
    const cplx* x = buf;
    if (NB == 2 && j >= S) {
      j -= S;
      x += column;
    }
    const int k = j % Ns;
    cplx v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[r] = x[small_fft_at(j + r * S)];
      if (r > 0) {
        const cplx w = tw[small_fft_at(r * k * ts)];   // r k < R Ns: below L
        v[r] = cmul(v[r], cplx{w.x, -sign * w.y});
      }
    }
    dft_small<R>(v, V[m], sign);
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m) {
    int j = threadIdx.x + m * kSmallFftThreads;
    if (j >= NB * S) break;
    cplx* x = buf;
    if (NB == 2 && j >= S) {
      j -= S;
      x += column;
    }
    const int k = j % Ns;
    const int d = (j - k) * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) x[small_fft_at(d + r * Ns)] = V[m][r];
  }
  __syncthreads();
}

// buf <- DFT(buf) (sign -1 forward, +1 inverse, unnormalised) of NB columns
template <int NB>
__device__ inline void small_fft(const SmallRadices& rad, const cplx* tw, cplx* buf, double sign) {
  const int L = rad.len;
  int Ns = 1;
  for (int i = 0; i < rad.passes; ++i) {
    const int R = rad.r[i];
    if (R == 8) small_fft_pass<8, NB>(L, Ns, tw, buf, sign);
    else if (R == 4) small_fft_pass<4, NB>(L, Ns, tw, buf, sign);
    else if (R == 5) small_fft_pass<5, NB>(L, Ns, tw, buf, sign);
    else if (R == 3) small_fft_pass<3, NB>(L, Ns, tw, buf, sign);
    else small_fft_pass<2, NB>(L, Ns, tw, buf, sign);
    Ns *= R;
  }
}

// real columns 2c, 2c + 1 of row i of src (n x p, row length ld), times rs[i]
template <typename T>
__device__ inline cplx small_pair(const T* src, int64_t ld, int p, int c, int i, const double* rs) {
  const double sc = rs ? rs[i] : 1.0;
  const T* s = src + int64_t(i) * ld + 2 * c;
  return {sc * double(s[0]), 2 * c + 1 < p ? sc * double(s[1]) : 0.0};
}
template <typename T>
__device__ inline void small_unpair(T* dst, int64_t ld, int p, int c, int i, double scale, cplx v) {
  T* d = dst + int64_t(i) * ld + 2 * c;
  d[0] = T(scale * v.x);
  if (2 * c + 1 < p) d[1] = T(scale * v.y);
}

// Y = scale * diag(dout) T diag(din) X by the circulant embedding (toeplitz_apply);
// scale includes 1 / L
template <typename T>
__global__ void __launch_bounds__(kSmallFftThreads)
k_small_toeplitz(SmallRadices rad, int n, int p, const T* X, int64_t ldx,
                 T* Y, int64_t ldy, const cplx* __restrict__ sym,
                 const double* __restrict__ din, const double* __restrict__ dout, double scale) {
  extern __shared__ char fft_lds[];
  const int L = rad.len, c = blockIdx.x;
  cplx* tw = reinterpret_cast<cplx*>(fft_lds);
  cplx* buf = tw + small_fft_at(L) + 1;
  small_fft_table(L, tw);
  for (int i = threadIdx.x; i < L; i += kSmallFftThreads)
    buf[small_fft_at(i)] = i < n ? small_pair(X, ldx, p, c, i, din) : cplx{0.0, 0.0};
  __syncthreads();
  small_fft<1>(rad, tw, buf, -1.0);
  for (int i = threadIdx.x; i < L; i += kSmallFftThreads) {
    cplx& b = buf[small_fft_at(i)];
    const cplx v = cmul(b, sym[i]);
    b = {scale * v.x, scale * v.y};
  }
  __syncthreads();
  small_fft<1>(rad, tw, buf, 1.0);
  for (int i = threadIdx.x; i < n; i += kSmallFftThreads)
    small_unpair(Y, ldy, p, c, i, dout ? dout[i] : 1.0, buf[small_fft_at(i)]);
}

// The length-n Gohberg-Semencul inverse (toeplitz_gsf_n: the same factors in
// the same order).  first, last: signs of the twists that open and close the
// skew-circulant factors (0: none).
template <typename T>
__global__ void __launch_bounds__(kSmallFftThreads)
k_small_gsf_n(SmallRadices rad, int p, const T* V, T* W,
              const cplx* __restrict__ f1, const cplx* __restrict__ f2,
              const cplx* __restrict__ g1, const cplx* __restrict__ g2,
              const double* __restrict__ din, const double* __restrict__ dout, double first,
              double last, double scale) {
  extern __shared__ char fft_lds[];
  const int n = rad.len, c = blockIdx.x;
  cplx* tw = reinterpret_cast<cplx*>(fft_lds);
  cplx* buf = tw + small_fft_at(n) + 1;   // two columns
  cplx* buf2 = buf + small_fft_at(n) + 1;
  const double inv = 1.0 / double(n);
  small_fft_table(n, tw);
  for (int i = threadIdx.x; i < n; i += kSmallFftThreads) {
    const cplx v = small_pair(V, p, p, c, i, din);
    buf[small_fft_at(i)] = first != 0.0 ? cmul(v, twist_factor(i, n, first)) : v;
  }
  __syncthreads();
  small_fft<1>(rad, tw, buf, -1.0);
  for (int i = threadIdx.x; i < n; i += kSmallFftThreads) {
    const int m = i == 0 ? 0 : n - i, at = small_fft_at(i);
    const cplx u = buf[at], a = cmul(u, f1[m]), b = cmul(u, f2[m]);
    buf[at] = {inv * a.x, inv * a.y};
    buf2[at] = {inv * b.x, inv * b.y};
  }
  __syncthreads();
  small_fft<2>(rad, tw, buf, 1.0);
  for (int i = threadIdx.x; i < n; i += kSmallFftThreads) {
    const cplx t = twist_factor(i, n, 1.0);
    const int at = small_fft_at(i);
    buf[at] = cmul(buf[at], t);
    buf2[at] = cmul(buf2[at], t);
  }
  __syncthreads();
  small_fft<2>(rad, tw, buf, -1.0);
  for (int i = threadIdx.x; i < n; i += kSmallFftThreads) {
    const int at = small_fft_at(i);
    const cplx a = cmul(buf[at], g1[i]), b = cmul(buf2[at], g2[i]);
    buf[at] = {inv * (a.x - b.x), inv * (a.y - b.y)};
  }
  __syncthreads();
  small_fft<1>(rad, tw, buf, 1.0);
  for (int i = threadIdx.x; i < n; i += kSmallFftThreads) {
    cplx v = buf[small_fft_at(i)];
    if (last != 0.0) v = cmul(v, twist_factor(i, n, last));
    small_unpair(W, p, p, c, i, dout ? scale * dout[i] : scale, v);
  }
}

// The embedding form of the inverse (toeplitz_gsf: triangular products of
// length L, for an n with a prime factor above 5)
template <typename T>
__global__ void __launch_bounds__(kSmallFftThreads)
k_small_gsf(SmallRadices rad, int n, int p, const T* V, T* W,
            const cplx* __restrict__ a1, const cplx* __restrict__ a2,
            const cplx* __restrict__ b1, const cplx* __restrict__ b2,
            const double* __restrict__ din, const double* __restrict__ dout, double scale) {
  extern __shared__ char fft_lds[];
  const int L = rad.len, c = blockIdx.x;
  cplx* tw = reinterpret_cast<cplx*>(fft_lds);
  cplx* buf = tw + small_fft_at(L) + 1;   // two columns
  cplx* buf2 = buf + small_fft_at(L) + 1;
  const double inv = 1.0 / double(L);
  small_fft_table(L, tw);
  for (int i = threadIdx.x; i < L; i += kSmallFftThreads)
    buf[small_fft_at(i)] = i < n ? small_pair(V, p, p, c, n - 1 - i, din) : cplx{0.0, 0.0};
  __syncthreads();
  small_fft<1>(rad, tw, buf, -1.0);
  for (int i = threadIdx.x; i < L; i += kSmallFftThreads) {
    const int at = small_fft_at(i);
    const cplx u = buf[at], a = cmul(u, a1[i]), b = cmul(u, a2[i]);
    buf[at] = {inv * a.x, inv * a.y};
    buf2[at] = {inv * b.x, inv * b.y};
  }
  __syncthreads();
  small_fft<2>(rad, tw, buf, 1.0);
  // reversed in place and cut to n rows
  for (int i = threadIdx.x; i < L; i += kSmallFftThreads) {
    const int m = n - 1 - i, at = small_fft_at(i);
    if (i < m) {
      const int am = small_fft_at(m);
      const cplx a = buf[at], b = buf2[at];
      buf[at] = buf[am];
      buf[am] = a;
      buf2[at] = buf2[am];
      buf2[am] = b;
    } else if (i >= n) {
      buf[at] = buf2[at] = {0.0, 0.0};
    }
  }
  __syncthreads();
  small_fft<2>(rad, tw, buf, -1.0);
  for (int i = threadIdx.x; i < L; i += kSmallFftThreads) {
    const int at = small_fft_at(i);
    const cplx a = cmul(buf[at], b1[i]), b = cmul(buf2[at], b2[i]);
    buf[at] = {inv * (a.x - b.x), inv * (a.y - b.y)};
  }
  __syncthreads();
  small_fft<1>(rad, tw, buf, 1.0);
  for (int i = threadIdx.x; i < n; i += kSmallFftThreads)
    small_unpair(W, p, p, c, i, dout ? scale * dout[i] : scale, buf[small_fft_at(i)]);
}

}  // namespace expmv
