// Block Gram-Schmidt and CholQR2 of a small block in one workgroup.
//
// The streaming passes (orth_mfma.hpp) take 14 launches per block step, 2 to 7
// us each plus the gaps, whatever the size.  Here one workgroup keeps the block
// W in LDS and reads the basis four times from L2: project, update, project
// again, update, then both Cholesky QR passes.  Bound: the latency of those
// sweeps (one CU's L2 bandwidth would allow 2.7 us each at n = 1,728, 30 columns)
// and of the p^2 wavefront sums per panel.  A step takes 34-37 us instead of
// 53-60 and its launches' gaps: the source-term solve at n = 1,000 11.5 -> 8.3 ms,
// 32^2, p = 4 4.3 -> 3.9, 12^3 upwind, p = 3 11.2 -> 10.1.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "kernels_dense.hpp"
#include "small_solve.hpp"

namespace expmv {

constexpr int kSmallOrthThreads = 512;
constexpr int kSmallOrthCols = 4;         // widest block (P^2 sums per panel)
constexpr int kSmallOrthBlock = 6144;     // entries of W (LDS)

// G = R^T R and R^{-1} as k_cholqr_factor forms them (its stages 1, 2 and 3),
// for a p x p Gram matrix in LDS; the whole workgroup calls it.  Returns
// whether a shifted factor was taken (stage 1: a third pass follows).
__device__ inline bool small_cholqr(int p, const double* G, double* R, double* Ri,
                                    const double* w0norm2, int stage, double shift_rel,
                                    int* __restrict__ flags, int* s_int) {
  const int tid = threadIdx.x;
  for (int i = tid; i < p * p; i += kSmallOrthThreads) R[i] = Ri[i] = 0.0;
  __syncthreads();
  if (tid == 0) {
    double tr = 0.0, wn = 0.0;
    for (int i = 0; i < p; ++i) tr += G[i * p + i];
    if (stage == 1 && w0norm2)
      for (int b = 0; b < p; ++b) wn += w0norm2[b];
    bool zero = (stage == 1 && w0norm2) ? (tr <= 1e-24 * wn) : (tr == 0.0);
    bool shifted = false;
    if (!zero) {
      int st = chol_upper(p, G, 0.0, tr, R);
      if (stage == 1 && st != 0) {
        st = chol_upper(p, G, shift_rel * tr, tr, R);
        shifted = st != 2;
      }
      if (st == 2) {
        flags[1] = 1;
        zero = true;
      }
    } else if (stage == 1 && w0norm2) {
      flags[0] = 1;
    }
    s_int[0] = zero;
    s_int[1] = shifted;
  }
  __syncthreads();
  if (s_int[0]) {
    for (int i = tid; i < p * p; i += kSmallOrthThreads) R[i] = 0.0;
  } else if (tid < p) {
    const int j = tid;
    Ri[j * p + j] = 1.0 / R[j * p + j];
    for (int i = j - 1; i >= 0; --i) {
      double acc = 0.0;
      for (int k = i + 1; k <= j; ++k) acc += R[i * p + k] * Ri[k * p + j];
      Ri[i * p + j] = -acc / R[i * p + i];
    }
  }
  const bool shifted = s_int[1] != 0;
  __syncthreads();
  return shifted;
}

// The block step of orthonormalize: W (n x P) against npan panels of V, the
// result to Vout; H(0 : npan P, col0 ..) += the coefficients and H(npan P ..,
// col0 ..) = the factor, or (H NULL) Rhat = the factor.
// Dynamic LDS: coefficients (npan P^2 doubles), W (n P entries).
template <typename T, int P>
__global__ void __launch_bounds__(kSmallOrthThreads)
k_orth_small(int n, int npan, const T* __restrict__ V, const T* W, T* __restrict__ Vout,
             double* __restrict__ H, int ldh, int col0, double* __restrict__ Rhat,
             double shift_rel, int* __restrict__ flags) {
  constexpr int NW = kSmallOrthThreads / 64, PP = P * P;
  extern __shared__ char orth_lds[];
  __shared__ double sG[PP], sR[PP], sRi[PP], sF[PP], s_w0[P], red[NW * PP];
  __shared__ int s_int[2];
  double* sc = reinterpret_cast<double*>(orth_lds);
  T* sw = reinterpret_cast<T*>(sc + npan * PP);
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  for (int i = tid; i < n * P; i += kSmallOrthThreads) sw[i] = W[i];
  __syncthreads();

  // sc = V^T W: panels over wavefronts, rows over lanes, four rows in flight
  auto project = [&]() {
    for (int i = wave; i < npan; i += NW) {
      const T* v = V + int64_t(i) * n * P;
      double acc[P][P];
#pragma unroll
      for (int a = 0; a < P; ++a)
#pragma unroll
        for (int b = 0; b < P; ++b) acc[a][b] = 0.0;
      constexpr int U = 4;
      for (int r0 = lane; r0 < n; r0 += 64 * U) {
        T x[U][P];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int a = 0; a < P; ++a) {
            const int r = r0 + 64 * u;
            x[u][a] = r < n ? v[r * P + a] : T(0);
          }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int r = r0 + 64 * u;
          if (r < n) {
#pragma unroll
            for (int b = 0; b < P; ++b) {
              const double w = double(sw[r * P + b]);
#pragma unroll
              for (int a = 0; a < P; ++a) acc[a][b] += double(x[u][a]) * w;
            }
          }
        }
      }
#pragma unroll
      for (int a = 0; a < P; ++a)
#pragma unroll
        for (int b = 0; b < P; ++b) {
          const double s = wave_sum(acc[a][b]);
          if (lane == 0) sc[(i * P + a) * P + b] = s;
        }
    }
    __syncthreads();
  };
  // W -= V sc, one row per thread and step, four panels in flight; H += sc
  auto update = [&]() {
    for (int r = tid; r < n; r += kSmallOrthThreads) {
      double w[P];
#pragma unroll
      for (int b = 0; b < P; ++b) w[b] = double(sw[r * P + b]);
      constexpr int U = 4;
      for (int i0 = 0; i0 < npan; i0 += U) {
        T x[U][P];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int a = 0; a < P; ++a)
            x[u][a] = i0 + u < npan ? V[(int64_t(i0 + u) * n + r) * P + a] : T(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (i0 + u >= npan) break;
#pragma unroll
          for (int a = 0; a < P; ++a)
#pragma unroll
            for (int b = 0; b < P; ++b)
              w[b] -= double(x[u][a]) * sc[((i0 + u) * P + a) * P + b];
        }
      }
#pragma unroll
      for (int b = 0; b < P; ++b) sw[r * P + b] = T(w[b]);
    }
    for (int o = tid; o < npan * PP; o += kSmallOrthThreads)
      H[int64_t(o / P) * ldh + col0 + o % P] += sc[o];
    __syncthreads();
  };
  // sG = W^T W; diag: only the squared norms, into s_w0
  auto gram = [&](bool diag) {
    double acc[P][P];
#pragma unroll
    for (int a = 0; a < P; ++a)
#pragma unroll
      for (int b = 0; b < P; ++b) acc[a][b] = 0.0;
    for (int r = tid; r < n; r += kSmallOrthThreads) {
      double w[P];
#pragma unroll
      for (int b = 0; b < P; ++b) w[b] = double(sw[r * P + b]);
#pragma unroll
      for (int a = 0; a < P; ++a)
#pragma unroll
        for (int b = a; b < P; ++b) acc[a][b] += w[a] * w[b];
    }
#pragma unroll
    for (int a = 0; a < P; ++a)
#pragma unroll
      for (int b = a; b < P; ++b) {
        const double s = wave_sum(acc[a][b]);
        if (lane == 0) red[wave * PP + a * P + b] = s;
      }
    __syncthreads();
    for (int o = tid; o < PP; o += kSmallOrthThreads) {
      const int a = min(o / P, o % P), b = max(o / P, o % P);
      double s = 0.0;
      for (int w = 0; w < NW; ++w) s += red[w * PP + a * P + b];
      if (!diag) sG[o] = s;
      else if (o / P == o % P) s_w0[a] = s;
    }
    __syncthreads();
  };
  // W <- W C, or out <- W C
  auto scale = [&](const double* C, T* out) {
    for (int r = tid; r < n; r += kSmallOrthThreads) {
      double w[P];
#pragma unroll
      for (int a = 0; a < P; ++a) w[a] = double(sw[r * P + a]);
#pragma unroll
      for (int b = 0; b < P; ++b) {
        double s = 0.0;
#pragma unroll
        for (int a = 0; a <= b; ++a) s += w[a] * C[a * P + b];   // C upper triangular
        out[r * P + b] = T(s);
      }
    }
    __syncthreads();
  };
  // sF <- sR sF
  auto chain = [&]() {
    double v = 0.0;
    if (tid < PP)
      for (int k = tid / P; k < P; ++k) v += sR[(tid / P) * P + k] * sF[k * P + tid % P];
    __syncthreads();
    if (tid < PP) sF[tid] = v;
    __syncthreads();
  };

  if (npan > 0) {
    gram(true);
    project();
    update();
    project();
    update();
  }
  gram(false);
  const bool third = small_cholqr(P, sG, sR, sRi, npan > 0 ? s_w0 : nullptr, 1, shift_rel, flags,
                                  s_int);
  if (tid < PP) sF[tid] = sR[tid];
  scale(sRi, sw);
  gram(false);
  small_cholqr(P, sG, sR, sRi, nullptr, 2, 0.0, flags, s_int);
  chain();
  if (third) {
    scale(sRi, sw);
    gram(false);
    small_cholqr(P, sG, sR, sRi, nullptr, 3, 0.0, flags, s_int);
    chain();
  }
  scale(sRi, Vout);
  if (tid < PP) {
    if (H) H[int64_t(npan * P + tid / P) * ldh + col0 + tid % P] = sF[tid];
    else Rhat[tid] = sF[tid];
  }
}

}  // namespace expmv
