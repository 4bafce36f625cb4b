// Inner solves of small operators: one workgroup runs a whole Jacobi-CG or
// Jacobi-BiCGStab solve of one column (the columns of a batched solve share
// nothing but the operator).
//
// The streaming kernels of kernels.hpp cost three (CG) or five (BiCGStab)
// launches per iteration, 3 to 5 us each plus the gap before it, whatever the
// size: at n = 1,024, p = 4 a CG iteration took 16 us for 0.16 MB of operands,
// and takes 1.2 us here (the whole e^{tA}B 31.9 -> 4.3 ms; the 7-point
// upwind operator at n = 1,728, p = 3: 37 -> 3.2 us, 60.2 -> 11.2 ms).
// Here the operator's rows (values and 16-bit column indices) stay in
// registers for the whole solve, the vectors in registers and LDS, and an
// iteration costs three (five) workgroup barriers and one LDS gather per
// nonzero.  The bound is that gather (4 cycles per wavefront of 64 values)
// and the latency of the two reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "kernels.hpp"

namespace expmv {

// largest n: 512 threads with eight rows each (CG: three vectors in LDS), or
// seven (BiCGStab: five vectors in the 160 KB)
constexpr int kSmallRowsCg = 4096, kSmallRowsBcg = 3584;
constexpr int kSmallWidth = 7;     // longest row kept in registers

// iterations and cap flag of each column
struct SmallResult {
  int iters[kMaxP];
  int hit_cap[kMaxP];
};

template <int Ctrl>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), Ctrl, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), Ctrl, 0xf, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
template <int Lane>
__device__ __forceinline__ double lane_value(double v) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), Lane),
                          __builtin_amdgcn_readlane(__double2loint(v), Lane));
}
// Sum over the 64 lanes (all active), the same in every lane: quad swaps,
// half-row and row mirrors, then the four rows of 16.
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0xB1>(v);    // quad_perm 1, 0, 3, 2
  v = dpp_add<0x4E>(v);    // quad_perm 2, 3, 0, 1
  v = dpp_add<0x141>(v);   // row_half_mirror
  v = dpp_add<0x140>(v);   // row_mirror
  return (lane_value<0>(v) + lane_value<16>(v)) + (lane_value<32>(v) + lane_value<48>(v));
}

// Sums of NV values over the NW wavefronts of a workgroup, the same bits in
// every thread (fixed order).  One barrier; red (NV x NW doubles) may be
// written again only after a later barrier.
template <int NV, int NW>
__device__ __forceinline__ void block_sums(double (&v)[NV], double* red) {
  const int wave = threadIdx.x / 64;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
  if (threadIdx.x % 64 == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) red[k * NW + wave] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double s[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) s[w] = red[k * NW + w];
#pragma unroll
    for (int h = NW / 2; h >= 1; h /= 2) {
#pragma unroll
      for (int w = 0; w < h; ++w) s[w] += s[w + h];
    }
    v[k] = s[0];
  }
}

// The rows tid + r NT (r < R) of an operator whose rows have at most W
// nonzeros.  Missing entries have value 0 and the row's own index, so that a
// row reads nothing that it does not depend on.
template <int W, int R, int NT>
struct SmallRows {
  double v[R][W];
  unsigned j[R][(W + 1) / 2];

  __device__ __forceinline__ void load(int n, const int32_t* __restrict__ rowptr,
                                       const int32_t* __restrict__ colind,
                                       const double* __restrict__ val) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = threadIdx.x + r * NT;
      const int e0 = row < n ? rowptr[row] : 0, e1 = row < n ? rowptr[row + 1] : 0;
#pragma unroll
      for (int u = 0; u < W; u += 2) {
        const bool a = e0 + u < e1, b = u + 1 < W && e0 + u + 1 < e1;
        const unsigned ja = a ? unsigned(colind[e0 + u]) : unsigned(row);
        const unsigned jb = b ? unsigned(colind[e0 + u + 1]) : unsigned(row);
        j[r][u / 2] = ja | (jb << 16);
        v[r][u] = a ? val[e0 + u] : 0.0;
        if (u + 1 < W) v[r][u + 1] = b ? val[e0 + u + 1] : 0.0;
      }
    }
  }
  // row r times x (LDS, NT R entries), summed in the row's order in FP64
  template <typename T>
  __device__ __forceinline__ double dot(int r, const T* x) const {
    T g[W];
#pragma unroll
    for (int u = 0; u < W; u += 2) {
      g[u] = x[j[r][u / 2] & 0xffffu];
      if (u + 1 < W) g[u + 1] = x[j[r][u / 2] >> 16];
    }
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < W; ++u) acc += v[r][u] * double(g[u]);
    return acc;
  }
};

// A vector's own entries (rows tid + r NT) of a thread: registers, or LDS
// where registers are short (R > 4: the operator's rows take 150 and more).
// In LDS at n = 1,024 they cost as many LDS cycles as the gathers.
template <typename T, int R, int NT, bool Lds>
struct OwnRows {
  T v[R];
  __device__ __forceinline__ T get(int r) const { return v[r]; }
  __device__ __forceinline__ void set(int r, T x) { v[r] = x; }
};
template <typename T, int R, int NT>
struct OwnRows<T, R, NT, true> {
  T* v;
  __device__ __forceinline__ T get(int r) const { return v[threadIdx.x + r * NT]; }
  __device__ __forceinline__ void set(int r, T x) { v[threadIdx.x + r * NT] = x; }
};
template <typename T, int R, int NT, bool Lds>
__device__ __forceinline__ void own_place(OwnRows<T, R, NT, Lds>& o, T*& lds) {
  if constexpr (Lds) {
    o.v = lds;
    lds += NT * R;
  }
}

// x = K^{-1} (sign * src), column blockIdx.x, by Jacobi-CG: the recurrences,
// the stopping test (|r| <= tol |b| on the recurrence residual) and the cap of
// k_cg_c / k_cg_a / k_cg_b.
template <typename T, int W, int R, int NT>
__global__ void __launch_bounds__(NT)
k_small_cg(int n, int p, double sign, const int32_t* __restrict__ rowptr,
           const int32_t* __restrict__ colind, const double* __restrict__ val,
           const T* __restrict__ dinv, const T* src, T* x, double tol2, int maxit,
           SmallResult* __restrict__ res) {
  constexpr int NW = NT / 64;
  extern __shared__ char small_lds[];
  double* red = reinterpret_cast<double*>(small_lds);   // 2 NW, NW
  T* sp = reinterpret_cast<T*>(red + 3 * NW);           // the direction
  T* more = sp + NT * R;
  OwnRows<T, R, NT, (R > 4)> dv, xv;                    // D^{-1}, the iterate
  own_place(dv, more);
  own_place(xv, more);
  const int c = blockIdx.x, tid = threadIdx.x;
  SmallRows<W, R, NT> A;
  A.load(n, rowptr, colind, val);
  T rv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = tid + r * NT;
    rv[r] = row < n ? T(sign * double(src[int64_t(row) * p + c])) : T(0);
    xv.set(r, T(0));
    dv.set(r, row < n ? dinv[row] : T(0));
    sp[row] = T(0);
  }
  double bn = 0.0, rho_prev = 0.0;
  int it = 0, hit = 0;
  for (int k = 0;; ++k) {
    double s[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double rd = double(rv[r]);
      s[0] += rd * double(dv.get(r)) * rd;
      s[1] += rd * rd;
    }
    block_sums<2, NW>(s, red);
    const double rho = s[0], rn = s[1];
    if (k == 0) bn = rn;
    if (!(bn > 0.0) || rn <= tol2 * bn) break;
    if (it >= maxit) {
      hit = 1;
      break;
    }
    ++it;
    const T beta = T(k > 0 && rho_prev != 0.0 ? rho / rho_prev : 0.0);
    rho_prev = rho;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = tid + r * NT;
      sp[row] = dv.get(r) * rv[r] + beta * sp[row];
    }
    __syncthreads();
    T q[R];
    double sig[1] = {0.0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      q[r] = T(A.dot(r, sp));
      sig[0] += double(sp[tid + r * NT]) * double(q[r]);
    }
    block_sums<1, NW>(sig, red + 2 * NW);
    const T alpha = T(sig[0] != 0.0 ? rho / sig[0] : 0.0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      xv.set(r, xv.get(r) + alpha * sp[tid + r * NT]);
      rv[r] = rv[r] - alpha * q[r];
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = tid + r * NT;
    if (row < n) x[int64_t(row) * p + c] = xv.get(r);
  }
  if (tid == 0) {
    res->iters[c] = it;
    res->hit_cap[c] = hit;
  }
}

// The same by right Jacobi-preconditioned BiCGStab (k_bcg_u1 / s / u2 / s / u3).
template <typename T, int W, int R, int NT>
__global__ void __launch_bounds__(NT)
k_small_bcg(int n, int p, double sign, const int32_t* __restrict__ rowptr,
            const int32_t* __restrict__ colind, const double* __restrict__ val,
            const T* __restrict__ dinv, const T* src, T* x, double tol2, int maxit,
            SmallResult* __restrict__ res) {
  constexpr int NW = NT / 64;
  extern __shared__ char small_lds[];
  double* red = reinterpret_cast<double*>(small_lds);   // 2 NW, NW, 2 NW
  T* sy = reinterpret_cast<T*>(red + 5 * NW);           // D^{-1} p, then D^{-1} s
  T* more = sy + NT * R;
  OwnRows<T, R, NT, (R > 4)> dv, hv, xv, pv;            // D^{-1}, r^ = b, iterate, direction
  own_place(dv, more);
  own_place(hv, more);
  own_place(xv, more);
  own_place(pv, more);
  const int c = blockIdx.x, tid = threadIdx.x;
  SmallRows<W, R, NT> A;
  A.load(n, rowptr, colind, val);
  T rv[R], vv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = tid + r * NT;
    rv[r] = row < n ? T(sign * double(src[int64_t(row) * p + c])) : T(0);
    vv[r] = T(0);
    dv.set(r, row < n ? dinv[row] : T(0));
    hv.set(r, rv[r]);
    xv.set(r, T(0));
    pv.set(r, T(0));
  }
  double bn = 0.0, rho_prev = 1.0, a_prev = 1.0, om_prev = 1.0;
  int it = 0, hit = 0;
  for (int i = 0;; ++i) {
    double s[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double rd = double(rv[r]);
      s[0] += double(hv.get(r)) * rd;
      s[1] += rd * rd;
    }
    block_sums<2, NW>(s, red);
    const double rho = s[0], rn = s[1];
    if (i == 0) bn = rn;
    if (!(bn > 0.0) || rn <= tol2 * bn) break;
    if (it >= maxit || rho == 0.0 || om_prev == 0.0 || rho_prev == 0.0) {
      hit = 1;
      break;
    }
    ++it;
    const T beta = T((rho / rho_prev) * (a_prev / om_prev)), om1 = T(om_prev);
    rho_prev = rho;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = tid + r * NT;
      const T pn = i == 0 ? rv[r] : rv[r] + beta * (pv.get(r) - om1 * vv[r]);
      pv.set(r, pn);
      sy[row] = dv.get(r) * pn;
    }
    __syncthreads();
    double d[1] = {0.0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      vv[r] = T(A.dot(r, sy));
      d[0] += double(hv.get(r)) * double(vv[r]);
    }
    block_sums<1, NW>(d, red + 2 * NW);
    const double alpha = d[0] != 0.0 ? rho / d[0] : 0.0;
    const T a = T(alpha);
    // s = r - alpha v in place of r; x += alpha y before y makes room
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = tid + r * NT;
      rv[r] = rv[r] - a * vv[r];
      xv.set(r, xv.get(r) + a * sy[row]);
      sy[row] = dv.get(r) * rv[r];
    }
    __syncthreads();
    T t[R];
    double e[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      t[r] = T(A.dot(r, sy));
      e[0] += double(rv[r]) * double(t[r]);
      e[1] += double(t[r]) * double(t[r]);
    }
    block_sums<2, NW>(e, red + 3 * NW);
    const double omega = e[1] != 0.0 ? e[0] / e[1] : 0.0;
    const T om = T(omega);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = tid + r * NT;
      xv.set(r, xv.get(r) + om * sy[row]);
      rv[r] = rv[r] - om * t[r];
    }
    a_prev = alpha;
    om_prev = omega;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = tid + r * NT;
    if (row < n) x[int64_t(row) * p + c] = xv.get(r);
  }
  if (tid == 0) {
    res->iters[c] = it;
    res->hit_cap[c] = hit;
  }
}

}  // namespace expmv
