// Host eigensolvers for the small projected matrix of the restart step.
#pragma once

#include <atomic>
#include <vector>

namespace expmv {

// Lets the thread that started a computation end it early: check(), called at
// every step of the loops below, throws Stopped once the flag is set.
struct Stopped {};
struct StopToken {
  const std::atomic<bool>* flag = nullptr;   // NULL: runs to its end
  void check() const {
    if (flag && flag->load(std::memory_order_relaxed)) throw Stopped{};
  }
};

// A (n x n, row-major) symmetric part -> eigenvalues w (n) and orthonormal
// eigenvectors in the columns of Q (n x n row-major): A = Q diag(w) Q^T.
// Returns false if the QR iteration did not deflate every off-diagonal
// entry within 60 n sweeps, or if the input or the result is not finite (w
// and Q then hold the unconverged iterate).
bool sym_eig(int n, const double* A, double* w, double* Q, StopToken stop = {});

// General real A (n x n row-major) -> eigenvalues wr + i wi and eigenvectors
// (column i of Vr + i Vi, unit 2-norm).  Complex eigenvalues come as exact
// conjugate pairs.  Returns false if the QR iteration did not converge or
// an eigenvalue is not finite.
bool general_eig(int n, const double* A, double* wr, double* wi, double* Vr, double* Vi);

// Upper Hessenberg form H = Q^T A Q of a general A (n x n row-major), handed
// from the first half of general_eig to the second.  Q = P_0 P_1 ... P_{n-3},
// P_k = I - beta[k] v v^T with v in row k of refl, columns k + 1 .. k + len[k].
struct HessForm {
  int n = 0;
  std::vector<double> H, refl, beta;
  std::vector<int> len;
};

// The two halves of general_eig: eigenvalues (exact conjugate pairs), then
// eigenvectors only for the indices with want[i] != 0 (want NULL: all; the
// other columns are zero).  With hf, general_eigvals leaves the Hessenberg
// form there and general_eigvecs starts from it; without, general_eigvecs
// reduces A again.
bool general_eigvals(int n, const double* A, double* wr, double* wi, HessForm* hf = nullptr,
                     StopToken stop = {});
void general_eigvecs(int n, const double* A, const double* wr, const double* wi,
                     const char* want, double* Vr, double* Vi, const HessForm* hf = nullptr,
                     StopToken stop = {});

}  // namespace expmv
