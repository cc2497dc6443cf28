// Factorization and triangular solves of the Newton matrices with N > 64
// (kernels in newton_blocked.hip, called by newton.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pyjac {

constexpr int ST_UNSET = -100;   // internal per-state status before convergence
constexpr int ST_SING32 = -4;    // zero pivot in the FP32 factor: re-solved in FP64

// Largest N of the blocked path.
constexpr int kBlockedMax = 608;

// LU of the states (or of the *count states of `list`): A holds one
// column-major N x N matrix per slot and is overwritten by the factor with its
// rows in pivot order; piv[k] is the matrix row that became row k.  A zero
// pivot sets the state's status to sing_code; states with status -3 are left
// alone.
template <typename T>
hipError_t launch_lu(int N, int64_t n, T* A, int* piv, const int* list, const int* count, int* status, int sing_code,
                     hipStream_t st);

// Solves with that factor.  direct: x = A^-1 b, b from rhs [N][ld], x to
// xout [N][ld], status 0 or -1.
template <typename T>
hipError_t launch_solve_direct(int N, int64_t n, int64_t ld, const T* A, const int* piv, const double* rhs,
                               double* xout, const int* list, const int* count, int* status, hipStream_t st);
// refine: sweep 0 x = A^-1 b into xs [N][n] (FP64); later sweeps d = A^-1 r
// with r from rbuf [N][n] and x += d; a state that converges by the tests of
// the kernel gets status = sweep and its x in xout [N][ld].
hipError_t launch_solve_refine(int N, int64_t n, int64_t ld, const float* A, const int* piv, const double* rhs,
                               const double* rbuf, double* xs, double* xout, int* status, int sweep, double rtol,
                               double* dprev, hipStream_t st);

}  // namespace pyjac
