// The root matrix and its pivots' row, shared by the root factorization alone (factor.hip) and
// with the root step of a solve (solve.hip).
#pragma once
#include "blockchol.h"
#include "bmpc_internal.h"

namespace bmpc {

// A (NMAX x NMAX, rows of LD, identity padded) = R - sum_g part[g] in group order, lower
// triangle (system sys of the batch); 1024 threads, all partials of an element in flight.
template <int NMAX, int LD>
__device__ __attribute__((always_inline)) inline void root_matrix(double* A, const RootStep& s,
                                                                  int sys) {
  const int n = s.n, groups = s.groups;
  const double* R = s.R + (size_t)sys * n * n;
  const double* part = s.part + (size_t)sys * groups * n * n;
  for (int e = threadIdx.x; e < NMAX * NMAX; e += 1024) {
    const int r = e / NMAX, c = e % NMAX;
    double v = (r == c) ? 1.0 : 0.0;
    if (r < n && c <= r) {
      constexpr int B = 32;
      double acc = 0.0;
      for (int g0 = 0; g0 < groups; g0 += B) {
        double t[B];
#pragma unroll
        for (int u = 0; u < B; ++u)
          t[u] = part[(size_t)min(g0 + u, groups - 1) * n * n + r * n + c];
#pragma unroll
        for (int u = 0; u < B; ++u) acc = (g0 + u < groups) ? acc + t[u] : acc;
      }
      v = R[r * n + c] - acc;
    }
    A[r * LD + c] = v;
  }
}

// L_R of system sys from A (after block_chol), and its first non-positive pivot (fail, valid on
// wave 1) into the factorization's info.  One system (s.info_out): its info is complete
// here, the last step of a factorization; it is published and the accumulator made
// ready for the next one.
template <int NMAX, int LD>
__device__ __attribute__((always_inline)) inline void root_store(const double* A,
                                                                 const RootStep& s, int sys,
                                                                 int fail) {
  const int n = s.n;
  if (threadIdx.x == 64) {
    const unsigned long long row =
        fail >= 0 && fail < n ? sys * s.sys_rows + s.root_row + fail + 1 : ~0ull;
    if (s.info_out) {
      const unsigned long long before = atomicExch(s.info, ~0ull);
      *s.info_out = before < row ? before : row;
      if (s.flags) s.flags[0] = s.flags[1] = 0;
    } else if (row != ~0ull) {
      atomicMin(s.info, row);
    }
  }
  double* LR = s.LR + (size_t)sys * n * n;
  for (int e = threadIdx.x; e < NMAX * NMAX; e += 1024) {
    const int r = e / NMAX, c = e % NMAX;
    if (r < n && c < n) LR[r * n + c] = c <= r ? A[r * LD + c] : 0.0;
  }
}

}  // namespace bmpc
