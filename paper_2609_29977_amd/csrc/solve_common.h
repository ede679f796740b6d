// Vector indexing and scenario sums shared by the solve and residual kernels.
#pragma once

#include "bmpc_internal.h"
#include "multi.h"

namespace bmpc {

// Vectors b, x, r are [B][nrhs][len], len = (S*N+1)*n: system sys, right-hand side q
// of the launch's chunk starts at sys*vsys + q*len (the pointers are offset to the
// chunk), its tails in stage order, its root last.  Chain g of the batch
// (0 <= g < B*S) is scenario g % S of system g / S.  vec_off gives the offset of
// (chain g, q = 0, stage); seg_of the first norm index of g's system in the chunk.
__device__ inline size_t vec_len(const SolveArgs& a) { return ((size_t)a.S * a.N + 1) * a.n; }
__device__ inline size_t vec_off(const SolveArgs& a, int g, int stage) {
  const int sys = g / a.S, sl = g - sys * a.S;
  return (size_t)sys * a.vsys + ((size_t)sl * a.N + stage) * a.n;
}
__device__ inline int seg_of(const SolveArgs& a, int g) { return (g / a.S) * a.seg_sys; }

// x[off + q*len] = d  or  x += rnorm * d with rnorm * d kept in dstore.
__device__ inline void scatter_value(const SolveArgs& a, int q, size_t off, int seg0, double d) {
  const size_t idx = (size_t)q * vec_len(a) + off;
  if (a.accumulate) {
    const double dd = a.rnorm[seg0 + q] * d;
    a.x[idx] += dd;
    a.dstore[idx] = dd;
  } else {
    a.x[idx] = d;
  }
}

// One system's arguments of a ragged launch on the caller's arrays.
__device__ inline SolveArgs relocate_solve(const SolveArgs& t, const Reloc& r) {
  SolveArgs a = t;
  a.b = rel(r.b, t.b);
  a.x = rel(r.x, t.x);
  a.dstore = rel(r.r, t.dstore);
  return a;
}

// Sum of v[s][q][i] over the scenarios s = g, g + G, .. < S for the QB right-hand sides
// q0 .. of nv (n elements each), B scenarios' loads in flight; then over the lanes of the
// wave that hold element i.
template <int NMAX, int QB, int B>
__device__ inline void scenario_sums(const double* __restrict__ v, int S, int n, int nv, int q0,
                                     double (&acc)[QB]) {
  constexpr int G = 1024 / NMAX;
  const int i = threadIdx.x % NMAX, g = threadIdx.x / NMAX;
#pragma unroll
  for (int q = 0; q < QB; ++q) acc[q] = 0.0;
  if (i < n) {
    for (int s0 = g; s0 < S; s0 += G * B) {
      double w[QB][B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const double* p = v + ((size_t)min(s0 + G * u, S - 1) * nv) * n + i;
#pragma unroll
        for (int q = 0; q < QB; ++q) w[q][u] = p[(size_t)min(q0 + q, nv - 1) * n];
      }
#pragma unroll
      for (int q = 0; q < QB; ++q)
#pragma unroll
        for (int u = 0; u < B; ++u) acc[q] += s0 + G * u < S ? w[q][u] : 0.0;
    }
  }
#pragma unroll
  for (int q = 0; q < QB; ++q)
    for (int off = NMAX; off < 64; off <<= 1) acc[q] += __shfl_xor(acc[q], off);
}

}  // namespace bmpc
