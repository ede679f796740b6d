// Cholesky of one block by 16 x 16 tiles, the waves of a workgroup together (gfx950).
#pragma once
#include "blockops.h"

namespace bmpc {

// In place: A (NT x NT tiles of 16 in LDS, rows of LD entries, lower tiles read, identity padded)
// := L^{-1} (INV) or L, with L L^T = A.  W waves call it, at least NT; the tiles above the
// diagonal are left as they were.  scratch: 16 x 17 entries (INV: not used).  Returns the row
// of the first non-positive pivot, or -1 (INV: on wave 0, else on wave 1).
//
// The chain is the NT diagonal tiles, one wave each (their 16 columns take 1.9 us in FP64);
// everything else is one or a few MFMA tile products per wave between them.  While a
// diagonal tile k is factored and inverted, the other waves form W_kj = sum_m L_km X_mj, the
// inverse's row k up to a factor; after it X_kj = -X_kk W_kj, taken from W's accumulator
// as it lies, and column k of L below the diagonal, L_ik = A_ik X_kk^T; then the remaining
// tiles lose L_ik L_jk^T.  (L itself: the diagonal tile is factored by one wave and, in
// scratch, inverted by another.)
template <typename T, int NT, int LD, int W, bool INV>
__device__ __attribute__((always_inline)) inline int block_chol(T* A, T* scratch) {
  static_assert(W >= NT, "a wave per tile of a row");
  typedef typename Mfma<T>::acc_t acc_t;
  const int wv = wave_id(), l = threadIdx.x & 63, g = l >> 4, i = l & 15;
  auto tile = [&](int r, int c) { return A + 16 * r * LD + 16 * c; };
  int fail = -1;
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    T* const Akk = tile(k, k);
    T* X = Akk;  // the inverse of the diagonal tile, rows of XLD
    constexpr int XLD = INV ? LD : 17;
    acc_t w = {0, 0, 0, 0};
    if constexpr (!INV) {
      X = scratch;
      if (wv == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) X[(4 * g + v) * 17 + i] = Akk[(4 * g + v) * LD + i];
      }
      __syncthreads();
      if (wv == 1) {
        const int f = wave_potrf<T, 16, LD>(Akk);
        if (fail < 0 && f >= 0) fail = 16 * k + f;
      }
      if (wv == 0 && k + 1 < NT) (void)wave_potrf_inv_leaf<T, 16, RowMajor<17>>(X);
    } else {
      if (wv == 0) {
        const int f = wave_potrf_inv_leaf<T, 16, RowMajor<LD>>(Akk);
        if (fail < 0 && f >= 0) fail = 16 * k + f;
      } else if (wv <= k) {
        const int j = wv - 1;
        for (int m = j; m < k; ++m) {
          const T* const L = tile(k, m);
          const T* const Xm = tile(m, j);
#pragma unroll
          for (int s = 0; s < 4; ++s)
            w = Mfma<T>::mma(L[i * LD + 4 * g + s], Xm[(4 * g + s) * LD + i], w);
        }
      }
    }
    __syncthreads();
    if (INV && wv >= 1 && wv <= k) {  // row k of the inverse
      acc_t x = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 4; ++s) x = Mfma<T>::mma(-X[i * XLD + Mfma<T>::row(l, s)], w[s], x);
      T* const out = tile(k, wv - 1);
#pragma unroll
      for (int v = 0; v < 4; ++v) out[Mfma<T>::row(l, v) * LD + i] = x[v];
    }
    if (wv > k && wv < NT) {  // column k of L
      T* const Aik = tile(wv, k);
      acc_t t = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        t = Mfma<T>::mma(Aik[i * LD + 4 * g + s], X[i * XLD + 4 * g + s], t);
#pragma unroll
      for (int v = 0; v < 4; ++v) Aik[Mfma<T>::row(l, v) * LD + i] = t[v];
    }
    if (k + 1 < NT) {
      __syncthreads();
      int task = 0;
#pragma unroll
      for (int r = k + 1; r < NT; ++r)
#pragma unroll
        for (int c = k + 1; c <= r; ++c, ++task) {
          if (wv != task % W) continue;
          T* const Arc = tile(r, c);
          const T* const Lr = tile(r, k);
          const T* const Lc = tile(c, k);
          acc_t t;
#pragma unroll
          for (int v = 0; v < 4; ++v) t[v] = Arc[Mfma<T>::row(l, v) * LD + i];
#pragma unroll
          for (int s = 0; s < 4; ++s)
            t = Mfma<T>::mma(-Lr[i * LD + 4 * g + s], Lc[i * LD + 4 * g + s], t);
#pragma unroll
          for (int v = 0; v < 4; ++v) Arc[Mfma<T>::row(l, v) * LD + i] = t[v];
        }
    }
    __syncthreads();
  }
  return fail;
}

}  // namespace bmpc
