// Device code of the solve steps (Algorithm 2) as matrix products (gfx950): a position of
// either sweep, the x_1 steps.
//
// The right-hand sides of a launch (at most 16) are the columns of 16 x 16 MFMA tiles, so a
// block is read once for all of them and every product costs the same for one or sixteen.  A
// wave holds all row tiles of a position (NT = ceil(n / 16)).  Blocks are read straight into
// the A operand layout (lane 16 g + i: row i of a tile, the contraction indices chosen so
// that a lane reads 16 consecutive bytes where it reads rows), the neighbours' vectors into
// the B layout (the scratch y holds a position's right-hand sides with their index fastest),
// and L_jj^{-1} is applied to the accumulators as they lie: the contraction indices of its
// product follow the accumulator layout, so nothing goes through LDS but the partial sums
// of the waves that share a position's pulls.  Every load of a round is issued before the
// first product.  Memory-bound while the levels are wide, latency-bound at the top.
//
#pragma once
#include "blockops.h"
#include "bmpc_internal.h"
#include "regblock.h"
#include "solve_common.h"

namespace bmpc {

// Which row of a block an MFMA row stands for.  An accumulator holds four rows of a tile per
// lane; they are made neighbours in memory (tile t, lane group g, register v: row
// 16 t + 4 g + v), so that vectors and the rows of L^{-1} move in runs of four.
template <typename T>
__device__ inline int a_row(int t, int i) {  // row i of tile t as the A operand
  return 16 * t + (sizeof(T) == 8 ? 4 * (i & 3) + (i >> 2) : i);
}
// (register v, group g) of tile t as an accumulator, or as the contraction index of step v
// in slab t of a product that takes that accumulator as its B operand.
__device__ inline int acc_row(int t, int v, int g) { return 16 * t + 4 * g + v; }
// f(row, t, v) over the rows of a lane (VEC: n is a multiple of four, so a run is in or out)
template <int NT, bool VEC, typename F>
__device__ __attribute__((always_inline)) inline void each_row(bool in, int n, int g, F&& f) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int base = acc_row(t, 0, g);
    if constexpr (VEC) {
      if (in && base < n) {
#pragma unroll
        for (int v = 0; v < 4; ++v) f(base + v, t, v);
      }
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (in && base + v < n) f(base + v, t, v);
    }
  }
}
// Contraction index of step s in a 16-wide slab of a pull: the steps of a lane are neighbours
// along a row.
template <typename T>
__device__ inline int pull_k(int s, int g) {
  return sizeof(T) == 8 ? 8 * (s >> 1) + 2 * g + (s & 1) : 4 * g + s;
}

template <typename T>
__device__ inline T buf_load(__amdgpu_buffer_rsrc_t rs, unsigned off) {
  if constexpr (sizeof(T) == 8)
    return buf_load_f64(rs, off);
  else
    return buf_load_f32(rs, off);
}
// K neighbouring values from byte offset off (16 or 32 bytes in all).  The whole offset goes
// through the range check: an offset on the side is taken off the range first, which a block
// of one entry (8 bytes) is shorter than.
template <typename T, int K>
__device__ inline void buf_load_run(__amdgpu_buffer_rsrc_t rs, unsigned off, T (&out)[K]) {
  static_assert(K * sizeof(T) % 16 == 0, "whole 16-byte pieces");
#pragma unroll
  for (int h = 0; h < (int)(K * sizeof(T)) / 16; ++h) {
    const auto w = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16u * h, 0, 0);
    __builtin_memcpy(&out[h * (16 / (int)sizeof(T))], &w, 16);
  }
}

// An n x n block (TRANS: transposed) as the A operand of NT row tiles by NT slabs of 16
// columns.  VEC: n is a multiple of four, so a run of neighbours is in the block or outside as
// a whole.
template <typename T, int NT, bool TRANS, bool VEC>
struct MmBlock {
  T v[NT][NT][4];
  __device__ void load(const T* __restrict__ M, int n) {
    const int l = threadIdx.x & 63, g = l >> 4, i = l & 15;
    const auto rs = block_rsrc(M, (unsigned)(n * n) * (unsigned)sizeof(T));
    constexpr int V = 16 / (int)sizeof(T);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int R = a_row<T>(t, i);
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        if constexpr (!TRANS && VEC) {
#pragma unroll
          for (int s = 0; s < 4; s += V) {
            const int k = 16 * c + pull_k<T>(s, g);
            T w[V];
            buf_load_run(
                rs, R < n && k < n ? (unsigned)(R * n + k) * (unsigned)sizeof(T) : kOutOfRange, w);
#pragma unroll
            for (int e = 0; e < V; ++e) v[t][c][s + e] = w[e];
          }
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int k = 16 * c + pull_k<T>(s, g);
            const unsigned o = (unsigned)(TRANS ? k * n + R : R * n + k) * (unsigned)sizeof(T);
            v[t][c][s] = buf_load<T>(rs, R < n && k < n ? o : kOutOfRange);
          }
        }
      }
    }
  }
};

// The vectors of a position (y: [n][nrhs]) as the B operand; lanes past nrhs read zero.
template <typename T, int NT>
struct MmVec {
  T v[NT][4];
  __device__ void load(const T* __restrict__ y, int n, int nrhs) {
    const int l = threadIdx.x & 63, g = l >> 4, i = l & 15;
    const auto rs = block_rsrc(y, (unsigned)(n * nrhs) * (unsigned)sizeof(T));
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const unsigned o = (unsigned)((16 * c + pull_k<T>(s, g)) * nrhs + i) * (unsigned)sizeof(T);
        v[c][s] = buf_load<T>(rs, i < nrhs ? o : kOutOfRange);  // rows past n: past the range
      }
  }
};

template <typename T, int NT, bool TRANS, bool VEC>
__device__ inline void mm_add(typename Mfma<T>::acc_t (&acc)[NT],
                              const MmBlock<T, NT, TRANS, VEC>& a, const MmVec<T, NT>& b, int n) {
#pragma unroll
  for (int c = 0; c < NT; ++c)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (sizeof(T) == 8 && 16 * c + 8 * (s >> 1) >= n) continue;  // uniform: zero columns
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = Mfma<T>::mma(a.v[t][c][s], b.v[c][s], acc[t]);
    }
}

// L^{-1} of a diagonal block, packed by rows, as the A operand of L^{-1} r or L^{-T} r with r
// in the accumulator layout.
template <typename T, int NT, bool TRANS>
struct MmLinv {
  static constexpr bool kept(int t, int c) { return TRANS ? c >= t : c <= t; }
  T v[NT][NT][4];
  __device__ void load(const T* __restrict__ Li, int n) {
    const int l = threadIdx.x & 63, g = l >> 4, i = l & 15;
    const auto rs = block_rsrc(Li, (unsigned)(n * (n + 1) / 2) * (unsigned)sizeof(T));
    auto at = [&](int row, int col) {
      return row < n && col <= row ? (unsigned)(row * (row + 1) / 2 + col) * (unsigned)sizeof(T)
                                   : kOutOfRange;
    };
#pragma unroll
    for (int c = 0; c < NT; ++c) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (!kept(t, c)) continue;
        const int o = a_row<T>(t, i);
        if constexpr (TRANS) {
#pragma unroll
          for (int s = 0; s < 4; ++s) v[t][c][s] = buf_load<T>(rs, at(acc_row(c, s, g), o));
        } else {
          const int k = acc_row(c, 0, g);
          T w[4];
          buf_load_run(rs, at(o, k), w);  // past the diagonal: the next row's
#pragma unroll
          for (int s = 0; s < 4; ++s) v[t][c][s] = k + s <= o ? w[s] : T(0);
        }
      }
    }
  }
  // FP64 takes a row's sum in one chain of matrix instructions per slab, two where there is
  // only one slab or registers are short (a single chain over 64 columns: the kernel of the last
  // backward levels stays under 512), and adds the chains at the end, as the other solve kernels
  // add their lanes' partial sums.  One chain over the whole row rounds more often on its way:
  // root mean square error against extended precision, 2 chains of 8 at n = 48 with one
  // right-hand side 1.05e-16 -> 9.7e-17, at n = 64 with twelve 8.6e-17 -> 7.9e-17, 2 chains of
  // 16 at n = 32 with twelve 6.7e-17 -> 6.3e-17, in the same time (within 1 %).
  static constexpr int kChains = sizeof(T) == 4 ? 1 : NT == 1 || (NT == 4 && TRANS) ? 2 : NT;
  static constexpr int chain(int c, int s) {
    return kChains == 1 ? 0 : NT == 1 ? s >> 1 : kChains < NT ? c >> 1 : c;
  }
  template <typename Vec>
  __device__ void apply(typename Mfma<T>::acc_t (&out)[NT], const Vec& r) const {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      typename Mfma<T>::acc_t sum[kChains];
#pragma unroll
      for (int k = 0; k < kChains; ++k) sum[k] = typename Mfma<T>::acc_t{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int c = 0; c < NT; ++c) {
          auto& to = sum[chain(c, s)];
          if (kept(t, c)) to = Mfma<T>::mma(v[t][c][s], static_cast<T>(r[c][s]), to);
        }
      out[t] = sum[0];
#pragma unroll
      for (int k = 1; k < kChains; ++k) out[t] += sum[k];
    }
  }
};

// A position of a forward level (MM_FWD), of a backward level (MM_BWD), or the x_1 forward
// step (MM_X): rhs minus the pulls' products, then L_jj^{-1} (L_jj^{-T}).  Pulls as in
// solve.hip: forward, the G_r of the left neighbours j - 2^t and the G_l of the right
// neighbours j + 2^t of the lower levels; backward, G_l^T with x of the left neighbour and
// G_r^T with x of the right one (or of X); x_1, the G_r of the last position of every level
// with an odd chain length.  P pulls are in flight per wave (mm_pulls_per_wave; both of a
// backward position up to n = 32).  W waves share the pulls, this
// one being wv; part (LDS) takes the partial sums of all but the first.  TOGETHER: the
// workgroup holds several positions, so that every wave goes through the barrier, the ones
// without a position (not active) too.  LEAN: fewer loads in flight (one pull, or L_jj^{-1} after
// the pulls), for a kernel that would spill otherwise.
enum MmKind { MM_FWD, MM_BWD, MM_X };

template <typename T, int NT, int KIND, bool VEC, bool TOGETHER, bool LEAN = false>
__device__ __attribute__((always_inline)) inline void mm_position_body(
    const SolveArgs& a, int level, int s, int j, int W, int wv,
    typename Mfma<T>::acc_t* part, bool active) {
  typedef typename Mfma<T>::acc_t acc_t;
  constexpr bool BWD = KIND == MM_BWD;
  constexpr int P = BWD && NT == 2 && !LEAN ? 2 : mm_pulls_per_wave(16 * NT, sizeof(T) == 8);
  constexpr bool LATE = LEAN && NT > 2;
  if (TOGETHER && !active) {
    __syncthreads();
    return;
  }
  const int n = a.n, N = a.N, nrhs = a.nrhs, m = a.m;
  const size_t nn = (size_t)n * n;
  const int l = threadIdx.x & 63, g = l >> 4, i = l & 15;
  const size_t gstride = g_chain_blocks(N);
  const T* Gl = reinterpret_cast<const T*>(a.Gl) + (size_t)s * gstride * nn;
  const T* Gr = reinterpret_cast<const T*>(a.Gr) + (size_t)s * gstride * nn;
  const T* Li = reinterpret_cast<const T*>(a.Linv) + ((size_t)s * N + (j - 1)) * nn;
  T* y = reinterpret_cast<T*>(a.y) + (size_t)s * N * nrhs * n;
  T* yj = y + (size_t)(j - 1) * nrhs * n;
  const int half = BWD ? 1 << (level - 1) : 0;
  const int npull = KIND == MM_FWD ? 2 * (level - 1) : BWD ? 2 : chain_levels(m);
  const size_t off = vec_off(a, s, N - j);
  const int seg0 = seg_of(a, s);
  const size_t len = vec_len(a);

  auto pull = [&](int p, const T*& blk, const T*& vec) -> bool {
    int c;
    if constexpr (KIND == MM_FWD) {
      const int t = p >> 1;
      c = (p & 1) ? j + (1 << t) : j - (1 << t);
      if (c > m) return false;
      blk = ((p & 1) ? Gl : Gr) + (size_t)(c - 1) * nn;
    } else if constexpr (BWD) {
      if (p == 0) {
        if (j - half < 1) return false;
        blk = Gl + (size_t)(j - 1) * nn;
        c = j - half;
      } else {
        blk = Gr + (size_t)(j - 1) * nn;
        c = j + half <= m ? j + half : N;
      }
    } else {
      if (((m >> p) & 1) == 0) return false;
      c = (m >> p) << p;
      blk = Gr + (size_t)(c - 1) * nn;
    }
    vec = y + (size_t)(c - 1) * nrhs * n;
    return true;
  };

  // wave 0's loads besides its pulls: L_jj^{-1}, the right-hand side in the accumulator
  // layout (row_of(t, v), this lane's right-hand side i), the x being updated
  MmLinv<T, NT, BWD> lin;
  double rb[NT][4] = {}, xo[BWD ? NT : 1][4] = {};
  const double rn = a.rnorm && i < nrhs ? a.rnorm[seg0 + i] : 1.0;
  const size_t ix = (size_t)i * len + off;
  if (wv == 0) {
    if constexpr (!LATE) lin.load(Li, n);
    each_row<NT, VEC>(i < nrhs, n, g, [&](int row, int t, int v) {
      if constexpr (BWD)
        rb[t][v] = static_cast<double>(yj[row * nrhs + i]);
      else
        rb[t][v] = a.b[ix + row];
    });
    if constexpr (BWD)
      if (a.accumulate)
        each_row<NT, VEC>(i < nrhs, n, g,
                           [&](int row, int t, int v) { xo[t][v] = a.x[ix + row]; });
  }
  acc_t acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = acc_t{0, 0, 0, 0};
  for (int base = wv * P; base < npull; base += W * P) {
    MmBlock<T, NT, BWD, VEC> blk[P];
    MmVec<T, NT> vec[P];
    bool has[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const T* bp = nullptr;
      const T* vp = nullptr;
      has[u] = base + u < npull && pull(base + u, bp, vp);
      if (has[u]) {
        blk[u].load(bp, n);
        vec[u].load(vp, n, nrhs);
      }
    }
#pragma unroll
    for (int u = 0; u < P; ++u)
      if (has[u]) mm_add<T, NT, BWD, VEC>(acc, blk[u], vec[u], n);
  }
  if (TOGETHER || W > 1) {
    if (wv > 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t) part[((wv - 1) * NT + t) * 64 + l] = acc[t];
    }
    __syncthreads();
    if (wv != 0) return;
    for (int w = 1; w < W; ++w)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] += part[((w - 1) * NT + t) * 64 + l];
  }
  if constexpr (LATE) lin.load(Li, n);
  acc_t r[NT], out[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double bv = rb[t][v];
      if (!BWD && a.rnorm) bv = rn > 0.0 ? bv / rn : 0.0;
      r[t][v] = static_cast<T>(bv) - acc[t][v];
    }
  lin.apply(out, r);
  each_row<NT, VEC>(i < nrhs, n, g, [&](int row, int t, int v) {
    yj[row * nrhs + i] = out[t][v];
    if constexpr (BWD)
      if (!a.accumulate) a.x[ix + row] = static_cast<double>(out[t][v]);
  });
  if constexpr (BWD)
    if (a.accumulate)
      each_row<NT, VEC>(i < nrhs, n, g, [&](int row, int t, int v) {
        const double dd = rn * static_cast<double>(out[t][v]);
        a.x[ix + row] = xo[t][v] + dd;
        a.dstore[ix + row] = dd;
      });
  if constexpr (KIND == MM_X) {
    // w_s = F_s y_X in FP64 (the root reduction input of Algorithm 2), with y_X taken from
    // the accumulators as it lies
    const T* F = reinterpret_cast<const T*>(a.F) + (size_t)s * nn;
    const auto rf = block_rsrc(F, (unsigned)nn * (unsigned)sizeof(T));
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int R = a_row<double>(t, i);
      T f[NT][4];
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        const int k = acc_row(c, 0, g);
        const unsigned o = (unsigned)(R * n + k) * (unsigned)sizeof(T);
        if constexpr (VEC) {
          buf_load_run(rf, R < n && k < n ? o : kOutOfRange, f[c]);
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            f[c][v] = buf_load<T>(
                rf, R < n && k + v < n ? o + (unsigned)(v * sizeof(T)) : kOutOfRange);
        }
      }
      typename Mfma<double>::acc_t w = {0, 0, 0, 0};
#pragma unroll
      for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          w = Mfma<double>::mma(static_cast<double>(f[c][v]), static_cast<double>(out[c][v]), w);
      const int row = acc_row(t, 0, g);
      double* const ws = a.w + ((size_t)s * nrhs + i) * n;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (i < nrhs && row + v < n) ws[row + v] = w[v];
    }
  }
}

// Root propagation and the x_1 backward step: dy_X -= F^T x_0 (FP64), x_X = L_X^{-T} dy_X.
template <typename T, int NT, bool VEC>
__device__ __attribute__((always_inline)) inline void mm_x_bwd_body(const SolveArgs& a, int s) {
  typedef typename Mfma<T>::acc_t acc_t;
  typedef typename Mfma<double>::acc_t dacc_t;
  const int n = a.n, N = a.N, nrhs = a.nrhs;
  const size_t nn = (size_t)n * n;
  const int l = threadIdx.x & 63, g = l >> 4, i = l & 15;
  const T* F = reinterpret_cast<const T*>(a.F) + (size_t)s * nn;
  T* yx = reinterpret_cast<T*>(a.y) + ((size_t)s * N + (N - 1)) * nrhs * n;
  const double* x0 = a.x0 + ((size_t)(s / a.S) * nrhs + i) * n;
  const auto rf = block_rsrc(F, (unsigned)nn * (unsigned)sizeof(T));
  T f[NT][NT][4];  // F^T: tile, slab, step
#pragma unroll
  for (int c = 0; c < NT; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = acc_row(c, v, g);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int R = a_row<double>(t, i);
        f[t][c][v] = buf_load<T>(
            rf, R < n && k < n ? (unsigned)(k * n + R) * (unsigned)sizeof(T) : kOutOfRange);
      }
    }
  double rb[NT][4] = {}, xv[NT][4] = {};
  each_row<NT, VEC>(i < nrhs, n, g, [&](int row, int t, int v) { xv[t][v] = x0[row]; });
  each_row<NT, VEC>(i < nrhs, n, g, [&](int row, int t, int v) {
    rb[t][v] = static_cast<double>(yx[row * nrhs + i]);
  });
  MmLinv<T, NT, true> lin;
  lin.load(reinterpret_cast<const T*>(a.Linv) + ((size_t)s * N + (N - 1)) * nn, n);
  dacc_t r[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    dacc_t acc = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        acc = Mfma<double>::mma(static_cast<double>(f[t][c][v]), xv[c][v], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) r[t][v] = rb[t][v] - acc[v];
  }
  acc_t out[NT];
  lin.apply(out, r);
  const size_t off = vec_off(a, s, 0);
  const int seg0 = seg_of(a, s);
  each_row<NT, VEC>(i < nrhs, n, g, [&](int row, int t, int v) {
    yx[row * nrhs + i] = out[t][v];
    scatter_value(a, i, off + row, seg0, static_cast<double>(out[t][v]));
  });
}

}  // namespace bmpc
