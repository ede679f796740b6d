// Two-level triangular solves (Algorithm 2) for gfx950.
//
// Forward substitution L dy = Pi r, one launch per Gamma level: a position j of
// level l pulls the contributions of the positions that precede it in the factor's
// row j -- the left neighbours j-2^t and right neighbours j+2^t of levels t+1 < l --
// so every factor block is read exactly once per sweep and no two work items write
// the same vector (no atomics, fixed summation order).  Then X (x_1), whose row holds
// the G_r blocks of the last position of every level with an odd chain length, and
// the FP64 root step (Algorithm 2, root step).  Backward substitution walks the
// levels in reverse; position j reads the already known x of its two neighbours.
// The permutation Pi_i (Algorithm 2, gather and scatter) is applied as an index map:
// chain position j reads and writes stage N-j of the natural-order vectors.
//
// This file: the sweeps of few right-hand sides at n <= 32 (few_rhs), and the root step.
// Factor blocks are held in registers (RegBlock) and read once for all right-hand sides;
// every block a position needs is loaded at once, spread over up to four waves.  More
// right-hand sides and blocks of 33..64: solve_rhs.hip, solve64.hip.
#include <algorithm>

#include <type_traits>

#include "bmpc_internal.h"
#include "blockops.h"
#include "multi.h"
#include "regblock.h"
#include "root.h"
#include "solve_common.h"

namespace bmpc {

namespace {

// A position applies its own L_jj^{-1} after subtracting the products of the factor blocks it
// pulls, each with the vector of a neighbour.  Forward (position j of level l): pull 2t is
// the G_r of the left neighbour j-2^t, pull 2t+1 the G_l of the right neighbour j+2^t
// (t < l-1).  Backward: pull 0 is G_l(j)^T with x of the left neighbour, pull 1 is G_r(j)^T
// with x of the right neighbour (or of X).  Each wave takes kPullsPerWave consecutive pulls
// and issues all of their loads at once (wave 0 also loads L_jj^{-1}); the workgroup
// has up to kLevelMaxWaves waves and further pulls go round in turns.  Partial sums
// are combined in wave order.
constexpr int kPullsPerWave = 2;
constexpr int kLevelMaxWaves = 4;

// waves of a forward position, and of the x_1 forward step of a chain of L levels
__host__ __device__ inline int fwd_one_waves(int level) {
  return level < 2 ? 1 : level - 1 < kLevelMaxWaves ? level - 1 : kLevelMaxWaves;
}
__host__ __device__ inline int x_fwd_waves(int L) {
  return L < 3 ? 1 : L < 2 * kLevelMaxWaves ? (L + 1) / 2 : kLevelMaxWaves;
}

// Dynamic LDS of a level workgroup with W waves:
// vbuf[W][kPullsPerWave][NR][NMAX], partial[W][NR][NMAX], rhs[NR][NMAX].
template <typename T, int NMAX>
inline size_t level_smem_bytes(int waves, int nrhs) {
  return (size_t)(waves * kPullsPerWave + waves + 1) * nrhs * NMAX * sizeof(T);
}

// What a wave or several do for NR right-hand sides: a position of a forward or backward level,
// or the x_1 forward step, whose pulls are the G_r of the last position of every level with
// an odd chain length and which also forms w_s = F_s y_X.
enum FewKind { FEW_FWD, FEW_BWD, FEW_X };

// One position (index i of the level, scenario sl, system sys) served by W waves, this
// thread's wave being wv; smem holds (W * kPullsPerWave + W + 1) * NR * NMAX elements.  FULL:
// n == NMAX (smaller n: padding read as zero).  Lane l holds element l % NMAX of each vector
// it stages, and each wave keeps its partial sums in registers across rounds.
// TOGETHER: the workgroup holds several positions, so that every wave goes through the
// barrier, the ones without a position (not active) too.
template <typename T, int NMAX, int KIND, bool FULL, int NR, bool TOGETHER = false>
__device__ __attribute__((always_inline)) inline void few_position(
    const SolveArgs& a, int level, int i, int sl, int sys, int W, int wv, unsigned char* smem,
    bool active = true) {
  if (TOGETHER && !active) {
    __syncthreads();
    return;
  }
  typedef RegBlock<T, NMAX> RB;
  constexpr bool BWD = KIND == FEW_BWD;
  constexpr int P = kPullsPerWave;
  const int n = FULL ? NMAX : a.n;
  const size_t nn = (size_t)n * n;
  const int N = a.N, m = a.m;
  const int lane = threadIdx.x & 63;
  typedef T Vec[NMAX];
  Vec* vbuf = reinterpret_cast<Vec*>(smem);  // [(w * P + u) * NR + q]
  Vec* partial = vbuf + W * P * NR;          // [w * NR + q]
  Vec* t = partial + W * NR;                 // [q]: right-hand side, then residual
  const size_t s = (size_t)sys * a.S + sl;
  const int j = KIND == FEW_X ? N : (2 * i + 1) << (level - 1);
  const size_t gstride = g_chain_blocks(N);
  const T* Gl = reinterpret_cast<const T*>(a.Gl) + s * gstride * nn;
  const T* Gr = reinterpret_cast<const T*>(a.Gr) + s * gstride * nn;
  const T* Linv = reinterpret_cast<const T*>(a.Linv) + s * N * nn;
  T* y = reinterpret_cast<T*>(a.y) + s * N * n * NR;
  T* yj = y + (size_t)(j - 1) * n * NR;
  const int half = BWD ? 1 << (level - 1) : 0;
  const int npull = KIND == FEW_FWD ? 2 * (level - 1) : BWD ? 2 : chain_levels(m);
  const size_t len = vec_len(a);
  const size_t off = (size_t)sys * a.vsys + ((size_t)sl * N + (N - j)) * n;
  const int seg = sys * a.seg_sys;
  const int o = RB::out_index();
  const bool writer = RB::base() == 0, out = writer && (FULL || o < n);
  const int vl = lane & (NMAX - 1);
  const bool vin = FULL || vl < n;

  auto pull = [&](int p, const T*& blk, const T*& vec) -> bool {
    int c;
    if constexpr (KIND == FEW_FWD) {
      const int tt = p >> 1;
      c = (p & 1) ? j + (1 << tt) : j - (1 << tt);
      if (c > m) return false;
      blk = ((p & 1) ? Gl : Gr) + (size_t)(c - 1) * nn;
    } else if constexpr (BWD) {
      if (p == 0) {
        if (j - half < 1) return false;
        blk = Gl + (size_t)(j - 1) * nn;
        c = j - half;
      } else {
        c = j + half <= m ? j + half : N;
        blk = Gr + (size_t)(j - 1) * nn;
      }
    } else {
      if (((m >> p) & 1) == 0) return false;
      c = (m >> p) << p;
      blk = Gr + (size_t)(c - 1) * nn;
    }
    vec = y + (size_t)(c - 1) * n * NR;
    return true;
  };

  // All loads of the first round are issued before the first wait.
  RB lin, fb;
  T rv[NR] = {};
  double rb[NR] = {}, xo[NR] = {};
  if (wv == 0) {
    if constexpr (FULL)
      lin.template load_packed_raw<BWD>(Linv + (size_t)(j - 1) * nn);
    else
      lin.template load_packed<BWD>(Linv + (size_t)(j - 1) * nn, n);
    if constexpr (KIND == FEW_X)
      fb.template load_fixed<false, FULL>(reinterpret_cast<const T*>(a.F) + s * nn, n);
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      if constexpr (BWD)
        rv[q] = vin ? yj[vl * NR + q] : T(0);
      else
        rb[q] = vin ? a.b[(size_t)q * len + off + vl] : 0.0;
      if (BWD && a.accumulate && (FULL || o < n)) xo[q] = a.x[(size_t)q * len + off + o];
    }
  }
  T tot[NR];
  auto round = [&](int base, bool first) {
    RB blk[P];
    T vv[P][NR];
    bool has[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const int p = base + wv * P + u;
      const T* bp = nullptr;
      const T* vp = nullptr;
      has[u] = p < npull && pull(p, bp, vp);
      if (has[u]) {
        blk[u].template load_fixed<BWD, FULL>(bp, n);
#pragma unroll
        for (int q = 0; q < NR; ++q) vv[u][q] = vin ? vp[vl * NR + q] : T(0);
      }
    }
    if (first && wv == 0 && lane < NMAX) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        if constexpr (BWD) {
          t[q][lane] = rv[q];
        } else {
          const double rn = a.rnorm ? a.rnorm[seg + q] : 1.0;
          t[q][lane] = static_cast<T>(rn > 0.0 ? rb[q] / rn : 0.0);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < P; ++u)
#pragma unroll
      for (int q = 0; q < NR; ++q)
        if (has[u] && lane < NMAX) vbuf[(wv * P + u) * NR + q][lane] = vv[u][q];
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      T acc = T(0);
#pragma unroll
      for (int u = 0; u < P; ++u)
        if (has[u]) acc += blk[u].dot(vbuf[(wv * P + u) * NR + q]);
      acc = lane_group_sum_dpp<RB::LPR>(acc);
      tot[q] = first ? acc : tot[q] + acc;
    }
    wave_lds_fence();
  };
  round(0, true);
  for (int base = W * P; base < npull; base += W * P) round(base, false);
  if (TOGETHER || W > 1) {
    if (writer)
#pragma unroll
      for (int q = 0; q < NR; ++q) partial[wv * NR + q][o] = tot[q];
    __syncthreads();
    if (wv != 0) return;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      T sum = partial[q][o];
      for (int w = 1; w < W; ++w) sum += partial[w * NR + q][o];
      tot[q] = sum;
    }
  }
  // residual of the position, then L_jj^{-1} (forward) or L_jj^{-T} (backward) on it
#pragma unroll
  for (int q = 0; q < NR; ++q) tot[q] = t[q][o] - tot[q];
  wave_lds_fence();
  if (writer)
#pragma unroll
    for (int q = 0; q < NR; ++q) t[q][o] = tot[q];
  wave_lds_fence();
  if constexpr (FULL) lin.template mask_packed<BWD>();
  T v[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) v[q] = lane_group_sum_dpp<RB::LPR>(lin.dot(t[q]));
  if (out) {
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      yj[o * NR + q] = v[q];
      if constexpr (BWD) {
        const size_t idx = (size_t)q * len + off + o;
        const double d = static_cast<double>(v[q]);
        if (a.accumulate) {
          const double dd = a.rnorm[seg + q] * d;
          a.x[idx] = xo[q] + dd;
          a.dstore[idx] = dd;
        } else {
          a.x[idx] = d;
        }
      }
    }
  }
  if constexpr (KIND == FEW_X) {
    // w_s = F_s y_X in FP64 (the root reduction input of Algorithm 2)
    if (writer)
#pragma unroll
      for (int q = 0; q < NR; ++q) vbuf[q][o] = v[q];
    wave_lds_fence();
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      double p = 0.0;
#pragma unroll
      for (int e = 0; e < RB::EPL; ++e)
        p += static_cast<double>(fb.v[e]) * static_cast<double>(vbuf[q][RB::base() + e]);
      p = lane_group_sum_dpp<RB::LPR>(p);
      if (out) a.w[(s * NR + q) * n + o] = p;
    }
  }
}

// Root propagation and the x_1 backward step on one wave: dy_X -= F^T x_0 (FP64), x_X = L_X^{-T}
// dy_X.  smem: NR * NMAX doubles, then as many T.
template <typename T, int NMAX, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void few_x_bwd(const SolveArgs& a, int sl,
                                                                int sys, unsigned char* smem) {
  typedef RegBlock<T, NMAX> RB;
  const int n = FULL ? NMAX : a.n, N = a.N;
  const size_t nn = (size_t)n * n, s = (size_t)sys * a.S + sl;
  double(*x0s)[NMAX] = reinterpret_cast<double(*)[NMAX]>(smem);
  T(*rhs)[NMAX] = reinterpret_cast<T(*)[NMAX]>(smem + NR * NMAX * sizeof(double));
  const int vl = threadIdx.x & (NMAX - 1), o = RB::out_index();
  const bool vin = FULL || vl < n, writer = RB::base() == 0, out = writer && (FULL || o < n);
  T* yx = reinterpret_cast<T*>(a.y) + (s * N + (N - 1)) * n * NR;
  const size_t len = vec_len(a), off = (size_t)sys * a.vsys + (size_t)sl * N * n;
  RB lin, fb;
  fb.template load_fixed<true, FULL>(reinterpret_cast<const T*>(a.F) + s * nn, n);
  if constexpr (FULL)
    lin.template load_packed_raw<true>(reinterpret_cast<const T*>(a.Linv) + (s * N + (N - 1)) * nn);
  else
    lin.template load_packed<true>(reinterpret_cast<const T*>(a.Linv) + (s * N + (N - 1)) * nn, n);
  double x0[NR], xo[NR] = {};
  T yv[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    x0[q] = vin ? a.x0[((size_t)sys * NR + q) * n + vl] : 0.0;
    yv[q] = vin ? yx[vl * NR + q] : T(0);
    if (a.accumulate && (FULL || o < n)) xo[q] = a.x[(size_t)q * len + off + o];
  }
  if ((threadIdx.x & 63) < NMAX)
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      x0s[q][vl] = x0[q];
      rhs[q][vl] = yv[q];
    }
  wave_lds_fence();
  T r[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    double p = 0.0;
#pragma unroll
    for (int e = 0; e < RB::EPL; ++e)
      p += static_cast<double>(fb.v[e]) * x0s[q][RB::base() + e];
    p = lane_group_sum_dpp<RB::LPR>(p);
    r[q] = static_cast<T>(static_cast<double>(rhs[q][o]) - p);
  }
  wave_lds_fence();
  if (writer)
#pragma unroll
    for (int q = 0; q < NR; ++q) rhs[q][o] = r[q];
  wave_lds_fence();
  if constexpr (FULL) lin.template mask_packed<true>();
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const T v = lane_group_sum_dpp<RB::LPR>(lin.dot(rhs[q]));
    if (out) {
      yx[o * NR + q] = v;
      const size_t idx = (size_t)q * len + off + o;
      const double d = static_cast<double>(v);
      if (a.accumulate) {
        const double dd = a.rnorm[sys * a.seg_sys + q] * d;
        a.x[idx] = xo[q] + dd;
        a.dstore[idx] = dd;
      } else {
        a.x[idx] = d;
      }
    }
  }
}

template <typename T, int NMAX, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void few_x_bwd_body(const SolveArgs& a, int s) {
  if (a.done && *a.done) return;
  __shared__ __align__(16) unsigned char sm[NR * NMAX * (sizeof(double) + sizeof(T))];
  const int sys = s / a.S;
  few_x_bwd<T, NMAX, FULL, NR>(a, s - sys * a.S, sys, sm);
}
template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64) solve_x_bwd_kernel(SolveArgs a) {
  few_x_bwd_body<T, NMAX, FULL, NR>(a, blockIdx.x);
}

// The place of a workgroup in a level's grid: (position, scenario, system), or flat (count
// positions per chain) beyond the y and z launch limits.
struct FewPlace {
  int i, sl, sys;
};
__device__ inline FewPlace few_place(const SolveArgs& a, int count, unsigned x, unsigned y,
                                     unsigned z) {
  if (count == 0) return {(int)x, (int)y, (int)z};
  const unsigned s = x / (unsigned)count, sys = s / (unsigned)a.S;
  return {(int)(x - s * count), (int)(s - sys * a.S), (int)sys};
}

template <typename T, int NMAX, bool FWD, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void few_level_body(const SolveArgs& a, int level,
                                                                     const FewPlace& w) {
  if (a.done && *a.done) return;
  extern __shared__ __align__(16) unsigned char level_smem[];
  few_position<T, NMAX, FWD ? FEW_FWD : FEW_BWD, FULL, NR>(
      a, level, w.i, w.sl, w.sys, (int)(blockDim.x >> 6), wave_id(), level_smem);
}
template <typename T, int NMAX, bool FWD, bool FULL, int NR>
__global__ void __launch_bounds__(64 * kLevelMaxWaves) solve_level_one_kernel(SolveArgs a,
                                                                             int level, int count) {
  few_level_body<T, NMAX, FWD, FULL, NR>(
      a, level, few_place(a, count, blockIdx.x, blockIdx.y, blockIdx.z));
}

// The x_1 forward step of every chain, a wave for two pulls.
template <typename T, int NMAX, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void few_x_fwd_body(const SolveArgs& a, int s,
                                                                     int W) {
  if (a.done && *a.done) return;
  extern __shared__ __align__(16) unsigned char level_smem[];
  const int sys = s / a.S, wv = wave_id();
  few_position<T, NMAX, FEW_X, FULL, NR, true>(a, 0, 0, s - sys * a.S, sys, W, wv, level_smem,
                                               wv < W);
}
template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64 * kLevelMaxWaves) solve_x_fwd_kernel(SolveArgs a) {
  few_x_fwd_body<T, NMAX, FULL, NR>(a, blockIdx.x, (int)(blockDim.x >> 6));
}

// Backward position for n of 17..32 (FULL: 32) that reads every block by
// rows: lane l holds the 16-byte piece (VEC elements) at columns VEC*q of rows
// mrow + RPI*k (q = l % QPR, mrow = l / QPR, k < K), so one load instruction covers RPI
// whole rows of a block, as in the forward sweep, instead of reading columns with
// dword loads.  The transposed products G^T x and L_jj^{-T} r sum over rows, i.e. over
// the lanes that share q (column_group_sum); the residual r, produced by columns, is
// re-indexed by rows through LDS.  Position j's own G_l slot is read even without a
// left neighbour (it is then never written and not used), so that no load waits on a
// branch.  Below 32, pieces of rows past the block's read zero and a lane's columns past it
// are dropped.  (At n = 24, S = 73, N = 100 in FP64 the seven levels took 59.5 us with the
// columns read by dwords, 65 us as matrix products with fifteen of sixteen columns empty,
// 40 us so with the top levels in one launch.)
template <typename T, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void bwd_rows_position(
    const SolveArgs& a, int level, int i, int sl, int sys, T (*xs)[32]) {
  constexpr int NMAX = 32;
  constexpr int VEC = 16 / (int)sizeof(T);
  constexpr int QPR = NMAX / VEC;
  constexpr int RPI = 64 / QPR;
  constexpr int K = NMAX / RPI;
  const int n = FULL ? NMAX : a.n;
  const size_t nn = (size_t)n * n;
  typedef T vt __attribute__((ext_vector_type(VEC)));
  // xs[3][NR][NMAX] (this wave's LDS): x of the left and right neighbours, y_j; then r by rows
  T(*const xl)[32] = xs;
  T(*const xr)[32] = xs + NR;
  T(*const yr)[32] = xs + 2 * NR;
  const int lane = threadIdx.x & 63, q = lane % QPR, mrow = lane / QPR;
  const int N = a.N, m = a.m;
  const size_t s = (size_t)sys * a.S + sl;
  const int j = (2 * i + 1) << (level - 1);
  const int half = 1 << (level - 1);
  const size_t gstride = g_chain_blocks(N);
  const T* Glb = reinterpret_cast<const T*>(a.Gl) + (s * gstride + (j - 1)) * nn;
  const T* Grb = reinterpret_cast<const T*>(a.Gr) + (s * gstride + (j - 1)) * nn;
  const T* Lb = reinterpret_cast<const T*>(a.Linv) + (s * N + (j - 1)) * nn;
  T* y = reinterpret_cast<T*>(a.y) + s * N * n * NR;
  T* yj = y + (size_t)(j - 1) * n * NR;
  const bool has_left = j - half >= 1;
  const int ir = j + half <= m ? j + half - 1 : N - 1;
  const size_t len = vec_len(a);
  const size_t off = (size_t)sys * a.vsys + ((size_t)sl * N + (N - j)) * n;
  vt gl[K], gr[K];
  T li[K][VEC];
  const auto rsL = block_rsrc(Lb, (unsigned)(n * (n + 1) / 2) * sizeof(T));
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int R = mrow + RPI * k;
    if constexpr (FULL) {
      gr[k] = *reinterpret_cast<const vt*>(Grb + R * NMAX + VEC * q);
      gl[k] = *reinterpret_cast<const vt*>(Glb + R * NMAX + VEC * q);
    } else {
      const unsigned o =
          R < n && VEC * q < n ? (unsigned)(R * n + VEC * q) * sizeof(T) : kOutOfRange;
      const auto wr = __builtin_amdgcn_raw_buffer_load_b128(
          block_rsrc(Grb, (unsigned)nn * (unsigned)sizeof(T)), o, 0, 0);
      const auto wl = __builtin_amdgcn_raw_buffer_load_b128(
          block_rsrc(Glb, (unsigned)nn * (unsigned)sizeof(T)), o, 0, 0);
      __builtin_memcpy(&gr[k], &wr, 16);
      __builtin_memcpy(&gl[k], &wl, 16);
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const unsigned o = (unsigned)(R * (R + 1) / 2 + VEC * q + e) * sizeof(T);
      if constexpr (sizeof(T) == 8)
        li[k][e] = buf_load_f64(rsL, o);
      else
        li[k][e] = buf_load_f32(rsL, o);
    }
  }
  const int vl = lane & (NMAX - 1);
  const bool vin = FULL || vl < n;
  T v0[NR], v1[NR], v2[NR];
  double xo[NR][VEC];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    v0[k] = vin ? y[((size_t)(has_left ? j - half - 1 : j - 1) * n + vl) * NR + k] : T(0);
    v1[k] = vin ? y[((size_t)ir * n + vl) * NR + k] : T(0);
    v2[k] = vin ? yj[vl * NR + k] : T(0);
    if (a.accumulate) {  // wave-uniform; the x being updated, at the output lanes' columns
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        xo[k][e] = FULL || VEC * q + e < n ? a.x[(size_t)k * len + off + VEC * q + e] : 0.0;
    }
  }
  if (lane < NMAX) {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      xl[k][lane] = has_left ? v0[k] : T(0);
      xr[k][lane] = v1[k];
      yr[k][lane] = v2[k];
    }
  }
  wave_lds_fence();
  // r = y_j - G_l^T x_l - G_r^T x_r, by columns c = VEC*q + e
  T r[NR][VEC];
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    T p[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) p[e] = T(0);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int R = mrow + RPI * k;
      const T al = xl[u][R], ar = xr[u][R];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if (has_left) p[e] += gl[k][e] * al;
        p[e] += gr[k][e] * ar;
      }
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) r[u][e] = yr[u][VEC * q + e] - column_group_sum<QPR>(p[e]);
  }
  wave_lds_fence();
  if (mrow == 0) {
#pragma unroll
    for (int u = 0; u < NR; ++u)
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        xl[u][VEC * q + e] = FULL || VEC * q + e < n ? r[u][e] : T(0);
  }
  wave_lds_fence();
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    // x_j = L_jj^{-T} r: sum over rows R >= c of L^{-1}[R][c] r[R]
    T x[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) x[e] = T(0);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int R = mrow + RPI * k;
      const T rr = xl[u][R];
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (VEC * q + e <= R) x[e] += li[k][e] * rr;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) x[e] = column_group_sum<QPR>(x[e]);
    if (mrow == 0) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const int c = VEC * q + e;
        if (!FULL && c >= n) break;
        yj[c * NR + u] = x[e];
        const size_t idx = (size_t)u * len + off + c;
        const double d = static_cast<double>(x[e]);
        if (a.accumulate) {
          const double dd = a.rnorm[sys * a.seg_sys + u] * d;
          a.x[idx] = xo[u][e] + dd;
          a.dstore[idx] = dd;
        } else {
          a.x[idx] = d;
        }
      }
    }
  }
}

template <typename T, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void bwd_rows_body(const SolveArgs& a, int level,
                                                                    const FewPlace& w) {
  if (a.done && *a.done) return;
  __shared__ T xs[3 * NR][32];
  bwd_rows_position<T, FULL, NR>(a, level, w.i, w.sl, w.sys, xs);
}
template <typename T, bool FULL, int NR>
__global__ void __launch_bounds__(64) solve_bwd_rows_kernel(SolveArgs a, int level, int count) {
  bwd_rows_body<T, FULL, NR>(a, level, few_place(a, count, blockIdx.x, blockIdx.y, blockIdx.z));
}

// The top backward levels of every chain in one launch, with_x after root propagation and the
// x_1 backward step, one workgroup per chain: wave 0 solves x_1, then wave w
// position w of each level from the top level down to level_lo (at most one per wave), with a
// barrier between levels.  A position reads the x of its neighbours from y, written by
// other waves of the workgroup at higher levels; the barrier orders those stores before
// the reads (the waves of a workgroup share one CU and its vector cache).  Each position
// runs the code of the single-level kernel (row reads at n > 16, one wave of the level
// kernel otherwise), so the results are bitwise those of the launches level by level.
template <typename T, int NMAX, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void solve_bwd_top_body(const SolveArgs& a,
                                                                         int level_lo,
                                                                         bool with_x, int s) {
  if (a.done && *a.done) return;
  constexpr int PER = (NMAX == 32 ? 3 : kPullsPerWave + 2) * NR * NMAX;  // per wave
  static_assert(PER * sizeof(T) >= NR * NMAX * (sizeof(double) + sizeof(T)), "x_1 fits too");
  constexpr int W = mm_top_waves(NMAX);
  __shared__ __align__(16) T sm[W * PER];
  const int w = threadIdx.x >> 6, sys = s / a.S, sl = s - sys * a.S;
  if (with_x && w == 0)
    few_x_bwd<T, NMAX, FULL, NR>(a, sl, sys, reinterpret_cast<unsigned char*>(sm));
  for (int level = chain_levels(a.m); level >= level_lo; --level) {
    __syncthreads();
    if (w < level_count(a.m, level)) {
      if constexpr (NMAX == 32)
        bwd_rows_position<T, FULL, NR>(a, level, w, sl, sys,
                                       reinterpret_cast<T(*)[NMAX]>(sm + w * PER));
      else
        few_position<T, NMAX, FEW_BWD, FULL, NR>(a, level, w, sl, sys, 1, 0,
                                                 reinterpret_cast<unsigned char*>(sm + w * PER));
    }
  }
}

template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64 * mm_top_waves(NMAX)) solve_bwd_top_kernel(
    SolveArgs a, int level_lo, bool with_x) {
  solve_bwd_top_body<T, NMAX, FULL, NR>(a, level_lo, with_x, blockIdx.x);
}

// The top forward levels (at most four positions) and the x_1 forward step of every chain in
// one launch, one workgroup of sixteen waves per chain: four waves for each position,
// of which as many take part as in the single-level kernel, so the results are bitwise
// those of the launches level by level.  In FP64 for n <= 16: at n = 32 a wave would spill (S
// = 128, N = 64: 96 us for the solve against 92 level by level).  In FP32 at n = 24, S = 4, N =
// 16, two right-hand sides, 42 us level by level, 36 so.
constexpr int kFwdTopWaves = 16;
template <typename T, int NMAX, bool FULL, int NR>
__device__ __attribute__((always_inline)) inline void solve_fwd_top_body(const SolveArgs& a,
                                                                         int level_lo, int s) {
  if (a.done && *a.done) return;
  constexpr size_t kPos =
      (size_t)(kLevelMaxWaves * (kPullsPerWave + 1) + 1) * NR * NMAX * sizeof(T);
  __shared__ __align__(16) unsigned char sm[kFwdTopWaves / kLevelMaxWaves * kPos];
  const int wv = wave_id(), sys = s / a.S, sl = s - sys * a.S, L = chain_levels(a.m);
  const int i = wv / kLevelMaxWaves, w = wv % kLevelMaxWaves;
  for (int level = level_lo; level <= L; ++level) {
    const int W = fwd_one_waves(level);
    few_position<T, NMAX, FEW_FWD, FULL, NR, true>(a, level, i, sl, sys, W, w, sm + i * kPos,
                                                   i < level_count(a.m, level) && w < W);
    __syncthreads();
  }
  const int W = x_fwd_waves(L);
  few_position<T, NMAX, FEW_X, FULL, NR, true>(a, 0, 0, sl, sys, W, wv, sm, wv < W);
}

template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64 * kFwdTopWaves) solve_fwd_top_kernel(SolveArgs a,
                                                                          int level_lo) {
  solve_fwd_top_body<T, NMAX, FULL, NR>(a, level_lo, blockIdx.x);
}

// Root step in FP64 (Algorithm 2, root step).  One workgroup of 1024 threads per
// system of the batch: r~_0 = r_0 - sum_s w_s (scenario_sums: the scenarios over the
// threads, up to eight right-hand sides at a time, the waves' sums combined in order); then
// the two triangular solves with L_R in LDS, one wave per right-hand side, lane i
// owning row i.
// FACTOR: L_R is factored here first (step), its 32 x 32 or smaller matrix read together with
// the w_s; one launch, and its latency, fewer where a factorization has the forward
// substitution inside (with the group sums and the info reset, which one system up to 32
// scenarios needs no launch for, S = 4, N = 16, n = 8 in FP64: 29.7 -> 25.6 us).
template <int NMAX, bool FACTOR>
__device__ __attribute__((always_inline)) inline void solve_root_body(const SolveArgs& a,
                                                                      const RootStep& step,
                                                                      unsigned bx) {
  if (a.done && *a.done) return;
  constexpr int W = 16, LD = NMAX + 1, QB = NMAX == 64 ? 2 : 8;
  __shared__ double part[QB][W][NMAX];
  __shared__ double L[NMAX * LD];
  __shared__ double r0[kSolveRhs][NMAX];
  const int n = a.n, S = a.S, nrhs = a.nrhs;
  const int sys = bx;
  const size_t len = vec_len(a);
  const size_t root_off = (size_t)sys * a.vsys + (size_t)S * a.N * n;
  const int seg0 = sys * a.seg_sys;
  const double* w = a.w + (size_t)sys * S * nrhs * n;  // this system's chains
  const int t = threadIdx.x, i = t % NMAX, q = t / NMAX;
  if constexpr (FACTOR) {
    root_matrix<NMAX, LD>(L, step, sys);
  } else {
    for (int e = t; e < NMAX * NMAX; e += 1024) {
      const int r = e / NMAX, c = e % NMAX;
      L[r * LD + c] = (r < n && c < n) ? a.LR[(size_t)sys * n * n + r * n + c]
                                       : (r == c ? 1.0 : 0.0);  // identity padding
    }
  }
  const bool mine = q < nrhs && i < n;  // this thread's row and right-hand side
  double bv = mine ? a.b[(size_t)q * len + root_off + i] : 0.0;
  if (a.rnorm && mine) {
    const double rn = a.rnorm[seg0 + q];
    bv = rn > 0.0 ? bv / rn : 0.0;
  }
  double sum = 0.0;
  for (int q0 = 0, taken; q0 < nrhs; q0 += taken) {
    if (q0) __syncthreads();
    auto partials = [&](auto qb, auto in_flight) {
      constexpr int Q = decltype(qb)::value;
      double acc[Q];
      scenario_sums<NMAX, Q, decltype(in_flight)::value>(w, S, n, nrhs, q0, acc);
      if ((t & 63) < NMAX)
#pragma unroll
        for (int u = 0; u < Q; ++u) part[u][t >> 6][i] = acc[u];
      return Q;
    };
    // with few scenarios (a round or some of loads) all right-hand sides at once, the last one
    // read again for those that are not there; beyond, as many as there are, a power of two,
    // with at least sixteen loads in flight per thread: S = 20000, n = 8 in FP64, two
    // right-hand sides, one solve 584 -> 441 us, five 858 -> 671; one right-hand side with a
    // round or some needs four (one solve at S = 40, N = 30, n = 8 3 % longer with sixteen)
    const int left = nrhs - q0;
    if (QB >= 8 && left >= (S <= 4 * (1024 / NMAX) ? 5 : 8))
      taken = partials(std::integral_constant<int, QB < 8 ? QB : 8>{},
                       std::integral_constant<int, 4>{});
    else if (QB >= 4 && left >= (S <= 16 * (1024 / NMAX) ? 3 : 4))
      taken = partials(std::integral_constant<int, QB < 4 ? QB : 4>{},
                       std::integral_constant<int, 4>{});
    else if (left >= 2)
      taken = partials(std::integral_constant<int, 2>{},
                       std::integral_constant<int, QB < 8 ? 4 : 8>{});
    else if (S <= 4 * (1024 / NMAX))
      taken = partials(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
    else
      taken = partials(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
    __syncthreads();
    if (mine && q >= q0 && q < q0 + taken) {
#pragma unroll
      for (int v = 0; v < W; ++v) sum += part[q - q0][v][i];
    }
  }
  if (q < nrhs) r0[q][i] = bv - sum;
  __syncthreads();
  if constexpr (FACTOR) {
    double* const scratch = &part[0][0][0];  // the sums are taken
    const int fail = n <= 16 ? block_chol<double, 1, LD, W, false>(L, scratch)
                             : block_chol<double, NMAX / 16, LD, W, false>(L, scratch);
    root_store<NMAX, LD>(L, step, sys, fail);
  }
  // L_R y = r, then L_R^T x = y: wave q handles right-hand side q, lane k row k.  L is
  // identity padded to NMAX x NMAX, so both sweeps run K (NMAX, or 16 for n <= 16) unrolled
  // steps (the padded unknowns stay 0); each lane holds the row (forward) or column
  // (backward) of L it updates with, and 1 / L[k][k] is formed once per lane and
  // broadcast with x_k.
  const int wv = t >> 6, lane = t & 63;
  auto sweeps = [&](auto steps) {
    constexpr int K = decltype(steps)::value;
    const int row = lane < K ? lane : K - 1;
    double v = (lane < n) ? r0[wv][lane] : 0.0;
    const double rd = 1.0 / L[row * LD + row];
    double lk[K];
#pragma unroll
    for (int k = 0; k < K; ++k) lk[k] = L[row * LD + k];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double xk = wave_bcast(v, k) * wave_bcast(rd, k);
      v = (lane == k) ? xk : (lane > k ? v - lk[k] * xk : v);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) lk[k] = L[k * LD + row];
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
      const double xk = wave_bcast(v, k) * wave_bcast(rd, k);
      v = (lane == k) ? xk : (lane < k ? v - lk[k] * xk : v);
    }
    if (lane < n) r0[wv][lane] = v;
  };
  if (wv < nrhs) {
    if (NMAX == 32 && n <= 16)
      sweeps(std::integral_constant<int, 16>{});
    else
      sweeps(std::integral_constant<int, NMAX>{});
  }
  __syncthreads();
  for (int idx = t; idx < n * nrhs; idx += 1024) {
    const int q = idx / n, ii = idx - (idx / n) * n;
    a.x0[(size_t)sys * nrhs * n + idx] = r0[q][ii];
    scatter_value(a, q, root_off + ii, seg0, r0[q][ii]);
  }
}

template <int NMAX>
__global__ void __launch_bounds__(1024) solve_root_kernel(SolveArgs a) {
  solve_root_body<NMAX, false>(a, RootStep{}, blockIdx.x);
}
__global__ void __launch_bounds__(1024) root_factor_solve_kernel(RootStep s, SolveArgs a) {
  solve_root_body<32, true>(a, s, blockIdx.x);
}

// ---- one launch over the systems of a ragged batch (see multi.h) ----
// Items of the level kinds carry (level, positions per chain of a flat grid or 0) in p0, p1; the
// merged backward top levels carry (level_lo, with_x).

template <typename T, int NMAX, bool FWD, bool FULL, int NR>
__global__ void __launch_bounds__(64 * kLevelMaxWaves) solve_level_one_multi(
    const MultiItem<SolveArgs>* items, int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  const LocalBlock lb = multi_local(it);
  const SolveArgs a = relocate_solve(it.a, r);
  few_level_body<T, NMAX, FWD, FULL, NR>(a, it.p0, few_place(a, it.p1, lb.x, lb.y, lb.z));
}

template <typename T, bool FULL, int NR>
__global__ void __launch_bounds__(64) solve_bwd_rows_multi(const MultiItem<SolveArgs>* items,
                                                           int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  const LocalBlock lb = multi_local(it);
  const SolveArgs a = relocate_solve(it.a, r);
  bwd_rows_body<T, FULL, NR>(a, it.p0, few_place(a, it.p1, lb.x, lb.y, lb.z));
}

template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64 * mm_top_waves(NMAX)) solve_bwd_top_multi(
    const MultiItem<SolveArgs>* items, int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  const SolveArgs a = relocate_solve(it.a, r);
  solve_bwd_top_body<T, NMAX, FULL, NR>(a, it.p0, it.p1 != 0, multi_local(it).x);
}

template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64 * kFwdTopWaves) solve_fwd_top_multi(
    const MultiItem<SolveArgs>* items, int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  solve_fwd_top_body<T, NMAX, FULL, NR>(relocate_solve(it.a, r), it.p0, multi_local(it).x);
}

template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64 * kLevelMaxWaves) solve_x_fwd_multi(
    const MultiItem<SolveArgs>* items, int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  few_x_fwd_body<T, NMAX, FULL, NR>(relocate_solve(it.a, r), multi_local(it).x,
                                    x_fwd_waves(chain_levels(it.a.m)));
}

template <typename T, int NMAX, bool FULL, int NR>
__global__ void __launch_bounds__(64) solve_x_bwd_multi(const MultiItem<SolveArgs>* items,
                                                        int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  few_x_bwd_body<T, NMAX, FULL, NR>(relocate_solve(it.a, r), multi_local(it).x);
}

template <int NMAX>
__global__ void __launch_bounds__(1024) solve_root_multi(const MultiItem<SolveArgs>* items,
                                                         int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  solve_root_body<NMAX, false>(relocate_solve(it.a, r), RootStep{}, multi_local(it).x);
}

template <typename T, int NMAX, bool FULL, int NR>
void solve_multi_t(int kind, bool fwd, const MultiItem<SolveArgs>* items, int nitems,
                   unsigned blocks, unsigned threads, size_t lds, const Reloc& r, hipStream_t st) {
  const dim3 g(blocks), b(threads);
  switch (kind) {
    case SK_LEVEL_ONE:
      if (fwd)
        hipLaunchKernelGGL((solve_level_one_multi<T, NMAX, true, FULL, NR>), g, b, lds, st, items,
                           nitems, r);
      else if constexpr (NMAX < 32)
        hipLaunchKernelGGL((solve_level_one_multi<T, NMAX, false, FULL, NR>), g, b, lds, st, items,
                           nitems, r);
      break;
    case SK_BWD_ROWS:
      if constexpr (NMAX == 32)
        hipLaunchKernelGGL((solve_bwd_rows_multi<T, FULL, NR>), g, b, 0, st, items, nitems, r);
      break;
    case SK_BWD_TOP:
      hipLaunchKernelGGL((solve_bwd_top_multi<T, NMAX, FULL, NR>), g, b, 0, st, items, nitems, r);
      break;
    case SK_FWD_TOP:
      if constexpr (few_fwd_top(NMAX, sizeof(T) == 8))
        hipLaunchKernelGGL((solve_fwd_top_multi<T, NMAX, FULL, NR>), g, dim3(64 * kFwdTopWaves), 0,
                           st, items, nitems, r);
      break;
    case SK_X_BWD:
      hipLaunchKernelGGL((solve_x_bwd_multi<T, NMAX, FULL, NR>), g, dim3(64), 0, st, items, nitems,
                         r);
      break;
    case SK_X_FWD:
      hipLaunchKernelGGL((solve_x_fwd_multi<T, NMAX, FULL, NR>), g, b, lds, st, items, nitems, r);
      break;
  }
}

template <typename T, int NMAX, bool FULL, int NR>
void level_t(const SolveArgs& a, int level, bool fwd, hipStream_t st) {
  const LevelCfg c = solve_level_config(a, level, fwd, NMAX, sizeof(T) == 8);
  if (c.count <= 0) return;
  const dim3 g(c.gx, c.gy, c.gz), b(c.threads);
  if (c.kind == SK_BWD_ROWS) {
    if constexpr (NMAX == 32)
      hipLaunchKernelGGL((solve_bwd_rows_kernel<T, FULL, NR>), g, b, 0, st, a, level, c.flat);
  } else if (fwd) {
    hipLaunchKernelGGL((solve_level_one_kernel<T, NMAX, true, FULL, NR>), g, b, c.lds, st, a, level,
                       c.flat);
  } else if constexpr (NMAX < 32) {
    hipLaunchKernelGGL((solve_level_one_kernel<T, NMAX, false, FULL, NR>), g, b, c.lds, st, a,
                       level, c.flat);
  }
}

// f(NMAX, FULL, NR as std::integral_constant) for a block size of at most 32 and few
// right-hand sides
template <typename F>
void by_size(int n, int nrhs, F&& f) {
  auto rhs = [&](auto nmax, auto full) {
    if (nrhs == 1)
      f(nmax, full, std::integral_constant<int, 1>{});
    else if (nrhs == 2)
      f(nmax, full, std::integral_constant<int, 2>{});
    else
      f(nmax, full, std::integral_constant<int, kFewRhs>{});
  };
  auto full = [&](auto nmax) {
    if (n == decltype(nmax)::value)
      rhs(nmax, std::true_type{});
    else
      rhs(nmax, std::false_type{});
  };
  if (n <= 8)
    full(std::integral_constant<int, 8>{});
  else if (n <= 16)
    full(std::integral_constant<int, 16>{});
  else
    full(std::integral_constant<int, 32>{});
}

}  // namespace

// Kernel, grid and LDS of one level of a sweep: register blocks for few right-hand sides
// (few_rhs; row reads backward for n > 16), matrix products (solve_rhs.hip) otherwise.
// Forward positions of level l pull 2 (l - 1) blocks, kPullsPerWave per wave, on up to
// kLevelMaxWaves waves (or a.fwd_waves: one wave per position when the plan asks for it).
LevelCfg solve_level_config(const SolveArgs& a, int level, bool fwd, int nmax, bool fp64) {
  if (!(fwd ? few_rhs : few_bwd)(a.S, a.N, a.n, a.nrhs, fp64))
    return mm_level_config(a, level, fwd, fp64);
  LevelCfg c{};
  c.count = level_count(a.m, level);
  const int waves = fwd && a.fwd_waves != 1 ? fwd_one_waves(level) : 1;
  c.threads = 64 * waves;
  c.kind = (!fwd && nmax == 32) ? SK_BWD_ROWS : SK_LEVEL_ONE;
  c.lds = c.kind == SK_BWD_ROWS ? 0 : solve_level_lds(fp64, nmax, waves, a.nrhs);
  if (a.S <= 65535 && a.B <= 65535) {
    c.gx = (unsigned)c.count;
    c.gy = (unsigned)a.S;
    c.gz = (unsigned)a.B;
  } else {
    c.flat = c.count;
    c.gx = (unsigned)(a.B * a.S) * (unsigned)std::max(c.count, 0);
    c.gy = c.gz = 1;
  }
  return c;
}
// Threads and LDS of the x_1 forward step alone.
MmTopCfg x_fwd_config(const SolveArgs& a, int nmax, bool fp64) {
  const int waves = x_fwd_waves(chain_levels(a.m));
  return {64u * waves, solve_level_lds(fp64, nmax, waves, a.nrhs)};
}

template <typename T>
static void launch_level(const SolveArgs& a, int level, bool fwd, hipStream_t st) {
  if (!(fwd ? few_rhs : few_bwd)(a.S, a.N, a.n, a.nrhs, sizeof(T) == 8))
    return launch_mm_level<T>(a, level, fwd, st);
  by_size(a.n, a.nrhs, [&](auto nmax, auto full, auto nr) {
    level_t<T, decltype(nmax)::value, decltype(full)::value, decltype(nr)::value>(a, level, fwd,
                                                                                 st);
  });
}
template <typename T>
void launch_solve_fwd_level(const SolveArgs& a, int level, hipStream_t st) {
  launch_level<T>(a, level, true, st);
}
template <typename T>
void launch_solve_bwd_level(const SolveArgs& a, int level, hipStream_t st) {
  launch_level<T>(a, level, false, st);
}
template <typename T>
void launch_solve_bwd_top(const SolveArgs& a, int level_lo, bool with_x, hipStream_t st) {
  const dim3 grid((unsigned)(a.B * a.S));
  by_size(a.n, a.nrhs, [&](auto nmax, auto full, auto nr) {
    constexpr int NMAX = decltype(nmax)::value, NR = decltype(nr)::value;
    constexpr bool FULL = decltype(full)::value;
    if (level_lo > chain_levels(a.m)) {  // x_1 alone
      if (with_x)
        hipLaunchKernelGGL((solve_x_bwd_kernel<T, NMAX, FULL, NR>), grid, dim3(64), 0, st, a);
    } else {
      hipLaunchKernelGGL((solve_bwd_top_kernel<T, NMAX, FULL, NR>), grid,
                         dim3(64 * level_count(a.m, level_lo)), 0, st, a, level_lo, with_x);
    }
  });
}
template <typename T>
void launch_solve_fwd_top(const SolveArgs& a, int level_lo, hipStream_t st) {
  const dim3 grid((unsigned)(a.B * a.S));
  by_size(a.n, a.nrhs, [&](auto nmax, auto full, auto nr) {
    constexpr int NMAX = decltype(nmax)::value, NR = decltype(nr)::value;
    constexpr bool FULL = decltype(full)::value;
    if (level_lo > chain_levels(a.m)) {  // x_1 alone
      const MmTopCfg c = x_fwd_config(a, NMAX, sizeof(T) == 8);
      hipLaunchKernelGGL((solve_x_fwd_kernel<T, NMAX, FULL, NR>), grid, dim3(c.threads), c.lds, st,
                         a);
    } else if constexpr (few_fwd_top(NMAX, sizeof(T) == 8)) {
      hipLaunchKernelGGL((solve_fwd_top_kernel<T, NMAX, FULL, NR>), grid, dim3(64 * kFwdTopWaves),
                         0, st, a, level_lo);
    }
  });
}
void launch_solve_root(const SolveArgs& a, hipStream_t st) {
  if (a.n > 32)
    hipLaunchKernelGGL(solve_root_kernel<64>, dim3(a.B), dim3(1024), 0, st, a);
  else
    hipLaunchKernelGGL(solve_root_kernel<32>, dim3(a.B), dim3(1024), 0, st, a);
}

void launch_root_factor_solve(const RootStep& s, const SolveArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(root_factor_solve_kernel, dim3(a.B), dim3(1024), 0, st, s, a);
}

size_t solve_level_lds(bool fp64, int nmax, int waves, int nrhs) {
  return fp64 ? (nmax <= 8 ? level_smem_bytes<double, 8>(waves, nrhs)
                          : nmax <= 16 ? level_smem_bytes<double, 16>(waves, nrhs)
                                       : level_smem_bytes<double, 32>(waves, nrhs))
              : (nmax <= 8 ? level_smem_bytes<float, 8>(waves, nrhs)
                           : nmax <= 16 ? level_smem_bytes<float, 16>(waves, nrhs)
                                        : level_smem_bytes<float, 32>(waves, nrhs));
}

template <typename T>
void launch_solve_multi(int kind, bool fwd, int n, int nrhs, const MultiItem<SolveArgs>* items,
                        int nitems, unsigned blocks, unsigned threads, size_t lds, const Reloc& r,
                        hipStream_t st) {
  if (kind == SK_ROOT)
    hipLaunchKernelGGL((solve_root_multi<32>), dim3(blocks), dim3(threads), 0, st, items, nitems,
                       r);
  else if (kind == SK_LEVEL || kind == SK_MM_TOP)
    launch_mm_multi<T>(kind, fwd, n, items, nitems, blocks, threads, lds, r, st);
  else
    by_size(n, nrhs, [&](auto nmax, auto full, auto nr) {
      solve_multi_t<T, decltype(nmax)::value, decltype(full)::value, decltype(nr)::value>(
          kind, fwd, items, nitems, blocks, threads, lds, r, st);
    });
}
template void launch_solve_multi<double>(int, bool, int, int, const MultiItem<SolveArgs>*, int,
                                         unsigned, unsigned, size_t, const Reloc&, hipStream_t);
template void launch_solve_multi<float>(int, bool, int, int, const MultiItem<SolveArgs>*, int,
                                        unsigned, unsigned, size_t, const Reloc&, hipStream_t);

template void launch_solve_fwd_level<double>(const SolveArgs&, int, hipStream_t);
template void launch_solve_fwd_level<float>(const SolveArgs&, int, hipStream_t);
template void launch_solve_bwd_level<double>(const SolveArgs&, int, hipStream_t);
template void launch_solve_bwd_level<float>(const SolveArgs&, int, hipStream_t);
template void launch_solve_fwd_top<double>(const SolveArgs&, int, hipStream_t);
template void launch_solve_fwd_top<float>(const SolveArgs&, int, hipStream_t);
template void launch_solve_bwd_top<double>(const SolveArgs&, int, bool, hipStream_t);
template void launch_solve_bwd_top<float>(const SolveArgs&, int, bool, hipStream_t);

}  // namespace bmpc
