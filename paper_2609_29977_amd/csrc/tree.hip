// Factor passes for block sizes up to 16 (gfx950): the windows of factor.hip's tail
// factorization (Algorithm 1, Section IV-B in block form), walked level by level.
//
// A pass splits the (reduced) chain into windows of 2^Tw positions.  Blocks this small let a
// whole window live in LDS, so the positions of a level are eliminated at the same time, one
// wave each, where factor.hip's depth-first walk (n > 16) takes the window's positions one
// after another.  Per level of the window, two phases with a barrier after each:
//   1. every position j of the level: L_jj^{-1} of A_j; G_r = K[r,j] L^{-T};
//      G_l = K[l,j] L^{-T} (l, r: its neighbours); y_j = L_jj^{-1} V_j with a fused forward
//      substitution;
//   2. every position p that stays: A_p -= G_r G_r^T of its left neighbour's
//      elimination and G_l G_l^T of its right one's, the fill -G_r G_l^T of the latter into
//      its coupling, V_p -= G_r y + G_l y.
// Each block has one writer per phase and the updates of a position are added in a fixed
// order (left, right), so results do not depend on the number of waves.  The window's
// boundaries (its first position lo and the next window's first) are not eliminated: their
// updates are kept in registers (the MFMA accumulators of one wave each) over all levels and
// handed to the next pass, as are the coupling between them and the right-hand sides; a
// boundary's updates from earlier passes ride in its left accumulator.  The last pass also
// eliminates x_1 (F = C L_X^{-T}, U = F F^T).
//
// Bound: with few windows, the latency of a level (the 16-column factorization chain, two
// dependent rounds of products); with many, HBM.  Factor passes with the forward
// substitution, serial walk of the windows -> this: 4 chains of 16 stages, FP64, n = 8: 34 ->
// 15 us; 20 of 30, n = 16: 59 -> 34 us; 100 of 160: 137 -> 91 us; 8192 of 64: 1694 -> 1475 us
// (4.3 GB, 2.9 TB/s); 8192 of 136, FP32, n = 16: 1970 -> 1901 us, n = 8: 765 -> 615 us.
#include <algorithm>
#include <type_traits>

#include "bmpc_internal.h"
#include "blockops.h"
#include "multi.h"
#include "regblock.h"

namespace bmpc {

namespace {

constexpr int kTreeWaves = 16;  // waves per workgroup at most
// Positions whose diagonal blocks one wave factors together, in groups of its lanes, for the
// instructions of one: four at NMAX = 8 (before a barrier, after which every position has a
// wave of its own again for the products).  At NMAX = 16 two would fit, but the barrier and
// the idle waves cost more than the instructions (8192 chains of 64 stages, FP64: 1475 us
// of factor passes with one, 1720 with two).
template <int NMAX>
constexpr int tree_leaf_group() {
  return NMAX == 8 ? 4 : 1;
}

// LDS of a pass: right-hand sides V[0 .. W] (V[0] and V[W] the boundaries'), blocks A[1 ..
// W-1] (diagonals) and C[0 .. W-1] (couplings to the successor; C[0] of the left boundary),
// two more for x_1 in the last pass; W = 2^Tw, or one more than the chain's positions if
// that is less (two at least: the last pass forms F in FP64 in place of the first blocks).
__host__ __device__ inline int tree_window(int Tw, int mk) {
  const int w = 1 << Tw;
  return w <= mk ? w : (mk > 0 ? mk + 1 : 2);
}
template <typename T, int NMAX>
size_t tree_lds_bytes(int W, int nrhs_fused, bool final) {
  return ((2 * W - 1 + (final ? 2 : 0)) * Lay<NMAX>::SZ + (W + 1) * nrhs_fused * NMAX) * sizeof(T);
}
// Waves per workgroup (the results do not depend on it): one per position of the first level,
// which is fastest while the GPU is not full (4 chains of 16, n = 8: 15 us of factor passes
// against 20 with two waves).  Beyond that, 8 x 8 blocks take two waves: their products are so
// small that independent windows hide latencies better than the waves of one, most of which
// idle at the upper levels (8192 chains of 136, FP64 / FP32: 1357 / 895 us with one wave per
// position, 1126 / 615 with two).
inline unsigned tree_threads(int W, int nmax, unsigned blocks) {
  constexpr unsigned kFull = 256 * 32;  // waves that fill the GPU
  const unsigned waves = (unsigned)std::min(kTreeWaves, std::max(1, W / 2));
  return 64 * (nmax <= 8 && (size_t)blocks * waves > kFull ? std::min(waves, 2u) : waves);
}

// Entries of a block in accumulator order (mfma_tile_nt's result on one wave).
template <typename T, int NMAX>
struct AccAt {
  static constexpr int AV = NMAX == 8 ? 1 : 4;
  __device__ static int row(int v) {
    const int l = threadIdx.x & 63;
    return NMAX == 8 ? l >> 3 : Mfma<T>::row(l, v);
  }
  __device__ static int col() {
    const int l = threadIdx.x & 63;
    return NMAX == 8 ? (l & 7) : (l & 15);
  }
};

// The blocks of two positions in registers: D (plus the carried updates after the first
// pass), and two couplings.
template <typename T, int NMAX, bool FIRST>
struct TreeLoad {
  static constexpr int EL = NMAX * NMAX / 64;
  static constexpr int LD = Lay<NMAX>::LD;
  typedef typename std::conditional<FIRST, double, T>::type CT;
  double d[2][EL];
  T ac[2][EL], al[2][EL];
  CT c[2][EL];

  __device__ static unsigned off(int u, int n, bool lower) {  // element index, or out of range
    const int e = (int)(threadIdx.x & 63) + 64 * u, r = e / NMAX, col = e % NMAX;
    return r < n && col < n && (!lower || col <= r) ? (unsigned)(r * n + col)
                                                    : kOutOfRange / 8u;
  }
  template <typename X>
  __device__ static X ld(__amdgpu_buffer_rsrc_t rs, unsigned o) {
    if constexpr (sizeof(X) == 8)
      return buf_load_f64(rs, o * 8u);
    else
      return buf_load_f32(rs, o * 4u);
  }
  __device__ void diag(int k, const FactorPassArgs& a, size_t s, int q) {
    const int n = a.n;
    const size_t nn = (size_t)n * n;
    const auto rd = block_rsrc(a.D + (s * a.N + (a.N - (q << a.shift))) * nn, (unsigned)nn * 8u);
#pragma unroll
    for (int u = 0; u < EL; ++u) d[k][u] = ld<double>(rd, off(u, n, true));
    if constexpr (!FIRST) {
      const size_t o = (s * a.stride + q) * nn;
      const auto rr = block_rsrc(reinterpret_cast<const T*>(a.accR_in) + o, (unsigned)nn * sizeof(T));
      const auto rl = block_rsrc(reinterpret_cast<const T*>(a.accL_in) + o, (unsigned)nn * sizeof(T));
#pragma unroll
      for (int u = 0; u < EL; ++u) {
        ac[k][u] = ld<T>(rr, off(u, n, true));
        al[k][u] = ld<T>(rl, off(u, n, true));
      }
    }
  }
  __device__ void put_diag(int k, T* A, int n) const {
#pragma unroll
    for (int u = 0; u < EL; ++u) {
      const int e = (int)(threadIdx.x & 63) + 64 * u, r = e / NMAX, col = e % NMAX;
      T v = static_cast<T>(d[k][u]);
      if constexpr (!FIRST) v = (v + ac[k][u]) + al[k][u];
      if (r >= n && r == col) v = T(1);  // identity padding
      A[r * LD + col] = v;
    }
  }
  // coupling of q to its successor: E^T of its stage, or the carried fill
  __device__ void coup(int k, const FactorPassArgs& a, size_t s, int q) {
    const int n = a.n;
    const size_t nn = (size_t)n * n;
    const CT* src;
    if constexpr (FIRST)
      src = a.E + (s * (a.N - 1) + (a.N - 1 - q)) * nn;
    else
      src = reinterpret_cast<const T*>(a.fill_in) + (s * a.stride + q) * nn;
    const auto rs = block_rsrc(src, (unsigned)(nn * sizeof(CT)));
#pragma unroll
    for (int u = 0; u < EL; ++u) c[k][u] = ld<CT>(rs, off(u, n, false));
  }
  __device__ void put_coup(int k, T* C) const {
#pragma unroll
    for (int u = 0; u < EL; ++u) {
      const int e = (int)(threadIdx.x & 63) + 64 * u, r = e / NMAX, col = e % NMAX;
      C[FIRST ? col * LD + r : r * LD + col] = static_cast<T>(c[k][u]);
    }
  }
};

// out[q][o] = sum_c M[o][c] v[q][c] on one wave (64 / NMAX lanes per row), put(q, o, value)
// on the first lane of each row.
template <typename T, int NMAX, typename Put>
__device__ inline void wave_matvec(const T* M, const T* v, int nrhs, Put put) {
  constexpr int LD = Lay<NMAX>::LD, TPR = 64 / NMAX, CPT = NMAX / TPR;
  const int l = threadIdx.x & 63, o = l / TPR, p = l % TPR;
  T m[CPT];
#pragma unroll
  for (int u = 0; u < CPT; ++u) m[u] = M[o * LD + p * CPT + u];
  for (int q = 0; q < nrhs; ++q) {
    T acc = T(0);
#pragma unroll
    for (int u = 0; u < CPT; ++u) acc += m[u] * v[q * NMAX + p * CPT + u];
    acc = lane_group_sum_dpp<TPR>(acc);
    if (p == 0) put(q, o, acc);
  }
}

// The right-hand side of a position: b at its stage plus (after the first pass) the updates
// carried from earlier passes, zero padded, by one wave.
template <typename T, int NMAX, bool FIRST>
__device__ inline void tree_load_rhs(const FactorPassArgs& a, size_t s, const double* b, size_t len,
                                     int q, bool with_b, T* V) {
  const int n = a.n, nr = a.nrhs;
  const double* bj = b + (size_t)(a.N - (q << a.shift)) * n;
  const size_t vo = (s * a.stride + q) * nr * n;
  for (int idx = threadIdx.x & 63; idx < nr * NMAX; idx += 64) {
    const int k = idx / NMAX, i = idx % NMAX;
    T v = T(0);
    if (i < n) {
      if (with_b) v = static_cast<T>(bj[(size_t)k * len + i]);
      if constexpr (!FIRST) {
        v += reinterpret_cast<const T*>(a.vaccR_in)[vo + k * n + i];
        v += reinterpret_cast<const T*>(a.vaccL_in)[vo + k * n + i];
      }
    }
    V[idx] = v;
  }
}

template <typename T, int NMAX, bool FIRST, bool FINAL, bool FWD, bool FULL>
__device__ __attribute__((always_inline)) inline void tree_pass_body(const FactorPassArgs& a_in,
                                                                    unsigned bx) {
  FactorPassArgs a = a_in;
  if constexpr (FULL) a.n = NMAX;
  typedef typename Mfma<T>::acc_t acc_t;
  typedef AccAt<T, NMAX> At;
  constexpr int AV = At::AV, LD = Lay<NMAX>::LD, SZ = Lay<NMAX>::SZ;
  constexpr int NP = NMAX * (NMAX + 1) / 2, LG = tree_leaf_group<NMAX>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* const smem = reinterpret_cast<T*>(smem_raw);
  const int W = tree_window(a.Tw, a.mk);
  const int VS = FWD ? a.nrhs * NMAX : 0;
  T* const blk = smem + (W + 1) * VS;  // hl <= W - 1
  auto V = [&](int p) { return smem + p * VS; };
  auto A = [&](int p) { return blk + (p - 1) * SZ; };
  auto C = [&](int p) { return blk + (W - 1 + p) * SZ; };
  T* const AX = blk + (2 * W - 1) * SZ;
  T* const CX = AX + SZ;
  const int n = a.n, N = a.N, nr = a.nrhs;
  const size_t nn = (size_t)n * n;
  const size_t s = bx / a.windows;
  const int w = (int)(bx - s * a.windows);
  const int lo = w << a.Tw;
  const int hl = min((1 << a.Tw) - 1, a.mk - lo);  // local positions 1 .. hl
  const bool has_left = lo >= 1;
  const bool rb_is_x = lo + (1 << a.Tw) > a.mk;
  const int NW = blockDim.x >> 6, wv = wave_id(), lane = threadIdx.x & 63;
  // the waves that keep the boundaries' updates
  const int wL = NW - 1, wR = NW > 1 ? NW - 2 : 0;
  const int sys = (int)(s / a.Ssys), sc = (int)(s - (size_t)sys * a.Ssys);
  const unsigned long long chain_row0 =
      (unsigned long long)sys * ((unsigned long long)a.Ssys * N + 1) * n +
      (unsigned long long)sc * N * n;
  const size_t len = ((size_t)a.Ssys * N + 1) * n;
  const double* bch = FWD ? a.b + (size_t)sys * a.vsys + (size_t)sc * N * n : nullptr;

  // ---- loads: wave i brings position 2 i + 1 (its block, its coupling, its predecessor's)
  // and the block of position 2 i + 2, which is all that phase 1 of level 1 needs for
  // position 2 i + 1.  The last position's coupling is its own wave's too when it is even,
  // and wave 0 brings the left boundary's.
  acc_t accL = {0, 0, 0, 0}, accR = {0, 0, 0, 0};
  if (!FIRST && has_left && wv == wL) {
    const size_t o = (s * a.stride + lo) * nn;
#pragma unroll
    for (int v = 0; v < AV; ++v) {
      const int r = At::row(v), c = At::col();
      if (r < n && c < n)
        accL[v] = reinterpret_cast<const T*>(a.accR_in)[o + r * n + c] +
                  reinterpret_cast<const T*>(a.accL_in)[o + r * n + c];
    }
  }
  for (int i = wv; i == wv || 2 * i + 1 <= hl; i += NW) {
    const int j = 2 * i + 1;
    const bool has = j <= hl, has2 = j + 1 <= hl, lastc = j + 1 == hl;
    const bool c0 = i > 0 ? has : has_left;
    TreeLoad<T, NMAX, FIRST> ld, le;
    if (c0) ld.coup(0, a, s, lo + j - 1);
    if (has) {
      ld.coup(1, a, s, lo + j);
      ld.diag(0, a, s, lo + j);
      if (has2) ld.diag(1, a, s, lo + j + 1);
      if (lastc) le.coup(0, a, s, lo + j + 1);
      if constexpr (FWD) {
        tree_load_rhs<T, NMAX, FIRST>(a, s, bch, len, lo + j, true, V(j));
        if (has2) tree_load_rhs<T, NMAX, FIRST>(a, s, bch, len, lo + j + 1, true, V(j + 1));
      }
    }
    if (c0) ld.put_coup(0, C(j - 1));
    if (has) {
      ld.put_coup(1, C(j));
      ld.put_diag(0, A(j), n);
      if (has2) ld.put_diag(1, A(j + 1), n);
      if (lastc) le.put_coup(0, C(j + 1));
    }
  }
  if constexpr (FWD) {
    if (wv == wL && has_left) tree_load_rhs<T, NMAX, FIRST>(a, s, bch, len, lo, false, V(0));
    if (wv == wR)
      for (int idx = lane; idx < VS; idx += 64) V(W)[idx] = T(0);
  }
  if constexpr (FINAL) {  // x_1: D of stage 0 plus the earlier passes' updates, and C
    if (wv == wR) {
      const double* D0 = a.D + s * N * nn;
#pragma unroll
      for (int v = 0; v < AV; ++v) {
        const int r = At::row(v), c = At::col();
        T t = r == c ? T(1) : T(0);
        if (r < n && c < n) {
          t = static_cast<T>(r >= c ? D0[r * n + c] : D0[c * n + r]);
          for (int p = 0; p < a.pass; ++p)
            t += reinterpret_cast<const T*>(a.accX)[(s * a.npass + p) * nn + r * n + c];
        }
        accR[v] = t;
        CX[r * LD + c] =
            r < n && c < n ? static_cast<T>(a.C[s * nn + r * n + c]) : T(0);
      }
    }
  }
  // packed entries lane, lane + 64, .. of an inverse: their LDS places
  constexpr int PR = (NP + 63) / 64;
  int pat[PR];
#pragma unroll
  for (int k = 0; k < PR; ++k) {
    const int p = min(lane + 64 * k, NP - 1);
    int r = (int)((__fsqrt_rn(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);
    r = (r * (r + 1) / 2 > p) ? r - 1 : r;
    r = ((r + 1) * (r + 2) / 2 <= p) ? r + 1 : r;
    pat[k] = r * LD + (p - r * (r + 1) / 2);
  }
  auto store_packed = [&](T* __restrict__ dst, const T* src) {
#pragma unroll
    for (int k = 0; k < PR; ++k) {
      const int p = lane + 64 * k;
      if (p < n * (n + 1) / 2) dst[p] = src[pat[k]];
    }
  };
  auto store_acc = [&](T* __restrict__ dst, const acc_t& g) {
#pragma unroll
    for (int v = 0; v < AV; ++v) {
      const int r = At::row(v), c = At::col();
      if (r < n && c < n) dst[r * n + c] = g[v];
    }
  };
  T* const Linv = reinterpret_cast<T*>(a.Linv) + s * N * nn;
  T* const Gl = reinterpret_cast<T*>(a.Gl) + s * g_chain_blocks(N) * nn;
  T* const Gr = reinterpret_cast<T*>(a.Gr) + s * g_chain_blocks(N) * nn;
  T* const ych = FWD ? reinterpret_cast<T*>(a.y) + s * N * nr * n : nullptr;

  auto report = [&](int j, int fail) {  // a failing pivot of local position j
    const int jc = (lo + j) << a.shift;
    atomicMin(a.info, chain_row0 + (unsigned long long)a.permpos[jc - 1] * n + fail + 1);
  };
  if constexpr (LG > 1) __syncthreads();  // a leaf's wave factors other waves' positions
  for (int t = 0; (1 << t) <= hl; ++t) {
    const int half = 1 << t;
    // phase 1: the positions of this level
    if constexpr (LG > 1) {
      for (int i = wv * LG; ((2 * i + 1) << t) <= hl; i += NW * LG) {
        // lanes past the level's last position repeat it (the same values stored again)
        const int ii = i + lane / (64 / LG);
        const bool mine = ((2 * ii + 1) << t) <= hl;
        const int j = mine ? (2 * ii + 1) << t : (((hl >> t) - 1) | 1) << t;
        wave_lds_fence();
        const int fail = wave_potrf_inv_leaf<T, NMAX, RowMajor<LD>, LG>(A(j));
        if (mine && lane % (64 / LG) == 0 && fail >= 0 && fail < n) report(j, fail);
      }
      __syncthreads();
    }
    for (int i = wv; ((2 * i + 1) << t) <= hl; i += NW) {
      const int j = (2 * i + 1) << t, l = j - half;
      const bool left = l > 0 || has_left;
      const size_t at = (size_t)(((lo + j) << a.shift) - 1);  // chain position, from 0
      T *Aj = A(j), *Cj = C(j), *Cl = C(l);
      if constexpr (LG == 1) {
        wave_lds_fence();
        const int fail = wave_potrf_inv_leaf<T, NMAX, RowMajor<LD>>(Aj);
        if (fail >= 0 && fail < n && lane == 0) report(j, fail);
        wave_lds_fence();
      }
      const acc_t gr = mfma_tile_nt<T, NMAX, false>(Cj, Aj);
      acc_t gl = {0, 0, 0, 0};
      if (left) gl = mfma_tile_nt<T, NMAX, true>(Cl, Aj);
      if constexpr (FWD) {
        T* yj = ych + at * nr * n;
        T* Vj = V(j);
        // each right-hand side is read before its place takes y
        wave_matvec<T, NMAX>(Aj, Vj, nr, [&](int q, int o, T v) {
          Vj[q * NMAX + o] = v;
          if (o < n) yj[o * nr + q] = v;
        });
      }
      wave_lds_fence();
      mfma_tile_store<T, NMAX, false>(Cj, gr, T(1));
      if (left) mfma_tile_store<T, NMAX, false>(Cl, gl, T(1));
      store_acc(Gr + at * nn, gr);
      if (left) store_acc(Gl + at * nn, gl);
      store_packed(Linv + at * nn, Aj);
    }
    __syncthreads();
    // phase 2: the positions that stay
    for (int i = wv + 1; (i << (t + 1)) <= hl; i += NW) {
      const int p = i << (t + 1), j1 = p - half, j2 = p + half;
      const bool right = j2 <= hl;
      acc_t u = mfma_tile_nt<T, NMAX, false>(C(j1), C(j1));
      acc_t f = {0, 0, 0, 0};
      if (right) {
        u = mfma_tile_nt<T, NMAX, false>(C(p), C(p), u);
        f = mfma_tile_nt<T, NMAX, false>(C(j2), C(p));
      }
      if constexpr (FWD) {
        T* Vp = V(p);
        wave_matvec<T, NMAX>(C(j1), V(j1), nr, [&](int q, int o, T v) { Vp[q * NMAX + o] -= v; });
        if (right)
          wave_matvec<T, NMAX>(C(p), V(j2), nr, [&](int q, int o, T v) { Vp[q * NMAX + o] -= v; });
      }
      wave_lds_fence();
      mfma_tile_store<T, NMAX, true>(A(p), u, T(-1));
      if (right) mfma_tile_store<T, NMAX, false>(C(p), f, T(-1));
    }
    if (wv == wL && has_left) {  // the left boundary, whose right neighbour half is eliminated
      const acc_t u = mfma_tile_nt<T, NMAX, false>(C(0), C(0));
      const acc_t f = mfma_tile_nt<T, NMAX, false>(C(half), C(0));
#pragma unroll
      for (int v = 0; v < AV; ++v) accL[v] -= u[v];
      if constexpr (FWD)
        wave_matvec<T, NMAX>(C(0), V(half), nr,
                             [&](int q, int o, T v) { V(0)[q * NMAX + o] -= v; });
      wave_lds_fence();
      mfma_tile_store<T, NMAX, false>(C(0), f, T(-1));
    }
    if (wv == wR && ((hl >> t) & 1)) {  // the right boundary (or X): the level's last position
      const int j1 = (hl >> t) << t;
      const acc_t u = mfma_tile_nt<T, NMAX, false>(C(j1), C(j1));
#pragma unroll
      for (int v = 0; v < AV; ++v) accR[v] -= u[v];
      if constexpr (FWD)
        wave_matvec<T, NMAX>(C(j1), V(j1), nr,
                             [&](int q, int o, T v) { V(W)[q * NMAX + o] -= v; });
    }
    __syncthreads();
  }

  if (LG == 1 && hl <= 0) __syncthreads();  // no position: the left boundary's coupling is wave 0's
  const size_t vs = (size_t)nr * n;
  auto store_vec = [&](T* __restrict__ dst, const T* src) {
    for (int idx = lane; idx < nr * n; idx += 64) dst[idx] = src[(idx / n) * NMAX + idx % n];
  };
  if constexpr (!FINAL) {
    const size_t base = s * a.stride;
    wave_lds_fence();
    if (wv == wL && has_left) {
      store_acc(reinterpret_cast<T*>(a.accL_out) + (base + w) * nn, accL);
      T* fo = reinterpret_cast<T*>(a.fill_out) + (base + w) * nn;
#pragma unroll
      for (int v = 0; v < AV; ++v) {
        const int r = At::row(v), c = At::col();
        if (r < n && c < n) fo[r * n + c] = C(0)[r * LD + c];
      }
      if constexpr (FWD) store_vec(reinterpret_cast<T*>(a.vaccL_out) + (base + w) * vs, V(0));
    }
    if (wv == wR) {
      store_acc(rb_is_x ? reinterpret_cast<T*>(a.accX) + (s * a.npass + a.pass) * nn
                        : reinterpret_cast<T*>(a.accR_out) + (base + w + 1) * nn,
                accR);
      if constexpr (FWD)
        store_vec(rb_is_x ? reinterpret_cast<T*>(a.vaccX) + (s * a.npass + a.pass) * vs
                          : reinterpret_cast<T*>(a.vaccR_out) + (base + w + 1) * vs,
                  V(W));
    }
  } else {
    // ---- x_1 (Algorithm 1, the tail steps for the terminal block), on the wave that holds
    // its updates
    if (wv != wR) return;
#pragma unroll
    for (int v = 0; v < AV; ++v) AX[At::row(v) * LD + At::col()] = accR[v];
    wave_lds_fence();
    const int fail = wave_potrf_inv_leaf<T, NMAX, RowMajor<LD>>(AX);
    if (fail >= 0 && fail < n && lane == 0)
      atomicMin(a.info, chain_row0 + (unsigned long long)a.permpos[N - 1] * n + fail + 1);
    wave_lds_fence();
    const acc_t f = mfma_tile_nt<T, NMAX, false>(CX, AX);  // F = C L_X^{-T}
    wave_lds_fence();
    // F in FP64 for U = F F^T (its place: the first blocks of the window, done with; two
    // FP32 blocks hold one of FP64)
    double* Fd = reinterpret_cast<double*>(blk);
#pragma unroll
    for (int v = 0; v < AV; ++v) Fd[At::row(v) * LD + At::col()] = static_cast<double>(f[v]);
    store_acc(reinterpret_cast<T*>(a.F) + s * nn, f);
    store_packed(Linv + (size_t)(N - 1) * nn, AX);
    wave_lds_fence();
    const typename Mfma<double>::acc_t u = mfma_tile_nt<double, NMAX, false>(Fd, Fd);
    double* U = a.U + s * nn;
#pragma unroll
    for (int v = 0; v < AV; ++v) {
      const int r = AccAt<double, NMAX>::row(v), c = At::col();
      if (r < n && c < n) U[r * n + c] = u[v];
    }
    if constexpr (FWD) {
      // the terminal forward step: b at stage 0 plus the X updates of every pass (same order
      // as its block), y_X = L_X^{-1} of it, w_s = F_s y_X in FP64
      T* Vx = V(W);
      for (int idx = lane; idx < VS; idx += 64) {
        const int q = idx / NMAX, i = idx % NMAX;
        T v = T(0);
        if (i < n) {
          v = static_cast<T>(bch[(size_t)q * len + i]);
          for (int p = 0; p < a.pass; ++p)
            v += reinterpret_cast<const T*>(a.vaccX)[(s * a.npass + p) * vs + q * n + i];
          v += Vx[idx];
        }
        Vx[idx] = v;
      }
      wave_lds_fence();
      T* yx = ych + (size_t)(N - 1) * vs;
      wave_matvec<T, NMAX>(AX, Vx, nr, [&](int q, int o, T v) {
        Vx[q * NMAX + o] = v;
        if (o < n) yx[o * nr + q] = v;
      });
      wave_lds_fence();
      constexpr int TPR = 64 / NMAX, CPT = NMAX / TPR;
      const int o = lane / TPR, p = lane % TPR;
      for (int q = 0; q < nr; ++q) {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < CPT; ++k)
          acc += Fd[o * LD + p * CPT + k] * static_cast<double>(Vx[q * NMAX + p * CPT + k]);
        acc = lane_group_sum_dpp<TPR>(acc);
        if (p == 0 && o < n) a.w[(s * nr + q) * n + o] = acc;
      }
    }
  }
}

template <typename T, int NMAX, bool FIRST, bool FINAL, bool FWD, bool FULL>
__global__ void __launch_bounds__(64 * kTreeWaves) tree_pass_kernel(FactorPassArgs a) {
  tree_pass_body<T, NMAX, FIRST, FINAL, FWD, FULL>(a, blockIdx.x);
}

// one launch over the systems of a ragged batch (see multi.h)
template <typename T, int NMAX, bool FIRST, bool FINAL, bool FWD, bool FULL>
__global__ void __launch_bounds__(64 * kTreeWaves) tree_pass_multi(
    const MultiItem<FactorPassArgs>* items, int nitems, Reloc r) {
  const MultiItem<FactorPassArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  FactorPassArgs a = it.a;
  a.D = rel(r.D, a.D);
  a.E = rel(r.E, a.E);
  a.C = rel(r.C, a.C);
  a.b = FWD ? rel(r.b, a.b) : nullptr;
  tree_pass_body<T, NMAX, FIRST, FINAL, FWD, FULL>(a, multi_local(it).x);
}

template <typename K>
void allow_lds(K kernel) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

// f(T, NMAX, FIRST, FINAL, FWD, FULL as std::integral_constant) for the run-time values
template <typename F>
void tree_dispatch(int nmax, bool first, bool final, bool fwd, bool full, F&& f) {
  auto b = [](bool v, auto&& g) {
    if (v)
      g(std::true_type{});
    else
      g(std::false_type{});
  };
  b(nmax <= 8, [&](auto small) {
    b(first, [&](auto fi) {
      b(final, [&](auto fn) {
        b(fwd, [&](auto fw) {
          b(full, [&](auto fu) {
            f(std::integral_constant<int, decltype(small)::value ? 8 : 16>{}, fi, fn, fw, fu);
          });
        });
      });
    });
  });
}

}  // namespace

size_t tree_pass_lds(bool fp64, int nmax, int Tw, int mk, int nrhs_fused, bool final) {
  const int W = tree_window(Tw, mk);
  if (fp64)
    return nmax <= 8 ? tree_lds_bytes<double, 8>(W, nrhs_fused, final)
                     : tree_lds_bytes<double, 16>(W, nrhs_fused, final);
  return nmax <= 8 ? tree_lds_bytes<float, 8>(W, nrhs_fused, final)
                   : tree_lds_bytes<float, 16>(W, nrhs_fused, final);
}

template <typename T>
void launch_tree_pass(const FactorPassArgs& a, int nmax, hipStream_t st) {
  const size_t lds = 
      tree_pass_lds(sizeof(T) == 8, nmax, a.Tw, a.mk, a.b ? a.nrhs : 0, a.is_final);
  const dim3 grid((unsigned)a.S * (unsigned)a.windows);
  const dim3 block(tree_threads(tree_window(a.Tw, a.mk), nmax, grid.x));
  tree_dispatch(nmax, a.pass == 0, a.is_final, a.b != nullptr, a.n == nmax,
                [&](auto nm, auto fi, auto fn, auto fw, auto fu) {
                  auto* k = &tree_pass_kernel<T, decltype(nm)::value, decltype(fi)::value,
                                              decltype(fn)::value, decltype(fw)::value,
                                              decltype(fu)::value>;
                  static const bool set = (allow_lds(k), true);
                  (void)set;
                  hipLaunchKernelGGL(k, grid, block, lds, st, a);
                });
}
template void launch_tree_pass<double>(const FactorPassArgs&, int, hipStream_t);
template void launch_tree_pass<float>(const FactorPassArgs&, int, hipStream_t);

template <typename T>
void launch_tree_pass_multi(const MultiItem<FactorPassArgs>* items, int nitems, unsigned blocks,
                            int nmax, bool first, bool final, bool fwd, bool full, int W,
                            size_t lds, const Reloc& r, hipStream_t st) {
  const unsigned threads = tree_threads(W, nmax, blocks);
  tree_dispatch(nmax, first, final, fwd, full, [&](auto nm, auto fi, auto fn, auto fw, auto fu) {
    auto* k = &tree_pass_multi<T, decltype(nm)::value, decltype(fi)::value, decltype(fn)::value,
                               decltype(fw)::value, decltype(fu)::value>;
    static const bool set = (allow_lds(k), true);
    (void)set;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(threads), lds, st, items, nitems, r);
  });
}
template void launch_tree_pass_multi<double>(const MultiItem<FactorPassArgs>*, int, unsigned, int,
                                             bool, bool, bool, bool, int, size_t,
                                             const Reloc&, hipStream_t);
template void launch_tree_pass_multi<float>(const MultiItem<FactorPassArgs>*, int, unsigned, int,
                                            bool, bool, bool, bool, int, size_t,
                                            const Reloc&, hipStream_t);

}  // namespace bmpc
