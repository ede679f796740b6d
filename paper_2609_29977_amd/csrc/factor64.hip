// Factor passes for block sizes 33..64 (gfx950).
//
// The same elimination as factor.hip (the tail factorization of Algorithm 1 in the
// Gamma level order; Section IV-B in block form), for blocks of 3 x 3 or 4 x 4 tiles of
// 16, which are 19 or 33 KB each in FP64 LDS: too large for the depth-first window walk,
// whose live set holds 2 Tw + 3 blocks.  Here every pass is one level (window depth 1): window
// w of a pass holds the pass-local position q = 2w + 1 with its left neighbour lo = 2w and its
// right neighbour 2w + 2 (X beyond the reduced chain).  The live set is three LDS
// blocks -- A_q and the two couplings K[q+1, q] and K[q, lo] -- and the Schur updates
// of the two neighbours (A_r -= G_r G_r^T, A_l -= G_l G_l^T, lower tiles, and the fill
// -G_r G_l^T) stay in the MFMA accumulators of the waves, one 16 x 16 output tile each,
// until they are written to the reduced-chain buffers that the next pass reads (the
// accumulator scheme of factor.hip: a boundary node's updates from earlier passes ride
// in its left accumulator).  The last pass (reduced chain of at most one position) also
// eliminates x_1 and forms F = C L_X^{-T} and U = F F^T in FP64.
//
// A position's time is the chain of its diagonal tiles (block_chol) plus the latency of its
// loads and stores, all of which are issued together, the couplings' before the
// factorization and waited for after it.  Every load and store follows the rows of the block
// in memory (E^T is transposed on the way into LDS).  n <= 48 runs on nine waves and 57 KB of
// LDS, two workgroups per CU.
// Against padding to 64 with 32 x 32 leaves on one wave, E read by columns and the stores
// divided by n: n = 48, S = N = 64 in FP64, first pass 256 -> 115 us, the five others 335 ->
// 180 us, one position alone 33 -> 20 us; in FP32 175 -> 83 and 256 ->
// 152. n = 64: 286 -> 227 and 409 -> 317 us in FP64.
#include "bmpc_internal.h"
#include "blockchol.h"

namespace bmpc {

namespace {

template <int NT>
struct Big {
  static constexpr int NB = 16 * NT;
  static constexpr int LD = NB + 1;
  static constexpr int SZ = NB * LD;
  static constexpr int W = NT * NT;  // one wave per 16 x 16 output tile
  static constexpr int TH = 64 * W;
  static constexpr int EL = NB * NB / TH;  // entries of a block per thread
  static_assert(EL * TH == NB * NB, "the block divides among the threads");
};

// A block's entries of this thread (e = threadIdx.x + u TH, row e / NB), zero beyond n.
template <typename S, int NT>
struct BigBlock {
  typedef Big<NT> G;
  S v[G::EL];
  __device__ void load(const S* __restrict__ src, int n, bool lower) {
#pragma unroll
    for (int u = 0; u < G::EL; ++u) {
      const int e = threadIdx.x + u * G::TH, r = e / G::NB, c = e % G::NB;
      v[u] = r < n && c < n && (!lower || c <= r) ? src[r * n + c] : S(0);
    }
  }
  template <typename T>
  __device__ void put(T* dst, bool trans) const {
#pragma unroll
    for (int u = 0; u < G::EL; ++u) {
      const int e = threadIdx.x + u * G::TH, r = e / G::NB, c = e % G::NB;
      dst[trans ? c * G::LD + r : r * G::LD + c] = static_cast<T>(v[u]);
    }
  }
};

// acc + tile (ti, tj) of X Y^T (TRANS: X^T Y^T) for slabs 0..last of 16.
template <typename T, int NT, bool TRANS>
__device__ inline typename Mfma<T>::acc_t big_tile(const T* X, const T* Y, int ti, int tj,
                                                   int last, typename Mfma<T>::acc_t acc = {}) {
  constexpr int LD = Big<NT>::LD;
  const int l = threadIdx.x & 63, g = l >> 4, i = l & 15;
  const int r = 16 * ti + i, c = 16 * tj + i;
#pragma unroll
  for (int m = 0; m < NT; ++m) {
    if (m > last) break;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 16 * m + 4 * g + s;
      acc = Mfma<T>::mma(TRANS ? X[k * LD + r] : X[r * LD + k], Y[c * LD + k], acc);
    }
  }
  return acc;
}
template <typename T, int NT>
__device__ inline void big_tile_put(T* X, const typename Mfma<T>::acc_t& t, int ti, int tj) {
  const int l = threadIdx.x & 63, i = l & 15;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    X[(16 * ti + Mfma<T>::row(l, v)) * Big<NT>::LD + 16 * tj + i] = t[v];
}
// This wave's tile of an accumulator block in global memory (n x n, the rest skipped).
template <typename T>
__device__ inline typename Mfma<T>::acc_t big_tile_read(const T* __restrict__ src, int ti, int tj,
                                                        int n) {
  const int l = threadIdx.x & 63, c = 16 * tj + (l & 15);
  typename Mfma<T>::acc_t t;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = 16 * ti + Mfma<T>::row(l, v);
    t[v] = r < n && c < n ? src[r * n + c] : T(0);
  }
  return t;
}
template <typename T>
__device__ inline void big_tile_write(T* __restrict__ dst, const typename Mfma<T>::acc_t& t,
                                      int ti, int tj, int n) {
  const int l = threadIdx.x & 63, c = 16 * tj + (l & 15);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = 16 * ti + Mfma<T>::row(l, v);
    if (r < n && c < n) dst[r * n + c] = t[v];
  }
}
// LDS block to global memory, rows of n; PACKED: its lower triangle packed by rows.
template <typename T, int NT, bool PACKED>
__device__ inline void big_store(T* __restrict__ dst, const T* src, int n) {
  typedef Big<NT> G;
#pragma unroll
  for (int u = 0; u < G::EL; ++u) {
    const int e = threadIdx.x + u * G::TH, r = e / G::NB, c = e % G::NB;
    const T v = src[r * G::LD + c];
    if (r < n && c < (PACKED ? r + 1 : n)) dst[PACKED ? r * (r + 1) / 2 + c : r * n + c] = v;
  }
}

template <typename T, int NT, bool FIRST, bool FINAL>
__global__ void __launch_bounds__(Big<NT>::TH) factor64_pass_kernel(FactorPassArgs a) {
  typedef typename Mfma<T>::acc_t acc_t;
  typedef Big<NT> G;
  extern __shared__ __align__(16) unsigned char smem64[];
  T* Aq = reinterpret_cast<T*>(smem64);
  T* Cr = Aq + G::SZ;  // K[rb, q], then G_r
  T* Cl = Cr + G::SZ;  // K[q, lo], then G_l
  const int n = a.n, N = a.N;
  const size_t nn = (size_t)n * n;
  const int s = blockIdx.x / a.windows;
  const int w = blockIdx.x - s * a.windows;
  const int lo = 2 * w, q = lo + 1;
  const bool has_q = q <= a.mk, has_left = lo >= 1;
  const bool rb_is_x = lo + 2 > a.mk;
  const int j = q << a.shift;  // chain position of q
  const int wv = wave_id(), ti = wv / NT, tj = wv % NT;
  T* Linv = reinterpret_cast<T*>(a.Linv) + (size_t)s * N * nn;
  T* Gl = reinterpret_cast<T*>(a.Gl) + (size_t)s * g_chain_blocks(N) * nn;
  T* Gr = reinterpret_cast<T*>(a.Gr) + (size_t)s * g_chain_blocks(N) * nn;
  const int sys = s / a.Ssys;
  const unsigned long long chain_row0 =
      (unsigned long long)sys * ((unsigned long long)a.Ssys * N + 1) * n +
      (unsigned long long)(s - sys * a.Ssys) * N * n;
  const size_t base = (size_t)s * a.stride;
  const T* accR_in = reinterpret_cast<const T*>(a.accR_in);
  const T* accL_in = reinterpret_cast<const T*>(a.accL_in);
  const T* fill_in = reinterpret_cast<const T*>(a.fill_in);
  typedef typename std::conditional<FIRST, double, T>::type CT;

  const acc_t z = {0, 0, 0, 0};
  acc_t AL = z, AR = z, FL = z;
  BigBlock<double, NT> d;
  BigBlock<T, NT> ar, al;
  BigBlock<CT, NT> cr, cl;
  if (has_q) {
    d.load(a.D + ((size_t)s * N + (N - j)) * nn, n, true);
    if constexpr (!FIRST) {
      ar.load(accR_in + (base + q) * nn, n, true);
      al.load(accL_in + (base + q) * nn, n, true);
    }
    if constexpr (FIRST)
      cr.load(a.E + ((size_t)s * (N - 1) + (N - 1 - q)) * nn, n, false);
    else
      cr.load(fill_in + (base + q) * nn, n, false);
  }
  if (has_left) {
    if constexpr (FIRST)
      cl.load(a.E + ((size_t)s * (N - 1) + (N - 1 - lo)) * nn, n, false);
    else
      cl.load(fill_in + (base + lo) * nn, n, false);
    if (!FIRST && tj <= ti)
      AL = big_tile_read<T>(accR_in + (base + lo) * nn, ti, tj, n) +
           big_tile_read<T>(accL_in + (base + lo) * nn, ti, tj, n);
  }
  if (has_q) {
#pragma unroll
    for (int u = 0; u < G::EL; ++u) {
      const int e = threadIdx.x + u * G::TH, r = e / G::NB, c = e % G::NB;
      T v = static_cast<T>(d.v[u]);
      if constexpr (!FIRST) v = (v + ar.v[u]) + al.v[u];
      Aq[r * G::LD + c] = r == c && r >= n ? T(1) : v;  // identity padding
    }
    __syncthreads();
    const int fail = block_chol<T, NT, G::LD, G::W, true>(Aq, nullptr);
    if (threadIdx.x == 0 && fail >= 0 && fail < n)
      atomicMin(a.info, chain_row0 + (unsigned long long)a.permpos[j - 1] * n + fail + 1);
    cr.put(Cr, FIRST);  // E is read by its rows: K[q+1, q] = E^T
  }
  if (has_left) cl.put(Cl, FIRST);
  __syncthreads();
  if (has_q) {
    const acc_t gr = big_tile<T, NT, false>(Cr, Aq, ti, tj, tj);  // G_r = K[rb,q] L^{-T}
    acc_t gl = z;
    if (has_left) gl = big_tile<T, NT, true>(Cl, Aq, ti, tj, tj);  // G_l = K[q,lo]^T L^{-T}
    __syncthreads();
    big_tile_put<T, NT>(Cr, gr, ti, tj);
    if (has_left) big_tile_put<T, NT>(Cl, gl, ti, tj);
    __syncthreads();
    big_store<T, NT, true>(Linv + (size_t)(j - 1) * nn, Aq, n);
    big_store<T, NT, false>(Gr + (size_t)(j - 1) * nn, Cr, n);
    if (has_left) big_store<T, NT, false>(Gl + (size_t)(j - 1) * nn, Cl, n);
    if (tj <= ti) {
      AR = -big_tile<T, NT, false>(Cr, Cr, ti, tj, NT - 1);
      if (has_left) AL = AL - big_tile<T, NT, false>(Cl, Cl, ti, tj, NT - 1);
    }
    if (has_left) FL = -big_tile<T, NT, false>(Cr, Cl, ti, tj, NT - 1);
  } else if (has_left) {  // no position: lo keeps its coupling to X
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      FL[v] = Cl[(16 * ti + Mfma<T>::row(l, v)) * G::LD + 16 * tj + (l & 15)];
  }

  if constexpr (!FINAL) {
    if (has_left) {
      if (tj <= ti)
        big_tile_write<T>(reinterpret_cast<T*>(a.accL_out) + (base + w) * nn, AL, ti, tj, n);
      big_tile_write<T>(reinterpret_cast<T*>(a.fill_out) + (base + w) * nn, FL, ti, tj, n);
    }
    if (tj <= ti)
      big_tile_write<T>(rb_is_x ? reinterpret_cast<T*>(a.accX) + ((size_t)s * a.npass + a.pass) * nn
                                : reinterpret_cast<T*>(a.accR_out) + (base + w + 1) * nn,
                        AR, ti, tj, n);
  } else {
    // ---- last pass: x_1 step (the coupling solve and local Schur update) ----
    BigBlock<double, NT> dx, cx;
    dx.load(a.D + (size_t)s * N * nn, n, true);
    cx.load(a.C + (size_t)s * nn, n, false);
    T v[G::EL];
#pragma unroll
    for (int u = 0; u < G::EL; ++u) v[u] = static_cast<T>(dx.v[u]);
    for (int p = 0; p < a.pass; ++p) {
      BigBlock<T, NT> x;
      x.load(reinterpret_cast<const T*>(a.accX) + ((size_t)s * a.npass + p) * nn, n, true);
#pragma unroll
      for (int u = 0; u < G::EL; ++u) v[u] += x.v[u];
    }
    __syncthreads();  // the position's blocks are stored; Aq and Cr are free
#pragma unroll
    for (int u = 0; u < G::EL; ++u) {
      const int e = threadIdx.x + u * G::TH, r = e / G::NB, c = e % G::NB;
      Aq[r * G::LD + c] = r == c && r >= n ? T(1) : v[u];
    }
    cx.put(Cr, false);
    __syncthreads();
    if (tj <= ti) {
      const int l = threadIdx.x & 63;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        Aq[(16 * ti + Mfma<T>::row(l, u)) * G::LD + 16 * tj + (l & 15)] += AR[u];
    }
    __syncthreads();
    const int fail = block_chol<T, NT, G::LD, G::W, true>(Aq, nullptr);
    if (threadIdx.x == 0 && fail >= 0 && fail < n)
      atomicMin(a.info, chain_row0 + (unsigned long long)a.permpos[N - 1] * n + fail + 1);
    big_store<T, NT, true>(Linv + (size_t)(N - 1) * nn, Aq, n);
    const acc_t f = big_tile<T, NT, false>(Cr, Aq, ti, tj, tj);  // F = C L_X^{-T}
    __syncthreads();
    big_tile_put<T, NT>(Cr, f, ti, tj);
    __syncthreads();
    big_store<T, NT, false>(reinterpret_cast<T*>(a.F) + (size_t)s * nn, Cr, n);
    // U = F F^T in FP64 from the stored F
    const int l = threadIdx.x & 63, g = l >> 4, i = l & 15;
    Mfma<double>::acc_t u = {0, 0, 0, 0};
#pragma unroll
    for (int k = 4 * g; k < G::NB; k += 16)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        u = Mfma<double>::mma(static_cast<double>(Cr[(16 * ti + i) * G::LD + k + e]),
                              static_cast<double>(Cr[(16 * tj + i) * G::LD + k + e]), u);
    big_tile_write<double>(a.U + (size_t)s * nn, u, ti, tj, n);
  }
}

template <typename T, int NT, bool FIRST, bool FINAL>
void launch64_k(const FactorPassArgs& a, hipStream_t st) {
  const size_t lds = 3 * (size_t)Big<NT>::SZ * sizeof(T);
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute(
        reinterpret_cast<const void*>(&factor64_pass_kernel<T, NT, FIRST, FINAL>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  hipLaunchKernelGGL((factor64_pass_kernel<T, NT, FIRST, FINAL>),
                     dim3((unsigned)a.S * (unsigned)a.windows), dim3(Big<NT>::TH), lds, st, a);
}
template <typename T, int NT>
void launch64_t(const FactorPassArgs& a, hipStream_t st) {
  const bool first = a.pass == 0;
  if (first && a.is_final)
    launch64_k<T, NT, true, true>(a, st);
  else if (first)
    launch64_k<T, NT, true, false>(a, st);
  else if (a.is_final)
    launch64_k<T, NT, false, true>(a, st);
  else
    launch64_k<T, NT, false, false>(a, st);
}

}  // namespace

size_t factor64_lds_bytes(bool fp64) { return 3 * (size_t)Big<4>::SZ * (fp64 ? 8 : 4); }

template <typename T>
void launch_factor_pass64(const FactorPassArgs& a, hipStream_t st) {
  if (a.n <= 48)
    launch64_t<T, 3>(a, st);
  else
    launch64_t<T, 4>(a, st);
}
template void launch_factor_pass64<double>(const FactorPassArgs&, hipStream_t);
template void launch_factor_pass64<float>(const FactorPassArgs&, hipStream_t);

}  // namespace bmpc
