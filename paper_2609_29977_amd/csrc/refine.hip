// Mixed-precision iterative refinement support (FP64 residual r = b - K x).
//
// The residual is formed from the caller's FP64 blocks exactly as K is defined in
// eq. (root_coupled_matrix) / eq. (tail_block_tridiagonal): row block (s,k) of a
// tail is D_{s,k} x_{s,k} + E_{s,k-1} x_{s,k-1} + E_{s,k}^T x_{s,k+1} (+ C_s^T x_0
// for k = 0); the root row block is R x_0 + sum_s C_s x_{s,0}, with the sum over s
// taken in scenario order.  Infinity norms are maxima taken by a two-stage reduction
// (per-block partial maxima, then one block), so they are deterministic and need no
// atomics.
#include <algorithm>
#include <type_traits>

#include "bmpc_internal.h"
#include "multi.h"
#include "regblock.h"
#include "solve_common.h"

namespace bmpc {

namespace {

// Maximum that propagates NaN (so a NaN residual or correction fails the stop test).
__device__ inline double nan_max(double a, double b) { return (a != a || a > b) ? a : b; }

__device__ inline double wave_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = nan_max(v, __shfl_xor(v, off));
  return v;
}

template <int M>
__device__ inline double pair_sum(const double (&v)[M]) {
  static_assert(M == 1 || M == 4, "one sum or four");
  if constexpr (M == 1) return v[0];
  else return (v[0] + v[2]) + (v[1] + v[3]);
}

// One workgroup walks res_stages consecutive stages of one tail: four waves for blocks of
// more than 16 rows, one wave for smaller ones, whose stages are too little work for four
// (a stage of a 16 x 16 block has one entry per thread there, and both barriers of a step
// are between waves).  The blocks of a stage (the lower triangle of D, all of E) are read
// with coalesced loads (16 bytes where the block is full) into registers two stages
// ahead, together with the x of the next stage and the b of the stage, then staged in
// double-buffered LDS, where the symmetric product with D and the product with E^T read
// them transposed; so each E block leaves HBM once and serves both rows it touches.
// Nothing fetched ahead is used before the step that needs it, so the loads of two stages
// stay in flight while a stage is applied.  Row o of the stage's result is summed by RT =
// RES_T / NMAX threads, each over NMAX / RT columns.
// On 64 systems of 2 K to 65 K stages: n = 8 405 -> 144 us, n = 16 584 -> 471 us
// (n = 32 keeps four waves); S = 256, N = 128, n = 16, one right-hand side 36 -> 31 us.
// Eight stages per walk there: four right-hand sides 58 -> 48 us against sixteen.
constexpr int res_stages(int n) { return n > 16 ? 16 : 8; }
template <int NMAX>
constexpr int res_threads() {
  return NMAX > 16 ? 256 : 64;
}

// LDS of a residual workgroup: Ds[2][NMAX][NMAX+1] (D of stage k in Ds[k & 1]),
// Es[2][NMAX][NMAX+1] (E of stage k in Es[k & 1]; C in Es[1] at stage 0), then
// xs[3][nrhs][NMAX], x0s[nrhs][NMAX], bs[2][nrhs][NMAX], rs[nrhs][NMAX] and
// ws[nrhs][NMAX] (dynamic, sized by nrhs).
template <int NMAX>
inline size_t residual_lds_bytes(int nrhs) {
  return (size_t)(4 * NMAX * (NMAX + 1) + 8 * nrhs * NMAX) * sizeof(double);
}

// The blocks and vectors of one stage k, in registers: D_k (lower triangle), E_k (if
// k + 1 < N), x_{k+1} and b_k.  With FULL (n == NMAX) the blocks are read through a
// buffer resource (entries above the diagonal of D at an out-of-range offset, so they
// read as zero and are not fetched); vector lanes past the data read a clamped
// in-range element.  commit() writes the stage into LDS, zero padded, so the LDS copy
// never holds stale values.
template <int NMAX, bool FULL>
struct StageFetch {
  static constexpr int RES_T = res_threads<NMAX>();
  static constexpr int PER = (NMAX * NMAX + RES_T - 1) / RES_T;
  static constexpr int VPER = (residual_chunk(NMAX) * NMAX + RES_T - 1) / RES_T;
  double d[PER], e[PER], xv[VPER], bv[VPER];

  // Element of the block held in v[u]: with PAIRS, v[2h] and v[2h+1] are two
  // consecutive elements of a row, read by one 16-byte load.
  static constexpr bool PAIRS = FULL && NMAX * NMAX % (2 * RES_T) == 0;
  __device__ static int elem(int u) {
    if constexpr (PAIRS)
      return 2 * ((int)threadIdx.x + (u >> 1) * RES_T) + (u & 1);
    else
      return (int)threadIdx.x + u * RES_T;
  }

  // A block that does not exist (exists = false) is read as zero without a memory
  // access, so every fetch issues the same loads.
  template <bool LOWER>
  __device__ static void block(double (&v)[PER], const double* __restrict__ g, int n,
                               bool exists) {
    if constexpr (PAIRS) {
      // pairs past the diagonal of a lower triangle are not fetched; a pair that starts
      // on the diagonal brings one entry above it, which is never read
      const auto rs = block_rsrc(g, exists ? (unsigned)(NMAX * NMAX) * 8u : 0u);
#pragma unroll
      for (int h = 0; h < PER / 2; ++h) {
        const int el = elem(2 * h);
        const int r = el / NMAX, c = el % NMAX;
        const bool ok = !LOWER || c <= r;
        const auto w = __builtin_amdgcn_raw_buffer_load_b128(rs, ok ? (unsigned)el * 8u
                                                                    : kOutOfRange, 0, 0);
        __builtin_memcpy(&v[2 * h], &w, 16);
      }
    } else if constexpr (FULL) {
      const auto rs = block_rsrc(g, exists ? (unsigned)(NMAX * NMAX) * 8u : 0u);
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int el = threadIdx.x + u * RES_T;
        const int r = el / NMAX, c = el % NMAX;
        const bool ok = el < NMAX * NMAX && (!LOWER || c <= r);
        v[u] = buf_load_f64(rs, ok ? (unsigned)el * 8u : kOutOfRange);
      }
    } else {
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int el = threadIdx.x + u * RES_T;
        const int r = el / NMAX, c = el % NMAX;
        const bool ok = exists && el < NMAX * NMAX && r < n && c < n && (!LOWER || c <= r);
        v[u] = ok ? g[r * n + c] : 0.0;
      }
    }
  }
  __device__ static void put(double* dst, const double (&v)[PER]) {
    constexpr int LD = NMAX + 1;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int el = elem(u);
      if (el < NMAX * NMAX) dst[(el / NMAX) * LD + el % NMAX] = v[u];
    }
  }
  // xk = offset of stage 0 of the chain's vectors (right-hand side 0).  Stages at or
  // past k1 (the end of the chunk) fetch nothing from the blocks and clamped vectors.
  __device__ void issue(const ResidualArgs& a, const double* Dc, const double* Ec, size_t xk,
                        size_t len, int k, int k1) {
    const int n = a.n, N = a.N, nrhs = a.nrhs;
    const size_t nn = (size_t)n * n;
    const int kc = min(k, N - 1);
    block<true>(d, Dc + (size_t)kc * nn, n, k < k1);
    block<false>(e, Ec + (size_t)min(kc, N - 2 < 0 ? 0 : N - 2) * nn, n, k < k1 && k + 1 < N);
#pragma unroll
    for (int u = 0; u < VPER; ++u) {
      if (u > 0 && u * RES_T >= nrhs * NMAX) continue;  // uniform
      const int idx = threadIdx.x + u * RES_T;
      const int q = min(idx / NMAX, nrhs - 1), i = min(idx % NMAX, n - 1);
      const size_t base = xk + (size_t)q * len + i;
      xv[u] = a.x[base + (size_t)min(k + 1, N - 1) * n];
      bv[u] = a.b[base + (size_t)kc * n];
    }
  }
  // stage k into D/E slots, x_{k+1} into xslot, b_k into bslot
  __device__ void commit(const ResidualArgs& a, int k, double* Dsl, double* Esl, double* xslot,
                         double* bslot) const {
    const int n = a.n, N = a.N, nrhs = a.nrhs;
    put(Dsl, d);
    if (k + 1 < N) put(Esl, e);
#pragma unroll
    for (int u = 0; u < VPER; ++u) {
      const int idx = threadIdx.x + u * RES_T;
      if (idx < nrhs * NMAX) {
        const bool ok = idx % NMAX < n;
        xslot[idx] = ok && k + 1 < N ? xv[u] : 0.0;
        bslot[idx] = ok ? bv[u] : 0.0;
      }
    }
  }
};

template <int NMAX, bool FULL>
__device__ __attribute__((always_inline)) inline void residual_body(const ResidualArgs& a,
                                                                    int chunks, unsigned bx) {
  if (a.done && *a.done) return;
  constexpr int LD = NMAX + 1;
  constexpr int BS = NMAX * LD;
  constexpr int RES_T = res_threads<NMAX>();
  constexpr int RT = RES_T / NMAX;  // threads per row
  constexpr int CPT = NMAX / RT;                                 // columns per thread
  static_assert(CPT >= 1 && RT * CPT == NMAX, "row split");
  typedef StageFetch<NMAX, FULL> SF;
  extern __shared__ __align__(16) double res_lds[];
  const int n = a.n, N = a.N, S = a.S, nrhs = a.nrhs;
  const int VS = nrhs * NMAX;          // one vector slot
  double* Ds = res_lds;                // [2][BS]
  double* Es = res_lds + 2 * BS;       // [2][BS]
  double* xs = res_lds + 4 * BS;       // [3][nrhs][NMAX]
  double* x0s = xs + 3 * VS;           // [nrhs][NMAX]
  double* bs = x0s + VS;               // [2][nrhs][NMAX]
  double* rs = bs + 2 * VS;            // [nrhs][NMAX] residual of the current stage
  double* ws = rs + VS;                // [nrhs][NMAX] C_s x_{s,0} (stage 0)
  const size_t nn = (size_t)n * n;
  const size_t len = ((size_t)S * N + 1) * n;
  const int s = bx / chunks;  // chain of the batch
  const int ch = bx - s * chunks;
  const int sys = s / S, sl = s - sys * S;
  const size_t vbase = (size_t)sys * a.vsys;
  const size_t xk = vbase + (size_t)sl * N * n;  // stage 0 of this chain, q = 0
  const int k0 = ch * res_stages(NMAX), k1 = min(N, k0 + res_stages(NMAX));
  const double* Dc = a.D + (size_t)s * N * nn;
  const double* Ec = a.E + (size_t)s * (N > 1 ? N - 1 : 0) * nn;
  const int t = threadIdx.x, orow = t / RT, p = t - orow * RT;
  const int o = orow;
  double kmax = 0.0;  // largest row sum of |K| over this workgroup's rows (knorm_part)
  double rmax[SF::VPER] = {};  // largest |r| of the right-hand sides this thread stores

  // Prologue: stage k0 with x_{k0+1} and b_{k0}, E_{k0-1} (or C_s at k0 = 0), x_{k0-1},
  // x_{k0} and (k0 = 0) the root x, all straight into LDS.
  {
    SF f0;
    double pv[SF::PER];
    f0.issue(a, Dc, Ec, xk, len, k0, k1);
    if (k0 > 0)
      SF::template block<false>(pv, Ec + (size_t)(k0 - 1) * nn, n, true);
    else
      SF::template block<false>(pv, a.C + (size_t)s * nn, n, true);
    for (int idx = t; idx < VS; idx += RES_T) {
      const int q = idx / NMAX, i = idx % NMAX;
      const size_t b0 = xk + (size_t)q * len + i;
      xs[((k0 + 2) % 3) * VS + idx] = (k0 > 0 && i < n) ? a.x[b0 + (size_t)(k0 - 1) * n] : 0.0;
      xs[(k0 % 3) * VS + idx] = i < n ? a.x[b0 + (size_t)k0 * n] : 0.0;
      if (k0 == 0)
        x0s[idx] = i < n ? a.x[vbase + (size_t)q * len + (size_t)S * N * n + i] : 0.0;
    }
    f0.commit(a, k0, Ds + (k0 & 1) * BS, Es + (k0 & 1) * BS, xs + ((k0 + 1) % 3) * VS,
              bs + (k0 & 1) * VS);
    SF::put(Es + ((k0 + 1) & 1) * BS, pv);
  }
  // Two stages in flight: fa holds stage k+1 and fb stage k+2 when step k starts.  Every
  // step issues the same loads (past the chunk they fetch nothing) and stores its
  // residual after the next fetch is issued, so the wait for a stage covers only the
  // loads issued before it.
  SF fa, fb;
  fa.issue(a, Dc, Ec, xk, len, k0 + 1, k1);
  __builtin_amdgcn_sched_barrier(0);  // keep stage k0+1 ahead of k0+2 in the load queue
  fb.issue(a, Dc, Ec, xk, len, k0 + 2, k1);
  auto step = [&](int k, SF& f) {
    __syncthreads();
    if (k < k1) {
      const double* D = Ds + (k & 1) * BS;
      const double* Ek = Es + (k & 1) * BS;
      const double* Ep = Es + ((k + 1) & 1) * BS;  // E of stage k-1 (or C at k = 0)
      const double* xm = xs + ((k + 2) % 3) * VS;
      const double* xkk = xs + (k % 3) * VS;
      const double* xp = xs + ((k + 1) % 3) * VS;
      const double* bk = bs + (k & 1) * VS;
      const bool has_prev = k > 0, has_next = k + 1 < N;
      // This thread's entries of the row, the same for every right-hand side: D, E_{k-1}
      // (or C^T at k = 0), E_k^T.  Blocks up to 16 keep them in registers (four right-hand
      // sides 54 -> 48 us, one as fast); at 32 the registers cost a wave per SIMD (5%).
      auto ld = [&](int u) {
        const int c = p * CPT + u;
        return c <= o ? D[o * LD + c] : D[c * LD + o];
      };
      auto lp = [&](int u) {
        const int c = p * CPT + u;
        return has_prev ? Ep[o * LD + c] : Ep[c * LD + o];
      };
      auto ln = [&](int u) { return has_next ? Ek[(p * CPT + u) * LD + o] : 0.0; };
      constexpr bool KEEP = NMAX <= 16;
      double md[KEEP ? CPT : 1], mp[KEEP ? CPT : 1], mn[KEEP ? CPT : 1];
      if constexpr (KEEP) {
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
          md[u] = ld(u);
          mp[u] = lp(u);
          mn[u] = ln(u);
        }
      }
      const double* xq0 = has_prev ? xm : x0s;
      // A row's partial sums, one per thread and, where four threads have a row of 16, one per
      // column: what 16 threads a row would sum, so the residual rounds no more than theirs
      // (root mean square error of the refined x of 2 chains of 16 with four right-hand sides
      // 4.5e-17 with one sum per thread, 4.0e-17 so), in the same time (within 1 %).
      constexpr int SUMS = KEEP ? CPT : 1;
#pragma unroll 1
      for (int q = 0; q < nrhs; ++q) {
        double acc[SUMS] = {};
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
          const int c = q * NMAX + p * CPT + u;
          double& to = acc[u % SUMS];
          to += (KEEP ? md[KEEP ? u : 0] : ld(u)) * xkk[c];
          to += (KEEP ? mp[KEEP ? u : 0] : lp(u)) * xq0[c];
          if (has_next) to += (KEEP ? mn[KEEP ? u : 0] : ln(u)) * xp[c];
        }
        const double row = lane_group_sum_dpp<RT>(pair_sum(acc));
        if (p == 0) rs[q * NMAX + o] = bk[q * NMAX + o] - row;
        if (!has_prev) {  // k = 0: C x_{s,0} for the root rows
          double accw[SUMS] = {};
#pragma unroll
          for (int u = 0; u < CPT; ++u) {
            const int c = p * CPT + u;
            accw[u % SUMS] += Ep[o * LD + c] * xkk[q * NMAX + c];
          }
          const double roww = lane_group_sum_dpp<RT>(pair_sum(accw));
          if (p == 0) ws[q * NMAX + o] = roww;
        }
      }
      if (a.knorm_part) {
        // row sums of |K| over the same entries (independent of the right-hand side):
        // the largest one goes into the norm; at stage 0 the rows of |C_s| are kept for
        // the root rows (zero padding adds nothing)
        double ab = 0.0, abc = 0.0;
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
          ab += fabs(ld(u));
          ab += fabs(lp(u));
          if (has_next) ab += fabs(ln(u));
          if (!has_prev) abc += fabs(Ep[o * LD + p * CPT + u]);
        }
        ab = lane_group_sum_dpp<RT>(ab);
        kmax = fmax(kmax, ab);
        if (!has_prev) {
          abc = lane_group_sum_dpp<RT>(abc);
          if (p == 0 && orow < n) a.crow[(size_t)s * n + o] = abc;
        }
      }
    }
    __syncthreads();
    f.commit(a, k + 1, Ds + ((k + 1) & 1) * BS, Es + ((k + 1) & 1) * BS,
             xs + ((k + 2) % 3) * VS, bs + ((k + 1) & 1) * VS);
    f.issue(a, Dc, Ec, xk, len, k + 3, k1);
#pragma unroll
    for (int u = 0; u < SF::VPER; ++u) {
      const int idx = t + u * RES_T;
      if (k < k1 && idx < VS && idx % NMAX < n) {
        const int q = idx / NMAX, i = idx % NMAX;
        a.r[xk + (size_t)q * len + (size_t)k * n + i] = rs[idx];
        rmax[u] = nan_max(fabs(rs[idx]), rmax[u]);
        if (k == 0) a.w[((size_t)s * nrhs + q) * n + i] = ws[idx];
      }
    }
  };
  for (int k = k0; k < k1; k += 2) {
    step(k, fa);
    step(k + 1, fb);
  }
#pragma unroll
  for (int u = 0; u < SF::VPER; ++u) {
    const int idx = t + u * RES_T;
    double m = rmax[u];  // over the NMAX lanes of a right-hand side (a group of one wave)
    for (int off = NMAX / 2; off > 0; off >>= 1) m = nan_max(m, __shfl_xor(m, off));
    if (idx < VS && idx % NMAX == 0) a.rpart[(size_t)bx * nrhs + idx / NMAX] = m;
  }
  if (a.knorm_part) {
    __shared__ double wmax[RES_T / 64];
    for (int off = 32; off > 0; off >>= 1) kmax = fmax(kmax, __shfl_xor(kmax, off));
    if ((t & 63) == 0) wmax[t >> 6] = kmax;
    __syncthreads();
    if (t == 0) {
      double m = 0.0;
      for (int i = 0; i < RES_T / 64; ++i) m = fmax(m, wmax[i]);
      a.knorm_part[bx] = m;
    }
  }
}

template <int NMAX, bool FULL>
__global__ void __launch_bounds__(res_threads<NMAX>()) residual_kernel(ResidualArgs a, int chunks) {
  residual_body<NMAX, FULL>(a, chunks, blockIdx.x);
}

// max of the non-negative (or NaN) p[i * st] over i = t0, t0 + step, .. < cnt, 0 if none.
// U loads are issued together per round (indices clamped into range, the extra ones
// not counted), so that a thread waits once per round rather than once per load.
template <int U>
__device__ inline double strided_max(const double* p, int cnt, int t0, int step, int st = 1) {
  double m = 0.0;
  for (int i0 = t0; i0 < cnt; i0 += U * step) {
    double t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = p[(size_t)min(i0 + u * step, cnt - 1) * st];
#pragma unroll
    for (int u = 0; u < U; ++u) m = i0 + u * step < cnt ? nan_max(t[u], m) : m;
  }
  return m;
}

// One workgroup per system: the root rows of r, and the largest |r| of each right-hand
// side (rnorm), from the tail workgroups' maxima and the root rows.  Thread (g, i) sums
// element i of the products C_s x_{s,0} over the scenarios s = g mod G (G = 1024 / NMAX
// groups), up to four right-hand sides at a time; the lanes of a wave are added by shuffles, the
// waves in order from LDS.  Latency-bound (one workgroup per system).
template <int NMAX>
__device__ __attribute__((always_inline)) inline void residual_root_body(const ResidualArgs& a,
                                                                         unsigned bx) {
  if (a.done && *a.done) return;
  constexpr int W = 16, QB = 4;
  __shared__ double part[QB][W][NMAX];
  __shared__ double xr[16][NMAX];
  __shared__ double wm[17][W];  // per wave: largest |r| (per right-hand side), |K| row
  const int n = a.n, N = a.N, S = a.S, nrhs = a.nrhs;
  const int sys = bx;
  const size_t len = ((size_t)S * N + 1) * n;
  const size_t root = (size_t)sys * a.vsys + (size_t)S * N * n;
  const double* R = a.R + (size_t)sys * n * n;
  const int t = threadIdx.x, i = t % NMAX, q = t / NMAX, wv = t >> 6;
  const bool mine = q < nrhs && i < n;  // this thread's root row and right-hand side
  const size_t o = root + (size_t)q * len + i;
  if (q < nrhs) xr[q][i] = i < n ? a.x[o] : 0.0;
  const double bv = mine ? a.b[o] : 0.0;
  // the tail workgroups' largest |r|, a.kper of them per system
  const double* rp = a.rpart + (size_t)sys * a.kper * nrhs;
  for (int k = 0; k < nrhs; ++k) {
    const double m = wave_max(strided_max<4>(rp + k, a.kper, t, 1024, nrhs));
    if ((t & 63) == 0) wm[k][wv] = m;
  }
  const double* w = a.w + (size_t)sys * S * nrhs * n;
  double sum = 0.0;
  for (int q0 = 0, taken; q0 < nrhs; q0 += taken) {
    if (q0) __syncthreads();
    auto partials = [&](auto qb, auto in_flight) {
      constexpr int Q = decltype(qb)::value;
      double acc[Q];
      scenario_sums<NMAX, Q, decltype(in_flight)::value>(w, S, n, nrhs, q0, acc);
      if ((t & 63) < NMAX)
#pragma unroll
        for (int u = 0; u < Q; ++u) part[u][wv][i] = acc[u];
      return Q;
    };
    // with few scenarios (some rounds of loads) four for three, the last one read again for the
    // one that is not there; beyond, as many as there are, a power of two
    if (nrhs - q0 >= (S <= 16 * (1024 / NMAX) ? 3 : QB))
      taken = partials(std::integral_constant<int, QB>{}, std::integral_constant<int, 4>{});
    else if (nrhs - q0 >= 2)
      taken = partials(std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
    else
      taken = partials(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
    __syncthreads();
    if (mine && q >= q0 && q < q0 + taken) {
#pragma unroll
      for (int v = 0; v < W; ++v) sum += part[q - q0][v][i];
    }
  }
  double rabs = 0.0;
  if (mine) {
    double rx = 0.0;
    for (int c = 0; c < n; ++c) rx += (i >= c ? R[i * n + c] : R[c * n + i]) * xr[q][c];
    const double r = bv - rx - sum;
    a.r[o] = r;
    rabs = fabs(r);
  }
  if (q < nrhs) {  // whole NMAX-lane groups
    for (int off = NMAX / 2; off > 0; off >>= 1) rabs = nan_max(rabs, __shfl_xor(rabs, off));
    if (i == 0) {
      double m = rabs;
#pragma unroll
      for (int v = 0; v < W; ++v) m = nan_max(wm[q][v], m);
      a.rnorm[(size_t)sys * a.seg_sys + q] = m;
    }
  }
  if (a.knorm_root) {
    // |K| of the system: the tail workgroups' largest row sums, and the root rows' (the
    // |C_s| row sums of the scenarios plus |R|)
    __syncthreads();
    double acc[1];
    scenario_sums<NMAX, 1, 16>(a.crow + (size_t)sys * S * n, S, n, 1, 0, acc);
    if ((t & 63) < NMAX) part[0][wv][i] = acc[0];
    const double m =
        wave_max(strided_max<4>(a.knorm_part + (size_t)sys * a.kper, a.kper, t, 1024));
    if ((t & 63) == 0) wm[16][wv] = m;
    __syncthreads();
    double k = 0.0;
    if (t < n) {
#pragma unroll
      for (int v = 0; v < W; ++v) k += part[0][v][t];
      for (int c = 0; c < n; ++c) k += fabs(t >= c ? R[t * n + c] : R[c * n + t]);
    }
    k = wave_max(k);  // n <= 64: the rows sit in wave 0
    if (t == 0) {
#pragma unroll
      for (int v = 0; v < W; ++v) k = nan_max(wm[16][v], k);
      a.knorm_root[sys] = k;
    }
  }
}

template <int NMAX>
__global__ void __launch_bounds__(1024) residual_root_kernel(ResidualArgs a) {
  residual_root_body<NMAX>(a, blockIdx.x);
}

__device__ inline double block_max(double v, double* sh) {
  v = wave_max(v);
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[wv] = v;
  __syncthreads();
  double m = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) m = nan_max(m, sh[i]);
  __syncthreads();
  return m;
}

// max |p[i]| over i = t0, t0 + stride, .. < len, eight independent loads in flight
__device__ inline double stream_maxabs(const double* __restrict__ p, size_t len, size_t t0,
                                       size_t stride) {
  constexpr int U = 8;
  double m[U] = {};
  size_t i = t0;
  for (; i + (U - 1) * stride < len; i += U * stride) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[i + u * stride];
#pragma unroll
    for (int u = 0; u < U; ++u) m[u] = nan_max(fabs(v[u]), m[u]);
  }
  for (; i < len; i += stride) m[0] = nan_max(fabs(p[i]), m[0]);
#pragma unroll
  for (int u = 1; u < U; ++u) m[0] = nan_max(m[u], m[0]);
  return m[0];
}

// partial[t][q][blk] = max over block blk's slice of |v_t[q][.]| (t = 0: v, 1: v2); grid
// (blk, q, t).  Streams its vectors once; the blocks per vector follow its length
// (norm_blocks), so that short vectors take one wait per block and long ones fill the
// GPU, and every right-hand side has blocks of its own.
__global__ void __launch_bounds__(256) maxabs_partial_kernel(const double* v, const double* v2,
                                                             size_t len, double* partial,
                                                             const int* done) {
  if (done && *done) return;
  __shared__ double sh[4];
  const size_t q = blockIdx.y, t = blockIdx.z;
  const double mx = block_max(
      stream_maxabs((t == 0 ? v : v2) + q * len, len,
                    (size_t)blockIdx.x * blockDim.x + threadIdx.x,
                    (size_t)gridDim.x * blockDim.x), sh);
  if (threadIdx.x == 0) partial[(t * gridDim.y + q) * gridDim.x + blockIdx.x] = mx;
}

// max over the block partials of one vector and right-hand side, on one wave
__device__ inline double wave_reduce_partials(const double* part, int blocks) {
  return wave_max(strided_max<16>(part, blocks, (int)threadIdx.x & 63, 64));
}

__global__ void __launch_bounds__(64) maxabs_final_kernel(const double* partial, int blocks,
                                                          double* out) {
  const double mx = wave_reduce_partials(partial + (size_t)blockIdx.x * blocks, blocks);
  if (threadIdx.x == 0) out[blockIdx.x] = mx;
}

// flags[0] = done, flags[1] = corrections applied
__global__ void refine_reset_kernel(int* flags) {
  if (threadIdx.x == 0) {
    flags[0] = 0;
    flags[1] = 0;
  }
}

// Stop test over all segments (one workgroup; segment k = system, right-hand side, on
// wave k mod 16): quantity(k) from the block partials, the largest into relcorr, and
// flags[0] = 1 (and the host's copy hflag) when every one passes.  count: corrections
// are counted always (1) or when the test fails (2) or not at all (0).
template <typename Q>
__device__ inline void stop_test(int segs, int count, int* flags, int* hflag, double* relcorr,
                                 Q quantity) {
  __shared__ double sworst[16];
  __shared__ int sok[16];
  const int wv = threadIdx.x >> 6, W = blockDim.x >> 6;
  bool ok = true;
  double worst = 0.0;
  for (int k = wv; k < segs; k += W) {
    bool pass;
    const double v = quantity(k, pass);
    worst = nan_max(v, worst);
    ok = ok && pass;
  }
  if ((threadIdx.x & 63) == 0) {
    sworst[wv] = worst;
    sok[wv] = ok;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < W; ++w) {
      worst = nan_max(sworst[w], worst);
      ok = ok && sok[w];
    }
    *relcorr = worst;
    if (count == 1 || (count == 2 && !ok)) flags[1] += 1;
    if (ok) flags[0] = 1;
    *hflag = ok;
  }
}

// |d|_inf and |x|_inf from the block partials, then the stop test
// |d_q|_inf <= tol |x_q|_inf for every right-hand side.
__global__ void __launch_bounds__(1024) refine_check_kernel(const double* partial, int blocks,
                                                            int segs, double tol, int* flags,
                                                            int* hflag, double* relcorr) {
  if (flags[0]) return;
  stop_test(segs, 1, flags, hflag, relcorr, [&](int q, bool& pass) {
    const double d = wave_reduce_partials(partial + (size_t)q * blocks, blocks);
    const double xv = wave_reduce_partials(partial + ((size_t)segs + q) * blocks, blocks);
    pass = d <= tol * xv;
    return xv > 0.0 ? d / xv : d;
  });
}

// Backward-error stop test.  For every segment (system sys, right-hand side): |r|_inf from
// the residual (rnorm), |x|_inf from the block partials, |b|_inf from bnorm and |K|_inf of
// the system from knorm; eta = |r| / (|K| |x| + |b|), the normwise backward error of x.
// The loop is done (flags[0] = 1) when eta <= tol for every segment; otherwise flags[1]
// counts one more correction if count is set.
__global__ void __launch_bounds__(1024) refine_be_check_kernel(
    const double* partial, int blocks, int segs, int nrhs, const double* rnorm,
    const double* knorm, const double* bnorm, double tol, int count, int* flags, int* hflag,
    double* relcorr) {
  if (flags[0]) return;
  stop_test(segs, count ? 2 : 0, flags, hflag, relcorr, [&](int seg, bool& pass) {
    const double mx = wave_reduce_partials(partial + (size_t)seg * blocks, blocks);
    const double den = knorm[seg / nrhs] * mx + bnorm[seg], mr = rnorm[seg];
    const double eta = den > 0.0 ? mr / den : (mr > 0.0 ? HUGE_VAL : mr);
    pass = eta <= tol;
    return eta;
  });
}

// ---- ragged batches (see multi.h) ----

__device__ inline ResidualArgs relocate_residual(const ResidualArgs& t, const Reloc& r) {
  ResidualArgs a = t;
  a.D = rel(r.D, t.D);
  a.E = rel(r.E, t.E);
  a.C = rel(r.C, t.C);
  a.R = rel(r.R, t.R);
  a.b = rel(r.b, t.b);
  a.x = rel(r.x, t.x);
  a.r = rel(r.r, t.r);
  return a;
}

template <int NMAX, bool FULL>
__global__ void __launch_bounds__(res_threads<NMAX>()) residual_multi(
    const MultiItem<ResidualArgs>* items, int nitems, Reloc r) {
  const MultiItem<ResidualArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  residual_body<NMAX, FULL>(relocate_residual(it.a, r), it.p0, multi_local(it).x);
}

template <int NMAX>
__global__ void __launch_bounds__(1024) residual_root_multi(const MultiItem<ResidualArgs>* items,
                                                            int nitems, Reloc r) {
  const MultiItem<ResidualArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  residual_root_body<NMAX>(relocate_residual(it.a, r), multi_local(it).x);
}

// part[slice] = max |v| over slice blockIdx.x of the concatenated vectors (and part[slices
// + slice] of v2, if set).  A segment is cut into slices of kNormSlice elements, so that
// the long systems of a batch are streamed by many workgroups: on 64 systems of 0.02 to
// 2.1 M elements, 2480 us with one workgroup per segment.
__global__ void __launch_bounds__(256) seg_maxabs_kernel(const double* v, const double* v2,
                                                         const SegRec* slices, double* part,
                                                         const int* done) {
  if (done && *done) return;
  __shared__ double sh[4];
  const SegRec sg = slices[blockIdx.x];
  for (int t = 0; t < (v2 ? 2 : 1); ++t) {
    const double mx =
        block_max(stream_maxabs((t == 0 ? v : v2) + sg.off, sg.len, threadIdx.x, 256), sh);
    if (threadIdx.x == 0) part[t * gridDim.x + blockIdx.x] = mx;
  }
}

// out[k] = max over the slices of segment k
__global__ void __launch_bounds__(64) seg_final_kernel(const double* part, const int* slice0,
                                                       double* out) {
  const int k = blockIdx.x, s0 = slice0[k];
  const double mx = wave_reduce_partials(part + s0, slice0[k + 1] - s0);
  if (threadIdx.x == 0) out[k] = mx;
}

// Per system (one workgroup each, a wave per segment in turn): whether all its segments
// pass; sys_worst = the largest test quantity.  part: slice maxima of d and x (mode 0), of
// x (mode 1, backward error).
__global__ void __launch_bounds__(256) ragged_sys_check_kernel(
    int mode, const double* part, const int* slice0, int nslice, int nrhs, const double* rnorm,
    const double* knorm, const double* bnorm, double tol, const int* flags, int* sys_ok,
    double* sys_worst) {
  if (flags[0]) return;
  __shared__ double sworst[4];
  __shared__ int sok[4];
  const int sys = blockIdx.x, wv = threadIdx.x >> 6;
  bool ok = true;
  double worst = 0.0;
  for (int k = sys * nrhs + wv; k < (sys + 1) * nrhs; k += 4) {
    const int s0 = slice0[k], cnt = slice0[k + 1] - s0;
    double q;
    if (mode == 1) {
      const double den = knorm[sys] * wave_reduce_partials(part + s0, cnt) + bnorm[k];
      const double mr = rnorm[k];
      q = den > 0.0 ? mr / den : (mr > 0.0 ? HUGE_VAL : mr);
    } else {
      const double d = wave_reduce_partials(part + s0, cnt);
      const double xv = wave_reduce_partials(part + nslice + s0, cnt);
      q = xv > 0.0 ? d / xv : d;
    }
    worst = nan_max(q, worst);
    if (!(q <= tol)) ok = false;
  }
  if ((threadIdx.x & 63) == 0) {
    sworst[wv] = worst;
    sok[wv] = ok;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      worst = nan_max(sworst[w], worst);
      ok = ok && sok[w];
    }
    sys_ok[sys] = ok;
    sys_worst[sys] = worst;
  }
}

__global__ void __launch_bounds__(256) ragged_final_check_kernel(int B, int count, int* flags,
                                                                 int* hflag, double* relcorr,
                                                                 const int* sys_ok,
                                                                 const double* sys_worst) {
  if (flags[0]) return;
  __shared__ double sh[4];
  double w = 0.0, bad = 0.0;
  for (int i = threadIdx.x; i < B; i += blockDim.x) {
    w = nan_max(sys_worst[i], w);
    if (!sys_ok[i]) bad = 1.0;
  }
  w = block_max(w, sh);
  bad = block_max(bad, sh);
  if (threadIdx.x == 0) {
    *relcorr = w;
    // count: 2 = a correction was applied before this test (correction-size test),
    // 1 = one is applied after it unless the test holds (backward error), 0 = none
    if (count == 2 || (count == 1 && bad != 0.0)) flags[1] += 1;
    if (bad == 0.0) flags[0] = 1;
    *hflag = bad == 0.0;
  }
}

}  // namespace

int residual_walks(int N, int n) { return (N + res_stages(n) - 1) / res_stages(n); }

size_t residual_lds(int nmax, int nrhs) {
  return nmax <= 8 ? residual_lds_bytes<8>(nrhs)
                   : nmax <= 16 ? residual_lds_bytes<16>(nrhs) : residual_lds_bytes<32>(nrhs);
}

void launch_residual_multi(int nmax, bool full, const MultiItem<ResidualArgs>* items, int nitems,
                           unsigned blocks, size_t lds, const Reloc& r, hipStream_t st) {
  const dim3 g(blocks), b(nmax > 16 ? res_threads<32>() : res_threads<16>());
#define BMPC_RES_MULTI(NM)                                                             \
  if (full)                                                                            \
    hipLaunchKernelGGL((residual_multi<NM, true>), g, b, lds, st, items, nitems, r);     \
  else                                                                                 \
    hipLaunchKernelGGL((residual_multi<NM, false>), g, b, lds, st, items, nitems, r);
  if (nmax <= 8) {
    BMPC_RES_MULTI(8)
  } else if (nmax <= 16) {
    BMPC_RES_MULTI(16)
  } else {
    BMPC_RES_MULTI(32)
  }
#undef BMPC_RES_MULTI
}

void launch_residual_root_multi(const MultiItem<ResidualArgs>* items, int nitems, unsigned blocks,
                                const Reloc& r, hipStream_t st) {
  hipLaunchKernelGGL(residual_root_multi<32>, dim3(blocks), dim3(1024), 0, st, items, nitems, r);
}

void launch_seg_maxabs(const double* v, const double* v2, const SegRec* slices, int nslice,
                       double* part, const int* done, hipStream_t st) {
  hipLaunchKernelGGL(seg_maxabs_kernel, dim3(nslice), dim3(256), 0, st, v, v2, slices, part, done);
}

void launch_seg_final(const double* part, const int* slice0, int nseg, double* out,
                      hipStream_t st) {
  hipLaunchKernelGGL(seg_final_kernel, dim3(nseg), dim3(64), 0, st, part, slice0, out);
}

void launch_ragged_check(int mode, const double* part, const int* slice0, int nslice, int B,
                         int nrhs, const double* rnorm, const double* knorm,
                         const double* bnorm, double tol, int count, int* flags, int* hflag,
                         double* relcorr, int* sys_ok, double* sys_worst, hipStream_t st) {
  hipLaunchKernelGGL(ragged_sys_check_kernel, dim3(B), dim3(256), 0, st, mode, part, slice0,
                     nslice, nrhs, rnorm, knorm, bnorm, tol, (const int*)flags, sys_ok,
                     sys_worst);
  hipLaunchKernelGGL(ragged_final_check_kernel, dim3(1), dim3(256), 0, st, B, count, flags,
                     hflag, relcorr, (const int*)sys_ok, (const double*)sys_worst);
}

// Blocks per vector of maxabs_partial_kernel: 2048 elements each (a round of eight loads
// per thread), at most kNormBlocks.
static int norm_blocks(size_t len) {
  return (int)std::min<size_t>(kNormBlocks, (len + 2047) / 2048);
}
static int check_threads(int segs) { return 64 * std::min(16, segs); }

// The launches take the segments in the y dimension of the grid; beyond its limit they go
// in rounds of 65535.
static void maxabs_partials(const double* v, const double* v2, int segs, size_t len,
                            double* partial, const int* done, hipStream_t st) {
  const int nb = norm_blocks(len);
  if (segs <= 65535) {
    hipLaunchKernelGGL(maxabs_partial_kernel, dim3(nb, segs, v2 ? 2 : 1), dim3(256), 0, st, v, v2,
                       len, partial, done);
    return;
  }
  for (int t = 0; t < (v2 ? 2 : 1); ++t)
    for (int k0 = 0; k0 < segs; k0 += 65535)
      hipLaunchKernelGGL(maxabs_partial_kernel, dim3(nb, std::min(65535, segs - k0), 1), dim3(256),
                         0, st, (t ? v2 : v) + (size_t)k0 * len, (const double*)nullptr, len,
                         partial + ((size_t)t * segs + k0) * nb, done);
}

void launch_refine_be_check(const double* x, int B, int nrhs, size_t len, double* partial,
                            const double* rnorm, const double* knorm, const double* bnorm,
                            double tol, int count, int* flags, int* hflag, double* relcorr,
                            hipStream_t st) {
  maxabs_partials(x, nullptr, B * nrhs, len, partial, flags, st);
  hipLaunchKernelGGL(refine_be_check_kernel, dim3(1), dim3(check_threads(B * nrhs)), 0, st,
                     (const double*)partial, norm_blocks(len), B * nrhs, nrhs, rnorm, knorm,
                     bnorm, tol, count, flags, hflag, relcorr);
}

template <int NMAX>
static void launch_residual_t(const ResidualArgs& a, dim3 grid, int chunks, hipStream_t st) {
  const size_t lds = residual_lds_bytes<NMAX>(a.nrhs);
  if (NMAX > 32) {  // beyond the default 64 KB of dynamic LDS
    static bool attr_set = false;
    if (!attr_set) {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&residual_kernel<NMAX, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)residual_lds_bytes<NMAX>(residual_chunk(NMAX)));
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&residual_kernel<NMAX, false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)residual_lds_bytes<NMAX>(residual_chunk(NMAX)));
      attr_set = true;
    }
  }
  if (a.n == NMAX)
    hipLaunchKernelGGL((residual_kernel<NMAX, true>), grid, dim3(res_threads<NMAX>()), lds, st, a,
                       chunks);
  else
    hipLaunchKernelGGL((residual_kernel<NMAX, false>), grid, dim3(res_threads<NMAX>()), lds, st, a,
                       chunks);
}

void launch_residual(const ResidualArgs& a, int nmax, hipStream_t st) {
  const int chunks = residual_walks(a.N, a.n);
  const dim3 grid((unsigned)(a.B * a.S) * (unsigned)chunks);
  if (nmax <= 8)
    launch_residual_t<8>(a, grid, chunks, st);
  else if (nmax <= 16)
    launch_residual_t<16>(a, grid, chunks, st);
  else if (nmax <= 32)
    launch_residual_t<32>(a, grid, chunks, st);
  else
    launch_residual_t<64>(a, grid, chunks, st);
}

void launch_residual_root(const ResidualArgs& a, hipStream_t st) {
  if (a.n > 32)
    hipLaunchKernelGGL(residual_root_kernel<64>, dim3(a.B), dim3(1024), 0, st, a);
  else
    hipLaunchKernelGGL(residual_root_kernel<32>, dim3(a.B), dim3(1024), 0, st, a);
}

void launch_maxabs(const double* v, int segs, size_t len, double* partial, double* out,
                   hipStream_t st) {
  maxabs_partials(v, nullptr, segs, len, partial, nullptr, st);
  hipLaunchKernelGGL(maxabs_final_kernel, dim3(segs), dim3(64), 0, st, partial, norm_blocks(len),
                     out);
}

void launch_refine_reset(int* flags, hipStream_t st) {
  hipLaunchKernelGGL(refine_reset_kernel, dim3(1), dim3(64), 0, st, flags);
}

void launch_refine_check(const double* d, const double* x, int segs, size_t len,
                         double* partial, double tol, int* flags, int* hflag, double* relcorr,
                         hipStream_t st) {
  maxabs_partials(d, x, segs, len, partial, flags, st);
  hipLaunchKernelGGL(refine_check_kernel, dim3(1), dim3(check_threads(segs)), 0, st,
                     (const double*)partial, norm_blocks(len), segs, tol, flags, hflag, relcorr);
}

}  // namespace bmpc
