// Assembly of the reduced IPM system of a branch-MPC QP (gfx950).
//
// The regularized primal-dual IPM KKT matrix [[P + tau I, A^T, G^T], [A, -delta I, 0],
// [G, 0, -(W + delta I)]] reduces, by eliminating its second and third block rows, to
// the SPD matrix K = P + tau I + delta^{-1} A^T A + G^T (W + delta I)^{-1} G (appendix
// on the linear systems of IPM and ADMM).  In branch MPC every cost and constraint
// term touches two neighbouring blocks, stored per link j of scenario s: link 0 couples
// (u, v) = (x_0, x_{s,0}), link k couples (x_{s,k-1}, x_{s,k}), link N is the terminal
// term on u = x_{s,N-1}.  The link's share of K is M_j = Q_j + delta^{-1} A_j^T A_j +
// G_j^T (w_j + delta)^{-1} G_j (2n x 2n, quadrants uu, uv, vu, vv):
//   D_{s,k} = tau I + M_{s,k}[vv] + M_{s,k+1}[uu]      E_{s,k} = M_{s,k+1}[vu]
//   C_s     = M_{s,0}[uv]                             R = tau I + sum_s M_{s,0}[uu]
// so K has exactly the root-coupled block structure the solver takes.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "bmpc.h"
#include "blockops.h"
#include "bmpc_internal.h"
#include "regblock.h"

namespace bmpc {

namespace {

struct QpArgs {
  int S, N, n, me, mi;
  const double* Q;
  const double* A;
  const double* G;
  const double* w;
  double tau, delta, sdelta;  // sdelta: 1 / sqrt(delta)
  double* D;
  double* E;
  double* C;
  double* Rpart;  // [S][n][n] link-0 uu parts
};

// One wave walks a chunk of consecutive stages of one scenario, a link at a time, so that a
// link is read once (the first link of a chunk twice, its v columns only): M_j[vv] of a
// link waits in the accumulators for the next link's uu.  The products X^T diag X are 16 x
// 16 x 4 FP64 MFMA tiles with the constraint rows as the contraction index: lane 16 g + i
// holds entry (4 k + g, 16 t + i) of the rows for both operands (one load serves a tile's
// rows and columns; both carry the square root of the weight, so that entries (p, q) and
// (q, p) are sums of the same products and D and R are exactly symmetric where Q is), and Q
// is read in the accumulator layout, so nothing is staged in LDS and all loads of a link
// are in flight together.  Memory-bound: 8 (3 n^2 + (me + mi) 2n + mi) bytes read per link
// and 16 n^2 written.  S = 256, N = 128, n = 16, 12 + 32 rows: 349 us with one workgroup
// per stage and scalar products from LDS (every link read twice), 169 us
// now (4.3 TB/s); S = 64, N = 128, n = 32, 24 + 64 rows: 690 -> 193 us.
template <int NT>  // 16-column tiles of u and of v: ceil(n / 16)
struct QpLink {
  typedef Mfma<double>::acc_t acc_t;
  const QpArgs& a;
  int g, i;

  // column 16 t + i of the u (off = 0) or v (off = n) part, or out of range
  __device__ unsigned col(int t, int off) const {
    const int c = 16 * t + i;
    return c < a.n ? (unsigned)(off + c) * 8u : kOutOfRange;
  }
  // M += sum over the rows r < rows of X of (wt(r) X[r][.])^T (wt(r) X[r][.]) for the tiles
  // asked for
  template <bool UU, bool VU, bool UV, typename Wt>
  __device__ void rows(__amdgpu_buffer_rsrc_t rs, int rows, Wt wt, acc_t (&uu)[NT][NT],
                       acc_t (&vu)[NT][NT], acc_t (&vv)[NT][NT]) const {
    constexpr int U = NT == 1 ? 8 : 3;  // steps whose loads go out together
    constexpr bool NU = UU || VU || UV;
    const unsigned ld = 2u * (unsigned)a.n * 8u;
    for (int k0 = 0; 4 * k0 < rows; k0 += U) {
      double xu[U][NT], xv[U][NT], w[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int r = 4 * (k0 + k) + g;
        w[k] = wt.load(r);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          // rows past the end read as zero: past the range of rs
          if (NU) xu[k][t] = buf_load_f64(rs, (unsigned)r * ld + col(t, 0));
          xv[k][t] = buf_load_f64(rs, (unsigned)r * ld + col(t, a.n));
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        if (4 * (k0 + k) >= rows) continue;  // uniform
        // rows past the end are zero, and their weight is finite: 1 / sqrt(delta) at most
        const double s = wt.scale(w[k]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (NU) xu[k][t] *= s;
          xv[k][t] *= s;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
          for (int c = 0; c < NT; ++c) {
            if (UU) uu[t][c] = Mfma<double>::mma(xu[k][t], xu[k][c], uu[t][c]);
            if (VU) vu[t][c] = Mfma<double>::mma(xv[k][t], xu[k][c], vu[t][c]);
            if (UV) vu[t][c] = Mfma<double>::mma(xu[k][t], xv[k][c], vu[t][c]);
            vv[t][c] = Mfma<double>::mma(xv[k][t], xv[k][c], vv[t][c]);
          }
        }
      }
    }
  }
  // one block (n x n at row offset ro, column offset co of a 2n x 2n array) in accumulator
  // order; place(t, c, v): its element index, or -1
  __device__ void quadrant(__amdgpu_buffer_rsrc_t rs, int ro, int co, acc_t (&m)[NT][NT]) const {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * t + 4 * v + g, cc = 16 * c + i;
          m[t][c][v] = buf_load_f64(rs, r < a.n && cc < a.n
                                            ? (unsigned)((ro + r) * 2 * a.n + co + cc) * 8u
                                            : kOutOfRange);
        }
  }
  __device__ void store(double* __restrict__ dst, const acc_t (&m)[NT][NT]) const {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * t + 4 * v + g, cc = 16 * c + i;
          if (r < a.n && cc < a.n) dst[r * a.n + cc] = m[t][c][v];
        }
  }

  struct ConstWt {
    double s;
    __device__ double load(int) const { return 0.0; }
    __device__ double scale(double) const { return s; }
  };
  struct RowWt {
    __amdgpu_buffer_rsrc_t rs;
    double delta;
    __device__ double load(int r) const { return buf_load_f64(rs, (unsigned)r * 8u); }
    __device__ double scale(double w) const { return rsqrt(w + delta); }
  };
  // the quadrants of M_j: uu (UU), vu (VU) or uv (UV) into m2, vv always
  template <bool UU, bool VU, bool UV>
  __device__ void link(size_t lk, acc_t (&uu)[NT][NT], acc_t (&m2)[NT][NT],
                       acc_t (&vv)[NT][NT]) const {
    const unsigned n = a.n, n2 = 2 * n;
    const auto rq = block_rsrc(a.Q + lk * n2 * n2, n2 * n2 * 8u);
    if (UU) quadrant(rq, 0, 0, uu);
    if (VU) quadrant(rq, n, 0, m2);
    if (UV) quadrant(rq, 0, n, m2);
    quadrant(rq, n, n, vv);
    if (a.me > 0)
      rows<UU, VU, UV>(block_rsrc(a.A + lk * a.me * n2, a.me * n2 * 8u), a.me,
                       ConstWt{a.sdelta}, uu, m2, vv);
    if (a.mi > 0)
      rows<UU, VU, UV>(block_rsrc(a.G + lk * a.mi * n2, a.mi * n2 * 8u), a.mi,
                       RowWt{block_rsrc(a.w + lk * a.mi, a.mi * 8u), a.delta}, uu, m2, vv);
  }
};

template <int NT>
__global__ void __launch_bounds__(256, 2) qp_stage_kernel(QpArgs a, int chunk, int chunks) {
  typedef Mfma<double>::acc_t acc_t;
  const unsigned item = blockIdx.x * 4u + (unsigned)wave_id();
  if (item >= (unsigned)a.S * (unsigned)chunks) return;  // no barrier follows
  const int s = (int)(item / chunks), k0 = (int)(item - (unsigned)s * chunks) * chunk;
  const int k1 = min(a.N, k0 + chunk);
  const int l = threadIdx.x & 63;
  const QpLink<NT> q{a, l >> 4, l & 15};
  const int N = a.N;
  const size_t nn = (size_t)a.n * a.n, lk0 = (size_t)s * (N + 1);
  acc_t uu[NT][NT], m2[NT][NT], vv[NT][NT], carry[NT][NT];
  // link k0: its vv waits for the next link; the scenario's first one also gives C and the
  // root's share
  if (k0 == 0) {
    q.template link<true, false, true>(lk0, uu, m2, carry);
    q.store(a.Rpart + (size_t)s * nn, uu);
    q.store(a.C + (size_t)s * nn, m2);
  } else {
    q.template link<false, false, false>(lk0 + k0, uu, m2, carry);
  }
  for (int k = k0; k < k1; ++k) {
    q.template link<true, true, false>(lk0 + k + 1, uu, m2, vv);
    // D_{s,k} = tau I + M_k[vv] + M_{k+1}[uu]
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double tau = 16 * t + 4 * v + q.g == 16 * c + q.i ? a.tau : 0.0;
          uu[t][c][v] += tau + carry[t][c][v];
          carry[t][c][v] = vv[t][c][v];
        }
    q.store(a.D + ((size_t)s * N + k) * nn, uu);
    if (k + 1 < N) q.store(a.E + ((size_t)s * (N - 1) + k) * nn, m2);
  }
}

// R = tau I + sum_s Rpart[s]: 64 entries per workgroup, their scenarios over 16 waves
// (consecutive groups, each in scenario order, the groups in order)
__global__ void __launch_bounds__(1024) qp_root_kernel(const double* Rpart, int S, int n,
                                                       double tau, double* R) {
  __shared__ double part[16][64];
  const int l = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + l, nn = n * n;
  const int per = (S + 15) / 16, s0 = g * per, s1 = min(S, s0 + per);
  double acc = 0.0;
  if (e < nn) {
    constexpr int U = 16;
    for (int s = s0; s < s1; s += U) {
      double v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = Rpart[(size_t)min(s + u, s1 - 1) * nn + e];
#pragma unroll
      for (int u = 0; u < U; ++u) acc += s + u < s1 ? v[u] : 0.0;
    }
  }
  part[g][l] = acc;
  __syncthreads();
  if (g == 0 && e < nn) {
#pragma unroll
    for (int w = 1; w < 16; ++w) acc += part[w][l];
    R[e] = acc + (e / n == e % n ? tau : 0.0);
  }
}

}  // namespace

}  // namespace bmpc

namespace {

// Scratch of bmpc_assemble_qp_noalloc: the per-scenario root shares (S * n * n doubles)
// in a file-scope device array, one copy per GPU, so that the entry point allocates
// nothing.  Host code never uses the array's name as an address: the device address of
// each GPU's copy is looked up once per device (hipGetSymbolAddress with that device
// current) and kept here.
constexpr size_t kQpScratchDoubles = (size_t)512 * 32 * 32;  // 4 MiB
static __device__ __align__(256) double scratch[kQpScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's scratch (null on failure).
double* device_scratch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = static_cast<double*>(ptr);
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" bmpc_status bmpc_assemble_qp(const bmpc_qp_dims* d, const double* Q, const double* A,
                                        const double* G, const double* w, double tau,
                                        double delta, double* D, double* E, double* C,
                                        double* R, double* work, void* stream) {
  using namespace bmpc;
  if (!d || d->S < 1 || d->N < 1 || d->n < 1 || d->n > 32 || d->me < 0 || d->me > 64 ||
      d->mi < 0 || d->mi > 128 || !(tau >= 0.0) || !(delta > 0.0) || !Q || !D || !C || !R ||
      !work || (d->N > 1 && !E) || (d->me > 0 && !A) || (d->mi > 0 && (!G || !w)))
    return BMPC_ERR_INVALID;
  QpArgs a{};
  a.S = d->S;
  a.N = d->N;
  a.n = d->n;
  a.me = d->me;
  a.mi = d->mi;
  a.Q = Q;
  a.A = A;
  a.G = G;
  a.w = w;
  a.tau = tau;
  a.delta = delta;
  a.sdelta = 1.0 / std::sqrt(delta);
  a.D = D;
  a.E = E;
  a.C = C;
  a.Rpart = work;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  // stages per wave: eight (a link in eight read twice), fewer where that would leave the GPU
  // with less than four waves on each of its 1024 SIMDs
  const int chunk = (int)std::min<int64_t>(8, std::max<int64_t>(1, (int64_t)d->S * d->N / 4096));
  const int chunks = (d->N + chunk - 1) / chunk;
  const dim3 grid((unsigned)(((int64_t)d->S * chunks + 3) / 4));
  if (d->n <= 16)
    hipLaunchKernelGGL(qp_stage_kernel<1>, grid, dim3(256), 0, st, a, chunk, chunks);
  else
    hipLaunchKernelGGL(qp_stage_kernel<2>, grid, dim3(256), 0, st, a, chunk, chunks);
  hipLaunchKernelGGL(qp_root_kernel, dim3((unsigned)((d->n * d->n + 63) / 64)), dim3(1024), 0, st,
                     (const double*)work, d->S, d->n, tau, R);
  return hipGetLastError() == hipSuccess ? BMPC_OK : BMPC_ERR_DEVICE;
}

extern "C" bmpc_status bmpc_assemble_qp_noalloc(const bmpc_qp_dims* d, const double* Q,
                                                const double* A, const double* G, const double* w,
                                                double tau, double delta, double* D, double* E,
                                                double* C, double* R, void* stream) {
  if (!d || d->S < 1 || d->n < 1 || d->n > 32 ||
      (size_t)d->S * d->n * d->n > kQpScratchDoubles)
    return BMPC_ERR_INVALID;
  double* work = device_scratch();
  if (!work) return BMPC_ERR_DEVICE;
  return bmpc_assemble_qp(d, Q, A, G, w, tau, delta, D, E, C, R, work, stream);
}
