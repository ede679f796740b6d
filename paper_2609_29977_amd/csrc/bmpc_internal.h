// Internal declarations of the bmpc HIP library (gfx950).
//
// Chain notation used by every kernel (Section IV-A).  Tail s is reversed
// (Omega_i) so that chain position j = 1..m, m = N-1, holds stage N-j; the
// root-coupled stage 0 (the paper's x_1) is kept last and is called X below
// (position N).  The coupling from chain position j to its successor is
// K[pos j+1, pos j] = E[s][N-1-j]^T (for j = m the successor is X).  Under
// Gamma_{N-1} position j is eliminated at level tz(j)+1 (tz = trailing zeros):
// level 1 takes the odd positions, level 2 the positions 2*odd, ... (the groups of
// the recursion in Section II), and X comes last.  When position j (level t+1) is
// eliminated, its current neighbours are j-2^t (left, if >= 1) and j+2^t (right,
// or X when j+2^t > m).
//
// Factor storage (plan-owned, precision T of the tail factor):
//   Linv[S][N][n][n]  L_jj^{-1} of position j at index j-1, X at index N-1, each
//                     block packed by rows (element (r, c), c <= r, at r(r+1)/2 + c)
//   Gl  [S][m][n][n]  factor block of the left neighbour's row, G_l = K[left,j] L_jj^{-T}
//   Gr  [S][m][n][n]  factor block of the right neighbour's row (or X's row)
//   F   [S][n][n]     F_{s,1} = C_s L_X^{-T} (the only block of the root row, Thm 1)
//   U   [S][n][n]     F F^T in FP64;  LR[n][n] = chol(R - sum U) in FP64
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bmpc {

constexpr int kFactorThreads = 256;
// Right-hand sides per kernel launch: a solve takes them in chunks of kSolveRhs (the columns
// of an MFMA tile), the residual in chunks of kMaxRhs (kMaxRhs64 at n > 32, where its LDS
// holds fewer vectors), and up to kMaxRhs of them go through the factorization with the
// forward substitution inside; a plan's nrhs has no such limit.
constexpr int kSolveRhs = 16;
constexpr int kMaxRhs = 8;
constexpr int kMaxRhs64 = 4;
// Solves of few right-hand sides at n > 32 that go level by level through solve64.hip (figures
// there): at n > 48, and of chains of one or two stages, where nothing hides the latency of
// the products' one wave per position, unless there are scenarios enough for that (in FP32
// with short runs of loads, n % 4, there hardly are).
constexpr bool few_rhs64(int S, int N, int n, int nrhs, bool fp64) {
  const bool runs = n % 4 == 0;
  return (n > 48 && nrhs <= kMaxRhs64) ||
         (n > 32 && N <= 2 && (nrhs == 1 || (nrhs == 2 && (N == 1 || !runs))) &&
          S <= (fp64 || runs ? 512 : 2048));
}
constexpr __host__ __device__ int residual_chunk(int nmax) {
  return nmax > 32 ? kMaxRhs64 : kMaxRhs;
}

// Blocks per chain in the G_l and G_r arrays: the N-1 blocks of the positions 1..N-1,
// padded to N so that every factor array (L^{-1} has N) shares one chain stride; the
// solve streams read the three arrays at the same offsets, which HBM serves faster than
// offsets that drift apart by one block per chain.
inline __host__ __device__ size_t g_chain_blocks(int N) { return (size_t)N; }
constexpr int kMaxWindowDepth = 6;

// Kernel classes for per-kernel event timing.
enum KernelClass : int {
  KC_FACTOR_INIT = 0,
  KC_FACTOR_FIRST,   // first factor pass when it is not also the last
  KC_FACTOR_MID,     // intermediate factor passes
  KC_FACTOR_FINAL,   // last factor pass + the x_1 step (F, U)
  KC_ROOT_REDUCE,    // partial sums of U over scenario groups
  KC_ROOT_POTRF,     // R~ = R - sum U, L_R = chol(R~)
  KC_SOLVE_FWD,      // tail forward substitution, one launch per level below the top ones
  KC_SOLVE_X_FWD,    // top forward levels, x_1 forward step + F y products
  KC_SOLVE_ROOT,     // root reduction and root triangular solves
  KC_SOLVE_X_BWD,    // root propagation, x_1 backward step, top backward levels
  KC_SOLVE_BWD,      // tail backward substitution, one launch per level below the top ones
  KC_RESIDUAL,       // FP64 tail residual b - K x
  KC_RESIDUAL_ROOT,  // FP64 root residual
  KC_REFINE_MISC,    // refinement bookkeeping (norm reset, stop test)
  KC_GRAD_BLOCKS,    // block gradients through the solve
  KC_FACTOR_L1INV,   // level-1 diagonal inverses before the first factor pass
  KC_COUNT
};

// Batches: B independent systems of one shape are factored and solved together.
// The tail kernels run over the B*S chains (chain g is scenario g % S of system
// g / S); the root steps run once per system.  Vectors b, x, r are [B][nrhs][len]
// with len = (S*N+1)*n.
struct FactorPassArgs {
  int S, N, n, m;       // S = chains of the batch (B * scenarios); m = N - 1
  int Ssys;             // scenarios per system (for natural row numbers)
  int Tw;               // window depth (levels per pass)
  int pass, npass;      // index of this pass and total passes
  int mk, shift;        // reduced chain length, position stride log2
  int windows;          // windows per chain
  int is_final;
  const double* D;
  const double* E;
  const double* C;
  // reduced-chain inputs written by the previous pass (null for pass 0)
  const void* accR_in;  // [S][stride] : update of a node from the window on its left
  const void* accL_in;  // [S][stride] : update of a node from the window on its right
  const void* fill_in;  // [S][stride] : coupling from node q to its successor
  void* accR_out;
  void* accL_out;
  void* fill_out;
  int stride;           // blocks per chain in the reduced-chain buffers
  void* accX;           // [S][npass] : X updates of each pass
  void* Linv;
  void* Gl;
  void* Gr;
  void* F;
  double* U;
  const int* permpos;   // [N] permuted position of chain position j at j-1 (X at N-1)
  unsigned long long* info;
  // Forward substitution fused into the elimination (null b: factor only).  b is the
  // FP64 right-hand side in the vector layout of the solve ([B][nrhs][len]); y
  // receives L^{-1} Pi b per chain position ([S][N][n][nrhs], precision T) and w the
  // FP64 products F_s y_X ([S][nrhs][n]).  The vector accumulators mirror accR /
  // accL / accX per right-hand side ([S][stride][nrhs][n] and [S][npass][nrhs][n]).
  const double* b;       // right-hand side q = 0 of this chunk (b + q0 * len)
  int nrhs;              // right-hand sides of this chunk
  size_t vsys;           // vector elements per system (all right-hand sides)
  void* y;
  double* w;
  const void* vaccR_in;
  const void* vaccL_in;
  void* vaccR_out;
  void* vaccL_out;
  void* vaccX;
};

// Vectors b, x, r are [B][nrhs][len]; a launch takes a chunk of the right-hand sides:
// its pointers are those of the chunk's first right-hand side in system 0 (offset by
// q0 * len), nrhs counts the chunk, vsys = (all right-hand sides) * len is the stride
// between systems and seg_sys the stride of the per-(system, right-hand side) norms.
// Root factorization of every system of a batch: L_R = chol(R - sum of the groups' partials).
struct RootStep {
  const double* R;
  const double* part;  // [B][groups][n][n]
  double* LR;
  unsigned long long* info;      // smallest failing row so far (permuted), ~0: none
  unsigned long long* info_out;  // one system: where the finished info goes (else null)
  int* flags;                    // refinement flags to reset (or null)
  int n, groups;
  unsigned long long sys_rows, root_row;
};

struct SolveArgs {
  int S, N, n, m, nrhs;  // S = scenarios per system, nrhs of this chunk
  int B;                 // systems in the batch
  size_t vsys;           // vector elements per system
  int seg_sys;           // norm entries per system
  const void* Linv;
  const void* Gl;
  const void* Gr;
  const void* F;
  const double* LR;
  const double* b;       // [nrhs][len] FP64 input
  double* x;             // [nrhs][len] FP64 output
  void* y;               // [S][N][n][nrhs] scratch, precision T
  double* w;             // [S][nrhs][n] FP64 products F_s y_X
  double* x0;            // [nrhs][n]
  const double* rnorm;   // refinement: input scale 1/rnorm, output x += rnorm * d
  double* dstore;        // refinement: rnorm * d stored here ([nrhs][len], may alias b)
  const int* done;       // refinement stop flag (null outside refinement)
  int accumulate;        // 0: x = d ; 1: x += rnorm * d (refinement update)
  int fwd_waves;         // forward level positions: at most this many waves (0: 4)
};

struct ResidualArgs {
  int S, N, n, nrhs;     // S = scenarios per system, nrhs of this chunk
  int B;                 // systems in the batch
  size_t vsys;           // vector elements per system (all right-hand sides)
  const double* D;
  const double* E;
  const double* C;
  const double* R;       // [B][n][n]
  const double* b;
  const double* x;
  double* r;             // [B][nrhs][len]
  double* w;             // [S][nrhs][n] products C_s x_{s,0}
  const int* done;
  int kper;              // tail workgroups per system
  double* rpart;         // [B * kper][nrhs] largest |r| of each tail workgroup
  double* rnorm;         // largest |r| of system sys, right-hand side q: [sys * seg_sys + q]
  int seg_sys;
  // Row sums of |K| (backward-error stop): per workgroup of the tail residual the
  // maximum over its rows (knorm_part), the per-chain |C_s| row sums (crow
  // [B*S][n]), and from these and the root rows |K| of each system (knorm_root[sys]).
  // Null: not computed.
  double* knorm_part;
  double* knorm_root;
  double* crow;
};

struct GradArgs {
  int S, N, n, nrhs;     // S = scenarios per system, all right-hand sides
  int B;                 // systems in the batch
  const double* x;       // [nrhs][len] solution
  const double* lam;     // [nrhs][len] adjoint K^{-1} g
  double* dD;            // [S][N][n][n] or null
  double* dE;            // [S][N-1][n][n] or null
  double* dC;            // [S][n][n] or null
  double* dR;            // [n][n] or null
};

// launchers (defined next to their kernels)
template <typename T>
void launch_factor_pass(const FactorPassArgs& a, int nmax, hipStream_t st);
// L^{-1} of the odd chain positions' diagonal blocks (D only), before the first pass
// (whose arguments a are); block sizes 17..32 only.
template <typename T>
void launch_level1_inverse(const FactorPassArgs& a, hipStream_t st);
// block sizes up to 16 (tree.hip): window LDS and threads of a pass of Tw levels
template <typename T>
void launch_tree_pass(const FactorPassArgs& a, int nmax, hipStream_t st);
// over mk chain positions
size_t tree_pass_lds(bool fp64, int nmax, int Tw, int mk, int nrhs_fused, bool final);
// block sizes 33..64: window depth 1, no fused forward substitution (factor64.hip)
template <typename T>
void launch_factor_pass64(const FactorPassArgs& a, hipStream_t st);
size_t factor64_lds_bytes(bool fp64);
void launch_factor_init(unsigned long long* info, hipStream_t st);
// part[sys][g] = sum of U over the scenarios of group g of system sys (B systems of S)
void launch_root_reduce(const double* U, double* part, int B, int S, int n, int groups,
                        hipStream_t st);
// LR[sys] = chol(R[sys] - sum_g part[sys][g]) for every system; row numbers of system
// sys start at sys * sys_rows, its root rows at root_row within it
void launch_root_potrf(const RootStep& s, int B, hipStream_t st);

template <typename T>
void launch_solve_fwd_level(const SolveArgs& a, int level, hipStream_t st);
void launch_solve_root(const SolveArgs& a, hipStream_t st);
// root factorization and the root step of a solve in one launch, n <= 32
void launch_root_factor_solve(const RootStep& s, const SolveArgs& a, hipStream_t st);
template <typename T>
void launch_solve_bwd_level(const SolveArgs& a, int level, hipStream_t st);
// The backward levels from the top down to level_lo in one launch (one workgroup per chain,
// one wave per position), for few right-hand sides; with_x: root propagation and
// the x_1 backward step before them (alone if level_lo is above the top).  level_lo as
// bwd_top_level has it or above.
template <typename T>
void launch_solve_bwd_top(const SolveArgs& a, int level_lo, bool with_x, hipStream_t st);
// The forward levels from level_lo up to the top (where few_fwd_top says so; else none, level_lo
// above the top) and the x_1 forward step in one launch, for few right-hand sides.
template <typename T>
void launch_solve_fwd_top(const SolveArgs& a, int level_lo, hipStream_t st);

// the same as matrix products over the right-hand sides (solve_rhs.hip): one level of either
// sweep; the x_1 forward step after the forward levels from level_lo on (fwd), or root
// propagation and the x_1 backward step before the backward levels down to level_lo
template <typename T>
void launch_mm_level(const SolveArgs& a, int level, bool fwd, hipStream_t st);
template <typename T>
void launch_mm_top(const SolveArgs& a, int level_lo, bool fwd, hipStream_t st);

// the same one level, or one x_1 step, at a time, where few_rhs64 (solve64.hip)
template <typename T>
void launch_solve64_level(const SolveArgs& a, int level, bool fwd, hipStream_t st);
template <typename T>
void launch_solve64_x(const SolveArgs& a, bool fwd, hipStream_t st);

// Workgroups of the tail residual per chain of N stages with blocks of n.
int residual_walks(int N, int n);
void launch_residual(const ResidualArgs& a, int nmax, hipStream_t st);
void launch_grad_blocks(const GradArgs& a, hipStream_t st);
void launch_residual_root(const ResidualArgs& a, hipStream_t st);
void launch_refine_reset(int* flags, hipStream_t st);
// Infinity norms by a two-stage maximum (at most kNormBlocks block partials per vector,
// then one wave), deterministic and NaN-propagating.
constexpr int kNormBlocks = 1024;
// out[k] = max_i |v[k][i]| of segs vectors, through partial[segs][kNormBlocks]
void launch_maxabs(const double* v, int segs, size_t len, double* partial, double* out,
                   hipStream_t st);
// The stop test |d_k|_inf <= tol |x_k|_inf for every segment k (partials in
// partial[2][segs][kNormBlocks]): flags[0] = 1 if it holds, flags[1] counts the
// corrections, *hflag (pinned host memory) = whether it holds; relcorr = max_k |d_k| /
// |x_k|.  Skipped when flags[0] is set.
void launch_refine_check(const double* d, const double* x, int segs, size_t len,
                         double* partial, double tol, int* flags, int* hflag, double* relcorr,
                         hipStream_t st);

// Backward-error stop test after a residual r = b - K x of B systems with nrhs
// right-hand sides each (see refine_be_check_kernel): |r| (rnorm) and |K| (knorm, per
// system) from the residual, |x| by block partials, |b| from bnorm.  Sets flags[0] when
// every normwise backward error is <= tol, else counts a correction (flags[1]) if count.
void launch_refine_be_check(const double* x, int B, int nrhs, size_t len, double* partial,
                            const double* rnorm, const double* knorm, const double* bnorm,
                            double tol, int count, int* flags, int* hflag, double* relcorr,
                            hipStream_t st);

// number of chain positions eliminated at level l (1-based) of a chain of length m
__host__ __device__ inline int level_count(int m, int l) {
  int ml = m >> (l - 1);
  return (ml + 1) >> 1;
}
__host__ __device__ inline int chain_levels(int m) {
  int L = 0;
  while ((m >> L) > 0) ++L;
  return L;  // floor(log2 m) + 1 for m >= 1, 0 for m = 0
}

// The top levels of a sweep have few positions per chain; they can share one launch with the
// x_1 step, mm_top_waves waves per chain (solve_rhs.hip).  How many of its waves are there for
// each of count positions; the pulls that a wave has in flight (as its registers allow: with two
// at n = 32 in FP64, a solve at S = N = 128 with twelve right-hand sides took 259 us instead of
// 254, at S = 300, N = 200 with three 652 instead of 633); the waves that the pulls occupy.
constexpr __host__ __device__ int mm_top_waves(int n) { return n <= 32 ? 8 : 4; }
constexpr __host__ __device__ int mm_top_share(int n, int count) {
  return mm_top_waves(n) / (count <= 1 ? 1 : count <= 2 ? 2 : count <= 4 ? 4 : 8);
}
constexpr __host__ __device__ int mm_pulls_per_wave(int n, bool fp64) {
  return n <= 16 || (n <= 32 && !fp64) ? 2 : 1;
}
constexpr __host__ __device__ int mm_pull_waves(int n, bool fp64, int pulls, int most) {
  const int w = mm_pulls_per_wave(n, fp64) == 2 ? (pulls + 1) / 2 : pulls;
  return w < 1 ? 1 : (w < most ? w : most);
}
// Lowest level of either sweep that may go into that launch (chain_levels(m) + 1: none):
// backward, as many positions per chain as it has waves; forward, half as many.
inline int bwd_top_level(int m, int n) {
  int l = chain_levels(m) + 1;
  while (l > 1 && level_count(m, l - 1) <= mm_top_waves(n)) --l;
  return l;
}
__host__ __device__ inline int fwd_top_level(int m, int n) {
  int l = chain_levels(m) + 1;
  while (l > 1 && level_count(m, l - 1) <= mm_top_waves(n) / 2) --l;
  return l;
}
// Waves of a forward level's workgroup: as many as its pulls occupy, at most four, or for the
// levels that may go into that launch as many as they would have there, so that the sums do
// not depend on whether they do.
__host__ __device__ inline int mm_fwd_waves(int m, int n, bool fp64, int level) {
  return mm_pull_waves(n, fp64, 2 * (level - 1), level >= fwd_top_level(m, n)
                                                     ? mm_top_share(n, level_count(m, level))
                                                     : 4);
}
// Few right-hand sides at n <= 32 go through the kernels that hold a block in a wave's registers
// (solve.hip), the others through matrix products, which read a block once for up to
// sixteen columns but cost the same for one of them, and pad n to 16 or 32 rows.  By a
// system's own sizes alone: its sums do not depend on the other systems of a launch.  One
// solve, products / registers, us:
//   two right-hand sides in FP64 at S = 60, N = 250 n = 8 82 / 59, n = 32 212 / 178, at S =
//   1500, N = 16 85 / 63 and 248 / 214; in FP32 at S = 20, N = 30 n = 12 31 / 34, n = 16 31 / 29, n
//   = 24 46 / 47.5, at S = 100, N = 20 44 / 46.5, at S = 60, N = 250 121 / 116, at S = 512, N = 32
//   107 / 92, n = 28 at S = 128, N = 200 154 / 159, at S = 512, N = 32 112 / 103;
//   three at S = 4, N = 16 n = 8 23.5 / 23 in FP64 and 22.5 / 23.5 in FP32, n = 16 25.5 / 27.5 in
//   FP64, at S = 400, N = 20 n = 16 50 / 55.5, at S = 1500, N = 16 n = 12 in FP64 97 / 92, n = 20
//   195 / 150 and in FP32 134 / 122, n = 12 84 / 83, n = 32 in FP64 265 / 242;
//   up to nine stages, where all forward levels are one launch of the products, two at S =
//   5, N = 9 in FP64 n = 24 34 / 40, n = 32 36 / 36, at S = 5000, N = 8 n = 24 304 / 245.
constexpr int kFewRhs = 3;
constexpr bool few_rhs(int S, int N, int n, int nrhs, bool fp64) {
  const bool one_launch = N <= 9 && S <= 256;
  if (n > 32 || nrhs > kFewRhs) return false;
  if (nrhs == 1 || (nrhs == 2 && (n <= 8 || n == 16 || n == 32))) return true;
  if (one_launch) return false;
  if (nrhs == 2)
    return fp64 || (n > 16 && (n % 4 != 0 || S > 256 || (n <= 24 && S > 32 && N > 32)));
  return n == 32 || (fp64 && n <= 8) || (n > 16 ? S > 256 : fp64 && S > 512);
}
// Backward, two right-hand sides of full 16 x 16 blocks in FP64 stay with the products, which
// need no padding there: both sweeps / the forward one in registers, one solve at S = 60, N = 100
// 55 / 53 us, at S = 256, N = 128 102 / 96, factor_solve at S = 4, N = 16 44.5 / 43.
constexpr bool few_bwd(int S, int N, int n, int nrhs, bool fp64) {
  return few_rhs(S, N, n, nrhs, fp64) && !(fp64 && nrhs == 2 && n == 16);
}
// The merged forward launch of these kernels, of sixteen waves, exists where a wave does with
// the 128 registers that it then has.
constexpr bool few_fwd_top(int n, bool fp64) { return n <= (fp64 ? 16 : 32); }
// Whether the top levels go into a launch with x_1, for so many chains in it: up to what the
// GPU holds at once (256 compute units with one workgroup each for n > 16, two below).
// Beyond that the barriers cost more than the launches they replace.  One solve, together /
// apart: one right-hand side at S = 100, N = 160, n = 16 in FP32 56 / 63 us, at S = 512, N = 64
// 62 / 65, at S = 768 81 / 81; four at n = 32, N = 64 in FP32 107 / 126 us at S = 256, 166 / 170
// at 384, in FP64 288 / 284; one at S = 5000, N = 16, n = 16 in FP64 277 / 205.
constexpr bool tops_together(int n, int64_t chains) { return chains <= (n <= 16 ? 512 : 256); }

}  // namespace bmpc
