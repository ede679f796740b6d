// Solve steps (Algorithm 2) as matrix products, for several right-hand sides and blocks of
// 33..64 (gfx950): the level kernel of both sweeps, and the x_1 steps together with the levels
// next to them.  (Few right-hand sides: solve.hip, solve64.hip.)  Layouts: solve_mm.h.
//
// Against scalar products per right-hand side with the vectors in LDS, in chunks of eight
// (four for n > 32), one solve: FP64 n = 32, S = N = 128, twelve right-hand sides 554 -> 254
// us (level 1 backward moves its blocks at 5.1 TB/s); FP32 n = 16, S = 100, N = 160, four
// 114 -> 72 us; FP64 n = 48, S = N = 64, one 213 -> 159 us; FP32 n = 64, S = N = 64, sixteen
// 676 -> 199 us.  Tried: tiles interleaved so that the transposed blocks come in 16-byte
// pieces (the backward levels above: 132 -> 149 us, the triangle's zeros are no longer whole
// tiles); one pull in flight and three waves per SIMD instead of two backward (132 -> 136
// us).
//
// The top levels have a few positions per chain and cost a launch's latency each (4.2 to 5
// us).  They share one launch with the x_1 step: a workgroup of eight waves (four for n > 32,
// where a wave takes more than half of a SIMD's registers) per chain, a barrier between
// levels.  Forward the waves divide among the positions of a level, which therefore have
// at most half as many, and share their pulls; backward every position (two pulls) has one
// wave.  One solve at S = 28, N = 214: FP32 n = 16 with four right-hand sides 77 -> 61 us, FP64
// n = 32 with twelve 158 -> 155 us.
#include <type_traits>

#include "bmpc_internal.h"
#include "multi.h"
#include "solve_mm.h"

namespace bmpc {

namespace {

// TOGETHER: a workgroup of a ragged launch, with as many waves as the launch's largest item
// asks for.
// Waves per SIMD that the registers of a level kernel leave room for.  FP64 at n <= 16 and the
// forward levels at n 33..48 come out just above such a limit when the compiler is left to
// itself: one wave instead of two costs the solve of 300 chains of 100 at n = 40 with four
// right-hand sides 19 %, four instead of five that of n = 8 2 %.  No bound makes a kernel spill.
constexpr int mm_level_waves_per_simd(bool fp64, int nt, bool bwd) {
  return !fp64 ? 1 : nt == 1 ? (bwd ? 6 : 5) : nt == 3 && !bwd ? 2 : 1;
}

template <typename T, int NT, int KIND, bool VEC, bool TOGETHER>
__device__ __attribute__((always_inline)) inline void mm_level_body(const SolveArgs& a, int level,
                                                                    int count, unsigned bx) {
  extern __shared__ __align__(16) unsigned char mm_smem[];
  if (a.done && *a.done) return;
  const int s = bx / count, i = (int)(bx - (unsigned)s * count), wv = wave_id();
  const int W = KIND == MM_BWD || a.fwd_waves == 1
                    ? 1
                    : mm_fwd_waves(a.m, a.n, sizeof(T) == 8, level);
  mm_position_body<T, NT, KIND, VEC, TOGETHER>(
      a, level, s, (2 * i + 1) << (level - 1), W, wv,
      reinterpret_cast<typename Mfma<T>::acc_t*>(mm_smem), wv < W);
}

// Forward levels level_lo.. of chain s, then its x_1 step.
template <typename T, int NT, bool VEC>
__device__ __attribute__((always_inline)) inline void mm_fwd_top_body(const SolveArgs& a,
                                                                      int level_lo, int s) {
  extern __shared__ __align__(16) unsigned char mm_smem[];
  if (a.done && *a.done) return;
  auto* const part = reinterpret_cast<typename Mfma<T>::acc_t*>(mm_smem);
  const int wv = wave_id(), L = chain_levels(a.m);
  for (int level = level_lo; level <= L; ++level) {
    const int count = level_count(a.m, level);
    const int per = mm_top_share(16 * NT, count), i = wv / per, w = wv - i * per;
    const int W = mm_pull_waves(16 * NT, sizeof(T) == 8, 2 * (level - 1), per);
    mm_position_body<T, NT, MM_FWD, VEC, true>(a, level, s, (2 * i + 1) << (level - 1), W, w,
                                               part + i * per * NT * 64, i < count && w < W);
    __syncthreads();
  }
  const int W = mm_pull_waves(16 * NT, sizeof(T) == 8, L, mm_top_waves(16 * NT));
  mm_position_body<T, NT, MM_X, VEC, true>(a, 0, s, a.N, W, wv, part, wv < W);
}

// The x_1 backward step of chain s, then its backward levels down to level_lo.
template <typename T, int NT, bool VEC>
__device__ __attribute__((always_inline)) inline void mm_bwd_top_body(const SolveArgs& a,
                                                                      int level_lo, int s) {
  if (a.done && *a.done) return;
  const int wv = wave_id();
  if (wv == 0) mm_x_bwd_body<T, NT, VEC>(a, s);
  for (int level = chain_levels(a.m); level >= level_lo; --level) {
    __syncthreads();
    if (wv < level_count(a.m, level))
      mm_position_body<T, NT, MM_BWD, VEC, false, sizeof(T) == 8 && NT % 2 == 0>(
          a, level, s, (2 * wv + 1) << (level - 1), 1, 0, nullptr, true);
  }
}

template <typename T, int NT, int KIND, bool VEC>
__global__ void __launch_bounds__(KIND == MM_BWD ? 64 : 64 * mm_top_waves(16 * NT),
                                  mm_level_waves_per_simd(sizeof(T) == 8, NT, KIND == MM_BWD))
    mm_level_kernel(SolveArgs a, int level, int count) {
  mm_level_body<T, NT, KIND, VEC, false>(a, level, count, blockIdx.x);
}
template <typename T, int NT, bool FWD, bool VEC>
__global__ void __launch_bounds__(64 * mm_top_waves(16 * NT))
    mm_top_kernel(SolveArgs a, int level_lo) {
  if constexpr (FWD)
    mm_fwd_top_body<T, NT, VEC>(a, level_lo, blockIdx.x);
  else
    mm_bwd_top_body<T, NT, VEC>(a, level_lo, blockIdx.x);
}

// one launch over the systems of a ragged batch (see multi.h); items carry (level, count) or
// level_lo in p0, p1
template <typename T, int NT, int KIND, bool VEC>
__global__ void __launch_bounds__(KIND == MM_BWD ? 64 : 64 * mm_top_waves(16 * NT),
                                  mm_level_waves_per_simd(sizeof(T) == 8, NT, KIND == MM_BWD))
    mm_level_multi(const MultiItem<SolveArgs>* items, int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  mm_level_body<T, NT, KIND, VEC, KIND == MM_FWD>(relocate_solve(it.a, r), it.p0, it.p1,
                                                  multi_local(it).x);
}
template <typename T, int NT, bool FWD, bool VEC>
__global__ void __launch_bounds__(64 * mm_top_waves(16 * NT))
    mm_top_multi(const MultiItem<SolveArgs>* items, int nitems, Reloc r) {
  const MultiItem<SolveArgs>& it = items[multi_find(items, nitems, blockIdx.x)];
  if constexpr (FWD)
    mm_fwd_top_body<T, NT, VEC>(relocate_solve(it.a, r), it.p0, multi_local(it).x);
  else
    mm_bwd_top_body<T, NT, VEC>(relocate_solve(it.a, r), it.p0, multi_local(it).x);
}

// f(NT, VEC as std::integral_constant) for block size n
template <int MAXNT, typename F>
void mm_dispatch(int n, F&& f) {
  auto vec = [&](auto nt) {
    if (n % 4 == 0)
      f(nt, std::true_type{});
    else
      f(nt, std::false_type{});
  };
  const int nt = (n + 15) / 16;
  if (nt == 1) return vec(std::integral_constant<int, 1>{});
  if (nt == 2) return vec(std::integral_constant<int, 2>{});
  if constexpr (MAXNT > 2) {
    if (nt == 3) return vec(std::integral_constant<int, 3>{});
    vec(std::integral_constant<int, 4>{});
  }
}

size_t mm_lds(bool fp64, int n, int slots) {
  return (size_t)slots * ((n + 15) / 16) * 64 * 4 * (fp64 ? 8 : 4);
}

}  // namespace

LevelCfg mm_level_config(const SolveArgs& a, int level, bool fwd, bool fp64) {
  LevelCfg c{};
  c.kind = SK_LEVEL;
  c.count = level_count(a.m, level);
  const int waves = fwd && a.fwd_waves != 1 ? mm_fwd_waves(a.m, a.n, fp64, level) : 1;
  c.threads = 64 * waves;
  c.lds = mm_lds(fp64, a.n, waves - 1);
  c.gx = (unsigned)(a.B * a.S) * (unsigned)std::max(c.count, 0);
  c.gy = c.gz = 1;
  return c;
}
// Threads and LDS of the launch with the x_1 step and the levels from level_lo on.
MmTopCfg mm_top_config(const SolveArgs& a, int level_lo, bool fwd, bool fp64) {
  const int L = chain_levels(a.m), most = mm_top_waves(a.n);
  int waves = most;
  if (level_lo > L)
    waves = fwd ? mm_pull_waves(a.n, fp64, L, most) : 1;
  else if (!fwd)
    waves = level_count(a.m, level_lo);
  return {64u * waves, fwd ? mm_lds(fp64, a.n, waves) : 0};
}

template <typename T>
void launch_mm_level(const SolveArgs& a, int level, bool fwd, hipStream_t st) {
  const LevelCfg c = mm_level_config(a, level, fwd, sizeof(T) == 8);
  if (c.count <= 0) return;
  const dim3 g(c.gx), b(c.threads);
  mm_dispatch<4>(a.n, [&](auto nt, auto vec) {
    constexpr int NT = decltype(nt)::value;
    constexpr bool V = decltype(vec)::value;
    if (fwd)
      hipLaunchKernelGGL((mm_level_kernel<T, NT, MM_FWD, V>), g, b, c.lds, st, a, level, c.count);
    else
      hipLaunchKernelGGL((mm_level_kernel<T, NT, MM_BWD, V>), g, b, c.lds, st, a, level, c.count);
  });
}
template <typename T>
void launch_mm_top(const SolveArgs& a, int level_lo, bool fwd, hipStream_t st) {
  const dim3 g((unsigned)(a.B * a.S));
  const MmTopCfg c = mm_top_config(a, level_lo, fwd, sizeof(T) == 8);
  const dim3 b(c.threads);
  mm_dispatch<4>(a.n, [&](auto nt, auto vec) {
    constexpr int NT = decltype(nt)::value;
    constexpr bool V = decltype(vec)::value;
    if (fwd)
      hipLaunchKernelGGL((mm_top_kernel<T, NT, true, V>), g, b, c.lds, st, a, level_lo);
    else
      hipLaunchKernelGGL((mm_top_kernel<T, NT, false, V>), g, b, c.lds, st, a, level_lo);
  });
}
template <typename T>
void launch_mm_multi(int kind, bool fwd, int n, const MultiItem<SolveArgs>* items, int nitems,
                     unsigned blocks, unsigned threads, size_t lds, const Reloc& r,
                     hipStream_t st) {
  const dim3 g(blocks), b(threads);
  mm_dispatch<2>(n, [&](auto nt, auto vec) {
    constexpr int NT = decltype(nt)::value;
    constexpr bool V = decltype(vec)::value;
    if (kind == SK_MM_TOP && fwd)
      hipLaunchKernelGGL((mm_top_multi<T, NT, true, V>), g, b, lds, st, items, nitems, r);
    else if (kind == SK_MM_TOP)
      hipLaunchKernelGGL((mm_top_multi<T, NT, false, V>), g, b, lds, st, items, nitems, r);
    else if (fwd)
      hipLaunchKernelGGL((mm_level_multi<T, NT, MM_FWD, V>), g, b, lds, st, items, nitems, r);
    else
      hipLaunchKernelGGL((mm_level_multi<T, NT, MM_BWD, V>), g, b, lds, st, items, nitems, r);
  });
}
#define BMPC_MM(T)                                                                              \
  template void launch_mm_level<T>(const SolveArgs&, int, bool, hipStream_t);                   \
  template void launch_mm_top<T>(const SolveArgs&, int, bool, hipStream_t);                     \
  template void launch_mm_multi<T>(int, bool, int, const MultiItem<SolveArgs>*, int, unsigned,  \
                                   unsigned, size_t, const Reloc&, hipStream_t);
BMPC_MM(double)
BMPC_MM(float)
#undef BMPC_MM

}  // namespace bmpc
