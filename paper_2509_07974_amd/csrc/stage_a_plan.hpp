// Shared by the two pair kernels of stage (a): the orders that each
// per-galaxy weight is summed over, and wave-level primitives.
#pragma once

#include "fpcf4_internal.hpp"

namespace fpcf4 {
namespace sa {

enum { FA = 0, FB, FC, FD, FW, FE, FV, NF };

// Order plan.  The plan index n is the record order nmax for the 4PCF; an
// index 3PCF_PLAN + m selects the plan of the shear 3PCF on records of order
// m: the same record layout, but only the orders the 3PCF reads are formed
// (G up to 2m + 3, W up to 2m, and of the same-neighbour families Q up to 6,
// A up to 2, V at 0: the blocks Q_-6, Q_-2, A_2, V_0 of its corrections),
// and no triple-counting blocks.
constexpr int PLAN3 = 100;
__host__ __device__ constexpr bool is3(int n) { return n >= PLAN3; }
__host__ __device__ constexpr int nord(int n) { return is3(n) ? n - PLAN3 : n; }
// special units of pass 0: P8, Q8, P4, Q4, EA4, EB4 (complex); EA0, EB0, U (real)
__host__ __device__ constexpr int nspecial(int n) { return is3(n) ? 0 : 15; }

__host__ __device__ constexpr int kmax_f(int n, int f) {
  return is3(n) ? ((f == FA || f == FB) ? 2 * nord(n) + 3
                 : (f == FC || f == FD) ? 6
                 : (f == FE)            ? 2
                 : (f == FW)            ? 2 * nord(n)
                                        : 0)
                : ((f == FA || f == FB) ? 2 * n + 3
                 : (f == FC || f == FD) ? imax(2 * n + 5, n + 6)
                 : (f == FE)            ? imax(2 * n + 1, n + 2)
                                        : 2 * n);
}
__host__ __device__ constexpr int ktop(int n) {
  return is3(n) ? imax(2 * nord(n) + 3, 6) : imax(2 * n + 5, n + 6);
}
__host__ __device__ constexpr int units_at(int n, int k) {
  int u = 0;
  for (int f = 0; f < NF; ++f)
    if (k <= kmax_f(n, f)) u += (k == 0 ? 1 : 2);
  return u;
}
__host__ __device__ constexpr int total_units(int n) {
  int u = nspecial(n);
  for (int k = 0; k <= ktop(n); ++k) u += units_at(n, k);
  return u;
}
__device__ __forceinline__ double r2_exact(double dx, double dy) {
#pragma clang fp contract(off)
  const double a = dx * dx;
  const double b = dy * dy;
  return a + b;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ unsigned lane_id() { return __lane_id(); }

__device__ __forceinline__ unsigned rank_in_mask(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Whether a launch is the one that findings of faint octets rule out (the same
// for every workgroup of it).
__device__ __forceinline__ bool ruled_out(const StageAArgs& a) {
  if (a.when == RUN_ALWAYS) return false;
  bool faint = false;
  for (int d = 0; d <= TREE_LEVELS_MAX; ++d)
    if ((a.faint_of >> d & 1u) != 0u) faint |= a.faint[d] != 0u;
  return faint != (a.when == RUN_IF_FAINT);
}

// Plans that the matrix-core kernel serves.
__host__ __device__ constexpr bool use_matrix(int n) { return matrix_order(is3(n) ? 3 : 4, nord(n)); }

}  // namespace sa
}  // namespace fpcf4
