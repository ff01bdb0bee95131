// Device helpers shared by the element and vector kernels: wave-level sums,
// the PCG scalars of a system, and the rigid-motion removal.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "mto_kernels.hpp"

namespace mto {

typedef const __attribute__((address_space(4))) double* cptr;  // read-only tables, through the scalar cache
__device__ __forceinline__ cptr scalar_table(const double* p) { return (cptr)(uintptr_t)p; }

// Sum of arr[a..b) by one wave: strided sequential sums per lane, then a xor
// butterfly.  Every lane ends with the same bits, and so does every wave that
// calls it on the same range.
__device__ __forceinline__ double wave_sum(const double* __restrict__ arr, int a, int b) {
  const int lane = threadIdx.x & 63;
  // four loads per lane are requested before any is added (a quarter of the
  // memory round trips); each lane still adds its terms in index order, an
  // absent term as +0.0, so the sum is the same as term by term
  double v = 0.0;
  for (int k = a + lane; k < b; k += 256) {
    double x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // unconditional (clamped) loads, absent terms zeroed after
      const double t = arr[min(k + 64 * u, b - 1)];
      x[u] = k + 64 * u < b ? t : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) v += x[u];
  }
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

// N wave_sum reductions over the same chunk range in one pass: each
// array's terms are added in wave_sum's order, so the results are identical
// to N calls, at one memory round trip instead of N.
template <int N>
__device__ __forceinline__ void wave_sum_n(const double* const (&arr)[N], int a, int b, double (&out)[N]) {
  const int lane = threadIdx.x & 63;
  double v[N];
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] = 0.0;
  for (int k = a + lane; k < b; k += 256) {
    double tv[N][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // unconditional (clamped) loads, absent terms zeroed after
      const int kk = min(k + 64 * u, b - 1);
      const bool in = k + 64 * u < b;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const double x = arr[j][kk];
        tv[j][u] = in ? x : 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int j = 0; j < N; ++j) v[j] += tv[j][u];
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] += __shfl_xor(v[j], m);
#pragma unroll
  for (int j = 0; j < N; ++j) out[j] = v[j];
}

// The stop threshold of a PCG cycle on r.r: rtol^2 f.f, or, when larger, the
// rounding floor of the cycle's residual recurrence, (4 eps ||D x||)^2 with
// D = diag(K) (xx = sum of (D x)_i^2 over the system).  Below that floor the
// recursive residual keeps falling but the true residual of x does not (the
// FP64 product K x carries errors of about eps |K| |x|, large where regions
// joined to the supports through void material move far); the cycle stops
// there and the refinement restart, from the double-double true residual,
// continues with a small correction.  4 eps ||D x|| is about the floor
// measured on the mixed batch (its true residual after the cycle is 2.6 to
// 3.9 times eps ||D x||), and far below rtol ||f|| where x stays moderate.
__device__ __forceinline__ double stop_thr2(const PcgDev& s, int sys, double xx) {
  constexpr double G2 = 16.0 * 0x1p-106;  // (4 eps)^2, eps = 2^-53
  return fmax(s.tol2[sys], G2 * xx);
}

struct Scal {
  bool active;
  double beta;
};

// Convergence state and beta of system `sys` (partial sums in chunks
// [pc_begin, pc_end)) at iteration `it`.  A newly converged system is latched
// by a designated thread of the caller.
__device__ __forceinline__ Scal pcg_state(const PcgDev& s, int sys, int pc_begin, int pc_end, int it,
                                          bool want_beta) {
  const int pi = it & 1;
  const int st = s.status[sys];
  double rr, xx, rz_new = 0.0, rz_old = 1.0;
  if (want_beta && it > 0) {
    const double* const arr[4] = {s.part_rr + pi * s.n_chunks, s.part_rz + pi * s.n_chunks,
                                  s.part_rz + (pi ^ 1) * s.n_chunks, s.part_xx + pi * s.n_chunks};
    double out[4];
    wave_sum_n<4>(arr, pc_begin, pc_end, out);
    rr = out[0];
    rz_new = out[1];
    rz_old = out[2];
    xx = out[3];
  } else {
    const double* const arr[2] = {s.part_rr + pi * s.n_chunks, s.part_xx + pi * s.n_chunks};
    double out[2];
    wave_sum_n<2>(arr, pc_begin, pc_end, out);
    rr = out[0];
    xx = out[1];
  }
  Scal o;
  o.active = (st == SYS_RUNNING) && !(rr <= stop_thr2(s, sys, xx));
  o.beta = (want_beta && it > 0) ? rz_new / rz_old : 0.0;
  return o;
}

// Removing an element's rigid motion (exact for the products: K_s annihilates
// rigid motions, its FP64 rounding does not, and a region joined to the
// supports through void material moves rigidly by ~1e9 times its
// deformation).  The rigid motion (a - th y, b + th x) takes the element
// vector's values at DOF 0 (vertex (0,0) x), 1 (its y) and 3 (vertex (1,0)
// y); only the four vertex functions carry it.  For local DOF `row` of an
// order-P element with value xv, x0 = value of DOF 0, x1 = of DOF 1,
// th = x3 - x1: the deformation part, formed as the difference of nearby
// values first ((xv - x0) and x3 - x1 are exact when the values are within a
// factor 2 of each other), so its rounding is relative to the deformation,
// not to the rigid motion.  Non-vertex DOFs are returned unchanged.
template <int P>
__device__ __forceinline__ double rigid_free(double xv, int row, double x0, double x1, double th) {
  const int a = row >> 1, i = a % (P + 1), j = a / (P + 1);
  if (i > 1 || j > 1) return xv;
  return (row & 1) ? (xv - x1) - th * i : (xv - x0) + th * j;
}

template <int P>
__device__ __forceinline__ int vertex_dof(int v) {  // v = 0..7: vertices (0,0), (1,0), (0,1), (1,1), x and y
  return v < 4 ? v : 2 * (P + 1) + (v - 4);
}

// Launches kernel k; with events the launch carries them on its own dispatch
// packet, so they time exactly this kernel (no separate marker packets).
template <typename K, typename... Args>
void launch_timed(K k, dim3 grid, dim3 block, uint32_t lds, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1,
                  Args... args) {
  if (ev0 || ev1)
    hipExtLaunchKernelGGL(k, grid, block, lds, st, ev0, ev1, 0u, args...);
  else
    hipLaunchKernelGGL(k, grid, block, lds, st, args...);
}

}  // namespace mto
