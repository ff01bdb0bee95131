// Refinement indicators of Sec. 3.2 and the dp update of Sec. 3.3.
//
// Analysis indicator (Sec. 3.2.1, Kelly): Gamma^a of an element is the sum
// over its interior edges F of c_F * integral_F |[du/dn]|^2 ds, c_F =
// h_F / (2 p_F), h_F the element diagonal (sqrt 2 in element units), p_F the
// larger order of the two elements.  Each element sums its own four edges, so
// an edge is integrated once from each side and no atomics or edge arrays are
// needed.
//
// Density indicator (Sec. 3.2.2): one thread per element sums the four
// cases over its cells.
//
// dp update (Sec. 3.3, steps 2-4): host code (ranking, flags, smoothing).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "mto_internal.hpp"
#include "mto_kernels.hpp"

namespace mto {
namespace {

constexpr int AD_BLOCK = 64;

// Kelly indicator on a patch of AD_X x AD_Y elements of one system, their
// neighbours around it (the halo) read with them.
//   Along an edge both sides use the same hierarchic functions of the tangent,
// so the jump is a polynomial whose coefficients are sums of element values
// (phi_i'(+-1) = -+1/2, 1/2, (+-1)^(i-1)), and its squared integral is a sum of
// squares of its Legendre coefficients: no quadrature, no basis evaluation.
//   The bytes are small (a 200 x 100 mesh: 17 MB with two systems), so the time
// is the chain of dependent loads (element -> group -> index -> value); the
// patch's values are therefore gathered by all threads at once, several loads
// in flight each, into LDS [row][element], where lanes are elements and the
// wave is the side: no divergence, and an edge within the patch costs no
// second gather.  200 x 100 mesh, p = 1..4, two systems: 350 us with a thread
// per element and its vectors in private arrays, 20 us with eight loads in
// flight per thread and two blocks per CU, 12.5 us with eleven and three.
constexpr int AD_X = 16, AD_Y = 4, AD_HX = AD_X + 2, AD_H = AD_HX * (AD_Y + 2);
static_assert(AD_X * AD_Y == 64, "a lane per element of the patch");

// Coefficients (x, y) of the outward normal derivative along one side of the
// element whose values are at w[((j N + i) 2 + c) AD_H], functions above its
// order zero; V: a vertical side (the normal is along x, i runs across it),
// HI: the side at +1.
template <int N, bool V, bool HI>
__device__ __forceinline__ void side_gradient(const double* w, double (&g)[N][2]) {
#pragma unroll
  for (int t = 0; t < N; ++t)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      auto at = [&](int k) { return w[((V ? t * N + k : k * N + t) * 2 + c) * AD_H]; };
      double v = at(1) - at(0);  // 2 phi': d/dx = 2 d/dxi on the unit element
#pragma unroll
      for (int k = 2; k < N; ++k) v = fma((HI || (k & 1)) ? 2.0 : -2.0, at(k), v);
      g[t][c] = HI ? v : -v;
    }
}

template <int N, int S>
__device__ __forceinline__ double edge_integral(const double* w, int h) {
  constexpr int NB = S == 0 ? -1 : S == 1 ? 1 : S == 2 ? -AD_HX : AD_HX;
  double own[N][2], nb[N][2];
  side_gradient<N, (S < 2), (S & 1) != 0>(w + h, own);
  side_gradient<N, (S < 2), (S & 1) == 0>(w + h + NB, nb);
  double sum = 0.0;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double J[7] = {};
#pragma unroll
    for (int t = 0; t < N; ++t) J[t] = own[t][c] + nb[t][c];  // outward normals are opposite
    // phi_k = (P_k - P_{k-2}) / (2 k - 1): the Legendre coefficients of the jump
    const double L[5] = {0.5 * (J[0] + J[1]) - J[2] * (1.0 / 3), 0.5 * (J[1] - J[0]) - J[3] * (1.0 / 5),
                         J[2] * (1.0 / 3) - J[4] * (1.0 / 7),
                         J[3] * (1.0 / 5), J[4] * (1.0 / 7)};
#pragma unroll
    for (int k = 0; k < N; ++k) sum = fma(L[k] * (1.0 / (2 * k + 1)), L[k], sum);  // ds = dt / 2
  }
  return sum;
}

template <int PM>
__global__ __launch_bounds__(256, 3) void k_kelly(AdaptDev a, const SysDesc* __restrict__ sys,
                                               const double* __restrict__ x, double* __restrict__ gamma) {
  constexpr int N = PM + 1, NV = 2 * N * N, TASKS = NV * AD_H, BATCH = 11;
  __shared__ double w[TASKS];
  __shared__ const int32_t* col[AD_H];  // the element's column of its group's index table
  __shared__ int npad[AD_H], order[AD_H];
  __shared__ double part[4][64];
  const SysDesc& sd = sys[blockIdx.y];
  const int inst = sd.inst, nelx = a.nelx[inst], nely = a.nely[inst], nel = nelx * nely;
  const int px = (nelx + AD_X - 1) / AD_X, bx = blockIdx.x % px, by = blockIdx.x / px;
  if (by * AD_Y >= nely) return;
  const int x0 = bx * AD_X - 1, y0 = by * AD_Y - 1;
  const double* __restrict__ xs = x + sd.dof_off;
  if (threadIdx.x < AD_H) {
    const int ex = x0 + (int)threadIdx.x % AD_HX, ey = y0 + (int)threadIdx.x / AD_HX;
    int p = 0;
    if (ex >= 0 && ex < nelx && ey >= 0 && ey < nely) {
      const int64_t gel = a.el_base[inst] + (int64_t)ey * nelx + ex;
      const GroupDev& G = a.groups[a.el_group[gel]];
      p = G.p;
      npad[threadIdx.x] = G.npad;
      col[threadIdx.x] = G.gidx + a.el_col[gel];
    }
    order[threadIdx.x] = p;
  }
  __syncthreads();
  for (int t0 = threadIdx.x; t0 < TASKS; t0 += 256 * BATCH) {
    int gi[BATCH];
#pragma unroll
    for (int q = 0; q < BATCH; ++q) {
      const int t = min(t0 + 256 * q, TASKS - 1), r = t / AD_H, h = t - r * AD_H;
      const int p = order[h], c = r & 1, i = (r >> 1) % N, j = (r >> 1) / N;
      const bool there = p > 0 && i <= p && j <= p;
      gi[q] = there ? col[h][(int64_t)(2 * (j * (p + 1) + i) + c) * npad[h]] : -1;
    }
#pragma unroll
    for (int q = 0; q < BATCH; ++q) {
      const double v = xs[max(gi[q], 0)];
      if (t0 + 256 * q < TASKS) w[t0 + 256 * q] = gi[q] >= 0 ? v : 0.0;
    }
  }
  __syncthreads();
  const int side = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int h = (lane / AD_X + 1) * AD_HX + lane % AD_X + 1;
  const int hf = h + (side == 0 ? -1 : side == 1 ? 1 : side == 2 ? -AD_HX : AD_HX);
  const int pe = order[h], pf = order[hf];
  double integral;
  switch (side) {
    case 0: integral = edge_integral<N, 0>(w, h); break;
    case 1: integral = edge_integral<N, 1>(w, h); break;
    case 2: integral = edge_integral<N, 2>(w, h); break;
    default: integral = edge_integral<N, 3>(w, h); break;
  }
  // c_F = h_F / (2 p_F); a boundary edge has no jump
  part[side][lane] = pf > 0 ? 1.4142135623730950488 / (2.0 * max(pe, pf)) * integral : 0.0;
  __syncthreads();
  if (side == 0 && pe > 0) {
    const int e = (y0 + 1 + lane / AD_X) * nelx + x0 + 1 + lane % AD_X;
    gamma[a.inst_eoff[inst] + (int64_t)sd.load * nel + e] =
        ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
  }
}

// Bound by its divisions and by the chain of its loads: 11.1 us on a 200 x 100
// mesh with d = 2..5 with a division per case and a load at a time, 8.0 as below.
__global__ __launch_bounds__(AD_BLOCK) void k_density_ind(AdaptDev a, const double* __restrict__ rho,
                                                          DensityBounds b, double* __restrict__ gamma,
                                                          int64_t n_el) {
  const int64_t gel = (int64_t)blockIdx.x * AD_BLOCK + threadIdx.x;
  if (gel >= n_el) return;
  const int g = a.el_group[gel], k = a.el_col[gel];
  const GroupDev& G = a.groups[g];
  const int n = G.S;
  const double* __restrict__ r = rho + G.cell[k];
  // x / n to the last bit: the quotient from the correctly rounded reciprocal
  // and one correction by its exact remainder (Markstein's division).  An
  // infinite x has no remainder and gives NaN here; the sum then goes by
  // divisions, which a test of every quotient would cost 1.5 us of 8.
  const double dn = (double)n, rn = 1.0 / dn;
  auto sum = [&](auto over_n) {
    double acc = 0.0;
    constexpr int BATCH = 9;  // loads in flight
    for (int j0 = 0; j0 < n; j0 += BATCH) {
      double vs[BATCH];
#pragma unroll
      for (int q = 0; q < BATCH; ++q) vs[q] = r[min(j0 + q, n - 1)];
#pragma unroll
      for (int q = 0; q < BATCH; ++q) {
        const double v = vs[q];
        if (j0 + q >= n) break;
        if (b.rl <= v && v <= b.avg) acc += over_n(v - b.rl);
        if (b.avg < v && v <= b.ru) acc += over_n(b.ru - v);
        if (v <= b.cl) acc -= over_n(b.cl - v);
        if (v >= b.cu) acc -= over_n(v - b.cu);
      }
    }
    return acc;
  };
  double acc = sum([&](double x) {
    const double q = x * rn;
    return fma(fma(-q, dn, x), rn, q);
  });
  if (__builtin_isnan(acc)) acc = sum([&](double x) { return x / dn; });
  gamma[gel] = acc;
}

}  // namespace

// n_patch: the most patches of any instance; p_max: the largest order
int kelly_patches(int nelx, int nely) { return (nelx + AD_X - 1) / AD_X * ((nely + AD_Y - 1) / AD_Y); }

void launch_kelly(const AdaptDev& a, const SysDesc* sys, int n_sys, int n_patch, int p_max, const double* x,
                  double* gamma, hipStream_t st) {
  if (n_sys == 0 || n_patch == 0) return;
  const dim3 grid(n_patch, n_sys), block(256);
  switch (p_max) {
    case 1: hipLaunchKernelGGL(k_kelly<1>, grid, block, 0, st, a, sys, x, gamma); break;
    case 2: hipLaunchKernelGGL(k_kelly<2>, grid, block, 0, st, a, sys, x, gamma); break;
    case 3: hipLaunchKernelGGL(k_kelly<3>, grid, block, 0, st, a, sys, x, gamma); break;
    default: hipLaunchKernelGGL(k_kelly<4>, grid, block, 0, st, a, sys, x, gamma); break;
  }
}

void launch_density_indicator(const AdaptDev& a, const double* rho, const DensityBounds& b, double* gamma,
                              int64_t n_el, hipStream_t st) {
  if (n_el == 0) return;
  hipLaunchKernelGGL(k_density_ind, dim3((unsigned)((n_el + AD_BLOCK - 1) / AD_BLOCK)), dim3(AD_BLOCK), 0, st, a,
                     rho, b, gamma, n_el);
}

}  // namespace mto

// ---- host: dp update (Sec. 3.3) ----

namespace {

// elements in ascending order of v, ties by element index
std::vector<int> ranking(const double* v, int n) {
  std::vector<int> o(n);
  std::iota(o.begin(), o.end(), 0);
  std::stable_sort(o.begin(), o.end(), [&](int a, int b) { return v[a] < v[b]; });
  return o;
}

// Raise the lower order of neighbours until they differ by at most 2:
// (p_max - p_min - 2) passes, rows bottom to top, each element against its
// right and upper neighbour, in place (Sec. 3.3, step 3c).
void smooth(std::vector<int>& p, int nelx, int nely) {
  const auto mm = std::minmax_element(p.begin(), p.end());
  const int passes = std::max(0, *mm.second - *mm.first - 2);
  for (int it = 0; it < passes; ++it)
    for (int ey = 0; ey < nely; ++ey)
      for (int ex = 0; ex < nelx; ++ex) {
        const int e = ey * nelx + ex;
        const int nb[2] = {ex + 1 < nelx ? e + 1 : -1, ey + 1 < nely ? e + nelx : -1};
        for (int f : nb) {
          if (f < 0) continue;
          if (p[e] < p[f] - 2) p[e] = p[f] - 2;
          else if (p[f] < p[e] - 2) p[f] = p[e] - 2;
        }
      }
}

}  // namespace

extern "C" {

int mto_dp_update(int32_t nelx, int32_t nely, const int8_t* p_in, const double* gamma_a, const double* gamma_d,
                  const mto_dp_params* prm, int8_t* p_out, int8_t* theta_out, int32_t* design_points,
                  int32_t* cells_per_element) {
  mto::clear_error();
  if (nelx < 1 || nely < 1 || !p_in || !gamma_a || !gamma_d || !prm || !p_out || !theta_out || !design_points ||
      !cells_per_element)
    return mto::set_error(MTO_EINVAL, "dp update: bad arguments");
  if (prm->p_max < 1 || prm->p_max > 126 || prm->d_max < 1 || !(prm->frac_a_refine >= 0 && prm->frac_a_refine <= 1) ||
      !(prm->frac_a_coarsen >= 0 && prm->frac_a_coarsen <= 1) || !(prm->frac_d_refine >= 0 && prm->frac_d_refine <= 1) ||
      !(prm->frac_d_coarsen >= 0 && prm->frac_d_coarsen <= 1))
    return mto::set_error(MTO_EINVAL, "dp update: parameters out of range");
  const int n = nelx * nely;
  std::vector<int> p(n), th(n, 0);
  for (int k = 0; k < n; ++k) {
    if (p_in[k] < 1) return mto::set_error(MTO_EINVAL, "dp update: p < 1");
    p[k] = p_in[k];
  }
  // step 2: analysis indicator, bottom fraction coarsened, top fraction refined
  {
    const std::vector<int> o = ranking(gamma_a, n);
    const int nc = (int)std::floor(prm->frac_a_coarsen * n), nr = (int)std::floor(prm->frac_a_refine * n);
    for (int k = 0; k < nc; ++k) th[o[k]] = -1;
    for (int k = n - nr; k < n; ++k) th[o[k]] = 1;
    for (int k = 0; k < n; ++k) p[k] = std::min(std::max(p[k] + th[k], 1), (int)prm->p_max);
  }
  // step 3: density indicator among the elements with Gamma^d < 0 (coarsen) and > 0 (refine)
  {
    const std::vector<int> o = ranking(gamma_d, n);
    std::vector<int> neg, pos;
    for (int k : o) {
      if (gamma_d[k] < 0.0) neg.push_back(k);
      else if (gamma_d[k] > 0.0) pos.push_back(k);
    }
    const int nc = (int)std::floor(prm->frac_d_coarsen * neg.size());
    const int nr = (int)std::floor(prm->frac_d_refine * pos.size());
    for (int m = 0; m < nc; ++m) {
      const int k = neg[m];
      if (p[k] == 1) th[k] = -2;
      else if (th[k] == 0) p[k] -= 1;
    }
    for (int m = (int)pos.size() - nr; m < (int)pos.size(); ++m) {
      const int k = pos[m];
      if (th[k] == 0 || th[k] == -1) p[k] = std::min(p[k] + 1, (int)prm->p_max);
    }
  }
  smooth(p, nelx, nely);
  int dmax = 0;
  for (int k = 0; k < n; ++k) {
    p_out[k] = (int8_t)p[k];
    theta_out[k] = (int8_t)th[k];
    const int dof = 2 * (p[k] + 1) * (p[k] + 1) - 3;  // element DOFs minus the rigid modes
    design_points[k] = th[k] == -2 ? 1 : std::min(dof, (int)prm->d_max);
    dmax = std::max(dmax, design_points[k]);
  }
  int side = 1;
  while (side * side < dmax) ++side;
  *cells_per_element = side * side;
  return MTO_OK;
}

int mto_qr_update(int32_t nel, const int8_t* p_in, const double* eps, double alpha_qr, int32_t p_max, int8_t* p_out) {
  mto::clear_error();
  if (nel < 0 || !p_in || !eps || !p_out || p_max < 1 || p_max > 126)
    return mto::set_error(MTO_EINVAL, "QR update: bad arguments");
  for (int k = 0; k < nel; ++k) p_out[k] = (int8_t)std::min((int)p_in[k] + (eps[k] > alpha_qr ? 1 : 0), (int)p_max);
  return MTO_OK;
}

}  // extern "C"
