// QR-error indicator of Sec. 3.2.3 (Eq. (9)): per element, the strain
// energy of the order-(p+1) element problem under the element's own load,
// against the order-p energy.
//
// One wave per element (all load cases of its instance share one
// factorisation):
//   1. K' = sum_s E_s K_s^(p+1) into LDS as a packed lower triangle, by sum
//      factorisation on the matrix cores (see k_qr);
//   2. per load case, u_e from the free-DOF vector, minus the rigid motion
//      that the three pinned DOFs carry (vertex (0,0) x and y, vertex (1,0)
//      y), so that the pinned values are zero; f = K^(p) u_e, read from the
//      embedded block of K' (the hierarchic order-p functions are order-(p+1)
//      functions, and both matrices are integrated exactly, so that block is
//      K^(p)); J^(p) = u_e . f / 2;
//   3. the pinned rows and columns of K' are replaced by identity rows and
//      K' is factored, U^T U, in registers (blocked Cholesky on the matrix
//      cores);
//   4. K' u' = f' is solved for all load cases at once (f on the embedded DOFs;
//      on the new ones the integrals of the order-p load field against the new
//      functions, by the tensor product of the 1D transfer t; zero on the
//      pinned ones), then u' is refined twice against a double-double residual
//      computed from K' in LDS, J^(p+1) = f' . u' / 2 (the load is
//      self-equilibrated, so the pinned DOFs carry no reaction and the rigid
//      motion removed in 2 changes neither energy), eps = 1 - J^(p) / J^(p+1),
//      or 0 if J^(p+1) = 0.
// eps is a small difference of two energies wherever the order-p field is
// already good, and the cell moduli inside one element can differ by 1e9, so
// f, both energies and the residuals are accumulated in double-double.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "mto_internal.hpp"
#include "mto_kernels.hpp"

namespace mto {
namespace {

constexpr int QR_LOADS = 4;  // load cases per pass over one factorisation (of the 16 columns of a solve)

__device__ __forceinline__ int tri(int i, int j) { return i >= j ? i * (i + 1) / 2 + j : j * (j + 1) / 2 + i; }

// order-(p+1) local DOF of order-p local DOF 2 (j (p+1) + i) + c
template <int P>
__device__ __forceinline__ int emb(int d) {
  const int a = d >> 1, i = a % (P + 1), j = a / (P + 1);
  return 2 * (j * (P + 2) + i) + (d & 1);
}

__device__ __forceinline__ double readlane_d(double v, int l) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(u & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(u >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

#pragma clang fp contract(off)
// (hi, lo) += a * b, error-free product and two-sum
__device__ __forceinline__ void dd_fma(double a, double b, double& hi, double& lo) {
  const double p = a * b;
  const double e = fma(a, b, -p);
  const double s = hi + p;
  const double bb = s - hi;
  const double t = (hi - (s - bb)) + (p - bb);
  hi = s;
  lo += t + e;
}
// (hi, lo) += v
__device__ __forceinline__ void dd_add(double v, double& hi, double& lo) {
  const double s = hi + v;
  const double bb = s - hi;
  lo += (hi - (s - bb)) + (v - bb);
  hi = s;
}
// sum over the wave of (hi, lo) pairs, rounded
__device__ __forceinline__ double wave_sum_dd(double hi, double lo) {
  for (int o = 32; o > 0; o >>= 1) {
    const double h2 = __shfl_xor(hi, o), l2 = __shfl_xor(lo, o);
    dd_add(h2, hi, lo);
    lo += l2;
  }
  return hi + lo;
}
#pragma clang fp contract(on)

constexpr int qr_steps(int p) { return ((p + 2) * (p + 2) + 1) / 2; }  // pivot steps: four of the 2 (p + 2)^2 rows each
constexpr uint32_t qr_lds_bytes(int p) {
  const int nq = 2 * (p + 2) * (p + 2);
  return 8 * (nq * (nq + 1) + 16 * qr_steps(p) + QR_LOADS + 3 * QR_LOADS * nq);
}

typedef double d4q __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) double* lds_cptr;
__device__ __forceinline__ d4q mfma(double a, double b, d4q c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// 1 / sqrt(d): the hardware estimate and two Newton steps
__device__ __forceinline__ double rsqrt_d(double d) {
  const double hd = 0.5 * d;
  double r = __builtin_amdgcn_rsq(d);
  r *= fma(-hd * r, r, 1.5);
  r *= fma(-hd * r, r, 1.5);
  return r;
}

// v_mfma_f64_16x16x4f64: D += A B with A[l % 16][l / 16], B[l / 16][l % 16]
// and D[l / 16 + 4 r][l % 16] (register r) in lane l.
//   K': with the 1D integrals t = a, b, c of each cell interval, K' is a sum of
// products t_x(i, k) t_y(j, l) (mto_factor.hip).  M_t[sy][(i, k)] = sum_sx
// E[sy, sx] t_x^(sx)(i, k) is one contraction over sx, K'[(j, l)][(i, k)] of
// each component pair two over sy (two terms); D of the first is B of the
// second as it stands, and A there and B here are tables in fragment order.
// 120 products at p = 4, d = 5, where the sum over the cells' dense matrices
// read 525 KB of them and took 66 k multiply-adds.
//   U: tiles of the upper triangle in registers, four pivot rows at a time: the
// rows are register r = kb % 4 of tile row kb / 4, B operand as they stand and,
// transposed, A operand of the same lanes; with L the 4 x 4 pivot block's factor,
// W = L^-1 R becomes the rows of U and the trailing tiles lose W^T W.
//   The solves keep 16 right-hand sides in the D layout; forward, U is read
// from the registers, backward (transposed) from a copy in LDS.
//   What bounds it is the chain of one wave (18 pivot steps, 6 x 18 solve steps
// at p = 4) with three elements per CU in LDS (50 KB each at p = 4).  200 x 100
// mesh, p = 1..4, one load case (us): p = 4 1690 -> 380, the other orders 740 ->
// 215; before, 256 threads per element kept the triangle in LDS behind two
// barriers per column and substituted with one wave per load case.  Of these
// 595: factorisation 90, a refinement 113 (its residual 41), the scatter of K'
// 18.  At p = 4 the compiler gets 512 registers (the LDS allows no more than
// one wave per SIMD): held to 256 it spills, 536.
template <int P>
__global__ __launch_bounds__(64, P == 4 ? 1 : 2) void k_qr(QrGroupDev g, const double* __restrict__ E, const double* __restrict__ x,
                                           const SysDesc* __restrict__ sys, const int32_t* __restrict__ inst_sys0,
                                           const int32_t* __restrict__ inst_L, const int64_t* __restrict__ inst_eoff,
                                           const int32_t* __restrict__ inst_nel, double* __restrict__ eps) {
  constexpr int N = P + 2, N1 = P + 1, NE = 2 * N1 * N1, NQ = 2 * N * N, NT = NQ * (NQ + 1) / 2;
  constexpr int MB = (NQ + 15) / 16, NKB = qr_steps(P);                        // tiles, pivot steps
  constexpr int NP = N * (N + 1) / 2, RT = (NP + 15) / 16, CT = (N * N + 15) / 16;  // pairs j >= l, their tiles; (i, k)
  constexpr int NX = NQ > 64 ? NQ - 64 : 0, XL = NX > 0 ? 64 / NX : 1, XJ = (NQ + XL - 1) / XL;
  static_assert(NE <= 64 && NQ <= 128 && (NX == 0 || XL * NX <= 64), "rows per lane");
  // dynamic: with its size unknown the compiler keeps to the register bound
  // above, without moves to and from accumulation registers
  extern __shared__ double lds[];
  double* Kc = lds;                              // [NT] K', later with the identity rows
  double* Us = Kc + NT;                          // [NT] U[a][b], a <= b, at b (b + 1) / 2 + a
  double* Li = Us + NT;                          // [NKB][16] L^-1 of the pivot blocks, [m][k]
  double(*RH)[NQ] = (double(*)[NQ])(Li + NKB * 16 + QR_LOADS);  // f', high and low parts
  double(*RL)[NQ] = RH + QR_LOADS;
  double* Jp = Li + NKB * 16;                    // [QR_LOADS] J^(p)
  double(*X)[NQ] = RL + QR_LOADS;                // u_e; then u' and the right-hand sides of its refinement
  const int k = blockIdx.x;
  const int inst = g.einst[k], e = g.eid[k];
  const int64_t c0 = g.cell[k];
  const int nL = inst_L[inst], s0 = inst_sys0[inst], nel = inst_nel[inst], d = g.d;
  const d4q zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int l0 = 0; l0 < nL; l0 += QR_LOADS) {  // uniform
    const int nl = min(QR_LOADS, nL - l0);
    int lane = threadIdx.x;
    asm volatile("" : "+v"(lane));  // else every address below is kept in registers over this loop
    const int lr = lane >> 4, lc = lane & 15;
    for (int idx = lane; idx < nl * NE; idx += 64) {
      const int l = idx / NE, j = idx - l * NE;
      const int gi = g.gidx[(size_t)j * g.npad + k];
      X[l][j] = gi >= 0 ? x[sys[s0 + l0 + l].dof_off + gi] : 0.0;
    }
    {
      double Ef[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int sx = 4 * h + lr;
        const double v = E[c0 + min(lc, d - 1) * d + min(sx, d - 1)];
        Ef[h] = lc < d && sx < d ? v : 0.0;
      }
      const double* __restrict__ xf = g.tab + lane;
      const double* __restrict__ yf = g.tab + 4 * CT * 2 * 64 + lane;
      d4q M[4][CT];  // a, b, c, c^T
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          M[t][ct] = mfma(Ef[1], xf[((t * CT + ct) * 2 + 1) * 64], mfma(Ef[0], xf[(t * CT + ct) * 2 * 64], zero));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {  // component of the row, of the column
          const int ta = cc == 0 || cc == 3 ? 0 : cc == 1 ? 2 : 3, tb = cc == 0 || cc == 3 ? 1 : cc == 1 ? 3 : 2;
          double yv[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) yv[q] = yf[((cc * RT + rt) * 4 + q) * 64];
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            d4q D = mfma(yv[0], M[ta][ct][0], zero);
            D = mfma(yv[1], M[ta][ct][1], D);
            D = mfma(yv[2], M[tb][ct][0], D);
            D = mfma(yv[3], M[tb][ct][1], D);
            const int ik = 16 * ct + lc, i = ik / N, kk = ik - i * N;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int pr = 16 * rt + 4 * r + lr;
              const int j = (pr >= 1) + (pr >= 3) + (pr >= 6) + (pr >= 10) + (pr >= 15), l = pr - j * (j + 1) / 2;
              const int row = 2 * (j * N + i) + (cc >> 1), col = 2 * (l * N + kk) + (cc & 1);
              if (pr < NP && ik < N * N && row >= col) Kc[row * (row + 1) / 2 + col] = D[r];
            }
          }
        }
    }
    __syncthreads();
    {  // rigid motion (a - th y, b + th x) through the pinned values: a = u_x(0,0), b = u_y(0,0), th = u_y(1,0) - b
      double ud[QR_LOADS];
#pragma unroll
      for (int l = 0; l < QR_LOADS; ++l) {
        const int j = min(lane, NE - 1);
        const double a = X[l][0], b = X[l][1], th = X[l][3] - X[l][1];
        const int as = j >> 1, i1 = as % N1, j1 = as / N1;
        ud[l] = X[l][j];
        if (i1 <= 1 && j1 <= 1) ud[l] -= (j & 1) ? b + th * i1 : a - th * j1;
      }
      __syncthreads();
#pragma unroll
      for (int l = 0; l < QR_LOADS; ++l)
        if (l < nl && lane < NE) X[l][lane] = ud[l];
    }
    __syncthreads();
    // NL cases at a time, which share the reads of K'
    auto by_pairs = [&](auto body) {
#pragma unroll 1
      for (int l = 0; l < nl;) {
        if (l + 1 < nl) {
          body(std::integral_constant<int, 2>{}, l);
          l += 2;
        } else {
          body(std::integral_constant<int, 1>{}, l);
          ++l;
        }
      }
    };
    by_pairs([&](auto cases, int l) {
      constexpr int NL = decltype(cases)::value;
      const int i = min(lane, NE - 1), ei = emb<P>(i), eb = ei * (ei + 1) / 2;
      double hi[NL] = {}, lo[NL] = {};
#pragma unroll 2
      for (int j = 0; j < NE; ++j) {
        const int ej = emb<P>(j);
        const double kj = Kc[ej <= ei ? eb + ej : ej * (ej + 1) / 2 + ei];
#pragma unroll
        for (int h = 0; h < NL; ++h) dd_fma(kj, X[l + h][j], hi[h], lo[h]);
      }
#pragma unroll
      for (int h = 0; h < NL; ++h) {
        const double sh = hi[h] + lo[h], sl = lo[h] - (sh - hi[h]);
        double ah = 0.0, al = 0.0;
        if (lane < NE) {
          RH[l + h][ei] = sh;
          RL[l + h][ei] = sl;
          dd_fma(X[l + h][i], sh, ah, al);
          dd_fma(X[l + h][i], sl, ah, al);
        }
        const double v = 0.5 * wave_sum_dd(ah, al);
        if (lane == 0) Jp[l + h] = v;
      }
    });
    __syncthreads();
    // f' on the new functions: phi_{P+1}(x) phi_m(y) and phi_m(x) phi_{P+1}(y), m <= P, the transfer t
    // along the row m of f, then phi_{P+1} phi_{P+1}, t along the first of these
    auto transfer = [&](const double* rh, const double* rl, int first, int stride, int l, int r) {
      double hi = 0.0, lo = 0.0;
#pragma unroll
      for (int m = 0; m <= P; ++m) {
        const double th = rh[first + m * stride], tl = rl[first + m * stride];
        dd_fma(g.t[m], th, hi, lo);
        lo = fma(g.t[m], tl, lo);
      }
      const double sh = hi + lo;
      RH[l][r] = sh;
      RL[l][r] = lo - (sh - hi);
    };
    for (int idx = lane; idx < 4 * N1 * nl; idx += 64) {
      const int l = idx / (4 * N1), q = idx - l * 4 * N1, c = q & 1, m = (q >> 2), alongy = (q >> 1) & 1;
      transfer(RH[l], RL[l], alongy ? 2 * m + c : 2 * m * N + c, alongy ? 2 * N : 2, l,
               alongy ? 2 * ((P + 1) * N + m) + c : 2 * (m * N + P + 1) + c);
    }
    __syncthreads();
    if (lane < 2 * nl) {
      const int l = lane >> 1, c = lane & 1;
      transfer(RH[l], RL[l], 2 * (P + 1) + c, 2 * N, l, 2 * ((P + 1) * N + P + 1) + c);
    }
    for (int i = lane; i < NQ; i += 64) {  // identity rows and columns at the pinned DOFs
      const int pins[3] = {0, 1, 3};
      for (int c : pins) Kc[tri(i, c)] = i == c ? 1.0 : 0.0;
    }
    __syncthreads();
    if (lane < 3 * nl) RH[lane / 3][lane % 3 == 2 ? 3 : lane % 3] = RL[lane / 3][lane % 3 == 2 ? 3 : lane % 3] = 0.0;
    d4q U[MB][MB];  // tiles bj >= bi
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int bj = bi; bj < MB; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * bi + lr + 4 * r, b = 16 * bj + lc;
          const double v = Kc[tri(min(a, NQ - 1), min(b, NQ - 1))];
          U[bi][bj][r] = a < NQ && b < NQ ? v : a == b ? 1.0 : 0.0;
        }
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      const int bk = kb / 4, rk = kb % 4, pc0 = 4 * rk;
      double m[4][4], ri[4], li[4][4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = q; c < 4; ++c) {
          m[q][c] = readlane_d(U[bk][bk][rk], 16 * q + pc0 + c);
          asm volatile("" : "+v"(m[q][c]));
        }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        ri[t] = rsqrt_d(m[t][t]);
#pragma unroll
        for (int c = t + 1; c < 4; ++c) m[t][c] *= ri[t];
#pragma unroll
        for (int q = t + 1; q < 4; ++q)
#pragma unroll
          for (int c = q; c < 4; ++c) m[q][c] = fma(-m[t][q], m[t][c], m[q][c]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        li[q][q] = ri[q];
#pragma unroll
        for (int c = q - 1; c >= 0; --c) {
          double v = 0.0;
#pragma unroll
          for (int t = c; t < q; ++t) v = fma(m[t][q], li[t][c], v);
          li[q][c] = -ri[q] * v;
        }
      }
      double la = 0.0;  // L^-1 as the A operand
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c <= q; ++c) la = lc == q && lr == c ? li[q][c] : la;
      if (lc < 4) Li[kb * 16 + lc * 4 + lr] = la;
      double W[MB];
#pragma unroll
      for (int bj = bk; bj < MB; ++bj) {
        const double w = mfma(la, U[bk][bj][rk], zero)[0];
        W[bj] = bj == bk && lc < pc0 ? 0.0 : w;
      }
#pragma unroll
      for (int bi = bk; bi < MB; ++bi)
#pragma unroll
        for (int bj = bi; bj < MB; ++bj) U[bi][bj] = mfma(-W[bi], W[bj], U[bi][bj]);
#pragma unroll
      for (int bj = bk; bj < MB; ++bj) U[bk][bj][rk] = W[bj];
    }
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int bj = bi; bj < MB; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * bi + lr + 4 * r, b = 16 * bj + lc;
          if (a <= b && b < NQ) Us[b * (b + 1) / 2 + a] = U[bi][bj][r];
        }
    __syncthreads();
    d4q xs[MB];
#pragma unroll
    for (int bi = 0; bi < MB; ++bi) xs[bi] = zero;
#pragma unroll 1
    for (int round = 0; round < 3; ++round) {  // a solve and two refinements
      if (round > 0) {  // b = f' - K' x in double-double, rounded
        by_pairs([&](auto cases, int l) {
          constexpr int NL = decltype(cases)::value;
          const int r = min(lane, NQ - 1), rb = r * (r + 1) / 2;
          double hi[NL], lo[NL], bx[NL];
#pragma unroll
          for (int h = 0; h < NL; ++h) hi[h] = RH[l + h][r], lo[h] = RL[l + h][r];
#pragma unroll 4
          for (int j = 0; j < NQ; ++j) {
            const double kj = -Kc[j <= r ? rb + j : j * (j + 1) / 2 + r];
#pragma unroll
            for (int h = 0; h < NL; ++h) dd_fma(kj, X[l + h][j], hi[h], lo[h]);
          }
          if constexpr (NX > 0) {  // rows 64.., XL lanes to a row
            const int r2 = 64 + min(lane / XL, NX - 1), j0 = (lane % XL) * XJ, rb2 = r2 * (r2 + 1) / 2;
            double h2[NL], o2[NL];
#pragma unroll
            for (int h = 0; h < NL; ++h) {
              h2[h] = lane % XL == 0 ? RH[l + h][r2] : 0.0;
              o2[h] = lane % XL == 0 ? RL[l + h][r2] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < XJ; ++q) {
              const int j = min(j0 + q, NQ - 1);
              const double kj = j0 + q < NQ ? -Kc[j <= r2 ? rb2 + j : j * (j + 1) / 2 + r2] : 0.0;
#pragma unroll
              for (int h = 0; h < NL; ++h) dd_fma(kj, X[l + h][j], h2[h], o2[h]);
            }
#pragma unroll
            for (int h = 0; h < NL; ++h) {
              for (int o = 1; o < XL; o <<= 1) {
                const double h3 = __shfl_xor(h2[h], o), l3 = __shfl_xor(o2[h], o);
                dd_add(h3, h2[h], o2[h]);
                o2[h] += l3;
              }
              bx[h] = h2[h] + o2[h];
            }
          }
          __syncthreads();
#pragma unroll
          for (int h = 0; h < NL; ++h) {
            if (lane < NQ) X[l + h][lane] = hi[h] + lo[h];
            if (NX > 0 && lane % XL == 0) X[l + h][64 + lane / XL] = bx[h];
          }
        });
        __syncthreads();
      }
      d4q y[MB];
      const double* __restrict__ B = round == 0 ? &RH[0][0] : &X[0][0];
#pragma unroll
      for (int bi = 0; bi < MB; ++bi)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * bi + lr + 4 * r;
          const double v = B[min(lc, nl - 1) * NQ + min(a, NQ - 1)];
          y[bi][r] = lc < nl && a < NQ ? v : 0.0;
        }
      // A tile's rows up to the step's are final: those registers are kept
      // from before its product, whose A operand needs no mask.
      lds_cptr li = (lds_cptr)Li, us = (lds_cptr)Us;
      asm volatile("" : "+v"(li), "+v"(us));  // else the loop's operands are all kept in registers
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {  // U^T y = b
        const int bk = kb / 4, rk = kb % 4;
        const double la = lc < 4 ? li[kb * 16 + min(lc, 3) * 4 + lr] : 0.0;
        const double yk = mfma(la, y[bk][rk], zero)[0], ny = -yk;
        const d4q old = y[bk];
#pragma unroll
        for (int bi = bk; bi < MB; ++bi) y[bi] = mfma(U[bk][bi][rk], ny, y[bi]);
#pragma unroll
        for (int r = 0; r < rk; ++r) y[bk][r] = old[r];
        y[bk][rk] = yk;
      }
#pragma unroll
      for (int kb = NKB - 1; kb >= 0; --kb) {  // U x = y
        const int bk = kb / 4, rk = kb % 4, col = min(4 * kb + lr, NQ - 1);
        const double la = lc < 4 ? li[kb * 16 + lr * 4 + min(lc, 3)] : 0.0;
        const double xk = mfma(la, y[bk][rk], zero)[0], nx = -xk;
        const d4q old = y[bk];
#pragma unroll
        for (int bi = bk; bi >= 0; --bi) y[bi] = mfma(us[col * (col + 1) / 2 + min(16 * bi + lc, col)], nx, y[bi]);
#pragma unroll
        for (int r = rk + 1; r < 4; ++r) y[bk][r] = old[r];
        y[bk][rk] = xk;
      }
#pragma unroll
      for (int bi = 0; bi < MB; ++bi) xs[bi] += y[bi];
      __syncthreads();
#pragma unroll
      for (int bi = 0; bi < MB; ++bi)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * bi + lr + 4 * r;
          if (lc < nl && a < NQ) X[lc][a] = xs[bi][r];
        }
      __syncthreads();
    }
#pragma unroll 1
    for (int l = 0; l < nl; ++l) {
      double jh = 0.0, jl = 0.0;
      for (int r = lane; r < NQ; r += 64) {
        dd_fma(RH[l][r], X[l][r], jh, jl);
        dd_fma(RL[l][r], X[l][r], jh, jl);
      }
      const double Jq = 0.5 * wave_sum_dd(jh, jl);
      if (lane == 0) eps[inst_eoff[inst] + (int64_t)(l0 + l) * nel + e] = Jq > 0.0 ? 1.0 - Jp[l] / Jq : 0.0;
    }
    __syncthreads();  // the next pass rebuilds K'
  }
}

}  // namespace

void launch_qr(const QrGroupDev& g, const double* E, const double* x, const SysDesc* sys, const int32_t* inst_sys0,
               const int32_t* inst_L, const int64_t* inst_eoff, const int32_t* inst_nel, double* eps,
               hipStream_t st) {
  if (g.n_elems == 0) return;
  const dim3 grid(g.n_elems), block(64);
  switch (g.p) {
    case 1: hipLaunchKernelGGL(k_qr<1>, grid, block, qr_lds_bytes(1), st, g, E, x, sys, inst_sys0, inst_L, inst_eoff, inst_nel, eps); break;
    case 2: hipLaunchKernelGGL(k_qr<2>, grid, block, qr_lds_bytes(2), st, g, E, x, sys, inst_sys0, inst_L, inst_eoff, inst_nel, eps); break;
    case 3: hipLaunchKernelGGL(k_qr<3>, grid, block, qr_lds_bytes(3), st, g, E, x, sys, inst_sys0, inst_L, inst_eoff, inst_nel, eps); break;
    default: hipLaunchKernelGGL(k_qr<4>, grid, block, qr_lds_bytes(4), st, g, E, x, sys, inst_sys0, inst_L, inst_eoff, inst_nel, eps); break;
  }
}

}  // namespace mto
