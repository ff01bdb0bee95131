// Element product by sum factorisation: y_e = sum_s E_{e,s} K_s u_e without
// the dense cell tables K_s.
//
// The basis is a tensor product and the cells of an element form a d x d
// grid, so every K_s is a sum of products of 1D integrals over one cell
// interval, a(i,k) = int phi_i' phi_k', b(i,k) = int phi_i phi_k,
// c(i,k) = int phi_i' phi_k (unit interval, n = p + 1 functions):
//   K_s[x,x] = D11 a_x b_y + D33 b_x a_y      K_s[x,y] = D12 c_x c_y^T + D33 c_x^T c_y
//   K_s[y,y] = D11 b_x a_y + D33 a_x b_y      K_s[y,x] = D12 c_x^T c_y + D33 c_x c_y^T
// For one row sy of cells the moduli enter the x factors only, M_t = sum_sx
// E[sx, sy] t_x^(sx) for t = a, b, c, after which the row costs two small
// matrix products (along x, then along y): d (8 n^3 + 8 n^3 + (2 n^2 + n) d)
// multiply-adds per element against d^2 (2 n^2)^2 for the dense contraction,
// 11.4 k against 62.5 k at p = 4, d = 5 and 4.7 k against 16.4 k at p = 3, d = 4.
//
// One lane takes one element column, so the 1D tables are the same for every
// lane: they come through the scalar cache and enter the FMAs as scalar
// operands, and no lane idles on padding.  Per lane: 2 n^2 accumulators in
// registers, the element vector in LDS ([row][lane], conflict free).  FP64
// vector FMAs run at the FP64 MFMA rate on gfx950, so nothing is lost by
// leaving the matrix cores, whose 16 x 16 tiles fit neither the 5 x 5 factors
// nor a per-element operand.
//
// The cell rows form fac_chains(d) chains (rows ch, ch + chains, ...), each
// summed in one accumulator, and the chains' sums are added in order: the
// same rounding however the work is split, so a design's results do not
// depend on what else is in its plan.  A split tile gives its 64 columns to a
// block of W waves, one chain (or, with waves to spare, one component of one
// chain) to a wave, which share the gather and the scatter and meet in LDS.
// The other tiles (small elements of large meshes) go one to a wave, from
// gather to scatter without a barrier, W of them to a block.  Plans of few tiles
// take tiles of 16 columns instead (narrow_tile).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "mto_device.hpp"
#include "mto_kernels.hpp"

namespace mto {
namespace {

typedef const __attribute__((address_space(3))) double* lds_vec;

__host__ __device__ constexpr int sym_index(int n, int i, int k) {  // packed upper triangle by rows
  return i <= k ? i * n - i * (i - 1) / 2 + (k - i) : k * n - k * (k - 1) / 2 + (i - k);
}

// acc += the product for the cell rows sy0, sy0 + step, ... of one column: u
// its element vector in LDS (rigid motion removed; row r at LS r), tab the
// group's 1D tables.  NC = 2: both components; NC = 1: component c0 alone.
// NK < n: u is nonzero only for the functions i, j < NK (the vertex
// functions, NK = 2).
// A single wave issues one instruction in 4 cycles whatever its kind, so the
// input rows are unrolled (no register moves, no loop control) with the next
// row's LDS and table reads ahead of the current one's products.  The empty
// asm statements hold each pass together: without them the compiler keeps u
// in registers across the passes, or sinks a pass's products below the next
// loop with all their operands live, and spills.
template <int P, int NK, int NC, int LS = 64>
__device__ __forceinline__ void factored_rows(int d, cptr tab, const double* __restrict__ Ecell, int sy0, int step,
                                              int c0, lds_vec u, double (&acc)[NC][P + 1][P + 1]) {
  constexpr int n = P + 1, NS = n * (n + 1) / 2, XT = fac_x_of(P), YT = fac_y_of(P);
  cptr yt = tab + d * XT;
#pragma unroll 1
  for (int sy = sy0; sy < d; sy += step) {
    cptr ys = yt + sy * n * YT;
    const double* __restrict__ Er = Ecell + sy * d;
    // M = sum_sx E t^(sx) for NM table entries from `off` on
    auto moduli = [&](auto& M, int off) {
      constexpr int NM = sizeof(M) / sizeof(double);
      double e = Er[0];
#pragma unroll
      for (int q = 0; q < NM; ++q) M[q] = 0.0;
#pragma unroll 1
      for (int sx = 0; sx < d; ++sx) {
        const double en = Er[min(sx + 1, d - 1)];
        cptr x = tab + sx * XT + off;
#pragma unroll
        for (int q = 0; q < NM; ++q) M[q] = fma(x[q], e, M[q]);
        e = en;
      }
    };
    // acc[c] += y_c (m u_c) along x, then y; entry(i, k) the x matrix, y
    // columns yo and yo + 1 for the components; `swap`: the other component's u
    auto pass = [&](int yo, bool swap, auto entry) {
      lds_vec up = u;
      asm volatile("" : "+v"(up));
      if (NC == 1) up += LS * (swap ? 1 - c0 : c0);
      cptr yc = ys + (NC == 1 ? yo + c0 : yo) * n;
      double ul[2][NK][NC], yv[2][NC][n];
      auto request = [&](int b, int l) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int j = 0; j < n; ++j) yv[b][c][j] = yc[l * YT + c * n + j];
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
          for (int c = 0; c < NC; ++c) ul[b][k][c] = up[(2 * (l * n + k) + c) * LS];
      };
      request(0, 0);
#pragma unroll
      for (int l = 0; l < NK; ++l) {
        const int b = l & 1;
        if (l + 1 < NK) request(b ^ 1, l + 1);
        __builtin_amdgcn_sched_barrier(0);
        double T[NC][n];
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
          for (int i = 0; i < n; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c)
              T[c][i] = k == 0 ? entry(i, k) * ul[b][0][c] : fma(entry(i, k), ul[b][k][c], T[c][i]);
#pragma unroll
        for (int j = 0; j < n; ++j)
#pragma unroll
          for (int i = 0; i < n; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c)
              acc[c][j][i] = fma(yv[b][c][j], T[NC == 2 && swap ? 1 - c : c][i], acc[c][j][i]);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int a = 0; a < n * n; ++a) asm volatile("" : "+v"(acc[c][a / n][a % n]));
    };
    // a_x: D11 b_y on x, D33 b_y on y; b_x: D33 a_y on x, D11 a_y on y; c_x and
    // its transpose couple the components.  The three x matrices are formed
    // together where the registers hold them.
    if constexpr (P <= 3) {
      double M[2 * NS + n * n];
      moduli(M, 0);
      pass(0, false, [&](int i, int k) { return M[sym_index(n, i, k)]; });
      pass(2, false, [&](int i, int k) { return M[NS + sym_index(n, i, k)]; });
      pass(4, true, [&](int i, int k) { return M[2 * NS + i * n + k]; });
      pass(6, true, [&](int i, int k) { return M[2 * NS + k * n + i]; });
    } else {
      {
        double M[2 * NS];
        moduli(M, 0);
        pass(0, false, [&](int i, int k) { return M[sym_index(n, i, k)]; });
        pass(2, false, [&](int i, int k) { return M[NS + sym_index(n, i, k)]; });
      }
      double C[n * n];
      moduli(C, 2 * NS);
      pass(4, true, [&](int i, int k) { return C[i * n + k]; });
      pass(6, true, [&](int i, int k) { return C[k * n + i]; });
    }
  }
}

template <int P, int NC>
__device__ __forceinline__ void clear(double (&acc)[NC][P + 1][P + 1]) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int a = 0; a < (P + 1) * (P + 1); ++a) acc[c][a / (P + 1)][a % (P + 1)] = 0.0;
}

// One tile by the W waves of a block (SPLIT), or by one wave (W = 1, no
// barrier); ush: its LDS, [NE][64] element vectors, then partial results.
// VERT: xin is nonzero at vertex DOFs only (read there alone) and the results
// are added to the slots: with the slots holding K z from before the V-cycle's
// coarse-grid correction, which changes z at vertex DOFs, this gives K z after
// it at a third of a full product's multiply-adds (3.8 k at p = 4, d = 5).
template <int P, bool SPLIT, bool VERT>
__device__ __forceinline__ void factored_tile(const FacTile& t, const double* __restrict__ E,
                                              const double* __restrict__ xin, const PcgDev& s, int mode, int it_k,
                                              double* ush) {
  constexpr int n = P + 1, NE = ne_of(P);
  // a stopped system has nothing to do (PCG mode also checks this iteration's residual below)
  if (mode != ELEM_APPLY && s.status[t.sys] != SYS_RUNNING) return;
  const bool pcg = mode == ELEM_PCG;
  const int W = SPLIT ? blockDim.x >> 6 : 1, lane = threadIdx.x & 63;
  const int wave = SPLIT ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const bool valid = lane < t.count;
  const int el = valid ? lane : t.count - 1;  // idle lanes repeat the last column, unstored
  const double* __restrict__ xs = xin + t.dof_off;
  const double* __restrict__ zs = s.z + t.dof_off;
  const int32_t* __restrict__ gi_ = t.gidx + el;
  const int cell = t.cell[el];
  // the column's moduli, one read per cache line: on their way during the gather
  double warm[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) warm[k] = E[cell + min(16 * k, t.d * t.d - 1)];
  // Rows wave, wave + W, ... (VERT: the eight vertex rows): GB index loads, then their values, all
  // unconditional (clamped row; an absent DOF reads the system's first).
  // Every wave reduces the PCG scalars itself, while its first values load: no
  // barrier, and no memory round trip more than the values take.
  double beta = 0.0;
  bool on = true;
  {
    constexpr int NG = VERT ? 8 : NE, GB = SPLIT ? (NG + 3) / 4 : VERT ? 8 : (NE + 1) / 2;
    auto row_of = [](int k) { return VERT ? vertex_dof<P>(k) : k; };
    int gi[GB];
    for (int r0 = wave; r0 < NG; r0 += W * GB) {
#pragma unroll
      for (int q = 0; q < GB; ++q) gi[q] = gi_[(int64_t)row_of(min(r0 + W * q, NG - 1)) * t.npad];
      const int it = pcg && r0 == wave ? *s.it_base + it_k : 0;
      double v[GB], z[GB];
#pragma unroll
      for (int q = 0; q < GB; ++q) {
        const int gc = max(gi[q], 0);
        v[q] = xs[gc];
        z[q] = pcg ? zs[gc] : 0.0;
      }
      if (pcg && r0 == wave) {
        const Scal sc = pcg_state(s, t.sys, t.pc_begin, t.pc_end, it, true);
        on = sc.active;  // the same in every wave
        beta = sc.beta;
      }
#pragma unroll
      for (int q = 0; q < GB; ++q) {
        const int k = r0 + W * q, row = row_of(k);
        // p = z + beta p_old formed as k_dof1 stores it
        if (k < NG) ush[row * 64 + lane] = gi[q] >= 0 ? (pcg ? fma(beta, v[q], z[q]) : v[q]) : 0.0;
      }
    }
  }
  // (an empty statement that uses them)
  asm volatile("" ::"v"(warm[0]), "v"(warm[1]), "v"(warm[2]), "v"(warm[3]), "v"(warm[4]));
  if (!on) return;
  if (SPLIT) __syncthreads();
  {  // rigid motion removed from the vertex rows
    const double x0 = ush[lane], x1 = ush[64 + lane], th = ush[3 * 64 + lane] - x1;
    if (SPLIT) __syncthreads();
    for (int v = wave; v < 8; v += W) {
      const int row = vertex_dof<P>(v);
      ush[row * 64 + lane] = rigid_free<P>(ush[row * 64 + lane], row, x0, x1, th);
    }
    if (SPLIT) __syncthreads();
  }
  constexpr int NK = VERT ? 2 : n;
  const cptr tab = scalar_table(t.kfac);
  const double* __restrict__ Ec = E + cell;
  const lds_vec u = (lds_vec)(ush + lane);
  const int nch = fac_chains(t.d);
  double* __restrict__ sl = s.slots + t.slot_off;
  const int32_t* __restrict__ si_ = t.sidx + el;
  if (!SPLIT) {
    double acc[2][n][n], tot[2][n][n];
    for (int ch = 0; ch < nch; ++ch) {
      clear<P, 2>(acc);
      factored_rows<P, NK, 2>(t.d, tab, Ec, ch, nch, 0, u, acc);
#pragma unroll
      for (int a = 0; a < NE; ++a) {
        double& v = tot[a & 1][(a >> 1) / n][(a >> 1) % n];
        const double w = acc[a & 1][(a >> 1) / n][(a >> 1) % n];
        v = ch == 0 ? w : v + w;
      }
    }
    int si[NE];
#pragma unroll
    for (int r = 0; r < NE; ++r) si[r] = si_[(int64_t)r * t.npad];
    double old[VERT ? NE : 1];
    if (VERT) {
#pragma unroll
      for (int r = 0; r < NE; ++r) old[VERT ? r : 0] = sl[max(si[r], 0)];
    }
#pragma unroll
    for (int r = 0; r < NE; ++r) {
      const double v = tot[r & 1][(r >> 1) / n][(r >> 1) % n];
      if (valid && si[r] >= 0) sl[si[r]] = VERT ? old[VERT ? r : 0] + v : v;
    }
    return;
  }
  // Partial results in LDS, [chain][CP n n][64]: both components at once
  // (CP = 2) or, where that takes too much, one after the other.  slots: the
  // scatter slots of the wave's rows a = wave, wave + W, ..., SB at a time.
  constexpr int CP = P <= 2 ? 2 : 1, NR = CP * n * n, SB = (NR + 3) / 4;
  int si[2][SB];
  double old[2][VERT ? SB : 1];
  auto slots_of = [&](int h, int a0) {  // row a of phase h: component h (CP = 1) or a % 2 (CP = 2)
#pragma unroll
    for (int q = 0; q < SB; ++q) {
      const int a = min(a0 + W * q, NR - 1);
      si[h][q] = si_[(int64_t)(CP == 2 ? a : 2 * a + h) * t.npad];
    }
    if (VERT) {
#pragma unroll
      for (int q = 0; q < SB; ++q) old[h][VERT ? q : 0] = sl[max(si[h][q], 0)];
    }
  };
  auto put = [&](int ch, int c, const double (&a)[n][n]) {
#pragma unroll
    for (int q = 0; q < n * n; ++q) ush[(ch * NR + (CP == 2 ? 2 * q + c : q)) * 64 + lane] = a[q / n][q % n];
  };
  auto scatter = [&](int h) {
    for (int a0 = wave; a0 < NR; a0 += W * SB) {
      if (a0 != wave) slots_of(h, a0);
#pragma unroll
      for (int q = 0; q < SB; ++q) {
        const int a = a0 + W * q;
        if (a >= NR) break;  // uniform
        double v = ush[a * 64 + lane];
        for (int ch = 1; ch < nch; ++ch) v += ush[(ch * NR + a) * 64 + lane];
        if (valid && si[h][q] >= 0) sl[si[h][q]] = VERT ? old[h][VERT ? q : 0] + v : v;
      }
    }
  };
  auto finish = [&](auto store) {  // store(h): this wave's part of phase h
#pragma unroll
    for (int h = 0; h < 2 / CP; ++h) slots_of(h, wave);
#pragma unroll
    for (int h = 0; h < 2 / CP; ++h) {
      __syncthreads();  // the previous contents are no longer read
      store(h);
      __syncthreads();
      scatter(h);
    }
  };
  if (2 * nch <= W) {  // one component of one chain per wave
    const int ch = wave >> 1, c = wave & 1;
    double acc[1][n][n];
    clear<P, 1>(acc);
    if (ch < nch) factored_rows<P, NK, 1>(t.d, tab, Ec, ch, nch, c, u, acc);
    finish([&](int h) {
      if (ch < nch && (CP == 2 || c == h)) put(ch, c, acc[0]);
    });
    return;
  }
  double acc[2][n][n];
  clear<P, 2>(acc);
  if (wave < nch) factored_rows<P, NK, 2>(t.d, tab, Ec, wave, nch, 0, u, acc);
  finish([&](int h) {
    if (wave >= nch) return;
    if (CP == 2) {
      put(wave, 0, acc[0]);
      put(wave, 1, acc[1]);
    } else {
      put(wave, h, acc[h]);
    }
  });
}

// One tile of at most FAC_NARROW = 16 columns by the four waves of a block, for
// plans whose tiles are few (fac_cols): the launch is one tile's latency then.
// Lane l holds column l % 16 and, in the gather and the scatter, row l / 16 of four
// rows of an instruction, which are a quarter of a 64-column tile's
// instructions; in between the lanes of the four sets compute the same sums, in
// the order of the other tiles.  What depends on the tile alone is requested
// before anything is waited for, the scatter slots (VERT: and their values) too,
// and both components' partial results meet in LDS at once.
//   Time of a product in the PCG loop, 2013 elements, a launch of 64-column tiles ->
// of these (us): p = 4, d = 5: 27.0 -> 21.9; p = 3, d = 2: 11.1 -> 8.6 (the dense
// contraction on its tiles of 16 columns: 29.8, 8.5).
template <int P, bool VERT>
__device__ __forceinline__ void narrow_tile(const FacTile& t, const double* __restrict__ E,
                                            const double* __restrict__ xin, const PcgDev& s, int mode, int it_k,
                                            double* ush) {
  constexpr int n = P + 1, NE = ne_of(P), C = FAC_NARROW, RP = 64 / C, W = FAC_MAX_W;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane % C, r0 = wave * RP + lane / C;  // this lane's rows r0, r0 + W RP, ...
  const bool pcg = mode == ELEM_PCG, valid = col < t.count;
  const int el = valid ? col : t.count - 1;  // idle lanes repeat the last column, unstored
  const double* __restrict__ xs = xin + t.dof_off;
  const double* __restrict__ zs = s.z + t.dof_off;
  constexpr int NG = VERT ? 8 : NE, GB = (NG + W * RP - 1) / (W * RP), SB = (NE + W * RP - 1) / (W * RP);
  auto row_of = [](int k) { return VERT ? vertex_dof<P>(k) : k; };
  int gi[GB], si[SB];
#pragma unroll
  for (int q = 0; q < GB; ++q) gi[q] = t.gidx[(int64_t)row_of(min(r0 + W * RP * q, NG - 1)) * t.npad + el];
  const int cell = t.cell[el];
#pragma unroll
  for (int q = 0; q < SB; ++q) si[q] = t.sidx[(int64_t)min(r0 + W * RP * q, NE - 1) * t.npad + el];
  const int it = pcg ? *s.it_base + it_k : 0;
  // a stopped system has nothing to do (PCG mode also checks this iteration's residual below)
  if (mode != ELEM_APPLY && s.status[t.sys] != SYS_RUNNING) return;
  // the column's moduli, one read per cache line: on their way during the gather
  double warm[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) warm[k] = E[cell + min(16 * k, t.d * t.d - 1)];
  double v[GB], z[GB];
#pragma unroll
  for (int q = 0; q < GB; ++q) {
    const int gc = max(gi[q], 0);
    v[q] = xs[gc];
    z[q] = pcg ? zs[gc] : 0.0;
  }
  double beta = 0.0;
  bool on = true;
  if (pcg) {  // by every wave, while its values load
    const Scal sc = pcg_state(s, t.sys, t.pc_begin, t.pc_end, it, true);
    on = sc.active;  // the same in every wave
    beta = sc.beta;
  }
#pragma unroll
  for (int q = 0; q < GB; ++q) {
    const int k = r0 + W * RP * q;
    // p = z + beta p_old formed as k_dof1 stores it
    if (k < NG) ush[row_of(k) * C + col] = gi[q] >= 0 ? (pcg ? fma(beta, v[q], z[q]) : v[q]) : 0.0;
  }
  // (an empty statement that uses them)
  asm volatile("" ::"v"(warm[0]), "v"(warm[1]), "v"(warm[2]), "v"(warm[3]), "v"(warm[4]));
  if (!on) return;
  __syncthreads();
  {  // rigid motion removed from the vertex rows
    const double x0 = ush[col], x1 = ush[C + col], th = ush[3 * C + col] - x1;
    __syncthreads();
    if (r0 < 8) {
      const int row = vertex_dof<P>(r0);
      ush[row * C + col] = rigid_free<P>(ush[row * C + col], row, x0, x1, th);
    }
    __syncthreads();
  }
  constexpr int NK = VERT ? 2 : n;
  const cptr tab = scalar_table(t.kfac);
  const double* __restrict__ Ec = E + cell;
  const lds_vec u = (lds_vec)(ush + col);
  const int nch = fac_chains(t.d);
  double* __restrict__ sl = s.slots + t.slot_off;
  double old[VERT ? SB : 1];
  if (VERT) {
#pragma unroll
    for (int q = 0; q < SB; ++q) old[VERT ? q : 0] = sl[max(si[q], 0)];
  }
  // partial results in LDS, [chain][NE][C]
  auto put = [&](int ch, int c, const double (&a)[n][n]) {
#pragma unroll
    for (int q = 0; q < n * n; ++q) ush[(ch * NE + 2 * q + c) * C + col] = a[q / n][q % n];
  };
  if (2 * nch <= W) {  // one component of one chain per wave
    const int ch = wave >> 1, c = wave & 1;
    double acc[1][n][n];
    clear<P, 1>(acc);
    if (ch < nch) factored_rows<P, NK, 1, C>(t.d, tab, Ec, ch, nch, c, u, acc);
    __syncthreads();  // u is no longer read
    if (ch < nch) put(ch, c, acc[0]);
  } else {
    double acc[2][n][n];
    clear<P, 2>(acc);
    if (wave < nch) factored_rows<P, NK, 2, C>(t.d, tab, Ec, wave, nch, 0, u, acc);
    __syncthreads();
    if (wave < nch) {
      put(wave, 0, acc[0]);
      put(wave, 1, acc[1]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < SB; ++q) {
    const int a = r0 + W * RP * q;
    if (a >= NE) break;
    double y = ush[a * C + col];
    for (int ch = 1; ch < nch; ++ch) y += ush[(ch * NE + a) * C + col];
    if (valid && si[q] >= 0) sl[si[q]] = VERT ? old[VERT ? q : 0] + y : y;
  }
}

// Tiles of 64 columns from any group, PM the largest order among them: n_split split tiles, one per block, then n_whole
// tiles of order <= 2, one per wave.  At most 256 registers: two waves per SIMD.
template <int PM, bool VERT>
__global__ __launch_bounds__(64 * FAC_MAX_W, 2) void k_elem_factored(const FacTile* __restrict__ tiles, int n_split,
                                                                    int n_whole, int xcd_run,
                                                                    const double* __restrict__ E,
                                                                    const double* __restrict__ xin, PcgDev s, int mode,
                                                                    int it_k) {
  extern __shared__ double lds[];
  if ((int)blockIdx.x >= n_split) {
    const int W = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = xcd_tile(blockIdx.x - n_split, gridDim.x - n_split, xcd_run) * W + wave;
    if (i >= n_whole) return;
    const FacTile t = tiles[n_split + i];
    double* mine = lds + wave * ne_of(PM < 2 ? PM : 2) * 64;  // waves of a block may hold different orders
    if (t.p == 1) return factored_tile<1, false, VERT>(t, E, xin, s, mode, it_k, mine);
    if constexpr (PM >= 2) factored_tile<2, false, VERT>(t, E, xin, s, mode, it_k, mine);
    return;
  }
  const FacTile t = tiles[xcd_tile(blockIdx.x, n_split, xcd_run)];
  if constexpr (PM >= 4)
    if (t.p == 4) return factored_tile<4, true, VERT>(t, E, xin, s, mode, it_k, lds);
  if constexpr (PM >= 3)
    if (t.p == 3) return factored_tile<3, true, VERT>(t, E, xin, s, mode, it_k, lds);
  if constexpr (PM >= 2)
    if (t.p == 2) return factored_tile<2, true, VERT>(t, E, xin, s, mode, it_k, lds);
  factored_tile<1, true, VERT>(t, E, xin, s, mode, it_k, lds);
}

template <int PM, bool VERT>
__global__ __launch_bounds__(64 * FAC_MAX_W, 2) void k_elem_narrow(const FacTile* __restrict__ tiles, int n_tiles,
                                                                  int xcd_run, const double* __restrict__ E,
                                                                  const double* __restrict__ xin, PcgDev s, int mode,
                                                                  int it_k) {
  extern __shared__ double lds[];
  const FacTile t = tiles[xcd_tile(blockIdx.x, n_tiles, xcd_run)];
  if constexpr (PM >= 4)
    if (t.p == 4) return narrow_tile<4, VERT>(t, E, xin, s, mode, it_k, lds);
  if constexpr (PM >= 3)
    if (t.p == 3) return narrow_tile<3, VERT>(t, E, xin, s, mode, it_k, lds);
  if constexpr (PM >= 2)
    if (t.p == 2) return narrow_tile<2, VERT>(t, E, xin, s, mode, it_k, lds);
  narrow_tile<1, VERT>(t, E, xin, s, mode, it_k, lds);
}

// Sensitivity: w_s = lam_e^T K_s u_e for every cell s of every column, g =
// -E'(rho) w.  With K_s as above, a row sy of cells needs for the x factors
// a, b, c the n x n matrices Z_t(i, k) = sum over j, l, components of lam_ij
// y_t(j, l) u_kl; then w = sum_t t_x^(sx) : Z_t, d of them from one Z: d (16 n^3
// + (2 n^2 + n) d) multiply-adds per column (11.4 k at p = 4, d = 5; 62.5 k for
// the cells' dense matrices).  One lane takes a column, the waves of a block
// take the rows of cells of its 64 columns in turn; a component of u and Z are
// in registers, u and lam in LDS (once where they are the same vector, SAME: the
// arithmetic does not differ).  Both have their rigid motions removed first, as in
// k_elem_dd: K_s annihilates them exactly, its FP64 rounding does not.
template <int P, bool SAME>
__device__ __forceinline__ void sens_tile(const FacTile& t, const double* __restrict__ dE,
                                          const double* __restrict__ x, const double* __restrict__ y,
                                          double* __restrict__ gout, const SysDesc* __restrict__ sys, double* ush) {
  constexpr int n = P + 1, NE = ne_of(P), NS = n * (n + 1) / 2, XT = fac_x_of(P), YT = fac_y_of(P);
  constexpr int NV = SAME ? 1 : 2, GB = (NE + 3) / 4;
  const int W = blockDim.x >> 6, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool valid = lane < t.count;
  const int el = valid ? lane : t.count - 1;  // idle lanes repeat the last column, unstored
  const double* __restrict__ xs = x + t.dof_off;
  const double* __restrict__ ys_ = y + t.dof_off;
  const int32_t* __restrict__ gi_ = t.gidx + el;
  const int64_t cell = t.cell[el];
  const int64_t g_off = sys[t.sys].g_off;
  for (int r0 = wave; r0 < NE; r0 += W * GB) {
    int gi[GB];
    double v[NV][GB];
#pragma unroll
    for (int q = 0; q < GB; ++q) gi[q] = gi_[(int64_t)min(r0 + W * q, NE - 1) * t.npad];
#pragma unroll
    for (int q = 0; q < GB; ++q) {
      v[0][q] = xs[max(gi[q], 0)];
      if (!SAME) v[NV - 1][q] = ys_[max(gi[q], 0)];
    }
#pragma unroll
    for (int q = 0; q < GB; ++q)
      if (r0 + W * q < NE)
#pragma unroll
        for (int h = 0; h < NV; ++h) ush[(h * NE + r0 + W * q) * 64 + lane] = gi[q] >= 0 ? v[h][q] : 0.0;
  }
  __syncthreads();
  {  // rigid motion removed from the vertex rows
    double x0[NV], x1[NV], th[NV];
#pragma unroll
    for (int h = 0; h < NV; ++h) {
      const double* b = ush + h * NE * 64 + lane;
      x0[h] = b[0];
      x1[h] = b[64];
      th[h] = b[3 * 64] - x1[h];
    }
    __syncthreads();
    for (int v = wave; v < 8; v += W) {
      const int row = vertex_dof<P>(v);
#pragma unroll
      for (int h = 0; h < NV; ++h) {
        double* b = ush + (h * NE + row) * 64 + lane;
        *b = rigid_free<P>(*b, row, x0[h], x1[h], th[h]);
      }
    }
    __syncthreads();
  }
  const cptr tab = scalar_table(t.kfac);
  const int d = t.d;
#pragma unroll 1
  for (int sy = wave; sy < d; sy += W) {
    double Z[2 * NS + n * n];
#pragma unroll
    for (int q = 0; q < 2 * NS + n * n; ++q) Z[q] = 0.0;
    cptr ys = tab + d * XT + sy * n * YT;
    auto half = [&](auto comp) {  // the part of u's component C
      constexpr int C = decltype(comp)::value;
      lds_vec up = (lds_vec)(ush + lane), lp = (lds_vec)(ush + (NV - 1) * NE * 64 + lane);
      asm volatile("" : "+v"(up));
      double u[n][n];
#pragma unroll
      for (int l = 0; l < n; ++l)
#pragma unroll
        for (int k = 0; k < n; ++k) u[l][k] = up[(2 * (l * n + k) + C) * 64];
#pragma unroll 1
      for (int j = 0; j < n; ++j) {
        double lm[2][n];  // lam's components C, 1 - C of function row j
#pragma unroll
        for (int i = 0; i < n; ++i) {
          lm[0][i] = lp[(2 * (j * n + i) + C) * 64];
          lm[1][i] = lp[(2 * (j * n + i) + 1 - C) * 64];
        }
        double T[4][n];
#pragma unroll
        for (int l = 0; l < n; ++l)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            // x: D11 b, D33 a, D12 c, D33 c^T; y: D33 b, D11 a, D33 c, D12 c^T (rows j, columns l)
            const double m = ys[j * YT + (2 * q + C) * n + l];
#pragma unroll
            for (int k = 0; k < n; ++k) T[q][k] = l == 0 ? m * u[0][k] : fma(m, u[l][k], T[q][k]);
          }
#pragma unroll
        for (int i = 0; i < n; ++i)
#pragma unroll
          for (int k = 0; k < n; ++k) {
            const int sym = sym_index(n, i, k);
            Z[sym] = fma(lm[0][i], T[0][k], Z[sym]);
            Z[NS + sym] = fma(lm[0][i], T[1][k], Z[NS + sym]);
            double &z1 = Z[2 * NS + k * n + i], &z2 = Z[2 * NS + i * n + k];
            z1 = fma(lm[1][i], T[2][k], z1);
            z2 = fma(lm[1][i], T[3][k], z2);
          }
      }
#pragma unroll
      for (int q = 0; q < 2 * NS + n * n; ++q) asm volatile("" : "+v"(Z[q]));
    };
    half(std::integral_constant<int, 0>{});
    half(std::integral_constant<int, 1>{});
    const int64_t c0 = cell + sy * d;
#pragma unroll 1
    for (int sx = 0; sx < d; ++sx) {
      const double de = dE[c0 + sx];
      cptr xt = tab + sx * XT;
      double w = 0.0;
#pragma unroll
      for (int q = 0; q < 2 * NS + n * n; ++q) w = fma(xt[q], Z[q], w);
      if (valid) gout[g_off + c0 + sx] = -de * w;
    }
  }
}

template <int PM, bool SAME>
__global__ __launch_bounds__(64 * SENS_MAX_W, 2) void k_sens(const FacTile* __restrict__ tiles, int n_tiles, int xcd_run,
                                                            const double* __restrict__ dE,
                                                            const double* __restrict__ x, const double* __restrict__ y,
                                                            double* __restrict__ gout,
                                                            const SysDesc* __restrict__ sys) {
  extern __shared__ double lds[];
  const FacTile t = tiles[xcd_tile(blockIdx.x, n_tiles, xcd_run)];
  if constexpr (PM >= 4)
    if (t.p == 4) return sens_tile<4, SAME>(t, dE, x, y, gout, sys, lds);
  if constexpr (PM >= 3)
    if (t.p == 3) return sens_tile<3, SAME>(t, dE, x, y, gout, sys, lds);
  if constexpr (PM >= 2)
    if (t.p == 2) return sens_tile<2, SAME>(t, dE, x, y, gout, sys, lds);
  sens_tile<1, SAME>(t, dE, x, y, gout, sys, lds);
}

}  // namespace

namespace {
template <bool VERT>
void launch_factored(const FacTile* tiles, const FactoredLaunch& f, int xcd_run, const double* E, const double* xin,
                     const PcgDev& s, int mode, int it_k, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (f.n_split + f.n_whole == 0) return;
  const int blocks = f.n_split + (f.n_whole + f.waves - 1) / f.waves;
  const dim3 grid(blocks), block(64 * f.waves);
  const FacTile* tl = tiles + f.tile_begin;
  const uint32_t lds = (uint32_t)f.lds;
  if (f.cols == FAC_NARROW) {
    auto go = [&](auto k) {
      launch_timed(k, grid, block, lds, st, ev0, ev1, tl, (int)f.n_split, xcd_run, E, xin, s, mode, it_k);
    };
    switch (f.p_max) {
      case 1: go(k_elem_narrow<1, VERT>); break;
      case 2: go(k_elem_narrow<2, VERT>); break;
      case 3: go(k_elem_narrow<3, VERT>); break;
      default: go(k_elem_narrow<4, VERT>); break;
    }
    return;
  }
  auto go = [&](auto k) {
    launch_timed(k, grid, block, lds, st, ev0, ev1, tl, (int)f.n_split, (int)f.n_whole, xcd_run, E, xin, s, mode, it_k);
  };
  switch (f.p_max) {
    case 1: go(k_elem_factored<1, VERT>); break;
    case 2: go(k_elem_factored<2, VERT>); break;
    case 3: go(k_elem_factored<3, VERT>); break;
    default: go(k_elem_factored<4, VERT>); break;
  }
}
}  // namespace

void launch_elem_factored(const FacTile* tiles, const FactoredLaunch& f, int xcd_run, const double* E,
                          const double* xin, const PcgDev& s, int mode, int it_k, hipStream_t st, hipEvent_t ev0,
                          hipEvent_t ev1) {
  launch_factored<false>(tiles, f, xcd_run, E, xin, s, mode, it_k, st, ev0, ev1);
}

void launch_vertex_factored(const FacTile* tiles, const FactoredLaunch& f, int xcd_run, const double* E,
                            const double* dz, const PcgDev& s, hipStream_t st) {
  launch_factored<true>(tiles, f, xcd_run, E, dz, s, ELEM_APPLY_RUNNING, 0, st, nullptr, nullptr);
}

// Up to 256 tiles (one per CU) each row of cells has its own wave, and at least
// four share the gather; up to 2048 four waves; beyond, two, which keep more columns'
// gathers in flight.  us with 2, 4 and a wave per row of cells (at 256 and 2048 the
// lines do not matter much, p = 4, d = 2 would take two waves from 700 tiles on):
//   16 x 8 mesh, p = 4, d = 1: 12.5, 11.6 and 14.7
//   110 x 55, p = 4, d = 5, 95 tiles: 27.6, 21.0 and 18.1
//   300 x 150, p = 3, d = 4, 704 tiles: 30.6, 23.4 and 23.4
//   400 x 200, p = 4, d = 5, 1250 tiles: 73.9, 70.7 and 85.2
//   400 x 200, p = 1..4, three systems, 3750 tiles: 58.0, 67.6 and 99.4
//   16 designs, p = 4 in the main, two systems, 9600 tiles: 136, 161 and 243
// A dense K_s contraction per cell and a launch per group took 21.9 us on a 160 x 80
// mesh, p = 3, d = 4 (now 9.4, half of it the gather), 250 and 560 on the last two.
void launch_sens(const FacTile* tiles, const FactoredLaunch& f, int d_max, int xcd_run, const double* dE,
                 const double* x, const double* y, double* gout, const SysDesc* sys, hipStream_t st) {
  const int n = f.n_split + f.n_whole;
  if (n == 0) return;
  const int waves = n <= 256 ? std::min(std::max(d_max, 4), SENS_MAX_W) : n <= 2048 ? 4 : 2;
  const bool same = x == y;
  const dim3 grid(n), block(64 * waves);
  const uint32_t lds = (uint32_t)(8 * 64 * ne_of(f.p_max) * (same ? 1 : 2));
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, grid, block, lds, st, tiles + f.tile_begin, n, xcd_run, dE, x, y, gout, sys);
  };
  switch (f.p_max) {
    case 1: same ? go(k_sens<1, true>) : go(k_sens<1, false>); break;
    case 2: same ? go(k_sens<2, true>) : go(k_sens<2, false>); break;
    case 3: same ? go(k_sens<3, true>) : go(k_sens<3, false>); break;
    default: same ? go(k_sens<4, true>) : go(k_sens<4, false>); break;
  }
}

}  // namespace mto
