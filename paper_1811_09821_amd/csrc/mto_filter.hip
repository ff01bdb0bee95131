// Density filter of Sec. 2.2 (Eqs. (4)-(5)) on the density cells and its
// transpose for the chain rule.
//
// H is symmetric (H_ij = R - |c_i - c_j| is the same float either way round),
// so one pattern serves both directions: with s_i = 1 / sum_j H_ij,
//   apply:  y_i = s_i sum_j H_ij x_j            (W = diag(s) H)
//   grad:   y_i = sum_j H_ij (s_j x_j)          (W^T = H diag(s))
// The pattern is stored sliced by 64 rows (one wavefront): slice t holds its
// rows' k-th entries side by side at sp[t] + 64 k + lane, padded to the
// slice's longest row with zero weights pointing at the row itself, so each
// load of a wave is one contiguous run and no lane diverges.  Both directions
// are plain gathers: no atomics, bit-reproducible.
//   The cells of a mesh lie in few relative positions, so H has few distinct
// values (60 on a 400 x 200 mesh with d = 1, 2, 5, R = 0.3) and short offsets
// j - i: an entry is one 32-bit word, the offset and the value's place in a
// table.  Where there are more than 65536 values or an offset exceeds 16 bits
// (about 32000 cells in the rows of elements that R spans), entries are a
// 32-bit index and the value itself.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <unordered_map>
#include <vector>

#include "mto_internal.hpp"

using namespace mto;

namespace {
constexpr int FSLICE = 64;  // rows per slice = wavefront width
}

struct mto_filter {
  int device = 0;
  double R = 0.0;
  int64_t n = 0, nnz = 0, stored = 0;
  int64_t* sp = nullptr;   // [n_slices + 1] slice starts (entries)
  uint32_t* word = nullptr;  // [stored] (j - i) & 0xffff, place of H_ij in tab << 16; or, NULL:
  int32_t* col = nullptr;    // [stored]
  double* h = nullptr;       // [stored] H_ij
  double* tab = nullptr;     // the distinct H_ij
  int32_t n_tab = 0;
  double* s = nullptr;     // [n] 1 / sum_j H_ij
};

namespace {

// Bound by the gathers (some 16 cycles of a CU's address unit per 64 of them)
// and by round trips: the entries of a slice go through in batches of equal
// size, at most FBATCH, without a load that is not needed, and a batch's loads,
// then the loads they point at, are in flight together.  The table of values is
// in LDS where it fits.  400 x 200 mesh, 584 k rows of 7 entries, apply / grad in
// us: 17.3 / 17.6 with 12 bytes an entry and an entry at a time; 9.3 / 9.9 as
// below (15.1 / 17.7 with batches filled up to eight and the table in memory).
constexpr int FBATCH = 8;
constexpr int FTAB = 512;  // table entries held in LDS
enum { F_PLAIN, F_PACKED, F_PACKED_LDS };

// The pattern, as one argument (a launch costs the host some 50 ns for each).
struct FilterDev {
  const int64_t* sp;
  const uint32_t* word;
  const double* tab;
  const int32_t* col;
  const double *h, *s;
  int64_t n;
  int32_t n_tab;
};

template <bool GRAD, int FORM>
__global__ __launch_bounds__(256) void k_filter(FilterDev f, const double* __restrict__ x, double* __restrict__ y) {
  const int64_t* __restrict__ sp = f.sp;
  const uint32_t* __restrict__ word = f.word;
  const double* __restrict__ tab = f.tab;
  const int32_t* __restrict__ col = f.col;
  const double* __restrict__ h = f.h;
  const double* __restrict__ s = f.s;
  const int64_t n = f.n;
  const int n_tab = f.n_tab;
  __shared__ double tl[FORM == F_PACKED_LDS ? FTAB : 1];
  // consecutive blocks go to the XCDs in turn: each XCD takes a contiguous
  // eighth of the rows, whose x its L2 then holds
  const int per = gridDim.x / 8, blk = (blockIdx.x % 8) * per + blockIdx.x / 8;
  const int64_t i = (int64_t)blk * 256 + threadIdx.x, ic = i < n ? i : n - 1;
  const int64_t t = __builtin_amdgcn_readfirstlane((int)(ic / FSLICE));
  const int lane = (int)(i % FSLICE);
  // the slice's bounds and the row's scale are on their way while the table is
  const int64_t b = sp[t];
  const int cnt = (int)((sp[t + 1] - b) / FSLICE);  // the same for every lane
  const double scale = GRAD ? 1.0 : s[ic];
  if (FORM == F_PACKED_LDS) {
    for (int k = threadIdx.x; k < n_tab; k += 256) tl[k] = tab[k];
    __syncthreads();
  }
  if (i >= n) return;
  // 32-bit byte offsets from the slice's first row less the furthest offset
  const uintptr_t x0 = (uintptr_t)x + 8 * (t * FSLICE - 32768), s0 = (uintptr_t)s + 8 * (t * FSLICE - 32768);
  double acc = 0.0;
  auto batch = [&](auto size, int k) {
    constexpr int B = decltype(size)::value;
    double hv[B], xv[B], sv[B];
    if (FORM == F_PLAIN) {
#pragma unroll
      for (int q = 0; q < B; ++q) {
        const int64_t at = b + FSLICE * (k + q) + lane;
        const int64_t j = col[at];
        hv[q] = h[at];
        xv[q] = x[j];
        sv[q] = GRAD ? s[j] : 1.0;
      }
    } else {
      uint32_t w[B];
#pragma unroll
      for (int q = 0; q < B; ++q) w[q] = (word + b + FSLICE * (k + q))[lane];
#pragma unroll
      for (int q = 0; q < B; ++q) {
        const uint32_t at = 8u * (uint32_t)(lane + 32768 + (int16_t)(w[q] & 0xffffu));
        xv[q] = *(const double*)(x0 + at);
        sv[q] = GRAD ? *(const double*)(s0 + at) : 1.0;
        hv[q] = FORM == F_PACKED_LDS ? tl[w[q] >> 16] : tab[w[q] >> 16];
      }
    }
#pragma unroll
    for (int q = 0; q < B; ++q) acc = fma(hv[q], GRAD ? sv[q] * xv[q] : xv[q], acc);
  };
  static_assert(FBATCH == 8, "one case per size");
  for (int k = 0, left = (cnt + FBATCH - 1) / FBATCH; left > 0; --left) {
    const int size = (cnt - k + left - 1) / left;
    switch (size) {
      case 8: batch(std::integral_constant<int, 8>{}, k); break;
      case 7: batch(std::integral_constant<int, 7>{}, k); break;
      case 6: batch(std::integral_constant<int, 6>{}, k); break;
      case 5: batch(std::integral_constant<int, 5>{}, k); break;
      case 4: batch(std::integral_constant<int, 4>{}, k); break;
      case 3: batch(std::integral_constant<int, 3>{}, k); break;
      case 2: batch(std::integral_constant<int, 2>{}, k); break;
      default: batch(std::integral_constant<int, 1>{}, k); break;
    }
    k += size;
  }
  y[i] = GRAD ? acc : scale * acc;
}

template <class T>
int upload(T** dst, const std::vector<T>& v) {
  const size_t bytes = std::max<size_t>(v.size(), 1) * sizeof(T);
  if (hipMalloc((void**)dst, bytes) != hipSuccess) return set_error(MTO_ENOMEM, "hipMalloc failed (density filter)");
  if (!v.empty() && hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess)
    return set_error(MTO_EHIP, "hipMemcpy failed (density filter)");
  return MTO_OK;
}

int launch(const mto_filter* F, bool grad, const double* x, double* y, void* stream) {
  if (F->n == 0) return MTO_OK;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != F->device)
    return set_error(MTO_EINVAL, "density filter used on a device other than the one it was created on");
  const unsigned blocks = (unsigned)((F->n + 255) / 256 + 7) / 8 * 8;
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                       FilterDev{F->sp, F->word, F->tab, F->col, F->h, F->s, F->n, F->n_tab}, x, y);
  };
  if (!F->word)
    grad ? go(k_filter<true, F_PLAIN>) : go(k_filter<false, F_PLAIN>);
  else if (F->n_tab > FTAB)
    grad ? go(k_filter<true, F_PACKED>) : go(k_filter<false, F_PACKED>);
  else
    grad ? go(k_filter<true, F_PACKED_LDS>) : go(k_filter<false, F_PACKED_LDS>);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(MTO_EHIP, std::string("density filter launch: ") + hipGetErrorString(e));
  return MTO_OK;
}

}  // namespace

static int filter_create(const mto_problem* probs, int32_t n_inst, double R, mto_filter** out) {
  if (!out) return set_error(MTO_EINVAL, "out is NULL");
  *out = nullptr;
  if (!probs || n_inst < 1) return set_error(MTO_EINVAL, "no problems");
  if (!(R > 0.0) || !std::isfinite(R)) return set_error(MTO_EINVAL, "filter radius must be positive and finite");
  // rows of H with global column indices, instance by instance (element-major, s = sy*d + sx)
  std::vector<int64_t> rowp{0};
  std::vector<int32_t> rcol;
  std::vector<double> rh, inv;
  int64_t base = 0;
  for (int i = 0; i < n_inst; ++i) {
    const mto_mesh& m = probs[i].mesh;
    if (m.nelx < 1 || m.nely < 1 || !m.d) return set_error(MTO_EINVAL, "instance " + std::to_string(i) + ": bad mesh");
    const int nel = m.nelx * m.nely;
    std::vector<int64_t> eoff(nel + 1, 0);
    for (int e = 0; e < nel; ++e) {
      if (m.d[e] < 1 || m.d[e] > MTO_MAX_D) return set_error(MTO_EINVAL, "instance " + std::to_string(i) + ": bad d");
      eoff[e + 1] = eoff[e] + (int64_t)m.d[e] * m.d[e];
    }
    if (base + eoff[nel] >= ((int64_t)1 << 31)) return set_error(MTO_EINVAL, "too many cells for 32-bit indices");
    auto centre = [&](int e, int s, double& x, double& y) {
      const int de = m.d[e], ex = e % m.nelx, ey = e / m.nelx, sx = s % de, sy = s / de;
      x = ex + (sx + 0.5) / de;
      y = ey + (sy + 0.5) / de;
    };
    // centres lie strictly inside their elements, so two cells k elements
    // apart (in x or y) are more than k - 1 apart: k <= ceil(R) suffices
    const int rr = (int)std::min<double>(std::ceil(R), (double)std::max(m.nelx, m.nely));
    std::vector<std::pair<int64_t, double>> nb;
    for (int e = 0; e < nel; ++e) {
      const int ex = e % m.nelx, ey = e / m.nelx;
      for (int s = 0; s < m.d[e] * m.d[e]; ++s) {
        double xi, yi;
        centre(e, s, xi, yi);
        nb.clear();
        for (int ey2 = std::max(0, ey - rr); ey2 <= std::min(m.nely - 1, ey + rr); ++ey2)
          for (int ex2 = std::max(0, ex - rr); ex2 <= std::min(m.nelx - 1, ex + rr); ++ex2) {
            const int e2 = ey2 * m.nelx + ex2;
            for (int s2 = 0; s2 < m.d[e2] * m.d[e2]; ++s2) {
              double xj, yj;
              centre(e2, s2, xj, yj);
              const double dx = xi - xj, dy = yi - yj;
              const double dist = (e2 == e && s2 == s) ? 0.0 : std::sqrt(dx * dx + dy * dy);
              if (dist < R) nb.emplace_back(base + eoff[e2] + s2, R - dist);
            }
          }
        std::sort(nb.begin(), nb.end());
        double sum = 0.0;
        for (auto& t : nb) sum += t.second;
        inv.push_back(1.0 / sum);
        for (auto& t : nb) {
          rcol.push_back((int32_t)t.first);
          rh.push_back(t.second);
        }
        rowp.push_back((int64_t)rcol.size());
      }
    }
    base += eoff[nel];
  }
  const int64_t n = base, nnz = (int64_t)rcol.size();
  // slice by 64 rows, entries of a slice interleaved by lane
  const int64_t nsl = (n + FSLICE - 1) / FSLICE;
  std::vector<int64_t> sp(nsl + 1, 0);
  for (int64_t t = 0; t < nsl; ++t) {
    int64_t wmax = 0;
    for (int64_t r = t * FSLICE; r < std::min(n, (t + 1) * FSLICE); ++r) wmax = std::max(wmax, rowp[r + 1] - rowp[r]);
    sp[t + 1] = sp[t] + wmax * FSLICE;
  }
  const int64_t stored = sp[nsl];
  // the distinct values, 0 (padding) first, in order of appearance; id[k] the place of rh[k].  Most are
  // found by their low bits in a direct-mapped cache of places.
  std::vector<double> tab{0.0};
  std::unordered_map<double, uint32_t> place{{0.0, 0u}};
  std::vector<uint32_t> id(nnz), cache(4096, 0u);
  bool packed = true;
  for (int64_t r = 0; r < n && packed; ++r)
    for (int64_t k = rowp[r]; k < rowp[r + 1] && packed; ++k) {
      const double v = rh[k];
      uint64_t bits;
      std::memcpy(&bits, &v, 8);
      uint32_t& c = cache[(bits * 0x9E3779B97F4A7C15ull) >> 52];
      if (tab[c] != v) {
        const auto [it, fresh] = place.emplace(v, (uint32_t)tab.size());
        if (fresh) tab.push_back(v);
        c = it->second;
      }
      id[k] = c;
      const int64_t off = rcol[k] - r;
      packed = off >= -32768 && off <= 32767 && tab.size() <= 65536;
    }
  std::vector<uint32_t> word(packed ? stored : 0);
  std::vector<int32_t> col(packed ? 0 : stored);
  std::vector<double> h(packed ? 0 : stored, 0.0);
  for (int64_t t = 0; t < nsl; ++t) {
    const int64_t wd = (sp[t + 1] - sp[t]) / FSLICE;
    for (int lane = 0; lane < FSLICE; ++lane) {
      const int64_t r = t * FSLICE + lane;
      for (int64_t k = 0; k < wd; ++k) {
        const int64_t dst = sp[t] + k * FSLICE + lane;
        const bool real = r < n && k < rowp[r + 1] - rowp[r];
        // padding: zero weight on the row's own cell (or cell 0 past the end)
        const int32_t j = real ? rcol[rowp[r] + k] : (int32_t)(r < n ? r : 0);
        if (packed) {
          word[dst] = real ? ((uint32_t)(j - r) & 0xffffu) | id[rowp[r] + k] << 16 : 0u;
        } else {
          col[dst] = j;
          h[dst] = real ? rh[rowp[r] + k] : 0.0;
        }
      }
    }
  }
  mto_filter* F = new mto_filter();
  if (hipGetDevice(&F->device) != hipSuccess) {
    delete F;
    return set_error(MTO_EHIP, "hipGetDevice failed");
  }
  F->R = R;
  F->n = n;
  F->nnz = nnz;
  F->stored = stored;
  F->n_tab = (int32_t)tab.size();
  int rc;
  if ((rc = upload(&F->sp, sp)) || (rc = upload(&F->s, inv)) ||
      (packed ? (rc = upload(&F->word, word)) || (rc = upload(&F->tab, tab))
              : (rc = upload(&F->col, col)) || (rc = upload(&F->h, h)))) {
    mto_filter_destroy(F);
    return rc;
  }
  *out = F;
  return MTO_OK;
}

extern "C" {

int mto_filter_create(const mto_problem* probs, int32_t n_inst, double R, mto_filter** out) {
  clear_error();
  try {
    return filter_create(probs, n_inst, R, out);
  } catch (const std::bad_alloc&) {
    return set_error(MTO_ENOMEM, "host memory exhausted building the density filter (radius too large?)");
  }
}

int mto_filter_apply(const mto_filter* F, const double* rho, double* rho_tilde, void* stream) {
  clear_error();
  if (!F || !rho || !rho_tilde) return set_error(MTO_EINVAL, "NULL argument");
  if (rho == rho_tilde) return set_error(MTO_EINVAL, "the filter cannot run in place");
  return launch(F, false, rho, rho_tilde, stream);
}

int mto_filter_grad(const mto_filter* F, const double* g_tilde, double* g, void* stream) {
  clear_error();
  if (!F || !g_tilde || !g) return set_error(MTO_EINVAL, "NULL argument");
  if (g == g_tilde) return set_error(MTO_EINVAL, "the filter cannot run in place");
  return launch(F, true, g_tilde, g, stream);
}

int mto_filter_info(const mto_filter* F, int64_t* n_cells, int64_t* nnz) {
  clear_error();
  if (!F) return set_error(MTO_EINVAL, "NULL filter");
  if (n_cells) *n_cells = F->n;
  if (nnz) *nnz = F->nnz;
  return MTO_OK;
}

void mto_filter_destroy(mto_filter* F) {
  if (!F) return;
  int prev = -1;
  (void)hipGetDevice(&prev);
  (void)hipSetDevice(F->device);
  (void)hipDeviceSynchronize();
  void* bufs[] = {F->sp, F->word, F->tab, F->col, F->h, F->s};
  for (void* b : bufs)
    if (b) (void)hipFree(b);
  if (prev >= 0) (void)hipSetDevice(prev);
  delete F;
}

}  // extern "C"
