// Hierarchy setup on the device: the finest Toeplitz-plus-Cross level from
// the row stencils (eq. (split01), eq. (ccs2.6)), the Galerkin coarse levels
// by the recurrences of Lemma 3.1, and the few scalars the host needs.  The
// same arithmetic as the host setup in amg_host.cpp, one thread per entry,
// so that a hierarchy of 2^22 intervals forms in milliseconds.
#include <hip/hip_runtime.h>

#include "amg_device.hpp"

namespace amg {

namespace {

__device__ __forceinline__ double stencil_at(const double* W, int64_t S, int64_t s2) {
  return (s2 < -S || s2 > S) ? 0.0 : W[s2 + S];
}

__device__ __forceinline__ void flag_bad(int* bad, double v) {
  if (!isfinite(v)) atomicOr(bad, 1);
}

constexpr int kSetupNT = 256;

inline unsigned setup_grid(int64_t count) {
  const int64_t g = (count + kSetupNT - 1) / kSetupNT;
  return (unsigned)(g < 1 ? 1 : (g > 65535 ? 65535 : g));
}

}  // namespace

// Finest level (N - 1 = n): generators a, b, c, d (2n - 1 entries, offsets
// -(n-1)..n-1) and Cross vectors from the node-row stencil Wn and the
// midpoint-row stencil Wm (half-grid offsets); then scale * (all) + shift on
// the diagonal entries a_0, d_0, o.
__global__ __launch_bounds__(kSetupNT) void k_finest_level(const double* Wn, int64_t Sn,
                                                           const double* Wm, int64_t Sm, int64_t n,
                                                           double scale, double shift, double* a,
                                                           double* b, double* c, double* d,
                                                           double* p, double* q, double* xi,
                                                           double* zeta, double* o, int* bad) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < 2 * n - 1; k += stride) {
    const int64_t dd = k - (n - 1);
    const double sh = dd == 0 ? shift : 0.0;
    a[k] = stencil_at(Wn, Sn, 2 * dd) * scale + sh;
    b[k] = stencil_at(Wn, Sn, 2 * dd + 1) * scale;
    c[k] = stencil_at(Wm, Sm, 2 * dd - 1) * scale;
    d[k] = stencil_at(Wm, Sm, 2 * dd) * scale + sh;
    flag_bad(bad, a[k] + b[k] + c[k] + d[k]);
  }
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    p[i] = stencil_at(Wn, Sn, -2 * i - 1) * scale;
    q[i] = stencil_at(Wm, Sm, 2 * i + 1) * scale;
    xi[i] = stencil_at(Wm, Sm, -2 * i - 2) * scale;
    zeta[i] = stencil_at(Wm, Sm, 2 * i + 2) * scale;
    flag_bad(bad, p[i] + q[i] + xi[i] + zeta[i]);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    o[0] = stencil_at(Wm, Sm, 0) * scale + shift;
    flag_bad(bad, o[0]);
  }
}

// Lemma 3.1, Toeplitz part: t'_i = (t_{2i-2} + 4 t_{2i-1} + 6 t_{2i} +
// 4 t_{2i+1} + t_{2i+2}) / 8.  The bodies below take their first entry and
// stride: one thread per entry over the whole chip, or one workgroup's share.
__device__ __forceinline__ void coarsen_toeplitz(const double* f, int64_t n, double* t, int64_t k0,
                                                 int64_t stride, int* bad) {
  const int64_t nc = (n - 1) / 2;
  for (int64_t k = k0; k < 2 * nc - 1; k += stride) {
    const int64_t i = k - (nc - 1);
    const double* g = f + (n - 1);  // g[off] = t_off
    t[k] = (g[2 * i - 2] + 4 * g[2 * i - 1] + 6 * g[2 * i] + 4 * g[2 * i + 1] + g[2 * i + 2]) / 8.0;
    flag_bad(bad, t[k]);
  }
}

// Lemma 3.1, Cross part, first step: the fine w_o column A z (z = P e_{w_o})
// and row rho^T A on the v and w_bar blocks (n entries each).
__device__ __forceinline__ void coarsen_cols(const DevTpx& f, int64_t n, double* scratch,
                                             int64_t i0, int64_t stride) {
  double *colv = scratch, *colw = scratch + n, *rowv = scratch + 2 * n, *roww = scratch + 3 * n;
  const double *ga = f.a + (n - 1), *gb = f.b + (n - 1), *gc = f.c + (n - 1), *gd = f.d + (n - 1);
  for (int64_t i = i0; i < n; i += stride) {
    colv[i] = 0.5 * ga[n - 1 - i] + f.p[i] + 0.5 * gb[-i];
    colw[i] = 0.5 * gc[n - 1 - i] + f.xi[i] + 0.5 * gd[-i];
    rowv[i] = 0.25 * ga[i - n + 1] + 0.5 * f.q[i] + 0.25 * gc[i];
    roww[i] = 0.25 * gb[i - n + 1] + 0.5 * f.zeta[i] + 0.25 * gd[i];
  }
}

// Lemma 3.1, Cross part, second step: restrictions of those vectors give the
// coarse p, xi (column) and q, zeta (row, times 2), and the coarse o.
__device__ __forceinline__ void coarsen_cross(const DevTpx& f, int64_t n, const double* scratch,
                                              const DevTpx& c, int64_t i0, int64_t stride,
                                              int* bad) {
  const double *colv = scratch, *colw = scratch + n, *rowv = scratch + 2 * n,
               *roww = scratch + 3 * n;
  const int64_t nc = (n - 1) / 2;
  auto R = [](const double* x, int64_t i) {
    return 0.25 * (x[2 * i] + 2 * x[2 * i + 1] + x[2 * i + 2]);
  };
  for (int64_t i = i0; i < nc; i += stride) {
    c.p[i] = R(colv, i);
    c.xi[i] = R(colw, i);
    c.q[i] = 2.0 * R(rowv, i);
    c.zeta[i] = 2.0 * R(roww, i);
    flag_bad(bad, c.p[i] + c.xi[i] + c.q[i] + c.zeta[i]);
  }
  if (i0 == 0) {
    const double colo = 0.5 * f.q[n - 1] + f.o[0] + 0.5 * f.zeta[0];
    c.o[0] = 0.25 * colv[n - 1] + 0.5 * colo + 0.25 * colw[0];
    flag_bad(bad, c.o[0]);
  }
}

// A symmetric level's coarse image: the recurrences give mirror entries that
// agree only up to rounding; their averages keep the level exactly symmetric
// (A = D, C = B mirrored, p = q, xi = zeta).  Entry i stands for the pair
// (i, m-1-i) of the generators (m = 2nc - 1) and entry i of the vectors.
__device__ __forceinline__ void symmetrize(const DevTpx& t, int64_t nc, int64_t i0,
                                           int64_t stride) {
  const int64_t m = 2 * nc - 1;
  for (int64_t i = i0; i <= (m - 1) / 2; i += stride) {
    const int64_t j = m - 1 - i;
    const double ai = t.a[i], aj = t.a[j], bi = t.b[i], bj = t.b[j], ci = t.c[i], cj = t.c[j];
    const double Ai = 0.5 * (ai + aj), Aj = 0.5 * (aj + ai);
    const double Bi = 0.5 * (bi + cj), Bj = 0.5 * (bj + ci);
    t.a[i] = Ai;
    t.a[j] = Aj;
    t.d[i] = Ai;
    t.d[j] = Aj;
    t.b[i] = Bi;
    t.b[j] = Bj;
    t.c[j] = Bi;
    t.c[i] = Bj;
  }
  for (int64_t i = i0; i < nc; i += stride) {
    const double pq = 0.5 * (t.p[i] + t.q[i]), xz = 0.5 * (t.xi[i] + t.zeta[i]);
    t.p[i] = pq;
    t.q[i] = pq;
    t.xi[i] = xz;
    t.zeta[i] = xz;
  }
}

// Large levels: one launch per step (blockIdx.y: the four Toeplitz blocks,
// then the Cross columns), bound by memory.
__global__ __launch_bounds__(kSetupNT) void k_coarsen_first(DevTpx f, int64_t n, DevTpx c,
                                                            double* scratch, int* bad) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  switch (blockIdx.y) {
    case 0: coarsen_toeplitz(f.a, n, c.a, i0, stride, bad); break;
    case 1: coarsen_toeplitz(f.b, n, c.b, i0, stride, bad); break;
    case 2: coarsen_toeplitz(f.c, n, c.c, i0, stride, bad); break;
    case 3: coarsen_toeplitz(f.d, n, c.d, i0, stride, bad); break;
    default: coarsen_cols(f, n, scratch, i0, stride); break;
  }
}
__global__ __launch_bounds__(kSetupNT) void k_coarsen_cross(DevTpx f, int64_t n,
                                                            const double* scratch, DevTpx c,
                                                            int* bad) {
  coarsen_cross(f, n, scratch, c, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
                (int64_t)gridDim.x * blockDim.x, bad);
}
__global__ __launch_bounds__(kSetupNT) void k_symmetrize(DevTpx t, int64_t nc) {
  symmetrize(t, nc, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
             (int64_t)gridDim.x * blockDim.x);
}

// Small levels (n <= kCoarsenSmall): every level below the table's first in
// one workgroup, whose barriers stand for the launches.  A launch of the
// kernels above costs 5 us from start to start whatever the level's size;
// here a step takes the time one CU needs for its bytes: under 4 us at
// n = 4095, less than 1 at 511.
__global__ __launch_bounds__(1024) void k_coarsen_small(CoarsenTable tab, double* scratch, int sym,
                                                        int* bad) {
  int64_t n = tab.n;
  const int64_t i0 = threadIdx.x;
  for (int l = 0; l < tab.count; ++l) {
    const DevTpx f = tab.lev[l], c = tab.lev[l + 1];
    const int64_t nc = (n - 1) / 2;
    coarsen_toeplitz(f.a, n, c.a, i0, 1024, bad);
    coarsen_toeplitz(f.b, n, c.b, i0, 1024, bad);
    coarsen_toeplitz(f.c, n, c.c, i0, 1024, bad);
    coarsen_toeplitz(f.d, n, c.d, i0, 1024, bad);
    coarsen_cols(f, n, scratch, i0, 1024);
    __syncthreads();
    coarsen_cross(f, n, scratch, c, i0, 1024, bad);
    __syncthreads();
    if (sym) symmetrize(c, nc, i0, 1024);
    __syncthreads();
    n = nc;
  }
}

// What the host needs of the hierarchy, written to its pinned block at `out`
// (the order that launch_setup_pack declares): one kernel in place of a launch per level and ten
// copies.
__global__ __launch_bounds__(kSetupNT) void k_setup_pack(PackTable t, const int* bad, double* out) {
  const int tid = threadIdx.x;
  if (tid == 0) out[0] = (double)*bad;
  if (tid < t.nl) {
    out[1 + 3 * tid] = *t.o[tid];
    out[2 + 3 * tid] = t.a[tid][t.n[tid] - 1];
    out[3 + 3 * tid] = t.d[tid][t.n[tid] - 1];
  }
  const int nc = t.n[t.nl - 1], g = 2 * nc - 1;
  const DevTpx& c = t.last;
  double* gen = out + 1 + 3 * t.nl;
  for (int i = tid; i < g; i += kSetupNT) {
    gen[i] = c.a[i];
    gen[g + i] = c.b[i];
    gen[2 * g + i] = c.c[i];
    gen[3 * g + i] = c.d[i];
  }
  double* vec = gen + 4 * g;
  for (int i = tid; i < nc; i += kSetupNT) {
    vec[i] = c.p[i];
    vec[nc + i] = c.q[i];
    vec[2 * nc + i] = c.xi[i];
    vec[3 * nc + i] = c.zeta[i];
  }
  __threadfence_system();
}

// Clears and FP32 copies of many arrays in one launch: a workgroup per
// kSpanBlock entries, found in the table by bisection.  Bound by memory; a
// setup's arrays are many and mostly small, and a launch or a memset apiece
// took the host 3 - 5 us (200 of them a third of a problem solved once at
// N = 2^14).
__global__ __launch_bounds__(kSetupNT) void k_spans(SpanTable t) {
  const int b = blockIdx.x;
  int lo = 0, hi = t.count;  // first[lo] <= b < first[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (t.first[mid] <= b) lo = mid;
    else hi = mid;
  }
  const Span sp = t.span[lo];
  const int64_t i0 = (int64_t)(b - t.first[lo]) * kSpanBlock;
  const int64_t i1 = i0 + kSpanBlock < sp.n ? i0 + kSpanBlock : sp.n;
  if (sp.src) {
    float* dst = static_cast<float*>(sp.dst);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kSetupNT) dst[i] = (float)sp.src[i];
  } else {
    double* dst = static_cast<double*>(sp.dst);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kSetupNT) dst[i] = 0.0;
  }
}

hipError_t launch_spans(const std::vector<Span>& spans, hipStream_t s) {
  for (size_t i = 0; i < spans.size();) {
    SpanTable t{};
    int64_t blocks = 0;
    for (; i < spans.size() && t.count < kSpanMax; ++i) {
      const int64_t nb = (spans[i].n + kSpanBlock - 1) / kSpanBlock;
      if (nb <= 0) continue;
      if (blocks + nb > INT32_MAX) break;
      t.span[t.count] = spans[i];
      t.first[t.count++] = (int)blocks;
      blocks += nb;
    }
    if (t.count == 0) {
      if (i < spans.size()) return hipErrorInvalidValue;  // one span beyond a grid
      break;
    }
    t.first[t.count] = (int)blocks;
    hipLaunchKernelGGL(k_spans, (unsigned)blocks, kSetupNT, 0, s, t);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Deterministic test data in [-1/2, 1/2) (a 32-bit integer hash of the
// index and the seed; inputs of the geometry tuner, whose results are only
// compared with each other).
__global__ __launch_bounds__(kSetupNT) void k_fill_hash(double* p, int64_t n, unsigned seed) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    unsigned h = (unsigned)i * 0x9E3779B1u ^ (unsigned)(i >> 32) ^ (seed * 0x85EBCA77u);
    h ^= h >> 16;
    h *= 0x7FEB352Du;
    h ^= h >> 15;
    h *= 0x846CA68Bu;
    h ^= h >> 16;
    p[i] = (double)(h >> 8) * (1.0 / 16777216.0) - 0.5;
  }
}

hipError_t launch_fill_hash(double* p, int64_t n, unsigned seed, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_hash, setup_grid(n), kSetupNT, 0, s, p, n, seed);
  return hipGetLastError();
}

hipError_t launch_finest_level(const double* Wn, int64_t Sn, const double* Wm, int64_t Sm,
                               int64_t n, double scale, double shift, const DevTpx& f, int* bad,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_finest_level, setup_grid(2 * n), kSetupNT, 0, s, Wn, Sn, Wm, Sm, n, scale,
                     shift, f.a, f.b, f.c, f.d, f.p, f.q, f.xi, f.zeta, f.o, bad);
  return hipGetLastError();
}

hipError_t launch_coarsen(const DevTpx& f, int64_t n, const DevTpx& c, double* scratch, bool sym,
                          int* bad, hipStream_t s) {
  const int64_t nc = (n - 1) / 2;
  if (n < 3 || (n & 1) == 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_coarsen_first, dim3(setup_grid(n), 5), kSetupNT, 0, s, f, n, c, scratch,
                     bad);
  hipLaunchKernelGGL(k_coarsen_cross, setup_grid(nc), kSetupNT, 0, s, f, n, scratch, c, bad);
  if (sym) hipLaunchKernelGGL(k_symmetrize, setup_grid(nc), kSetupNT, 0, s, c, nc);
  return hipGetLastError();
}

hipError_t launch_coarsen_small(const CoarsenTable& tab, double* scratch, bool sym, int* bad,
                                hipStream_t s) {
  int64_t n = tab.n;
  if (n > kCoarsenSmall || tab.count < 1 || tab.count >= kCoarsenLevels) return hipErrorInvalidValue;
  for (int l = 0; l < tab.count; ++l, n = (n - 1) / 2)
    if (n < 3 || (n & 1) == 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_coarsen_small, 1, 1024, 0, s, tab, scratch, sym ? 1 : 0, bad);
  return hipGetLastError();
}

hipError_t launch_setup_pack(const PackTable& t, const int* bad, double* out, hipStream_t s) {
  if (t.nl < 1 || t.nl > kPackLevels) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_setup_pack, 1, kSetupNT, 0, s, t, bad, out);
  return hipGetLastError();
}

}  // namespace amg
