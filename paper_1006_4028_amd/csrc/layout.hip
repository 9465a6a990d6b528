// Layout kernels: host-order (x0 slowest, complex128 interleaved) fields to the
// structure-of-arrays parity layout and back, precision conversion, the source
// redefinition eta' = beta eta, the restoration S = S'/beta and the per-
// timeslice correlator C_PP(y0) = -sum_y tr[S^+ S] (heavy-quark section,
// restoration eq. backcorrection in the form C = C'/alpha^2).  beta(y) =
// alpha(y0) a_1(y1) a_2(y2) a_3(y3): the time profile alpha of eq. redeft and
// the spatial factors of the light-quark factorisation (eqs. redefa, betaa),
// which must be divided out site by site before the contraction.
#include <algorithm>

#include "dp_device.h"

namespace dp {

namespace {

// a_1(x1) a_2(x2) a_3(x3), or 1 without spatial profiles
__device__ __forceinline__ double space_factor(const Geom& g, const double* sprof, int x1, int x2, int x3) {
  return sprof ? sprof[x1] * sprof[g.L1 + x2] * sprof[g.L1 + g.L2 + x3] : 1.0;
}

// ------------------------------------------------------------ transposes
//
// Between the host order (all components of a site together, both parities
// interleaved) and the parity fields (one array per component) every wave
// transposes 64 consecutive sites through LDS, so that it reads and writes
// whole cache lines on both sides: with a site per thread, whose 16-byte
// accesses lie 192 (spinors) or 576 (links) bytes apart, the export of 12
// columns at 24^3x48 took 1058 us, the two imports 652.  Extents are even, so
// sites 2 j and 2 j + 1 have one of each parity and index j in it: lanes 0..31
// take the even parity's sites of the 32 pairs, lanes 32..63 the odd one's.

constexpr int kPairs = 32;  // site pairs of one wave

// the pair's even site: x1, x2, x3 and its parity
struct Pair {
  int x0, x1, x2, x3, q;
};
__device__ __forceinline__ Pair pair_coords(const Geom& g, int i) {
  Pair c;
  const int row = i / g.L3h;
  c.x3 = 2 * (i - row * g.L3h);
  const int t = row / g.L2;
  c.x2 = row - t * g.L2;
  c.x0 = t / g.L1;
  c.x1 = t - c.x0 * g.L1;
  c.q = (c.x0 + c.x1 + c.x2) & 1;
  return c;
}

// host-order links -> parity fields in the three precisions, one read for all.
// A wave takes 16 pairs (18 KB of LDS).  LDS rows of 37 units: a column of 16
// lanes then touches every bank group once.
constexpr int kLinkPairs = 16;
struct GaugeDst {
  double2* f64[2];
  float2* f32[2];
  unsigned* f16[2];
};
__global__ void __launch_bounds__(64) gauge_reorder_kernel(Geom g, const double2* __restrict__ U, GaugeDst o) {
  __shared__ double2 t[2 * kLinkPairs * 37];
  const int lane = threadIdx.x, i0 = blockIdx.x * kLinkPairs;
  const long base = 2L * i0 * 36, total = 2L * g.Vh * 36;
#pragma unroll
  for (int m = 0; m < 2 * kLinkPairs * 36 / 64; ++m) {
    const int k = lane + 64 * m;
    double2 v = make_double2(0.0, 0.0);
    if (base + k < total) v = U ? vld<true>(U + base + k) : make_double2((k % 36) % 9 % 4 == 0 ? 1.0 : 0.0, 0.0);
    t[(k / 36) * 37 + k % 36] = v;
  }
  __syncthreads();
  // lanes: 16 pairs, 2 parities, 2 components at a time
  const int j = lane & 15, p = (lane >> 4) & 1, i = i0 + j;
  if (i >= g.Vh) return;
  const Pair c = pair_coords(g, i);
  const double2* src = t + (2 * j + (c.q ^ p)) * 37;
  for (int k = lane >> 5; k < 36; k += 2) {
    const double2 v = src[k];
    const long at = (long)k * g.Vp + i;
    if (o.f64[p]) o.f64[p][at] = v;
    if (o.f32[p]) o.f32[p][at] = make_float2((float)v.x, (float)v.y);
    if (o.f16[p]) o.f16[p][at] = f2h((float)v.x, (float)v.y);
  }
}

// host-order spinors -> FP64 parity fields (both), optionally times beta(x)
__global__ void __launch_bounds__(64) spinor_import_kernel(Geom g, const double2* __restrict__ aos, long aos_ss,
                                                           SpinorRef e, SpinorRef o, const double* __restrict__ amul,
                                                           const double* __restrict__ sprof) {
  __shared__ double2 t[2 * kPairs * 13];
  const int lane = threadIdx.x, i0 = blockIdx.x * kPairs, slot = blockIdx.y;
  const double2* src = aos + slot * aos_ss + 2L * i0 * 12;
  const int n = min(kPairs, g.Vh - i0) * 24;
#pragma unroll
  for (int m = 0; m < 12; ++m) {
    const int k = lane + 64 * m;
    if (k < n) t[(k / 12) * 13 + k % 12] = vld<true>(src + k);
  }
  __syncthreads();
  const int j = lane & 31, p = lane >> 5, i = i0 + j;
  if (i >= g.Vh) return;
  const Pair c = pair_coords(g, i);
  const int odd = c.q ^ p;  // the pair's second site has the other parity
  const double f = (amul ? amul[(long)slot * g.T + c.x0] : 1.0) * space_factor(g, sprof, c.x1, c.x2, c.x3 + odd);
  const SpinorRef& d = p ? o : e;
  double2* dst = static_cast<double2*>(d.data) + slot * d.slot_stride + i;
  const double2* q = t + (2 * j + odd) * 13;
#pragma unroll
  for (int k = 0; k < 12; ++k) dst[(long)k * g.Vp] = make_double2(f * q[k].x, f * q[k].y);
}

// FP64 parity fields -> host-order spinors, optionally divided by beta(x)
__global__ void __launch_bounds__(64) spinor_export_kernel(Geom g, SpinorRef e, SpinorRef o,
                                                           const double* __restrict__ adiv,
                                                           const double* __restrict__ sprof,
                                                           double2* __restrict__ aos, long aos_ss) {
  __shared__ double2 t[2 * kPairs * 13];
  const int lane = threadIdx.x, i0 = blockIdx.x * kPairs, slot = blockIdx.y;
  const int j = lane & 31, p = lane >> 5, i = i0 + j;
  if (i < g.Vh) {
    const Pair c = pair_coords(g, i);
    const int odd = c.q ^ p;
    const SpinorRef& f = p ? o : e;
    const double2* src = static_cast<const double2*>(f.data) + slot * f.slot_stride + i;
    const double inv =
        1.0 / ((adiv ? adiv[(long)slot * g.T + c.x0] : 1.0) * space_factor(g, sprof, c.x1, c.x2, c.x3 + odd));
    double2* q = t + (2 * j + odd) * 13;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const double2 v = vld<true>(src + (long)k * g.Vp);
      q[k] = make_double2(v.x * inv, v.y * inv);
    }
  }
  __syncthreads();
  double2* dst = aos + slot * aos_ss + 2L * i0 * 12;
  const int n = min(kPairs, g.Vh - i0) * 24;
#pragma unroll
  for (int m = 0; m < 12; ++m) {
    const int k = lane + 64 * m;
    if (k < n) vst<true>(dst + k, t[(k / 12) * 13 + k % 12]);
  }
}

// One block per (timeslice, slot): -sum over both parities of |psi|^2 / beta^2
// (the time factor alpha^2 after the sum, the spatial ones per site).
__global__ void __launch_bounds__(kBlock) cpp_kernel(Geom g, SpinorRef e, SpinorRef o,
                                                     const double* __restrict__ alpha, const double* __restrict__ sprof,
                                                     const int* __restrict__ x0src, const int* __restrict__ mask,
                                                     double* __restrict__ cpp) {
  const int x0 = blockIdx.x, slot = blockIdx.y;
  if (mask && !mask[slot]) return;
  __shared__ double lds[kBlock / 64];
  double acc = 0.0;
  for (int par = 0; par < 2; ++par) {
    const SpinorRef& f = par ? o : e;
    const double2* src = static_cast<const double2*>(f.data) + slot * f.slot_stride;
    for (int k = threadIdx.x; k < g.Vsh; k += kBlock) {
      const int i = x0 * g.Vsh + k;
      double site = 0.0;
      for (int c = 0; c < 12; ++c) {
        const double2 v = src[(long)c * g.Vp + i];
        site += v.x * v.x + v.y * v.y;
      }
      if (sprof) {
        int y0, y1, y2, y3;
        eo_coords(g, par, i, y0, y1, y2, y3);
        const double f = space_factor(g, sprof, y1, y2, y3);
        site /= f * f;
      }
      acc += site;
    }
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) s += lds[w];
    const double a = alpha ? alpha[(long)slot * g.T + x0] : 1.0;
    const int t = ((x0 - (x0src ? x0src[slot] : 0)) % g.T + g.T) % g.T;
    cpp[(long)slot * g.T + t] = -s / (a * a);
  }
}

// Fill of ncols point-source columns (every entry written: no memset, so the
// launch may sit in a captured graph).  Grid-stride over the 12 V ncols
// complex entries.
__global__ void __launch_bounds__(kBlock) point_source_kernel(long per_col, long at, int c0, int ncols,
                                                              double2* __restrict__ out) {
  const long total = per_col * ncols;
  for (long k = (long)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (long)gridDim.x * blockDim.x) {
    const long j = k / per_col, r = k - j * per_col;
    out[k] = make_double2(r == at + c0 + j ? 1.0 : 0.0, 0.0);
  }
}

// The boundary sources of the Schroedinger functional, column j for
// c = c0 + j: side 0, U_0(x0 = 0, xs)^+ P+ e_c on the first interior
// timeslice, P+ = (1 + gamma_0)/2 (the projector of the backward time hop,
// so that this is the hop from a boundary field P+ psi(0) = e_c); side 1,
// U_0(x0 = T, xs) P- e_c on the last interior timeslice, P- = (1 -
// gamma_0)/2 (the forward time hop into the boundary field at x0 = T + 1);
// 0 elsewhere.  In the chiral basis gamma_0 has -1 between spins s and
// s +- 2, so P+- is 1/2 on the diagonal and -+1/2 between those spins.
// Ut: the time links of the boundary-adjacent timeslice, host layout
// [xs][mu][3][3]; the source timeslice starts at element site0 * 12.
__global__ void __launch_bounds__(kBlock) sf_wall_source_kernel(long per_col, long Vs, long site0, int side, int c0,
                                                                int ncols, const double2* __restrict__ Ut,
                                                                double2* __restrict__ out) {
  const long total = per_col * ncols;
  for (long k = (long)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (long)gridDim.x * blockDim.x) {
    const long j = k / per_col, r = k - j * per_col;
    const long site = r / 12 - site0;
    const int comp = (int)(r % 12), s = comp / 3, a = comp % 3;
    double2 v = make_double2(0.0, 0.0);
    if (site >= 0 && site < Vs) {  // the source timeslice
      const int c = c0 + (int)j, sc = c / 3, ac = c % 3;
      const double off = side == 0 ? -0.5 : 0.5;
      const double pp = s == sc ? 0.5 : ((s & 1) == (sc & 1) ? off : 0.0);
      if (side == 0) {  // (U^+)[a][ac] = conj(U[ac][a])
        const double2 u = Ut[(site * 4 + 0) * 9 + ac * 3 + a];
        v = make_double2(pp * u.x, -pp * u.y);
      } else {  // U[a][ac]
        const double2 u = Ut[(site * 4 + 0) * 9 + a * 3 + ac];
        v = make_double2(pp * u.x, pp * u.y);
      }
    }
    out[k] = v;
  }
}

}  // namespace

hipError_t launch_sf_wall_sources(const Geom& g, const double2* Ut, int side, int c0, int ncols, double2* out,
                                  hipStream_t st) {
  if (ncols <= 0 || c0 < 0 || c0 + ncols > 12 || (side != 0 && side != 1)) return hipErrorInvalidValue;
  const long per_col = 2L * g.Vh * 12;
  const long Vs = 2L * g.Vsh;
  const long site0 = side == 0 ? 0 : (long)(g.T - 1) * Vs;
  const long total = per_col * ncols;
  const long blocks = std::min<long>((total + kBlock - 1) / kBlock, 8L * 1024);
  hipLaunchKernelGGL(sf_wall_source_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st, per_col, Vs, site0, side, c0,
                     ncols, Ut, out);
  return hipGetLastError();
}

hipError_t launch_point_sources(const Geom& g, const int site[4], int c0, int ncols, double2* out, hipStream_t st) {
  if (ncols <= 0 || c0 < 0 || c0 + ncols > 12) return hipErrorInvalidValue;
  const long per_col = 2L * g.Vh * 12;
  const long at = ((((long)site[0] * g.L1 + site[1]) * g.L2 + site[2]) * g.L3 + site[3]) * 12;
  const long total = per_col * ncols;
  const long blocks = std::min<long>((total + kBlock - 1) / kBlock, 8L * 1024);
  hipLaunchKernelGGL(point_source_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st, per_col, at, c0, ncols, out);
  return hipGetLastError();
}

hipError_t launch_gauge_reorder(const Geom& g, const double2* U_aos, void* const U64[2], void* const U32[2],
                                void* const U16[2], hipStream_t st) {
  GaugeDst o;
  for (int p = 0; p < 2; ++p) {
    o.f64[p] = static_cast<double2*>(U64[p]);
    o.f32[p] = U32 ? static_cast<float2*>(U32[p]) : nullptr;
    o.f16[p] = U16 ? static_cast<unsigned*>(U16[p]) : nullptr;
  }
  hipLaunchKernelGGL(gauge_reorder_kernel, dim3((g.Vh + kLinkPairs - 1) / kLinkPairs), dim3(64), 0, st, g, U_aos, o);
  return hipGetLastError();
}

hipError_t launch_spinor_import(const Geom& g, const double2* aos, int nslots, long aos_ss, SpinorRef even,
                                SpinorRef odd, const double* alpha_mul, const double* sprof, hipStream_t st) {
  if (even.prec != F64 || odd.prec != F64 || nslots <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(spinor_import_kernel, dim3((g.Vh + kPairs - 1) / kPairs, nslots), dim3(64), 0, st, g, aos, aos_ss,
                     even, odd, alpha_mul, sprof);
  return hipGetLastError();
}

hipError_t launch_spinor_export(const Geom& g, SpinorRef even, SpinorRef odd, int nslots, const double* alpha_div,
                                const double* sprof, double2* aos, long aos_ss, hipStream_t st) {
  if (even.prec != F64 || odd.prec != F64 || nslots <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(spinor_export_kernel, dim3((g.Vh + kPairs - 1) / kPairs, nslots), dim3(64), 0, st, g, even, odd,
                     alpha_div, sprof, aos, aos_ss);
  return hipGetLastError();
}

hipError_t launch_cpp(const Geom& g, SpinorRef even, SpinorRef odd, int nslots, const double* alpha,
                      const double* sprof, const int* x0src, const int* mask, double* cpp, hipStream_t st) {
  if (even.prec != F64 || odd.prec != F64 || nslots <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(cpp_kernel, dim3(g.T, nslots), dim3(kBlock), 0, st, g, even, odd, alpha, sprof, x0src, mask, cpp);
  return hipGetLastError();
}

}  // namespace dp
