// SAP+GCR: the domain-decomposition solver of the paper's light-quark
// iteration counts (Table 1, the Schwarz alternating procedure of the
// reference the paper cites for it) on the distance-preconditioned operator
// D' (time profile and the spatial profiles of the light-quark factorisation).
//
// The lattice is cut into blocks (an even number per direction) coloured by
// the parity of their block coordinates.  One application of the
// preconditioner, psi = M r, runs ncy cycles; each cycle treats colour 0, then
// colour 1: rho = (r - D' psi) on the blocks of that colour (zero elsewhere),
// then nmr minimal-residual steps on every block of the colour at once:
// a = D' rho (with rho zero off the colour, a on the colour's sites is the
// direct sum of the Dirichlet block operators, since touching blocks differ
// in colour), w_B = <a, rho>_B / <a, a>_B per block, psi += w_B rho,
// rho -= w_B a.  The block solves run in FP32 (or FP64); flexible GCR in FP64
// (restart length nkv) solves D' x = eta' with M on the right.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <complex>
#include <vector>

#include "dp_device.h"
#include "runtime.h"

using namespace dp;
using namespace dp::rt;

namespace dp {

namespace {

struct Blocking {
  int bs[4];     // block extents
  int nb[4];     // blocks per direction
  int vol;       // sites per block
  int nhalf;     // blocks of one colour
};

// the site's block colour
__device__ __forceinline__ int colour_of(const Blocking& b, int x0, int x1, int x2, int x3) {
  return (x0 / b.bs[0] + x1 / b.bs[1] + x2 / b.bs[2] + x3 / b.bs[3]) & 1;
}

// rho = colour-c part of (r - a) (a = D' psi; a null means psi = 0), zero
// elsewhere; grid over (sites of one parity, 2 parities)
template <int P>
__global__ void __launch_bounds__(kBlock) sap_residual_kernel(Geom g, Blocking b, int colour, SpinorRef r,
                                                              SpinorRef a, SpinorRef rho, int have_a) {
  using R = typename Tr<P>::R;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (i >= g.Vh) return;
  int x0, x1, x2, x3;
  eo_coords(g, p, i, x0, x1, x2, x3);
  cx<R> v[12];
  if (colour_of(b, x0, x1, x2, x3) == colour) {
    SpinorIO<P>::load(r, p, i, g.Vp, v);
    if (have_a) {
      cx<R> w[12];
      SpinorIO<P>::load(a, p, i, g.Vp, w);
#pragma unroll
      for (int c = 0; c < 12; ++c) v[c] = v[c] - w[c];
    }
  } else {
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = cx<R>{R(0), R(0)};
  }
  SpinorIO<P>::store(rho, p, i, g.Vp, v);
}

// One minimal-residual step on every block of one colour: one workgroup per
// block, the block sums in FP64 in a fixed order, then psi += w rho, rho -= w a.
template <int P>
__global__ void __launch_bounds__(kBlock) sap_mr_kernel(Geom g, Blocking b, int colour, SpinorRef a, SpinorRef rho,
                                                        SpinorRef psi) {
  using R = typename Tr<P>::R;
  // the k-th block of this colour: the last block coordinate takes the parity
  int k = blockIdx.x;
  const int h3 = b.nb[3] / 2;
  int c3 = k % h3;
  k /= h3;
  const int c2 = k % b.nb[2];
  k /= b.nb[2];
  const int c1 = k % b.nb[1];
  const int c0 = k / b.nb[1];
  c3 = 2 * c3 + ((colour + c0 + c1 + c2) & 1);
  const int o0 = c0 * b.bs[0], o1 = c1 * b.bs[1], o2 = c2 * b.bs[2], o3 = c3 * b.bs[3];
  __shared__ double lds[3][kBlock / 64];
  __shared__ double wsh[2];
  double num_re = 0.0, num_im = 0.0, den = 0.0;
  for (int s = threadIdx.x; s < b.vol; s += kBlock) {
    int t = s;
    const int l3 = t % b.bs[3];
    t /= b.bs[3];
    const int l2 = t % b.bs[2];
    t /= b.bs[2];
    const int l1 = t % b.bs[1];
    const int l0 = t / b.bs[1];
    const int x0 = o0 + l0, x1 = o1 + l1, x2 = o2 + l2, x3 = o3 + l3;
    const int p = (x0 + x1 + x2 + x3) & 1;
    const int i = eo_index(g, x0, x1, x2, x3);
    cx<R> va[12], vr[12];
    SpinorIO<P>::load(a, p, i, g.Vp, va);
    SpinorIO<P>::load(rho, p, i, g.Vp, vr);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      num_re += (double)va[c].x * (double)vr[c].x + (double)va[c].y * (double)vr[c].y;
      num_im += (double)va[c].x * (double)vr[c].y - (double)va[c].y * (double)vr[c].x;
      den += (double)va[c].x * (double)va[c].x + (double)va[c].y * (double)va[c].y;
    }
  }
  num_re = wave_sum(num_re);
  num_im = wave_sum(num_im);
  den = wave_sum(den);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
    lds[0][wv] = num_re;
    lds[1][wv] = num_im;
    lds[2][wv] = den;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double nr = 0.0, ni = 0.0, d = 0.0;
    for (int q = 0; q < kBlock / 64; ++q) {
      nr += lds[0][q];
      ni += lds[1][q];
      d += lds[2][q];
    }
    wsh[0] = d > 0.0 ? nr / d : 0.0;
    wsh[1] = d > 0.0 ? ni / d : 0.0;
  }
  __syncthreads();
  const cx<R> w{(R)wsh[0], (R)wsh[1]};
  for (int s = threadIdx.x; s < b.vol; s += kBlock) {
    int t = s;
    const int l3 = t % b.bs[3];
    t /= b.bs[3];
    const int l2 = t % b.bs[2];
    t /= b.bs[2];
    const int l1 = t % b.bs[1];
    const int l0 = t / b.bs[1];
    const int x0 = o0 + l0, x1 = o1 + l1, x2 = o2 + l2, x3 = o3 + l3;
    const int p = (x0 + x1 + x2 + x3) & 1;
    const int i = eo_index(g, x0, x1, x2, x3);
    cx<R> va[12], vr[12], vp[12];
    SpinorIO<P>::load(a, p, i, g.Vp, va);
    SpinorIO<P>::load(rho, p, i, g.Vp, vr);
    SpinorIO<P>::load(psi, p, i, g.Vp, vp);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      vp[c] = vp[c] + cmul(w, vr[c]);
      vr[c] = vr[c] - cmul(w, va[c]);
    }
    SpinorIO<P>::store(psi, p, i, g.Vp, vp);
    SpinorIO<P>::store(rho, p, i, g.Vp, vr);
  }
}

// ------------------------------------------------------------ vector kernels
// Full-lattice vectors are two-slot fields: slot p holds the sites of parity p.

// y = x converted between precisions
template <int PI, int PO>
__global__ void __launch_bounds__(kBlock) vec_convert_kernel(Geom g, SpinorRef x, SpinorRef y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (i >= g.Vh) return;
  cx<double> v[12];
  SpinorIO<PI>::load(x, p, i, g.Vp, v);
  SpinorIO<PO>::store(y, p, i, g.Vp, v);
}

// y = x, or y = 0 without x (y is not read, so that whatever a failed solve
// left in it is overwritten, not carried: 0 * NaN is NaN)
__global__ void __launch_bounds__(kBlock) vec_set_kernel(Geom g, SpinorRef x, SpinorRef y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (i >= g.Vh) return;
  cx<double> v[12];
  if (x.data) {
    SpinorIO<F64>::load(x, p, i, g.Vp, v);
  } else {
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = cx<double>{0.0, 0.0};
  }
  SpinorIO<F64>::store(y, p, i, g.Vp, v);
}

// block partials of <x, y> (complex) over both parities: partials[blockIdx][2]
__global__ void __launch_bounds__(kBlock) vec_dot_kernel(Geom g, SpinorRef x, SpinorRef y, double* partials) {
  __shared__ double lds[2][kBlock / 64];
  double re = 0.0, im = 0.0;
  const long n = 2L * g.Vh;
  for (long s = (long)blockIdx.x * blockDim.x + threadIdx.x; s < n; s += (long)gridDim.x * blockDim.x) {
    const int p = (int)(s / g.Vh), i = (int)(s - (long)p * g.Vh);
    cx<double> vx[12], vy[12];
    SpinorIO<F64>::load(x, p, i, g.Vp, vx);
    SpinorIO<F64>::load(y, p, i, g.Vp, vy);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      re += vx[c].x * vy[c].x + vx[c].y * vy[c].y;
      im += vx[c].x * vy[c].y - vx[c].y * vy[c].x;
    }
  }
  re = wave_sum(re);
  im = wave_sum(im);
  if ((threadIdx.x & 63) == 0) {
    lds[0][threadIdx.x >> 6] = re;
    lds[1][threadIdx.x >> 6] = im;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int q = 0; q < kBlock / 64; ++q) {
      a += lds[0][q];
      b += lds[1][q];
    }
    partials[2 * blockIdx.x] = a;
    partials[2 * blockIdx.x + 1] = b;
  }
}

// ------------------------------------------------------- fused block solves
//
// The whole pass over one colour (the block residual, then nmr
// minimal-residual steps) runs as one kernel, a workgroup per block.  Hops that
// leave the block drop in the minimal-residual steps (Dirichlet block
// boundaries); the residual is r - D'_B psi, with the same block operator, minus
// the hops from the neighbour blocks, which touch only the sites of the faces.
// Three kernels, by what of a block fits on the chip:
//  - sap_slice_kernel: at most kSapThreads sites and a whole number of time
//    slices in a wave; links, clover and residual stay on the chip
//  - sap_block_kernel: at most kSapThreads sites; links and residual
//  - sap_block_big_kernel: at most kSapBigSites sites; the residual
//
// The fields of the pass are stored block by block ("block layout"): the
// blocks of colour 0 in the order of their index k, then those of colour 1;
// each block as component arrays over its sites s = ((l0 b1 + l1) b2 + l2) b3
// + l3 (l = coordinates within the block), so that the lanes of a wave, one
// site each, read consecutive addresses.  Spinors: float4 [6][vol] per block
// (components 2q, 2q + 1); links: float2 [4][9][vol]; clover: float4 [18][vol]
// (the packed blocks of the parity fields).

constexpr int kSapThreads = 256;

struct BLoc {
  int blk, s;
};

// block-layout position of site x
__device__ __forceinline__ BLoc bl_locate(const Blocking& b, int x0, int x1, int x2, int x3) {
  const int c0 = x0 / b.bs[0], c1 = x1 / b.bs[1], c2 = x2 / b.bs[2], c3 = x3 / b.bs[3];
  const int colour = (c0 + c1 + c2 + c3) & 1;
  const int k = ((c0 * b.nb[1] + c1) * b.nb[2] + c2) * (b.nb[3] / 2) + c3 / 2;
  const int s = (((x0 - c0 * b.bs[0]) * b.bs[1] + (x1 - c1 * b.bs[1])) * b.bs[2] + (x2 - c2 * b.bs[2])) * b.bs[3] +
                (x3 - c3 * b.bs[3]);
  return {colour * b.nhalf + k, s};
}

// The site of position n of the blocks in lexicographic order: its place in
// the block layout (blk, s) and in the parity fields (p, i).  Neighbouring
// threads are neighbouring sites of a block, so that the block layout is
// written in whole lines, and neighbouring workgroups of an XCD (xcd_tile)
// neighbouring blocks, which share the lines of the parity fields (a thread
// per parity site wrote 16 scattered bytes a line: 251 us for one vector at
// 64x32^3, 1296 us for the links and blocks).
struct BSite {
  int blk, s, p, i;
};
__device__ __forceinline__ BSite bl_site(const Geom& g, const Blocking& b, long n) {
  int k = (int)(n / b.vol), s = (int)(n - (long)k * b.vol);
  BSite r;
  r.s = s;
  const int c3 = k % b.nb[3];
  k /= b.nb[3];
  const int c2 = k % b.nb[2];
  k /= b.nb[2];
  const int c1 = k % b.nb[1], c0 = k / b.nb[1];
  r.blk = ((c0 + c1 + c2 + c3) & 1) * b.nhalf + ((c0 * b.nb[1] + c1) * b.nb[2] + c2) * (b.nb[3] / 2) + c3 / 2;
  const int x3 = c3 * b.bs[3] + s % b.bs[3];
  s /= b.bs[3];
  const int x2 = c2 * b.bs[2] + s % b.bs[2];
  s /= b.bs[2];
  const int x1 = c1 * b.bs[1] + s % b.bs[1], x0 = c0 * b.bs[0] + s / b.bs[1];
  r.p = (x0 + x1 + x2 + x3) & 1;
  r.i = eo_index(g, x0, x1, x2, x3);
  return r;
}

// FP32 links and clover of both parities -> block layout
__global__ void __launch_bounds__(kBlock) sap_gather_kernel(Geom g, Blocking b, const float2* __restrict__ U0,
                                                            const float2* __restrict__ U1,
                                                            const float4* __restrict__ C0,
                                                            const float4* __restrict__ C1, float2* __restrict__ ubl,
                                                            float4* __restrict__ cbl) {
  const long n = (long)xcd_tile(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (n >= 2L * g.Vh) return;
  const BSite q = bl_site(g, b, n);
  const float2* U = q.p ? U1 : U0;
  const float4* C = q.p ? C1 : C0;
#pragma unroll 9
  for (int k = 0; k < 36; ++k) ubl[((long)q.blk * 36 + k) * b.vol + q.s] = U[(long)k * g.Vp + q.i];
#pragma unroll 9
  for (int k = 0; k < 18; ++k) cbl[((long)q.blk * 18 + k) * b.vol + q.s] = C[(long)k * g.Vp + q.i];
}

// FP64 parity fields -> FP32 block layout
__global__ void __launch_bounds__(kBlock) sap_to_block_kernel(Geom g, Blocking b, SpinorRef x,
                                                              float4* __restrict__ out) {
  const long n = (long)xcd_tile(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (n >= 2L * g.Vh) return;
  const BSite q = bl_site(g, b, n);
  cx<double> v[12];
  SpinorIO<F64>::load(x, q.p, q.i, g.Vp, v);
#pragma unroll
  for (int k = 0; k < 6; ++k)
    out[((long)q.blk * 6 + k) * b.vol + q.s] =
        make_float4((float)v[2 * k].x, (float)v[2 * k].y, (float)v[2 * k + 1].x, (float)v[2 * k + 1].y);
}

// FP32 block layout -> FP64 parity fields
__global__ void __launch_bounds__(kBlock) sap_from_block_kernel(Geom g, Blocking b, const float4* __restrict__ in,
                                                                SpinorRef y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (i >= g.Vh) return;
  int x0, x1, x2, x3;
  eo_coords(g, p, i, x0, x1, x2, x3);
  const BLoc q = bl_locate(b, x0, x1, x2, x3);
  cx<double> v[12];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const float4 f = in[((long)q.blk * 6 + k) * b.vol + q.s];
    v[2 * k] = cx<double>{f.x, f.y};
    v[2 * k + 1] = cx<double>{f.z, f.w};
  }
  SpinorIO<F64>::store(y, p, i, g.Vp, v);
}

// Spin projection in the chiral basis (psi = (u0, u1, l0, l1) in spin, as in
// the hop kernels): (1 - sg gamma_mu) psi is determined by its upper half h;
// the lower half is a fixed spin rotation of h.
template <int MU, int SG>
__device__ __forceinline__ void bl_proj(const cx<float> (&v)[12], cx<float> (&h)[6]) {
  constexpr float sg = (float)SG;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cx<float> u0 = v[a], u1 = v[3 + a], l0 = v[6 + a], l1 = v[9 + a];
    if constexpr (MU == 0) {
      h[a] = u0 + sg * l0;
      h[3 + a] = u1 + sg * l1;
    } else if constexpr (MU == 1) {
      h[a] = u0 + sg * ti(l1);
      h[3 + a] = u1 + sg * ti(l0);
    } else if constexpr (MU == 2) {
      h[a] = u0 + sg * l1;
      h[3 + a] = u1 - sg * l0;
    } else {
      h[a] = u0 + sg * ti(l0);
      h[3 + a] = u1 - sg * ti(l1);
    }
  }
}

// acc += c * (the full spinor whose upper half is w, of projector (1 - sg
// gamma_mu)), one fused multiply-add a component
template <int MU, int SG>
__device__ __forceinline__ void bl_recon(cx<float> (&acc)[12], const cx<float> (&w)[6], float c) {
  const float d = SG > 0 ? c : -c;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cx<float> w0 = w[a], w1 = w[3 + a];
    rfma(acc[a], c, w0);
    rfma(acc[3 + a], c, w1);
    if constexpr (MU == 0) {
      rfma(acc[6 + a], d, w0);
      rfma(acc[9 + a], d, w1);
    } else if constexpr (MU == 1) {
      rfma(acc[6 + a], -d, ti(w1));
      rfma(acc[9 + a], -d, ti(w0));
    } else if constexpr (MU == 2) {
      rfma(acc[6 + a], -d, w1);
      rfma(acc[9 + a], d, w0);
    } else {
      rfma(acc[6 + a], -d, ti(w0));
      rfma(acc[9 + a], d, ti(w1));
    }
  }
}

// o = U h (DAG: U^+ h) on both spin components of a half spinor
template <bool DAG>
__device__ __forceinline__ void bl_link(const cx<float> (&u)[9], const cx<float> (&h)[6], cx<float> (&o)[6]) {
#pragma unroll
  for (int sp = 0; sp < 2; ++sp)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cx<float> t;
      if constexpr (DAG) {
        t = cjmul(u[a], h[3 * sp]);
        cjfma2(t, u[3 + a], h[3 * sp + 1]);
        cjfma2(t, u[6 + a], h[3 * sp + 2]);
      } else {
        t = cmul(u[3 * a], h[3 * sp]);
        cfma2(t, u[3 * a + 1], h[3 * sp + 1]);
        cfma2(t, u[3 * a + 2], h[3 * sp + 2]);
      }
      o[3 * sp + a] = t;
    }
}

struct SapPass {
  Geom g;
  Blocking b;
  int colour;
  int nmr;
  int own_zero;  // psi of the pass's blocks is still zero (not read)
  const float4* r;
  float4* psi;
  const float2* U;
  const float4* C;
  const double* rt;      // time hop ratios [4][T] (fwd, bwd, ...; boundary sign folded in)
  const double* sratio;  // spatial hop ratios of the light-quark factorisation, or null
  float m4;              // 4 + M
};

// Element s of component array k of block blk (blk is the same for the whole
// wave): scalar base, lane offset.
template <typename T>
__device__ __forceinline__ const T* bl_at(const T* f, int ncomp, int blk, int k, int vol, int s) {
  return at(scalar_base(f + ((long)blk * ncomp + k) * vol), s);
}

__device__ __forceinline__ void bl_load_spinor(const float4* f, int blk, int vol, int s, cx<float> (&v)[12]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const float4 q = *bl_at(f, 6, blk, k, vol, s);
    v[2 * k] = cx<float>{q.x, q.y};
    v[2 * k + 1] = cx<float>{q.z, q.w};
  }
}

__device__ __forceinline__ void bl_store_spinor(float4* f, int blk, int vol, int s, const cx<float> (&v)[12]) {
#pragma unroll
  for (int k = 0; k < 6; ++k)
    *const_cast<float4*>(bl_at(f, 6, blk, k, vol, s)) = make_float4(v[2 * k].x, v[2 * k].y, v[2 * k + 1].x, v[2 * k + 1].y);
}

__device__ __forceinline__ void bl_load_link(const float2* U, int blk, int mu, int vol, int s, cx<float> (&u)[9]) {
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const float2 v = *bl_at(U, 36, blk, mu * 9 + q, vol, s);
    u[q] = cx<float>{v.x, v.y};
  }
}

__device__ __forceinline__ HermBlock<float> bl_herm(const float4 (&raw)[9]) {
  const float f[36] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y, raw[1].z, raw[1].w, raw[2].x,
                       raw[2].y, raw[2].z, raw[2].w, raw[3].x, raw[3].y, raw[3].z, raw[3].w, raw[4].x, raw[4].y,
                       raw[4].z, raw[4].w, raw[5].x, raw[5].y, raw[5].z, raw[5].w, raw[6].x, raw[6].y, raw[6].z,
                       raw[6].w, raw[7].x, raw[7].y, raw[7].z, raw[7].w, raw[8].x, raw[8].y, raw[8].z, raw[8].w};
  HermBlock<float> B;
#pragma unroll
  for (int q = 0; q < 6; ++q) B.d[q] = f[q];
#pragma unroll
  for (int q = 0; q < 15; ++q) B.o[q] = cx<float>{f[6 + 2 * q], f[7 + 2 * q]};
  return B;
}

// y = (C + m4) x with the site's clover blocks read from the block layout,
// one chirality at a time
__device__ __forceinline__ void bl_diag(const float4* C, int blk, int vol, int s, float m4, const cx<float> (&x)[12],
                                        cx<float> (&y)[12]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float4 raw[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) raw[q] = *bl_at(C, 18, blk, 9 * h + q, vol, s);
    herm_apply(bl_herm(raw), m4, &x[6 * h], &y[6 * h]);
  }
}

// Coordinates (in blocks) of the kidx-th block of a colour; the last one takes
// the parity.  The divisions run on the vector unit: back to scalar registers,
// so that what follows from the coordinates (block indices, base addresses) is
// scalar arithmetic.
struct BCoord {
  int c[4];
};
__device__ __forceinline__ BCoord bl_coord(const Blocking& b, int colour, int kidx) {
  BCoord r;
  const int h3 = b.nb[3] / 2;
  r.c[3] = kidx % h3;
  kidx /= h3;
  r.c[2] = kidx % b.nb[2];
  kidx /= b.nb[2];
  r.c[1] = kidx % b.nb[1];
  r.c[0] = kidx / b.nb[1];
  r.c[3] = 2 * r.c[3] + ((colour + r.c[0] + r.c[1] + r.c[2]) & 1);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) r.c[mu] = __builtin_amdgcn_readfirstlane(r.c[mu]);
  return r;
}
// index of the block next to it in direction MU
template <int MU, int SG>
__device__ __forceinline__ int bl_next(const Blocking& b, const BCoord& o) {
  int y[4] = {o.c[0], o.c[1], o.c[2], o.c[3]};
  y[MU] = SG > 0 ? (y[MU] + 1 == b.nb[MU] ? 0 : y[MU] + 1) : (y[MU] == 0 ? b.nb[MU] - 1 : y[MU] - 1);
  return ((y[0] + y[1] + y[2] + y[3]) & 1) * b.nhalf + ((y[0] * b.nb[1] + y[1]) * b.nb[2] + y[2]) * (b.nb[3] / 2) +
         y[3] / 2;
}

// coordinates within its block of the block's site s
__device__ __forceinline__ void bl_local(const Blocking& b, int s, int (&l)[4]) {
  l[3] = s % b.bs[3];
  s /= b.bs[3];
  l[2] = s % b.bs[2];
  s /= b.bs[2];
  l[1] = s % b.bs[1];
  l[0] = s / b.bs[1];
}

// hop coefficients at site l of block o, with the -1/2 of the hops: time
// ratios, spatial ratios (or 1)
__device__ __forceinline__ void bl_coefs(const SapPass& a, const BCoord& o, const int (&l)[4], float (&cf)[4],
                                         float (&cb)[4]) {
  const Geom& g = a.g;
  const int Ls[4] = {g.T, g.L1, g.L2, g.L3};
  const int x0 = o.c[0] * a.b.bs[0] + l[0];
  cf[0] = -0.5f * (float)a.rt[x0];
  cb[0] = -0.5f * (float)a.rt[g.T + x0];
  int off = 0;
#pragma unroll
  for (int mu = 1; mu < 4; ++mu) {
    const int x = o.c[mu] * a.b.bs[mu] + l[mu];
    cf[mu] = a.sratio ? -0.5f * (float)a.sratio[off + x] : -0.5f;
    cb[mu] = a.sratio ? -0.5f * (float)a.sratio[off + Ls[mu] + x] : -0.5f;
    off += 4 * Ls[mu];
  }
}

// strides of a block's site index
__device__ __forceinline__ int bl_stride(const Blocking& b, int mu) {
  return mu == 0 ? b.bs[1] * b.bs[2] * b.bs[3] : mu == 1 ? b.bs[2] * b.bs[3] : mu == 2 ? b.bs[3] : 1;
}

// out += the hops in direction MU that reach site s of block blk from the
// neighbour blocks (the sites of the block's faces).  REG: U holds the site's
// forward link.
template <bool REG, int MU>
__device__ __forceinline__ void bl_face(const SapPass& a, const BCoord& o, int blk, int s, const int (&l)[4],
                                        const cx<float> (&U)[9], float cf, float cb, cx<float> (&out)[12]) {
  const Blocking& b = a.b;
  const int span = (b.bs[MU] - 1) * bl_stride(b, MU);
  cx<float> v[12], h[6], w[6], u[9];
  if (l[MU] + 1 == b.bs[MU]) {
    bl_load_spinor(a.psi, bl_next<MU, 1>(b, o), b.vol, s - span, v);
    bl_proj<MU, 1>(v, h);
    if constexpr (REG) {
      bl_link<false>(U, h, w);
    } else {
      bl_load_link(a.U, blk, MU, b.vol, s, u);
      bl_link<false>(u, h, w);
    }
    bl_recon<MU, 1>(out, w, cf);
  }
  if (l[MU] == 0) {
    const int nb = bl_next<MU, -1>(b, o);
    bl_load_link(a.U, nb, MU, b.vol, s + span, u);
    bl_load_spinor(a.psi, nb, b.vol, s + span, v);
    bl_proj<MU, -1>(v, h);
    bl_link<true>(u, h, w);
    bl_recon<MU, -1>(out, w, cb);
  }
}

// per-thread FP64 terms of <a, rho>_B and |a|^2_B
__device__ __forceinline__ void bl_mr_sums(const cx<float> (&av)[12], const cx<float> (&rv)[12], double& nr,
                                           double& ni, double& dn) {
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const double ax = av[c].x, ay = av[c].y, rx = rv[c].x, ry = rv[c].y;
    nr = fmar(ay, ry, fmar(ax, rx, nr));
    ni = fmar(-ay, rx, fmar(ax, ry, ni));
    dn = fmar(ay, ay, fmar(ax, ax, dn));
  }
}

// The minimal-residual coefficient w = <a, rho>_B / |a|^2_B from per-thread
// FP64 terms: wave sums, then the waves in order.  Every thread calls it and
// forms w itself, so there is one barrier; a second call must have a barrier
// after the first one's return.
template <int NW>
__device__ __forceinline__ cx<float> bl_mr_coef(double nr, double ni, double dn, double (&red)[4][NW]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const double v = wave_sum4(nr, ni, dn, 0.0);
  if ((lane & 15) == 0) red[wave_row_value(lane >> 4)][wv] = v;
  __syncthreads();
  double sr = 0.0, si = 0.0, sd = 0.0;
  for (int q = 0; q < nw; ++q) {
    sr += red[0][q];
    si += red[1][q];
    sd += red[2][q];
  }
  return sd > 0.0 ? cx<float>{(float)(sr / sd), (float)(si / sd)} : cx<float>{0.f, 0.f};
}

// dpsi += w rho, rho -= w a.  The sum that is returned pairs its products (see
// cfma): the application of the preconditioner in FP32 is 1.8e-7 of the result
// off the FP64 one, 1.9e-7 without, for 0.3% of the solve at 64x32^3.
__device__ __forceinline__ void bl_mr_step(cx<float> w, const cx<float> (&av)[12], cx<float> (&rv)[12],
                                           cx<float> (&dpsi)[12]) {
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    cfma(dpsi[c], w, rv[c]);
    cfma2(rv[c], cx<float>{-w.x, -w.y}, av[c]);
  }
}

// ---- blocks with whole time slices in a wave
//
// A thread per site.  The spatial neighbours of a site are in the same wave, so
// the hops 1..3 exchange half spinors by lane permutes; the hops in time hand
// them over in LDS.  That leaves the LDS to one chirality of the clover blocks;
// the other one, the links, the residual and psi stay in registers, so that a
// pass reads each of them once.  The backward hop at x needs U_mu(x - mu)^+
// applied to the spinor at x - mu, which the thread of x - mu forms with its
// own link.  Two workgroups per CU.  (One with the clover blocks read again in
// each step, four directions through LDS: 426 us a pass at 64x32^3 with 4^4
// blocks, 2.8 GB past L2, half of the vector issue; this one 348 us, 1.2 GB,
// 0.64 of the issue.)  Workgroups of an XCD take neighbouring blocks, which read
// the same faces.
__host__ __device__ inline size_t sap_slice_lds(int nt) { return sizeof(float4) * (9 + 6) * (size_t)nt; }

// value of lane `from` / 4
__device__ __forceinline__ void bl_permute(int from, cx<float> (&h)[6]) {
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    h[e].x = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(h[e].x)));
    h[e].y = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(h[e].y)));
  }
}

__device__ __forceinline__ void bl_put_half(float4* buf, int nt, int s, const cx<float> (&h)[6]) {
#pragma unroll
  for (int e = 0; e < 3; ++e) buf[e * nt + s] = make_float4(h[2 * e].x, h[2 * e].y, h[2 * e + 1].x, h[2 * e + 1].y);
}
__device__ __forceinline__ void bl_get_half(const float4* buf, int nt, int s, cx<float> (&h)[6]) {
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const float4 q = buf[e * nt + s];
    h[2 * e] = cx<float>{q.x, q.y};
    h[2 * e + 1] = cx<float>{q.z, q.w};
  }
}

template <int MU>
__device__ __forceinline__ void bl_slice_hop(const Blocking& b, const int (&l)[4], const cx<float> (&U)[9],
                                             const cx<float> (&v)[12], float cf, float cb, cx<float> (&out)[12]) {
  const int lane = threadIdx.x & 63, st = bl_stride(b, MU);
  cx<float> h[6], g[6], w[6];
  bl_proj<MU, 1>(v, h);
  bl_permute(((lane + st) & 63) << 2, h);
  bl_proj<MU, -1>(v, g);
  bl_link<true>(U, g, w);
  bl_permute(((lane - st) & 63) << 2, w);
  bl_link<false>(U, h, g);
  bl_recon<MU, 1>(out, g, l[MU] + 1 < b.bs[MU] ? cf : 0.f);
  bl_recon<MU, -1>(out, w, l[MU] > 0 ? cb : 0.f);
}

// The on-chip part of a site: links, clover (one chirality at cl + k nt + s),
// coefficients (zero beyond the block's sites), buffers of the time hops.
struct SliceSite {
  cx<float> U[4][9];
  float4 c0[9];
  const float4* cl;
  float4 *hf, *hb;
  int l[4], s, nt;
  float cf[4], cb[4];
};

// out = D'_B v
__device__ __forceinline__ void bl_slice_dprime(const SapPass& a, const SliceSite& t, const cx<float> (&v)[12],
                                                cx<float> (&out)[12]) {
  const Blocking& b = a.b;
  cx<float> h[6], w[6];
  bl_proj<0, 1>(v, h);
  bl_put_half(t.hf, t.nt, t.s, h);
  bl_proj<0, -1>(v, h);
  bl_link<true>(t.U[0], h, w);
  bl_put_half(t.hb, t.nt, t.s, w);
  herm_apply(bl_herm(t.c0), a.m4, &v[0], &out[0]);
  {
    float4 raw[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) raw[q] = t.cl[q * t.nt + t.s];
    herm_apply(bl_herm(raw), a.m4, &v[6], &out[6]);
  }
  bl_slice_hop<1>(b, t.l, t.U[1], v, t.cf[1], t.cb[1], out);
  bl_slice_hop<2>(b, t.l, t.U[2], v, t.cf[2], t.cb[2], out);
  bl_slice_hop<3>(b, t.l, t.U[3], v, t.cf[3], t.cb[3], out);
  __syncthreads();
  const int st = bl_stride(b, 0);
  if (t.l[0] + 1 < b.bs[0]) {
    bl_get_half(t.hf, t.nt, t.s + st, h);
    bl_link<false>(t.U[0], h, w);
    bl_recon<0, 1>(out, w, t.cf[0]);
  }
  if (t.l[0] > 0) {
    bl_get_half(t.hb, t.nt, t.s - st, w);
    bl_recon<0, -1>(out, w, t.cb[0]);
  }
}

// One pass of the Schwarz procedure over the blocks of one colour:
// rho = r - D' psi on the block (NB_ZERO: psi = 0 everywhere, rho = r), nmr
// minimal-residual steps with the Dirichlet block operator, psi += the
// accumulated correction.  Block sums in FP64, reduced in a fixed order.
template <bool NB_ZERO>
__global__ void __launch_bounds__(kSapThreads, 2) sap_slice_kernel(SapPass a) {
  extern __shared__ float4 slice_lds[];
  __shared__ double red[4][kSapThreads / 64];
  const Blocking& b = a.b;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int blk = a.colour * b.nhalf + tile;
  const bool valid = (int)threadIdx.x < b.vol;
  const int s = valid ? threadIdx.x : 0;
  const BCoord o = bl_coord(b, a.colour, tile);
  SliceSite t;
  t.nt = blockDim.x;
  t.s = threadIdx.x;
  t.hf = slice_lds + 9 * t.nt;
  t.hb = slice_lds + 12 * t.nt;
  t.cl = slice_lds;
  bl_local(b, s, t.l);
  bl_coefs(a, o, t.l, t.cf, t.cb);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) bl_load_link(a.U, blk, mu, b.vol, s, t.U[mu]);
#pragma unroll
  for (int q = 0; q < 9; ++q) t.c0[q] = *bl_at(a.C, 18, blk, q, b.vol, s);
#pragma unroll
  for (int q = 0; q < 9; ++q) slice_lds[q * t.nt + t.s] = *bl_at(a.C, 18, blk, 9 + q, b.vol, s);
  // beyond the block's sites: no hops, zero spinors
  if (!valid) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) t.cf[mu] = t.cb[mu] = 0.f;
  }
  cx<float> dpsi[12], rv[12], av[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) dpsi[c] = rv[c] = av[c] = cx<float>{0.f, 0.f};
  if constexpr (!NB_ZERO) {
    if (!a.own_zero) {
      if (valid) bl_load_spinor(a.psi, blk, b.vol, s, dpsi);
      bl_slice_dprime(a, t, dpsi, av);
      __syncthreads();  // the buffers of the time hops are free again
    }
    if (valid) {
      bl_face<true, 0>(a, o, blk, s, t.l, t.U[0], t.cf[0], t.cb[0], av);
      bl_face<true, 1>(a, o, blk, s, t.l, t.U[1], t.cf[1], t.cb[1], av);
      bl_face<true, 2>(a, o, blk, s, t.l, t.U[2], t.cf[2], t.cb[2], av);
      bl_face<true, 3>(a, o, blk, s, t.l, t.U[3], t.cf[3], t.cb[3], av);
    }
  }
  if (valid) {
    bl_load_spinor(a.r, blk, b.vol, s, rv);
#pragma unroll
    for (int c = 0; c < 12; ++c) rv[c] = rv[c] - av[c];
  }
  for (int it = 0; it < a.nmr; ++it) {
    bl_slice_dprime(a, t, rv, av);
    double nr = 0.0, ni = 0.0, dn = 0.0;
    bl_mr_sums(av, rv, nr, ni, dn);
    bl_mr_step(bl_mr_coef(nr, ni, dn, red), av, rv, dpsi);
  }
  if (valid) bl_store_spinor(a.psi, blk, b.vol, s, dpsi);
}

// ---- other blocks of at most kSapThreads sites
//
// A thread per site; the links in registers, the residual in LDS, where the
// forward hops read it and the backward hops are handed over; the clover blocks
// are read again in each step.

struct BlockLds {
  float v[24 * kSapThreads];       // the spinors D'_B is applied to
  float hb[4 * 12 * kSapThreads];  // backward hops handed to x + mu
};
template <int MU>
__device__ __forceinline__ void bl_push(const Blocking& b, BlockLds& m, int s, const int (&l)[4],
                                        const cx<float> (&U)[9], const cx<float> (&v)[12]) {
  if (l[MU] + 1 < b.bs[MU]) {
    cx<float> h[6], w[6];
    bl_proj<MU, -1>(v, h);
    bl_link<true>(U, h, w);
    const int n = s + bl_stride(b, MU);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      m.hb[((MU * 12) + 2 * e) * kSapThreads + n] = w[e].x;
      m.hb[((MU * 12) + 2 * e + 1) * kSapThreads + n] = w[e].y;
    }
  }
}
template <int MU>
__device__ __forceinline__ void bl_pull(const Blocking& b, const BlockLds& m, int s, const int (&l)[4],
                                        const cx<float> (&U)[9], float cf, float cb, cx<float> (&out)[12]) {
  cx<float> v[12], h[6], w[6];
  if (l[MU] + 1 < b.bs[MU]) {
    const int n = s + bl_stride(b, MU);
#pragma unroll
    for (int c = 0; c < 12; ++c)
      v[c] = cx<float>{m.v[(2 * c) * kSapThreads + n], m.v[(2 * c + 1) * kSapThreads + n]};
    bl_proj<MU, 1>(v, h);
    bl_link<false>(U, h, w);
    bl_recon<MU, 1>(out, w, cf);
  }
  if (l[MU] > 0) {
#pragma unroll
    for (int e = 0; e < 6; ++e)
      w[e] = cx<float>{m.hb[((MU * 12) + 2 * e) * kSapThreads + s], m.hb[((MU * 12) + 2 * e + 1) * kSapThreads + s]};
    bl_recon<MU, -1>(out, w, cb);
  }
}
// out = D'_B v (v: the thread's site).  Every thread calls it; a second call must
// have a barrier after the first one's return.
__device__ __forceinline__ void bl_block_dprime(const SapPass& a, BlockLds& m, int blk, bool valid, int s,
                                                const int (&l)[4], const cx<float> (&U)[4][9], const float (&cf)[4],
                                                const float (&cb)[4], const cx<float> (&v)[12],
                                                cx<float> (&out)[12]) {
  const Blocking& b = a.b;
  if (valid) {
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      m.v[(2 * c) * kSapThreads + s] = v[c].x;
      m.v[(2 * c + 1) * kSapThreads + s] = v[c].y;
    }
    bl_push<0>(b, m, s, l, U[0], v);
    bl_push<1>(b, m, s, l, U[1], v);
    bl_push<2>(b, m, s, l, U[2], v);
    bl_push<3>(b, m, s, l, U[3], v);
  }
  __syncthreads();
  if (valid) {
    bl_diag(a.C, blk, b.vol, s, a.m4, v, out);
    bl_pull<0>(b, m, s, l, U[0], cf[0], cb[0], out);
    bl_pull<1>(b, m, s, l, U[1], cf[1], cb[1], out);
    bl_pull<2>(b, m, s, l, U[2], cf[2], cb[2], out);
    bl_pull<3>(b, m, s, l, U[3], cf[3], cb[3], out);
  }
}

template <bool NB_ZERO>
__global__ void __launch_bounds__(kSapThreads, 2) sap_block_kernel(SapPass a) {
  __shared__ BlockLds m;
  __shared__ double red[4][kSapThreads / 64];
  const Blocking& b = a.b;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int blk = a.colour * b.nhalf + tile;
  const bool valid = (int)threadIdx.x < b.vol;
  const int s = valid ? threadIdx.x : 0;
  const BCoord o = bl_coord(b, a.colour, tile);
  int l[4];
  bl_local(b, s, l);
  float cf[4], cb[4];
  bl_coefs(a, o, l, cf, cb);
  cx<float> U[4][9];
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) bl_load_link(a.U, blk, mu, b.vol, s, U[mu]);
  cx<float> dpsi[12], rv[12], av[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) dpsi[c] = rv[c] = av[c] = cx<float>{0.f, 0.f};
  if constexpr (!NB_ZERO) {
    if (!a.own_zero) {
      if (valid) bl_load_spinor(a.psi, blk, b.vol, s, dpsi);
      bl_block_dprime(a, m, blk, valid, s, l, U, cf, cb, dpsi, av);
      __syncthreads();  // the LDS buffers are free again
    }
    if (valid) {
      bl_face<true, 0>(a, o, blk, s, l, U[0], cf[0], cb[0], av);
      bl_face<true, 1>(a, o, blk, s, l, U[1], cf[1], cb[1], av);
      bl_face<true, 2>(a, o, blk, s, l, U[2], cf[2], cb[2], av);
      bl_face<true, 3>(a, o, blk, s, l, U[3], cf[3], cb[3], av);
    }
  }
  if (valid) {
    bl_load_spinor(a.r, blk, b.vol, s, rv);
#pragma unroll
    for (int c = 0; c < 12; ++c) rv[c] = rv[c] - av[c];
  }
  for (int it = 0; it < a.nmr; ++it) {
    bl_block_dprime(a, m, blk, valid, s, l, U, cf, cb, rv, av);
    double nr = 0.0, ni = 0.0, dn = 0.0;
    if (valid) bl_mr_sums(av, rv, nr, ni, dn);
    bl_mr_step(bl_mr_coef(nr, ni, dn, red), av, rv, dpsi);
  }
  if (valid) bl_store_spinor(a.psi, blk, b.vol, s, dpsi);
}

// ---- blocks of kSapThreads + 1 .. kSapBigSites sites
//
// kSapBigThreads threads with kSapBigPer sites each (site s = thread + q
// kSapBigThreads).  The residual is in LDS, where both hops of a site read it;
// D'_B rho and psi stay in registers, the links and clover blocks (1.1 MB for
// 6^4 sites) are read again in each step.  (With D'_B rho and psi in memory
// between the phases of a step: 262 us a pass at 48x24^3 with 6^4 blocks, 5.4 kB
// a site at 5.7 TB/s; this one 230 us, 3.6 kB at 5.1 TB/s.)
constexpr int kSapBigThreads = 512;
constexpr int kSapBigPer = 3;
constexpr int kSapBigSites = kSapBigThreads * kSapBigPer;

template <int MU>
__device__ __forceinline__ void bl_big_hop(const SapPass& a, const float* v_l, int blk, int s, const int (&l)[4],
                                           float cf, float cb, cx<float> (&out)[12]) {
  const Blocking& b = a.b;
  cx<float> v[12], h[6], w[6], u[9];
  if (l[MU] + 1 < b.bs[MU]) {
    const int n = s + bl_stride(b, MU);
    bl_load_link(a.U, blk, MU, b.vol, s, u);
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = cx<float>{v_l[(2 * c) * kSapBigSites + n], v_l[(2 * c + 1) * kSapBigSites + n]};
    bl_proj<MU, 1>(v, h);
    bl_link<false>(u, h, w);
    bl_recon<MU, 1>(out, w, cf);
  }
  if (l[MU] > 0) {
    const int n = s - bl_stride(b, MU);
    bl_load_link(a.U, blk, MU, b.vol, n, u);
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = cx<float>{v_l[(2 * c) * kSapBigSites + n], v_l[(2 * c + 1) * kSapBigSites + n]};
    bl_proj<MU, -1>(v, h);
    bl_link<true>(u, h, w);
    bl_recon<MU, -1>(out, w, cb);
  }
}

// out is complete here: else the compiler interleaves the hops and sites and
// spills
__device__ __forceinline__ void bl_pin(cx<float> (&out)[12]) {
#pragma unroll
  for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(out[c].x), "+v"(out[c].y));
  __builtin_amdgcn_sched_barrier(0);
}

// out = D'_B at site s of the spinors in v_l; v: the site's own one
__device__ __forceinline__ void bl_big_dprime(const SapPass& a, const float* v_l, const BCoord& o, int blk, int s,
                                              const cx<float> (&v)[12], cx<float> (&out)[12]) {
  // opaque: the coordinates and coefficients of kSapBigPer sites would
  // otherwise be kept through the steps, in registers that are not there
  asm volatile("" : "+v"(s));
  int l[4];
  bl_local(a.b, s, l);
  float cf[4], cb[4];
  bl_coefs(a, o, l, cf, cb);
  bl_diag(a.C, blk, a.b.vol, s, a.m4, v, out);
  bl_big_hop<0>(a, v_l, blk, s, l, cf[0], cb[0], out);
  bl_pin(out);
  bl_big_hop<1>(a, v_l, blk, s, l, cf[1], cb[1], out);
  bl_pin(out);
  bl_big_hop<2>(a, v_l, blk, s, l, cf[2], cb[2], out);
  bl_pin(out);
  bl_big_hop<3>(a, v_l, blk, s, l, cf[3], cb[3], out);
  bl_pin(out);
}

__device__ __forceinline__ void bl_big_put(float* v_l, int s, const cx<float> (&v)[12]) {
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    v_l[(2 * c) * kSapBigSites + s] = v[c].x;
    v_l[(2 * c + 1) * kSapBigSites + s] = v[c].y;
  }
}
__device__ __forceinline__ void bl_big_get(const float* v_l, int s, cx<float> (&v)[12]) {
#pragma unroll
  for (int c = 0; c < 12; ++c) v[c] = cx<float>{v_l[(2 * c) * kSapBigSites + s], v_l[(2 * c + 1) * kSapBigSites + s]};
}

template <bool NB_ZERO>
__global__ void __launch_bounds__(kSapBigThreads, 2) sap_block_big_kernel(SapPass a) {
  __shared__ float v_l[24 * kSapBigSites];
  __shared__ double red[4][kSapBigThreads / 64];
  const Blocking& b = a.b;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int blk = a.colour * b.nhalf + tile;
  const BCoord o = bl_coord(b, a.colour, tile);
  cx<float> av[kSapBigPer][12], dpsi[kSapBigPer][12];
#pragma unroll
  for (int q = 0; q < kSapBigPer; ++q)
#pragma unroll
    for (int c = 0; c < 12; ++c) dpsi[q][c] = av[q][c] = cx<float>{0.f, 0.f};
  if constexpr (!NB_ZERO) {
    if (!a.own_zero) {
#pragma unroll
      for (int q = 0; q < kSapBigPer; ++q) {
        const int s = threadIdx.x + q * kSapBigThreads;
        if (s < b.vol) {
          cx<float> pv[12];
          bl_load_spinor(a.psi, blk, b.vol, s, pv);
          bl_big_put(v_l, s, pv);
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kSapBigPer; ++q) {
        const int s = threadIdx.x + q * kSapBigThreads;
        if (s < b.vol) {
          cx<float> pv[12];
          bl_big_get(v_l, s, pv);
          bl_big_dprime(a, v_l, o, blk, s, pv, av[q]);
        }
      }
      __syncthreads();  // every site's hops are done: v_l is free for rho, site by site
    }
#pragma unroll
    for (int q = 0; q < kSapBigPer; ++q) {
      int s = threadIdx.x + q * kSapBigThreads;
      if (s < b.vol) {
        asm volatile("" : "+v"(s));
        int l[4];
        bl_local(b, s, l);
        float cf[4], cb[4];
        bl_coefs(a, o, l, cf, cb);
        const cx<float> none[9] = {};
        bl_face<false, 0>(a, o, blk, s, l, none, cf[0], cb[0], av[q]);
        bl_face<false, 1>(a, o, blk, s, l, none, cf[1], cb[1], av[q]);
        bl_face<false, 2>(a, o, blk, s, l, none, cf[2], cb[2], av[q]);
        bl_face<false, 3>(a, o, blk, s, l, none, cf[3], cb[3], av[q]);
        bl_pin(av[q]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kSapBigPer; ++q) {
    const int s = threadIdx.x + q * kSapBigThreads;
    if (s < b.vol) {
      cx<float> rv[12];
      bl_load_spinor(a.r, blk, b.vol, s, rv);
#pragma unroll
      for (int c = 0; c < 12; ++c) rv[c] = rv[c] - av[q][c];
      if constexpr (!NB_ZERO) {
        if (!a.own_zero) bl_big_get(v_l, s, dpsi[q]);
      }
      bl_big_put(v_l, s, rv);
      bl_pin(dpsi[q]);
    }
  }
  for (int it = 0; it < a.nmr; ++it) {
    __syncthreads();  // rho complete
    double nr = 0.0, ni = 0.0, dn = 0.0;
#pragma unroll
    for (int q = 0; q < kSapBigPer; ++q) {
      const int s = threadIdx.x + q * kSapBigThreads;
      if (s < b.vol) {
        cx<float> rv[12];
        bl_big_get(v_l, s, rv);
        bl_big_dprime(a, v_l, o, blk, s, rv, av[q]);
        bl_mr_sums(av[q], rv, nr, ni, dn);
        bl_pin(av[q]);
      }
    }
    const cx<float> w = bl_mr_coef(nr, ni, dn, red);
#pragma unroll
    for (int q = 0; q < kSapBigPer; ++q) {
      const int s = threadIdx.x + q * kSapBigThreads;
      if (s < b.vol) {
        cx<float> rv[12];
        bl_big_get(v_l, s, rv);
        bl_mr_step(w, av[q], rv, dpsi[q]);
        bl_big_put(v_l, s, rv);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kSapBigPer; ++q) {
    const int s = threadIdx.x + q * kSapBigThreads;
    if (s < b.vol) bl_store_spinor(a.psi, blk, b.vol, s, dpsi[q]);
  }
}

constexpr int kDotBlocks = 1024;

// ------------------------------------------------------------ GCR vectors
//
// The Gram-Schmidt step of GCR works on whole FP64 vectors, so what it costs is
// how often they pass through the memory.  The coefficients against up to
// kGcrGroup earlier vectors are formed in one pass and subtracted in a second
// one, which also takes the new vector's norm and its product with the
// residual (classical Gram-Schmidt within a group, modified between groups):
// 2 k + 7 vector passes for the k-th vector against 4 k + 7 one coefficient at
// a time.  No solve needs more iterations for it: restart lengths 16, 40 and
// 64, residues 1e-10 and 1e-13, masses from 0.05 to where 600 iterations do not
// converge, strong and weak preconditioners, 16x8^3 and 32x16^3, all counts equal.
// The earlier vectors stay unnormalised, their squared norms enter the
// coefficients.  A vector is 24 component rows (2 parities) of Vh entries,
// Vp apart; blockIdx.y is the row, so neighbouring threads and loop steps read
// neighbouring entries of every vector.

constexpr int kGcrGroup = 16;
constexpr int kGcrBlocksX = 85;  // at most 24 * 85 = 2040 blocks

struct VecList {
  const double2* v[kGcrGroup];
};

// block sums of n values -> partials[value][block]
template <int N>
__device__ __forceinline__ void gcr_store_sums(const double (&v)[N], double* partials) {
  __shared__ double lds[kBlock / 64][(N + 3) / 4 * 4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < N; k += 4) {
    const double w = wave_sum4(v[k], k + 1 < N ? v[k + 1] : 0.0, k + 2 < N ? v[k + 2] : 0.0, k + 3 < N ? v[k + 3] : 0.0);
    if ((lane & 15) == 0) lds[wv][k + wave_row_value(lane >> 4)] = w;
  }
  __syncthreads();
  const int nb = gridDim.x * gridDim.y, blk = blockIdx.y * gridDim.x + blockIdx.x;
  if (threadIdx.x < N) {
    double t = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) t += lds[w][threadIdx.x];
    partials[(long)threadIdx.x * nb + blk] = t;
  }
}

// <x_j, y> for N vectors: values 2 j, 2 j + 1
template <int N>
__global__ void __launch_bounds__(kBlock) gcr_dots_kernel(int Vh, int Vp, VecList x, const double2* __restrict__ y,
                                                          double* __restrict__ partials) {
  double v[2 * N] = {};
  const long row = (long)blockIdx.y * Vp;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < Vh; i += gridDim.x * kBlock) {
    const double2 b = y[row + i];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double2 a = x.v[j][row + i];
      v[2 * j] = fmar(a.y, b.y, fmar(a.x, b.x, v[2 * j]));
      v[2 * j + 1] = fmar(-a.y, b.x, fmar(a.x, b.y, v[2 * j + 1]));
    }
  }
  gcr_store_sums(v, partials);
}

enum GcrPass {
  GCR_UPDATE = 0,     // y += sum_j coef_j x_j
  GCR_ORTHO = 1,      // ... then |y|^2 and <y, z>
  GCR_RESIDUAL = 2,   // ... then |y|^2
  GCR_SUBTRACT = 3,   // y = z - y, then |y|^2
};

// N vectors x_j with complex coefficients on the device
template <int N, int MODE>
__global__ void __launch_bounds__(kBlock) gcr_update_kernel(int Vh, int Vp, VecList x, const double* __restrict__ coef,
                                                            double2* __restrict__ y, const double2* __restrict__ z,
                                                            double* __restrict__ partials) {
  constexpr int NV = MODE == GCR_ORTHO ? 3 : 1;
  double v[NV] = {};
  double c[2 * N + 1];
#pragma unroll
  for (int k = 0; k < 2 * N; ++k) c[k] = coef[k];
  const long row = (long)blockIdx.y * Vp;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < Vh; i += gridDim.x * kBlock) {
    double2 t = y[row + i], q;
    if constexpr (MODE == GCR_ORTHO || MODE == GCR_SUBTRACT) q = z[row + i];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double2 a = x.v[j][row + i];
      t.x = fmar(-c[2 * j + 1], a.y, fmar(c[2 * j], a.x, t.x));
      t.y = fmar(c[2 * j + 1], a.x, fmar(c[2 * j], a.y, t.y));
    }
    if constexpr (MODE == GCR_SUBTRACT) t = make_double2(q.x - t.x, q.y - t.y);
    if constexpr (N > 0 || MODE == GCR_SUBTRACT) y[row + i] = t;
    if constexpr (MODE != GCR_UPDATE) v[0] = fmar(t.y, t.y, fmar(t.x, t.x, v[0]));
    if constexpr (MODE == GCR_ORTHO) {
      v[1] = fmar(t.y, q.y, fmar(t.x, q.x, v[1]));
      v[2] = fmar(-t.y, q.x, fmar(t.x, q.y, v[2]));
    }
  }
  if constexpr (MODE != GCR_UPDATE) gcr_store_sums(v, partials);
}

// Folds the block sums in a fixed order and forms the coefficients.
//   mode 0 (block j): c = <w_j, w_k> / |w_j| for the host, coef_j = -<w_j, w_k> / |w_j|^2
//   mode 1: b = |w_k|, gamma = <w_k, r> / b for the host, coef_0 = -<w_k, r> / b^2,
//           both 0 unless b is finite and positive; b2 = b^2
//   mode 2: out = the sum
__global__ void __launch_bounds__(kBlock) gcr_finish_kernel(const double* __restrict__ partials, int nb, int mode,
                                                            const double* __restrict__ b2, long out_stride,
                                                            double* __restrict__ out, double* __restrict__ out2,
                                                            double* __restrict__ coef, double* __restrict__ b2_out) {
  __shared__ double lds[kBlock / 64][4];
  const int j = blockIdx.x, nv = mode == 0 ? 2 : mode == 1 ? 3 : 1;
  const double* p = partials + (long)(mode == 0 ? 2 * j : 0) * nb;
  double v[3] = {};
  for (int b = threadIdx.x; b < nb; b += kBlock)
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < nv) v[k] += p[(long)k * nb + b];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double w = wave_sum4(v[0], v[1], v[2], 0.0);
  if ((lane & 15) == 0) lds[wv][wave_row_value(lane >> 4)] = w;
  __syncthreads();
  if (threadIdx.x != 0) return;
  double s[3] = {};
  for (int q = 0; q < kBlock / 64; ++q)
    for (int k = 0; k < 3; ++k) s[k] += lds[q][k];
  if (mode == 0) {
    const double n2 = b2[j], n = sqrt(n2);
    out[j * out_stride] = s[0] / n;
    out[j * out_stride + 1] = s[1] / n;
    coef[2 * j] = -s[0] / n2;
    coef[2 * j + 1] = -s[1] / n2;
  } else if (mode == 1) {
    const double b = sqrt(s[0]);
    const bool ok = b > 0.0 && isfinite(b);
    out[0] = b;
    out2[0] = ok ? s[1] / b : 0.0;
    out2[1] = ok ? s[2] / b : 0.0;
    coef[0] = ok ? -s[1] / s[0] : 0.0;
    coef[1] = ok ? -s[2] / s[0] : 0.0;
    *b2_out = s[0];
  } else {
    out[0] = s[0];
  }
}

}  // namespace

// -------------------------------------------------------------- host driver

struct SapState {
  Geom g{};
  int nkv = 0;
  int prec = F32;
  Field eta, x, r, t;      // FP64 full-lattice vectors
  std::vector<Field> z, w;  // FP64, nkv each
  Field q_r, q_psi, q_rho, q_a;  // block-solve precision
  DevBuf ratio, m4, partials, alpha, cpp;
  // GCR coefficients on the device: c_jk [nkv][nkv], gamma_k [nkv], b_k
  // [nkv] (complex pairs), |r|^2, and their host copy; then |w_k|^2 [nkv] and
  // the coefficients of the next update [nkv]
  DevBuf gcr;
  std::vector<double> h_gcr;
  // fused block solves: links, clover, r and psi in block layout (FP32)
  bool fused = false;
  DevBuf ubl, cbl, rbl, pbl;
  std::vector<double> h_part;
};

namespace {

using zc = std::complex<double>;

size_t gcr_len(int nkv) { return (size_t)2 * nkv * nkv + 4 * nkv + 2; }
size_t gcr_cc(int nkv, int j, int k) { return (size_t)2 * (j * nkv + k); }
size_t gcr_gam(int nkv, int k) { return (size_t)2 * nkv * nkv + 2 * k; }
size_t gcr_bn(int nkv, int k) { return (size_t)2 * nkv * nkv + 2 * nkv + 2 * k; }
size_t gcr_rn(int nkv) { return (size_t)2 * nkv * nkv + 4 * nkv; }
size_t gcr_b2(int nkv, int k) { return gcr_len(nkv) + k; }
size_t gcr_coef(int nkv) { return gcr_len(nkv) + nkv; }
size_t gcr_dev_len(int nkv) { return gcr_len(nkv) + 3 * nkv; }

int sap_alloc(dp_ctx* c, SapState& s, int nkv, int prec) {
  const Geom& g = c->g;
  Field* f64[] = {&s.eta, &s.x, &s.r, &s.t};
  for (Field* f : f64) DP_HIP(c, alloc(c, *f, F64, 2));
  if ((int)s.z.size() < nkv) {
    s.z = std::vector<Field>(nkv);
    s.w = std::vector<Field>(nkv);
  }
  for (int k = 0; k < nkv; ++k) {
    DP_HIP(c, alloc(c, s.z[k], F64, 2));
    DP_HIP(c, alloc(c, s.w[k], F64, 2));
  }
  Field* fq[] = {&s.q_r, &s.q_psi, &s.q_rho, &s.q_a};
  for (Field* f : fq) DP_HIP(c, alloc(c, *f, prec, 2));
  DP_HIP(c, reserve(c, s.ratio, sizeof(double) * 4 * g.T));
  DP_HIP(c, reserve(c, s.m4, sizeof(double)));
  DP_HIP(c, reserve(c, s.alpha, sizeof(double) * g.T));
  DP_HIP(c, reserve(c, s.partials, sizeof(double) * std::max(2 * kDotBlocks, 2 * kGcrGroup * 24 * kGcrBlocksX)));
  s.h_gcr.resize(gcr_len(nkv));
  DP_HIP(c, reserve(c, s.gcr, sizeof(double) * gcr_dev_len(nkv)));
  s.h_part.resize(2 * kDotBlocks);
  s.g = g;
  s.nkv = nkv;
  s.prec = prec;
  return DP_OK;
}

// out = D' in on the whole lattice, both parities (full operator, not Schur)
int apply_full(dp_ctx* c, SapState& s, int prec, const Field& in, const Field& out) {
  HopArgs a = full_args(c, prec, 0, in.ref(0), in.ref(1), out.ref(0), out.ref(1));
  a.slots.ratio = s.ratio.as<double>();
  a.slots.m4 = s.m4.as<double>();
  a.red.red = RED_NONE;
  a.nslots = 1;
  a.sratio = space_hop_ratios(c);
  int nparts = 0;
  DP_HIP(c, launch_hop(a, c->stream, &nparts));
  return DP_OK;
}

dim3 site_grid(const Geom& g) { return dim3((g.Vh + kBlock - 1) / kBlock, 2); }
dim3 block_grid(const Geom& g) { return dim3((unsigned)((2L * g.Vh + kBlock - 1) / kBlock)); }

int vec_set(dp_ctx* c, const SpinorRef& x, const Field& y) {
  hipLaunchKernelGGL(vec_set_kernel, site_grid(c->g), dim3(kBlock), 0, c->stream, c->g, x, y.ref());
  DP_HIP(c, hipGetLastError());
  return DP_OK;
}

// <x, y> summed on the host in block order
int vec_dot(dp_ctx* c, SapState& s, const Field& x, const Field& y, zc* out) {
  hipLaunchKernelGGL(vec_dot_kernel, dim3(kDotBlocks), dim3(kBlock), 0, c->stream, c->g, x.ref(), y.ref(),
                     s.partials.as<double>());
  DP_HIP(c, hipGetLastError());
  DP_HIP(c, hipMemcpyAsync(s.h_part.data(), s.partials.p, sizeof(double) * 2 * kDotBlocks, hipMemcpyDeviceToHost,
                           c->stream));
  DP_HIP(c, hipStreamSynchronize(c->stream));
  double re = 0.0, im = 0.0;
  for (int k = 0; k < kDotBlocks; ++k) {
    re += s.h_part[2 * k];
    im += s.h_part[2 * k + 1];
  }
  *out = zc(re, im);
  return DP_OK;
}

dim3 gcr_grid(const Geom& g) { return dim3(std::min(kGcrBlocksX, (g.Vh + kBlock - 1) / kBlock), 24); }
int gcr_blocks(const Geom& g) { return (int)gcr_grid(g).x * 24; }

// <x_j, y> for the n vectors of the list
template <int N = 1>
hipError_t gcr_dots(dp_ctx* c, SapState& s, int n, const VecList& x, const Field& y) {
  if constexpr (N > kGcrGroup) {
    return hipErrorInvalidValue;
  } else {
    if (n != N) return gcr_dots<N + 1>(c, s, n, x, y);
    hipLaunchKernelGGL((gcr_dots_kernel<N>), gcr_grid(c->g), dim3(kBlock), 0, c->stream, c->g.Vh, c->g.Vp, x,
                       y.data.as<double2>(), s.partials.as<double>());
    return hipGetLastError();
  }
}

template <int MODE, int N>
hipError_t gcr_pass(dp_ctx* c, SapState& s, const VecList& x, const double* coef, const Field& y, const Field* z) {
  hipLaunchKernelGGL((gcr_update_kernel<N, MODE>), gcr_grid(c->g), dim3(kBlock), 0, c->stream, c->g.Vh, c->g.Vp, x, coef,
                     y.data.as<double2>(), z ? z->data.as<double2>() : nullptr, s.partials.as<double>());
  return hipGetLastError();
}

// a pass over n vectors, 0 <= n <= kGcrGroup
template <int MODE, int N = 0>
hipError_t gcr_update(dp_ctx* c, SapState& s, int n, const VecList& x, const double* coef, const Field& y,
                      const Field* z) {
  if constexpr (N > kGcrGroup) {
    return hipErrorInvalidValue;
  } else {
    return n == N ? gcr_pass<MODE, N>(c, s, x, coef, y, z) : gcr_update<MODE, N + 1>(c, s, n, x, coef, y, z);
  }
}

// the sum of the last pass on the host
int gcr_sum(dp_ctx* c, SapState& s, double* out) {
  double* rn = s.gcr.as<double>() + gcr_rn(s.nkv);
  hipLaunchKernelGGL(gcr_finish_kernel, dim3(1), dim3(kBlock), 0, c->stream, s.partials.as<double>(), gcr_blocks(c->g),
                     2, nullptr, 0L, rn, nullptr, nullptr, nullptr);
  DP_HIP(c, hipGetLastError());
  DP_HIP(c, hipMemcpyAsync(out, rn, sizeof(double), hipMemcpyDeviceToHost, c->stream));
  DP_HIP(c, hipStreamSynchronize(c->stream));
  return DP_OK;
}

// w_k against the earlier w_j, then b_k, gamma_k and r -= gamma_k w_k: every
// coefficient is formed and used on the device
int gcr_orthogonalise(dp_ctx* c, SapState& s, int k) {
  const int nkv = s.nkv, nb = gcr_blocks(c->g);
  double* gd = s.gcr.as<double>();
  double* part = s.partials.as<double>();
  double* coef = gd + gcr_coef(nkv);
  VecList x{};
  int n = 0;
  for (int j0 = 0; j0 < k; j0 += n) {
    n = std::min(kGcrGroup, k - j0);
    for (int j = 0; j < n; ++j) x.v[j] = s.w[j0 + j].data.as<double2>();
    DP_HIP(c, gcr_dots(c, s, n, x, s.w[k]));
    hipLaunchKernelGGL(gcr_finish_kernel, dim3(n), dim3(kBlock), 0, c->stream, part, nb, 0, gd + gcr_b2(nkv, j0),
                       (long)2 * nkv, gd + gcr_cc(nkv, j0, k), nullptr, coef, nullptr);
    DP_HIP(c, hipGetLastError());
    if (j0 + n < k) DP_HIP(c, gcr_update<GCR_UPDATE>(c, s, n, x, coef, s.w[k], nullptr));
  }
  DP_HIP(c, gcr_update<GCR_ORTHO>(c, s, n, x, coef, s.w[k], &s.r));
  hipLaunchKernelGGL(gcr_finish_kernel, dim3(1), dim3(kBlock), 0, c->stream, part, nb, 1, nullptr, 0L,
                     gd + gcr_bn(nkv, k), gd + gcr_gam(nkv, k), coef, gd + gcr_b2(nkv, k));
  DP_HIP(c, hipGetLastError());
  x.v[0] = s.w[k].data.as<double2>();
  DP_HIP(c, (gcr_pass<GCR_RESIDUAL, 1>(c, s, x, coef, s.r, nullptr)));
  hipLaunchKernelGGL(gcr_finish_kernel, dim3(1), dim3(kBlock), 0, c->stream, part, nb, 2, nullptr, 0L,
                     gd + gcr_rn(nkv), nullptr, nullptr, nullptr);
  DP_HIP(c, hipGetLastError());
  return DP_OK;
}

template <int PI, int PO>
int convert(dp_ctx* c, const Field& x, const Field& y) {
  hipLaunchKernelGGL((vec_convert_kernel<PI, PO>), site_grid(c->g), dim3(kBlock), 0, c->stream, c->g, x.ref(),
                     y.ref());
  DP_HIP(c, hipGetLastError());
  return DP_OK;
}

template <int P>
int sap_apply(dp_ctx* c, SapState& s, const Blocking& b, int ncy, int nmr) {
  const dim3 mr_grid(b.nhalf);
  bool psi_zero = true;
  for (int cy = 0; cy < ncy; ++cy)
    for (int colour = 0; colour < 2; ++colour) {
      if (!psi_zero) DP_TRY(apply_full(c, s, P, s.q_psi, s.q_a));
      hipLaunchKernelGGL((sap_residual_kernel<P>), site_grid(c->g), dim3(kBlock), 0, c->stream, c->g, b, colour,
                         s.q_r.ref(), s.q_a.ref(), s.q_rho.ref(), psi_zero ? 0 : 1);
      DP_HIP(c, hipGetLastError());
      if (psi_zero) {  // psi = 0 before the first block solve (no site has colour -1)
        hipLaunchKernelGGL((sap_residual_kernel<P>), site_grid(c->g), dim3(kBlock), 0, c->stream, c->g, b, -1,
                           s.q_r.ref(), s.q_a.ref(), s.q_psi.ref(), 0);
        DP_HIP(c, hipGetLastError());
        psi_zero = false;
      }
      for (int k = 0; k < nmr; ++k) {
        DP_TRY(apply_full(c, s, P, s.q_rho, s.q_a));
        hipLaunchKernelGGL((sap_mr_kernel<P>), mr_grid, dim3(kBlock), 0, c->stream, c->g, b, colour, s.q_a.ref(),
                           s.q_rho.ref(), s.q_psi.ref());
        DP_HIP(c, hipGetLastError());
      }
    }
  return DP_OK;
}

// The fused block solves take FP32 block solves on blocks of at most
// kSapBigSites sites (DP_SAP_FUSED=0 keeps the launch-per-step path).
bool sap_fused_enabled(int prec, const Blocking& b) {
  if (prec != F32 || b.vol > kSapBigSites) return false;
  const char* e = std::getenv("DP_SAP_FUSED");
  return !(e && e[0] == '0');
}

// Whole time slices in a wave: a slice of 1, 2, 4, .. or 64 sites.  The other
// small blocks (slices across waves) would have to hand over all directions in
// LDS, which then has no room for clover blocks.
bool sap_slices_in_wave(const Blocking& b) {
  return b.vol <= kSapThreads && 64 % (b.bs[1] * b.bs[2] * b.bs[3]) == 0;
}

// block-layout buffers and the links and clover gathered into them
int sap_fused_setup(dp_ctx* c, SapState& s, const Blocking& b) {
  const long V = 2L * c->g.Vh;
  DP_HIP(c, reserve(c, s.ubl, sizeof(float2) * 36 * V));
  DP_HIP(c, reserve(c, s.cbl, sizeof(float4) * 18 * V));
  DP_HIP(c, reserve(c, s.rbl, sizeof(float4) * 6 * V));
  DP_HIP(c, reserve(c, s.pbl, sizeof(float4) * 6 * V));
  hipLaunchKernelGGL(sap_gather_kernel, block_grid(c->g), dim3(kBlock), 0, c->stream, c->g, b,
                     c->U[F32][0].as<float2>(), c->U[F32][1].as<float2>(), c->C32[0].as<float4>(),
                     c->C32[1].as<float4>(), s.ubl.as<float2>(), s.cbl.as<float4>());
  DP_HIP(c, hipGetLastError());
  return DP_OK;
}

// psi = M r with one kernel per colour pass (r, psi in s.rbl, s.pbl)
int sap_apply_fused(dp_ctx* c, SapState& s, const Blocking& b, int ncy, int nmr) {
  SapPass a;
  a.g = c->g;
  a.b = b;
  a.nmr = nmr;
  a.r = s.rbl.as<float4>();
  a.psi = s.pbl.as<float4>();
  a.U = s.ubl.as<float2>();
  a.C = s.cbl.as<float4>();
  a.rt = s.ratio.as<double>();
  a.sratio = space_hop_ratios(c);
  a.m4 = (float)(4.0 + c->M);
  for (int cy = 0; cy < ncy; ++cy)
    for (int colour = 0; colour < 2; ++colour) {
      a.colour = colour;
      a.own_zero = cy == 0;
      const bool first = cy == 0 && colour == 0;
      if (sap_slices_in_wave(b)) {
        const int nt = (b.vol + 63) / 64 * 64;
        if (first)
          hipLaunchKernelGGL(sap_slice_kernel<true>, dim3(b.nhalf), dim3(nt), sap_slice_lds(nt), c->stream, a);
        else
          hipLaunchKernelGGL(sap_slice_kernel<false>, dim3(b.nhalf), dim3(nt), sap_slice_lds(nt), c->stream, a);
      } else if (b.vol <= kSapThreads) {
        if (first)
          hipLaunchKernelGGL(sap_block_kernel<true>, dim3(b.nhalf), dim3(kSapThreads), 0, c->stream, a);
        else
          hipLaunchKernelGGL(sap_block_kernel<false>, dim3(b.nhalf), dim3(kSapThreads), 0, c->stream, a);
      } else {
        if (first)
          hipLaunchKernelGGL(sap_block_big_kernel<true>, dim3(b.nhalf), dim3(kSapBigThreads), 0, c->stream, a);
        else
          hipLaunchKernelGGL(sap_block_big_kernel<false>, dim3(b.nhalf), dim3(kSapBigThreads), 0, c->stream, a);
      }
      DP_HIP(c, hipGetLastError());
    }
  return DP_OK;
}

// z = M r (r, z FP64)
int precondition(dp_ctx* c, SapState& s, const Blocking& b, int ncy, int nmr, const Field& r, const Field& z) {
  TraceRange tr("sap_precondition");
  if (s.fused) {
    hipLaunchKernelGGL(sap_to_block_kernel, block_grid(c->g), dim3(kBlock), 0, c->stream, c->g, b, r.ref(),
                       s.rbl.as<float4>());
    DP_HIP(c, hipGetLastError());
    DP_TRY(sap_apply_fused(c, s, b, ncy, nmr));
    hipLaunchKernelGGL(sap_from_block_kernel, site_grid(c->g), dim3(kBlock), 0, c->stream, c->g, b,
                       s.pbl.as<float4>(), z.ref());
    DP_HIP(c, hipGetLastError());
  } else if (s.prec == F64) {
    DP_TRY((convert<F64, F64>(c, r, s.q_r)));
    DP_TRY(sap_apply<F64>(c, s, b, ncy, nmr));
    DP_TRY((convert<F64, F64>(c, s.q_psi, z)));
  } else {
    DP_TRY((convert<F64, F32>(c, r, s.q_r)));
    DP_TRY(sap_apply<F32>(c, s, b, ncy, nmr));
    DP_TRY((convert<F32, F64>(c, s.q_psi, z)));
  }
  return DP_OK;
}

}  // namespace

void sap_free(SapState* s) { delete s; }

}  // namespace dp

namespace dp {
namespace {

// Shared set-up of dp_solve_sap and dp_sap_precondition: the blocking, the
// work space, the tables of the one right-hand side (time ratios, 4 + M,
// alpha) and, for fused block solves, the block-layout links and clover.
int sap_prepare(dp_ctx* c, const dp_sap_params* p, int nkv, Blocking* bo) {
  const Geom& g = c->g;
  Blocking& b = *bo;
  b.vol = 1;
  int nblocks = 1;
  for (int mu = 0; mu < 4; ++mu) {
    const int L = mu == 0 ? g.T : mu == 1 ? g.L1 : mu == 2 ? g.L2 : g.L3;
    b.bs[mu] = p->block[mu];
    if (b.bs[mu] < 1 || L % b.bs[mu] || (L / b.bs[mu]) % 2)
      return fail(c, DP_ERR_INVALID_ARG, "each block extent must divide its lattice extent an even number of times");
    b.nb[mu] = L / b.bs[mu];
    b.vol *= b.bs[mu];
    nblocks *= b.nb[mu];
  }
  b.nhalf = nblocks / 2;
  if (p->ncy < 1 || p->nmr < 1) return fail(c, DP_ERR_INVALID_ARG, "bad ncy or nmr");
  if (p->precision != DP_PREC_F64 && p->precision != DP_PREC_F32)
    return fail(c, DP_ERR_INVALID_ARG, "the block solves run in FP64 or FP32");
  DP_HIP(c, hipSetDevice(c->device));
  if (!c->have_U[F64]) return fail(c, DP_ERR_BAD_STATE, "gauge field not set");
  if (!c->sap) {
    c->sap = new (std::nothrow) SapState;
    if (!c->sap) return fail(c, DP_ERR_OOM, "host allocation failed");
  }
  SapState& s = *c->sap;
  DP_TRY(sap_alloc(c, s, nkv, p->precision));
  std::vector<double> rt(4 * g.T);
  ratio_tables(g.T, c->bc_t, c->alpha.data(), rt.data());
  DP_TRY(h2d(c, s.ratio.p, rt.data(), sizeof(double) * 4 * g.T));
  const double m4 = 4.0 + c->M;
  DP_TRY(h2d(c, s.m4.p, &m4, sizeof(double)));
  DP_TRY(h2d(c, s.alpha.p, c->alpha.data(), sizeof(double) * g.T));
  s.fused = sap_fused_enabled(p->precision, b);
  if (s.fused) DP_TRY(sap_fused_setup(c, s, b));
  return DP_OK;
}

}  // namespace
}  // namespace dp

extern "C" int dp_sap_precondition(dp_ctx* c, const double* r, const dp_sap_params* p, double* psi) {
  if (!c || !r || !p || !psi) return DP_ERR_INVALID_ARG;
  const Geom& g = c->g;
  Blocking b;
  DP_TRY(sap_prepare(c, p, 1, &b));
  SapState& s = *c->sap;
  const size_t bytes = (size_t)2 * g.Vh * 12 * sizeof(double2);
  DP_HIP(c, reserve(c, c->scratch_aos, bytes));
  DP_HIP(c, hipMemcpyAsync(c->scratch_aos.p, r, bytes, hipMemcpyHostToDevice, c->stream));
  DP_HIP(c, launch_spinor_import(g, c->scratch_aos.as<double2>(), 1, 0, s.r.ref(0), s.r.ref(1), nullptr, nullptr,
                                 c->stream));
  DP_TRY(precondition(c, s, b, p->ncy, p->nmr, s.r, s.z[0]));
  DP_HIP(c, launch_spinor_export(g, s.z[0].ref(0), s.z[0].ref(1), 1, nullptr, nullptr, c->scratch_aos.as<double2>(),
                                 0, c->stream));
  DP_HIP(c, hipMemcpyAsync(psi, c->scratch_aos.p, bytes, hipMemcpyDeviceToHost, c->stream));
  DP_HIP(c, hipStreamSynchronize(c->stream));
  return DP_OK;
}

namespace dp {
namespace {

// The SAP+GCR solve (after sap_prepare) from a source in device memory (host
// layout); the solution goes to S_dev (device, host layout) if not null, then
// to S_host; t0 is the start of the timed solve.
int sap_solve(dp_ctx* c, const Blocking& b, const double2* eta_dev, const dp_sap_params* p, double2* S_dev,
              double* S_host, double* cpp, dp_info* info, double t0) {
  const Geom& g = c->g;
  SapState& s = *c->sap;
  const size_t bytes = (size_t)2 * g.Vh * 12 * sizeof(double2);
  // eta' = beta eta
  DP_HIP(c, launch_spinor_import(g, eta_dev, 1, 0, s.eta.ref(0), s.eta.ref(1), s.alpha.as<double>(),
                                 space_profile(c), c->stream));
  zc e2;
  DP_TRY(vec_dot(c, s, s.eta, s.eta, &e2));
  const double target = p->r * std::sqrt(e2.real());
  // x = 0, r = eta'
  DP_TRY(vec_set(c, SpinorRef(), s.x));
  DP_TRY(vec_set(c, s.eta.ref(), s.r));
  int iters = 0, status = DP_ERR_NOT_CONVERGED, outer = 0;
  double rn = std::sqrt(e2.real());
  if (!std::isfinite(rn)) status = DP_ERR_NONFINITE;
  else if (rn <= target) status = DP_OK;
  const int nkv = p->nkv;
  std::vector<zc> cc((size_t)nkv * nkv), gam(nkv), al(nkv);
  std::vector<double> bn(nkv);
  while (status == DP_ERR_NOT_CONVERGED && iters < p->max_iter) {
    int k = 0;
    bool breakdown = false;
    for (; k < nkv && iters < p->max_iter; ++k) {
      DP_TRY(precondition(c, s, b, p->ncy, p->nmr, s.r, s.z[k]));
      DP_TRY(apply_full(c, s, F64, s.z[k], s.w[k]));
      ++iters;
      DP_TRY(gcr_orthogonalise(c, s, k));
      double* gd = s.gcr.as<double>();
      DP_HIP(c, hipMemcpyAsync(s.h_gcr.data(), gd, sizeof(double) * gcr_len(nkv), hipMemcpyDeviceToHost, c->stream));
      DP_HIP(c, hipStreamSynchronize(c->stream));
      const double* hg = s.h_gcr.data();
      for (int j = 0; j < k; ++j)
        cc[(size_t)j * nkv + k] = zc(hg[gcr_cc(nkv, j, k)], hg[gcr_cc(nkv, j, k) + 1]);
      bn[k] = hg[gcr_bn(nkv, k)];
      if (!(bn[k] > 0) || !std::isfinite(bn[k])) {
        breakdown = true;
        break;
      }
      gam[k] = zc(hg[gcr_gam(nkv, k)], hg[gcr_gam(nkv, k) + 1]);
      rn = std::sqrt(hg[gcr_rn(nkv)]);
      if (rn <= target) {
        ++k;
        break;
      }
    }
    if (breakdown) {
      status = std::isfinite(bn[k]) ? DP_ERR_BREAKDOWN : DP_ERR_NONFINITE;
      break;
    }
    for (int j = k - 1; j >= 0; --j) {
      zc v = gam[j];
      for (int l = j + 1; l < k; ++l) v -= cc[(size_t)j * nkv + l] * al[l];
      al[j] = v / bn[j];
    }
    // x += sum_j al_j z_j
    double* coef = s.gcr.as<double>() + gcr_coef(nkv);
    DP_TRY(h2d(c, coef, al.data(), sizeof(zc) * k));
    for (int j0 = 0; j0 < k; j0 += kGcrGroup) {
      const int n = std::min(kGcrGroup, k - j0);
      VecList x{};
      for (int j = 0; j < n; ++j) x.v[j] = s.z[j0 + j].data.as<double2>();
      DP_HIP(c, gcr_update<GCR_UPDATE>(c, s, n, x, coef + 2 * j0, s.x, nullptr));
    }
    // true residual r = eta' - D' x
    DP_TRY(apply_full(c, s, F64, s.x, s.r));
    DP_HIP(c, (gcr_pass<GCR_SUBTRACT, 0>(c, s, VecList{}, coef, s.r, &s.eta)));
    double r2 = 0.0;
    DP_TRY(gcr_sum(c, s, &r2));
    rn = std::sqrt(r2);
    ++outer;
    if (!std::isfinite(rn)) status = DP_ERR_NONFINITE;
    else if (rn <= target) status = DP_OK;
  }
  // S = x / beta, C_PP
  if (S_dev) {
    DP_HIP(c, launch_spinor_export(g, s.x.ref(0), s.x.ref(1), 1, s.alpha.as<double>(), space_profile(c), S_dev, 0,
                                   c->stream));
    if (S_host) DP_HIP(c, hipMemcpyAsync(S_host, S_dev, bytes, hipMemcpyDeviceToHost, c->stream));
  }
  if (cpp) {
    DP_HIP(c, reserve(c, s.cpp, sizeof(double) * g.T));
    DP_HIP(c, launch_cpp(g, s.x.ref(0), s.x.ref(1), 1, s.alpha.as<double>(), space_profile(c), nullptr, nullptr,
                         s.cpp.as<double>(), c->stream));
    DP_HIP(c, hipMemcpyAsync(cpp, s.cpp.p, sizeof(double) * g.T, hipMemcpyDeviceToHost, c->stream));
  }
  DP_HIP(c, hipStreamSynchronize(c->stream));
  DP_TRY(timing_harvest(c));
  if (info) {
    dp_info& o = *info;
    o.status = status;
    o.iters = iters;
    o.outer = outer;
    o.hop_calls = 0;
    o.restarts = 0;
    o.fallback = 0;
    o.true_res = e2.real() > 0 ? rn / std::sqrt(e2.real()) : 0.0;
    o.seconds = now_s() - t0;
  }
  if (status == DP_ERR_NOT_CONVERGED) return fail(c, status, "SAP+GCR did not converge within max_iter");
  if (status == DP_ERR_BREAKDOWN) return fail(c, status, "GCR broke down (zero preconditioned direction)");
  if (status == DP_ERR_NONFINITE) return fail(c, status, "a residual became NaN or Inf");
  return DP_OK;
}

int sap_check(dp_ctx* c, const dp_sap_params* p) {
  if (!(p->r > 0) || !std::isfinite(p->r) || p->nkv < 1 || p->nkv > 64 || p->max_iter < 1)
    return fail(c, DP_ERR_INVALID_ARG, "bad residue, ncy, nmr, nkv (1..64) or max_iter");
  return DP_OK;
}

}  // namespace
}  // namespace dp

extern "C" int dp_solve_sap(dp_ctx* c, const double* eta, const dp_sap_params* p, double* S, double* cpp,
                            dp_info* info) {
  if (!c || !eta || !p) return DP_ERR_INVALID_ARG;
  TraceRange tr("dp_solve_sap");
  DP_TRY(sap_check(c, p));
  Blocking b;
  DP_TRY(sap_prepare(c, p, p->nkv, &b));
  const double t0 = now_s();
  // the source through the context's staging buffer, which takes the
  // solution afterwards
  const size_t bytes = (size_t)2 * c->g.Vh * 12 * sizeof(double2);
  DP_HIP(c, reserve(c, c->scratch_aos, bytes));
  DP_HIP(c, hipMemcpyAsync(c->scratch_aos.p, eta, bytes, hipMemcpyHostToDevice, c->stream));
  double2* st = c->scratch_aos.as<double2>();
  return sap_solve(c, b, st, p, S ? st : nullptr, S, cpp, info, t0);
}

extern "C" int dp_solve_sap_dev(dp_ctx* c, const void* eta_dev, const dp_sap_params* p, void* S_dev, double* cpp,
                                dp_info* info, void* hip_stream) {
  if (!c || !eta_dev || !p) return DP_ERR_INVALID_ARG;
  TraceRange tr("dp_solve_sap_dev");
  DP_TRY(sap_check(c, p));
  const size_t bytes = (size_t)2 * c->g.Vh * 12 * sizeof(double2);
  const char* e0 = static_cast<const char*>(eta_dev);
  const char* s0 = static_cast<const char*>(S_dev);
  if (S_dev && e0 < s0 + bytes && s0 < e0 + bytes) return fail(c, DP_ERR_INVALID_ARG, "eta and S overlap");
  DP_HIP(c, hipSetDevice(c->device));
  DP_TRY(wait_caller(c, hip_stream));
  Blocking b;
  DP_TRY(sap_prepare(c, p, p->nkv, &b));
  const double t0 = now_s();
  return sap_solve(c, b, static_cast<const double2*>(eta_dev), p, static_cast<double2*>(S_dev), nullptr, cpp, info,
                   t0);
}
