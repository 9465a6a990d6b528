// The alpha-hop Wilson kernels with clover epilogues (templates; one
// translation unit per storage precision instantiates them).
//
// For an output site x of parity p they compute the hopping term of the
// preconditioned operator D' = alpha (D + M) alpha^-1 (eq. linsysprec),
//
//   H psi(x) = -1/2 sum_mu [ c+_mu(x) (1 - gamma_mu) U_mu(x) psi(x+mu)
//                          + c-_mu(x) (1 + gamma_mu) U_mu(x-mu)^+ psi(x-mu) ]
//
// where the time factors are the ratios of the modified time derivatives
// (heavy-quark section): c+_0(x) = alpha(x0)/alpha(x0+1) and c-_0(x) =
// alpha(x0)/alpha(x0-1), per slot, with the fermion boundary sign folded in at
// the wrap-around (the boundary rule eq. redeftbc reduces to exactly this),
// and the spatial factors are 1, or the same ratios of the spatial profiles
// of the light-quark factorisation (eqs. betaa, redefcovs; periodic).
// The adjoint hop (dag = 1) swaps the projectors and uses the reciprocal
// ratios; it is the hopping part of gamma5 D'(1/alpha) gamma5 = D'(alpha)^+.
//
// Spin projection in the chiral basis, with psi = (u0, u1, l0, l1) in spin and
// s = +1 for (1 - gamma_mu), s = -1 for (1 + gamma_mu):
//   mu = 0: h = u + s l,                 lower = s h
//   mu = k: h = u + s (i sigma_k) l,     lower = -s (i sigma_k) h
// so only the two upper spins are multiplied by the link.
//
// One thread per output site and right-hand side ("slot").  What bounds the
// kernels: with one slot the traffic of links and blocks; with many slots the
// traffic of the spinors past L2 (FP64, FP32) or the instructions (FP16).
// Multiply-adds are therefore fused ones, written out (FP32 link products but
// for one pair, see lfma); FP16 values enter the arithmetic through
// mixed-precision multiply-adds, which convert for free; the slot and with it
// every base address is a scalar; links and blocks stay in LDS as stored.
// 24^3x48, 12 slots, median launch of the solve, odd / even sites with one and
// with four dot products, before -> with these: FP16 247 / 317 / 344 -> 185 / 229 /
// 241 us (2040 .. 2510 -> 1330 .. 1680 instructions a wave and slot, 0.74 of the
// issue rate), FP32 305 / 373 / 402 -> 297 / 368 / 376 us (5.1 .. 5.6 TB/s fetched
// and written).  FP64 read its links from L2 once per slot (even sites) or pair
// of slots, and now once per launch (shared tile, the common blocks in LDS too):
// 787 / 1007 / 1011 -> 637 / 804 / 809 us.
#pragma once
#include <algorithm>
#include <cstdlib>

#include "dp_device.h"

namespace dp {

namespace {

template <typename R>
struct Half {
  cx<R> h[2][3];
};

// u + sg l for stored components: one add, or one mixed-precision
// multiply-add by `one` (1.0f, opaque to the compiler, which would otherwise
// convert and add).
template <int SG, typename R>
__device__ __forceinline__ R pm(R u, R l, float) {
  return SG > 0 ? u + l : u - l;
}
template <int SG>
__device__ __forceinline__ float pm(_Float16 u, _Float16 l, float one) {
  return __builtin_fmaf(SG > 0 ? (float)l : -(float)l, one, (float)u);
}

template <int MU, int S, typename R, int P>
__device__ __forceinline__ void project(const RawSpinor<P>& r, float one, Half<R>& o) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const auto u0 = raw_comp(r, a), u1 = raw_comp(r, 3 + a), l0 = raw_comp(r, 6 + a), l1 = raw_comp(r, 9 + a);
    if constexpr (MU == 0) {
      o.h[0][a] = cx<R>{pm<S>(u0.x, l0.x, one), pm<S>(u0.y, l0.y, one)};
      o.h[1][a] = cx<R>{pm<S>(u1.x, l1.x, one), pm<S>(u1.y, l1.y, one)};
    } else if constexpr (MU == 1) {  // i sigma_1 l = (i l1, i l0)
      o.h[0][a] = cx<R>{pm<-S>(u0.x, l1.y, one), pm<S>(u0.y, l1.x, one)};
      o.h[1][a] = cx<R>{pm<-S>(u1.x, l0.y, one), pm<S>(u1.y, l0.x, one)};
    } else if constexpr (MU == 2) {  // i sigma_2 l = (l1, -l0)
      o.h[0][a] = cx<R>{pm<S>(u0.x, l1.x, one), pm<S>(u0.y, l1.y, one)};
      o.h[1][a] = cx<R>{pm<-S>(u1.x, l0.x, one), pm<-S>(u1.y, l0.y, one)};
    } else {  // i sigma_3 l = (i l0, -i l1)
      o.h[0][a] = cx<R>{pm<-S>(u0.x, l0.y, one), pm<S>(u0.y, l0.x, one)};
      o.h[1][a] = cx<R>{pm<S>(u1.x, l1.y, one), pm<-S>(u1.y, l1.x, one)};
    }
  }
}

// acc += c * (1 - s gamma_mu)-reconstruction of colour a of the
// link-multiplied half spinor (w0, w1)
template <int MU, int S, typename R>
__device__ __forceinline__ void accumulate(cx<R> (&acc)[12], int a, cx<R> w0, cx<R> w1, R c) {
  const R p = S > 0 ? c : -c;
  rfma(acc[a], c, w0);
  rfma(acc[3 + a], c, w1);
  if constexpr (MU == 0) {
    rfma(acc[6 + a], p, w0);
    rfma(acc[9 + a], p, w1);
  } else if constexpr (MU == 1) {  // -s i sigma_1 w = -s (i w1, i w0)
    rfma(acc[6 + a], -p, ti(w1));
    rfma(acc[9 + a], -p, ti(w0));
  } else if constexpr (MU == 2) {  // -s i sigma_2 w = -s (w1, -w0)
    rfma(acc[6 + a], -p, w1);
    rfma(acc[9 + a], p, w0);
  } else {  // -s i sigma_3 w = -s (i w0, -i w1)
    rfma(acc[6 + a], -p, ti(w0));
    rfma(acc[9 + a], p, ti(w1));
  }
}

// ------------------------------------------------------------ links

// A link as stored; FP16 links are used as stored halves by mixed-precision
// multiply-adds.
template <int P>
struct RawLink;
template <>
struct RawLink<F64> {
  double2 v[9];
};
template <>
struct RawLink<F32> {
  float2 v[9];
};
template <>
struct RawLink<F16> {
  unsigned v[9];
};
template <int P>
using LinkElem = typename std::remove_reference<decltype(RawLink<P>().v[0])>::type;

template <int P, bool NT = false>
__device__ __forceinline__ void load_raw_link(const void* base, int mu, int i, int Vh, RawLink<P>& r) {
  using E = LinkElem<P>;
  const E* b = static_cast<const E*>(base) + (long)mu * 9 * Vh;
#pragma unroll
  for (int k = 0; k < 9; ++k) r.v[k] = vld<NT>(at(scalar_base(b + (long)k * Vh), i));
}
__device__ __forceinline__ cx<double> elem(double2 v) { return {v.x, v.y}; }
__device__ __forceinline__ cx<float> elem(float2 v) { return {v.x, v.y}; }
__device__ __forceinline__ h2v elem(unsigned v) { return as_h2(v); }

// t = u h, t += u h (CONJ: conj(u) h), u a stored link entry.  FP32 pairs the
// products: with two fused multiply-adds a component the hop's error against
// FP64 was 8.5e-8 of the result, 8.2e-8 with the pairs, at the same times (12
// columns at 48x24^3: 87.1 ms a solve either way).
template <bool CONJ, typename R>
__device__ __forceinline__ cx<R> lmul(cx<R> u, cx<R> h) { return CONJ ? cjmul(u, h) : cmul(u, h); }
template <bool CONJ, typename R>
__device__ __forceinline__ void lfma(cx<R>& t, cx<R> u, cx<R> h) {
  if constexpr (CONJ) cjfma(t, u, h);
  else cfma(t, u, h);
}
template <bool CONJ>
__device__ __forceinline__ void lfma(cx<float>& t, h2v u, cx<float> h) {
  const float ux = (float)u.x, uy = CONJ ? -(float)u.y : (float)u.y;
  t.x = __builtin_fmaf(-uy, h.y, __builtin_fmaf(ux, h.x, t.x));
  t.y = __builtin_fmaf(uy, h.x, __builtin_fmaf(ux, h.y, t.y));
}
template <bool CONJ>
__device__ __forceinline__ cx<float> lmul(h2v u, cx<float> h) {
  cx<float> t{0.f, 0.f};
  lfma<CONJ>(t, u, h);
  return t;
}

// the same for an entry u of a clover or A^-1 block (see cfma2)
template <bool CONJ, typename U, typename R>
__device__ __forceinline__ void bfma(cx<R>& t, U u, cx<R> h) {
  if constexpr (!std::is_same<U, cx<R>>::value) lfma<CONJ>(t, u, h);
  else if constexpr (CONJ) cjfma2(t, u, h);
  else cfma2(t, u, h);
}

// ------------------------------------------------------------ neighbours

// acc += the hop from neighbour K = 2 mu (forward) or 2 mu + 1 (backward);
// an FP16 spinor's per-site scale multiplies the hop's coefficient (the
// projection and the link product are linear).  DAG selects the adjoint's
// projectors at compile time.
template <int P, int K, bool DAG>
__device__ __forceinline__ void nb_compute(const RawSpinor<P>& raw, const RawLink<P>& rl, typename Tr<P>::R coef,
                                           float one, cx<typename Tr<P>::R> (&acc)[12]) {
  using R = typename Tr<P>::R;
  constexpr int MU = K >> 1;
  constexpr bool FWD = (K & 1) == 0;
  constexpr int S = (DAG ? -1 : 1) * (FWD ? 1 : -1);
  Half<R> h;
  project<MU, S>(raw, one, h);
  const R c = P == F16 ? coef * (R)raw_scale(raw) : coef;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    cx<R> w[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if constexpr (FWD) {
        w[s] = lmul<false>(elem(rl.v[3 * a]), h.h[s][0]);
        lfma<false>(w[s], elem(rl.v[3 * a + 1]), h.h[s][1]);
        lfma<false>(w[s], elem(rl.v[3 * a + 2]), h.h[s][2]);
      } else {
        w[s] = lmul<true>(elem(rl.v[a]), h.h[s][0]);
        lfma<true>(w[s], elem(rl.v[3 + a]), h.h[s][1]);
        lfma<true>(w[s], elem(rl.v[6 + a]), h.h[s][2]);
      }
    }
    accumulate<MU, S>(acc, a, w[0], w[1], c);
  }
}

// The eight neighbours in order through a ring of PF raw spinors: the load of
// neighbour K + PF is issued as soon as neighbour K is used, so that PF - 1 or
// more stay in flight (the scheduling barriers keep the compiler from moving
// the loads).  LDSL: links from the workgroup's LDS copy lu[8][9][64] (lane =
// site), else loaded with the spinors (forward hops from U_out at the output
// site, backward ones from U_in at the neighbour).
template <int P, int PF, bool DAG, bool LDSL>
struct Neighbours {
  using R = typename Tr<P>::R;
  RawSpinor<P> raw[PF];
  RawLink<P> rl[LDSL ? 1 : PF];

  template <int K>
  __device__ __forceinline__ void load(const HopArgs& a, int slot, int i, const int (&nb)[8]) {
    load_raw_spinor<P>(a.in, slot, nb[K], a.g.Vp, raw[K % PF]);
    if constexpr (!LDSL) {
      if constexpr ((K & 1) == 0) load_raw_link<P>(a.U_out, K >> 1, i, a.g.Vp, rl[K % PF]);
      else load_raw_link<P>(a.U_in, K >> 1, nb[K], a.g.Vp, rl[K % PF]);
    }
  }
  template <int K>
  __device__ __forceinline__ void fill(const HopArgs& a, int slot, int i, const int (&nb)[8]) {
    if constexpr (K < PF) {
      load<K>(a, slot, i, nb);
      fill<K + 1>(a, slot, i, nb);
    } else {
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  template <int K, typename E>
  __device__ __forceinline__ void step(const HopArgs& a, int slot, int i, const int (&nb)[8], const R (&coef)[8],
                                       float one, const LinkElem<P>* lu, int lane, cx<R> (&acc)[12], E& epi) {
    if constexpr (K < 8) {
      if constexpr (LDSL) {
        RawLink<P> u;
#pragma unroll
        for (int k = 0; k < 9; ++k) u.v[k] = lu[(K * 9 + k) * 64 + lane];
        nb_compute<P, K, DAG>(raw[K % PF], u, coef[K], one, acc);
      } else {
        nb_compute<P, K, DAG>(raw[K % PF], rl[K % PF], coef[K], one, acc);
      }
      // the sums are complete here: the compiler would otherwise put the
      // multiply-adds of several neighbours off to the epilogue and spill
#pragma unroll
      for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(acc[c].x), "+v"(acc[c].y));
      if constexpr (K + PF < 8) {
        __builtin_amdgcn_sched_barrier(0);
        load<K + PF>(a, slot, i, nb);
        __builtin_amdgcn_sched_barrier(0);
      } else if constexpr (K + PF == 8) {
        __builtin_amdgcn_sched_barrier(0);
        epi.load(a, slot, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      step<K + 1>(a, slot, i, nb, coef, one, lu, lane, acc, epi);
    }
  }
};

// ------------------------------------------------------------ epilogue

// One chirality's clover block as stored: 6 diagonal reals, then the 15 upper
// entries (FP16: halves, to be multiplied by the site's scale).
template <int P>
struct Blk;
template <>
struct Blk<F64> {
  double2 v[18];
  __device__ __forceinline__ double d(int r) const { return (r & 1) ? v[r >> 1].y : v[r >> 1].x; }
  __device__ __forceinline__ cx<double> o(int k) const { return {v[3 + k].x, v[3 + k].y}; }
};
template <>
struct Blk<F32> {
  float v[36];
  __device__ __forceinline__ float d(int r) const { return v[r]; }
  __device__ __forceinline__ cx<float> o(int k) const { return {v[6 + 2 * k], v[7 + 2 * k]}; }
};
template <>
struct Blk<F16> {
  unsigned v[18];
  __device__ __forceinline__ _Float16 d(int r) const { return (r & 1) ? as_h2(v[r >> 1]).y : as_h2(v[r >> 1]).x; }
  __device__ __forceinline__ h2v o(int k) const { return as_h2(v[3 + k]); }
};

// block h of a stored field at site i (FP16 blocks straddle a 16-byte unit:
// the middle one is read for both)
template <int P>
__device__ __forceinline__ void load_blk(const void* base, int h, int i, int Vh, Blk<P>& b) {
  if constexpr (P == F64) {
    const double2* q = static_cast<const double2*>(base);
#pragma unroll
    for (int k = 0; k < 18; ++k) b.v[k] = *at(scalar_base(q + (long)(18 * h + k) * Vh), i);
  } else if constexpr (P == F32) {
    const float4* q = static_cast<const float4*>(base);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const float4 t = *at(scalar_base(q + (long)(9 * h + k) * Vh), i);
      b.v[4 * k] = t.x;
      b.v[4 * k + 1] = t.y;
      b.v[4 * k + 2] = t.z;
      b.v[4 * k + 3] = t.w;
    }
  } else {
    const uint4* q = static_cast<const uint4*>(base);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const uint4 t = *at(scalar_base(q + (long)(4 * h + k) * Vh), i);
      const unsigned w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * k + e - 2 * h;
        if (j >= 0 && j < 18) b.v[j] = w[e];
      }
    }
  }
}

// y = (B + shift) x (FP32, FP64) or y = B x (FP16, without the scale); the
// order of herm_apply.
template <int P, typename R>
__device__ __forceinline__ void blk_apply(const Blk<P>& B, R shift, const cx<R>* x, cx<R>* y) {
  y[0] = lmul<false>(B.o(herm_off(0, 1)), x[1]);
#pragma unroll
  for (int c = 1; c < 6; ++c) y[c] = lmul<true>(B.o(herm_off(0, c)), x[0]);
#pragma unroll
  for (int r = 0; r < 6; ++r)
#pragma unroll
    for (int c = r + 1; c < 6; ++c) {
      if (r > 0 || c > 1) bfma<false>(y[r], B.o(herm_off(r, c)), x[c]);  // A_rc x_c
      if (r > 0) bfma<true>(y[c], B.o(herm_off(r, c)), x[r]);            // A_cr = conj(A_rc)
    }
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    if constexpr (P == F16) rfma(y[r], (float)B.d(r), x[r]);
    else rfma(y[r], B.d(r) + shift, x[r]);
  }
}

// components 6h .. 6h+5 of a stored spinor in the arithmetic type
template <int P, typename R>
__device__ __forceinline__ void decode_half(const RawSpinor<P>& r, int h, cx<R> (&x)[6]) {
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const auto q = raw_comp(r, 6 * h + c);
    if constexpr (P == F16) x[c] = cx<R>{(R)((float)q.x * r.sc), (R)((float)q.y * r.sc)};
    else x[c] = cx<R>{(R)q.x, (R)q.y};
  }
}

__device__ __forceinline__ void load_half64(const SpinorRef& f, int slot, int h, int i, int Vh, cx<double> (&x)[6]) {
  const double2* b = static_cast<const double2*>(f.data) + (long)slot * f.slot_stride;
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const double2 v = vld<true>(at(scalar_base(b + (long)(6 * h + c) * Vh), i));
    x[c] = cx<double>{v.x, v.y};
  }
}

template <int P, typename R>
__device__ __forceinline__ void store_half(const SpinorRef& f, int slot, int h, int i, int Vh, const cx<R>* s) {
  static_assert(P != F16, "an FP16 site is stored whole (its scale is the maximum over the site)");
  if constexpr (P == F64) {
    double2* b = static_cast<double2*>(f.data) + (long)slot * f.slot_stride;
#pragma unroll
    for (int c = 0; c < 6; ++c) vst<true>(at(scalar_base(b + (long)(6 * h + c) * Vh), i), make_double2(s[c].x, s[c].y));
  } else {
    float4* b = static_cast<float4*>(f.data) + (long)slot * f.slot_stride;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      vst<true>(at(scalar_base(b + (long)(3 * h + k) * Vh), i), make_float4(s[2 * k].x, s[2 * k].y, s[2 * k + 1].x, s[2 * k + 1].y));
  }
}

// s += <a, b> (real and imaginary part), s += |a|^2
template <typename R>
__device__ __forceinline__ void dot_add(R& re, R& im, cx<R> a, cx<R> b) {
  re = fmar(a.y, b.y, fmar(a.x, b.x, re));
  im = fmar(-a.y, b.x, fmar(a.x, b.y, im));
}

// The stored copy of the clover or A^-1 blocks the epilogue uses in LDS: units of
// 32 bits [72 (FP32) or 36 (FP16)][64], then the FP16 scales [64]; FP64:
// double2 [36][64].
constexpr int blk_units(int p) { return p == F64 ? 144 : p == F32 ? 72 : 36; }

// A thread's output site: its index, spatial coordinates and neighbours
// (2 mu forward, 2 mu + 1 backward).
struct Site {
  int i, x1, x2, x3;
  // of the wave (host order): its first site within the timeslice, the odd x3
  int sp0;
  unsigned long long odd;
  int nb[8];
};

// the epilogue an output parity sees
constexpr int site_epi(int epi) { return epi == EPI_FULL || epi == EPI_FULL_HOST ? EPI_DIAG : epi; }

// Spinors of a wave's 64 sites, a site per lane, stored in host order: site q at
// dst + (2 q + odd(q)) 12, odd(q) the bits of `odd` (sites of the other parity lie
// between), the first n sites.  Register k of four and the row of 16 lanes change
// places by register swaps (four components of site 16 k + m in the lanes m of
// the four rows), then a permute brings the four components of a site to
// neighbouring lanes, which store 64 bytes of it.  No LDS, which the links fill.
// (The full operator on 12 columns at 48x24^3: 1620 us and 530 of a separate
// export pass; 1720 with this.)  Every lane of the wave calls it.
__device__ __forceinline__ void store_host_order(double2* dst, unsigned long long odd, int n, const cx<double> (&v)[12],
                                                 int lane) {
  asm volatile("" : "+v"(lane));  // or the offsets stay in registers through the slots
  const int m = lane >> 2, r = lane & 3, from = (16 * r + m) << 2;
  dst = scalar_base(dst);
#pragma unroll
  for (int c = 0; c < 12; c += 4) {
    unsigned w[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned long long x = __builtin_bit_cast(unsigned long long, v[c + k].x);
      const unsigned long long y = __builtin_bit_cast(unsigned long long, v[c + k].y);
      w[k][0] = (unsigned)x;
      w[k][1] = (unsigned)(x >> 32);
      w[k][2] = (unsigned)y;
      w[k][3] = (unsigned)(y >> 32);
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const auto a = __builtin_amdgcn_permlane32_swap(w[0][d], w[2][d], false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(w[1][d], w[3][d], false, false);
      const auto e = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
      const auto f = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
      w[0][d] = e[0];
      w[1][d] = e[1];
      w[2][d] = f[0];
      w[3][d] = f[1];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      u4v u;
      u.x = __builtin_amdgcn_ds_bpermute(from, w[k][0]);
      u.y = __builtin_amdgcn_ds_bpermute(from, w[k][1]);
      u.z = __builtin_amdgcn_ds_bpermute(from, w[k][2]);
      u.w = __builtin_amdgcn_ds_bpermute(from, w[k][3]);
      const int q = 16 * k + m;
      if (q < n) *const_cast<u4v*>(at(reinterpret_cast<const u4v*>(dst), (2 * q + (int)((odd >> q) & 1)) * 12 + c + r)) = u;
    }
  }
}

// Epilogue and fused reduction terms for one slot, one chirality at a time
// (fewer live registers).  The epilogue's own inputs and the output are
// streamed past L2 (read or written once per launch: 3% at 24^3x48 with 12
// FP32 slots).  The 12 components of a dot product are summed in the
// arithmetic precision per lane and added to the FP64 partial once.
// load() issues the streams' loads (while the last neighbours are computed),
// finish() does the rest.
template <int P, int EPIL, int RED, bool LDSB>
struct Epilogue {
  using R = typename Tr<P>::R;
  static constexpr int EPI = site_epi(EPIL);
  static constexpr bool HOST = EPIL == EPI_FULL_HOST;
  static constexpr bool WHOLE = P == F16 || HOST;  // the output is stored when both chiralities are there
  static constexpr int PW = rh_prec(P);
  static constexpr bool XIN = EPI == EPI_DIAG || EPI == EPI_SUB || EPI == EPI_INV_SUB;
  static constexpr bool INV = EPI == EPI_INV || EPI == EPI_INV_SUB;
  static constexpr bool DOTW = RED == RED_DOT_EXT || RED == RED_TS4;
  RawSpinor<P> xr;
  RawSpinor<PW> wr;

  __device__ __forceinline__ void load(const HopArgs& a, int slot, int i) {
    if constexpr (XIN) load_raw_spinor<P, true>(a.xin, slot, i, a.g.Vp, xr);
    if constexpr (DOTW && P != F64) load_raw_spinor<PW, true>(a.red.w, slot, i, a.g.Vp, wr);
  }

  // HOST: x0, s of the wave's sites
  __device__ __forceinline__ void finish(const HopArgs& a, int slot, int i, cx<R> (&acc)[12], double (&red)[kRedMax],
                                         const unsigned* lc, int lane, int x0, const Site& s) const {
    const Geom& g = a.g;
    R s0 = R(0), s1 = R(0), s2 = R(0), s3 = R(0), s4 = R(0), s5 = R(0), s6 = R(0);
    cx<R> out[WHOLE ? 12 : 6];
    R bsc = R(1);  // FP16 block scale
    if constexpr (P == F16 && (EPI == EPI_DIAG || INV)) {
      if constexpr (LDSB) {
        bsc = __builtin_bit_cast(float, lc[blk_units(P) * 64 + lane]);
      } else if constexpr (INV) {
        bsc = *at(uniform_ptr(a.slots.ainv_scale[slot]), i);
      } else {
        bsc = *at(a.clov.scale, i);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      __builtin_amdgcn_sched_barrier(0);
      cx<R>* o = &out[WHOLE ? 6 * h : 0];
      cx<R>* ac = &acc[6 * h];
      cx<R> xh[6], wh[6];
      if constexpr (XIN) decode_half<P>(xr, h, xh);
      Blk<P> B;
      if constexpr (EPI == EPI_DIAG || INV) {
        if constexpr (LDSB && P == F64) {
          const double2* l = reinterpret_cast<const double2*>(lc);
#pragma unroll
          for (int k = 0; k < 18; ++k) B.v[k] = l[(18 * h + k) * 64 + lane];
        } else if constexpr (LDSB) {
          constexpr int n = blk_units(P) / 2;
#pragma unroll
          for (int k = 0; k < n; ++k)
            B.v[k] = __builtin_bit_cast(typename std::remove_reference<decltype(B.v[0])>::type,
                                        lc[(n * h + k) * 64 + lane]);
        } else if constexpr (INV) {
          load_blk<P>(uniform_ptr(a.slots.ainv[slot]), h, i, g.Vp, B);
        } else {
          load_blk<P>(a.clov.data, h, i, g.Vp, B);
        }
      }
      if constexpr (EPI == EPI_HOP) {
#pragma unroll
        for (int c = 0; c < 6; ++c) o[c] = R(-0.5) * ac[c];
      } else if constexpr (EPI == EPI_DIAG) {
        const R m4 = (R)a.slots.m4[slot];
        const R hs = (R)(-0.5 * a.sign);
        blk_apply<P>(B, m4, xh, o);
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          if constexpr (P == F16) {
            cx<R> t = m4 * xh[c];
            rfma(t, bsc, o[c]);
            o[c] = t;
          }
          rfma(o[c], hs, ac[c]);
        }
      } else if constexpr (EPI == EPI_SUB) {
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          o[c] = xh[c];
          rfma(o[c], R(0.5), ac[c]);
        }
      } else {  // EPI_INV, EPI_INV_SUB
        cx<R> t[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          if constexpr (EPI == EPI_INV_SUB) {
            t[c] = xh[c];
            rfma(t[c], R(0.5), ac[c]);
          } else {
            t[c] = R(-0.5) * ac[c];
          }
          if constexpr (P == F16) t[c] = bsc * t[c];
        }
        blk_apply<P>(B, R(0), t, o);
      }
      if constexpr (!WHOLE) store_half<P>(a.out, slot, h, i, g.Vp, o);
      if constexpr (DOTW) {
        if constexpr (P == F64) load_half64(a.red.w, slot, h, i, g.Vp, wh);  // here: fewer live registers
        else decode_half<PW>(wr, h, wh);
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        if constexpr (RED == RED_DOT_EXT) dot_add(s0, s1, wh[c], o[c]);
        if constexpr (RED == RED_TS || RED == RED_TS4) {
          dot_add(s0, s1, o[c], xh[c]);
          s2 = fmar(o[c].y, o[c].y, fmar(o[c].x, o[c].x, s2));
        }
        if constexpr (RED == RED_TS4) {
          dot_add(s3, s4, wh[c], xh[c]);
          dot_add(s5, s6, wh[c], o[c]);
        }
        if constexpr (RED == RED_NORM) s0 = fmar(o[c].y, o[c].y, fmar(o[c].x, o[c].x, s0));
      }
    }
    if constexpr (HOST)
      store_host_order(a.aos + slot * a.aos_ss + 24L * ((long)x0 * g.Vsh + s.sp0),
                       s.odd, g.Vsh - s.sp0, out, lane);
    else if constexpr (WHOLE)
      SpinorIO<P>::template store<true>(a.out, slot, i, g.Vp, out);
    if constexpr (RED != RED_NONE) red[0] = (double)s0;
    if constexpr (RED == RED_DOT_EXT || RED == RED_TS || RED == RED_TS4) red[1] = (double)s1;
    if constexpr (RED == RED_TS || RED == RED_TS4) red[2] = (double)s2;
    if constexpr (RED == RED_TS4) {
      red[3] = (double)s3;
      red[4] = (double)s4;
      red[5] = (double)s5;
      red[6] = (double)s6;
    }
  }
};

// ------------------------------------------------------------ sites

// Mapping of the blocks: every XCD (block b runs on XCD b mod 8) owns either
// a spatial slab, a fixed range of 64-site chunks of each timeslice that it
// sweeps in x0 (tmap 0), or the timeslices [T k / 8, T (k+1) / 8) of every
// chunk, chunk by chunk with the timeslices innermost (tmap 1); the x0 +- 1
// neighbour spinors are then re-read from that XCD's L2.  The reduction
// partial of an item is x0 nch + chunk (nparts = T nch) whatever the mapping.
// mL3h, mL2: reciprocals for the site coordinates (div_by).
struct SlabMap {
  int nch, maxc;
  int tmap, tlen;  // tlen: the longest XCD time range
  unsigned mL3h, mL2;
};

// n / d for n < 2^31 with m = min(2^32 - 1, floor(2^32 / d)): the product is
// short of the quotient by at most one
__device__ __forceinline__ int div_by(int n, int d, unsigned m) {
  const unsigned q = __umulhi((unsigned)n, m);
  return (int)(q + ((unsigned)n - q * (unsigned)d >= (unsigned)d ? 1u : 0u));
}

__device__ __forceinline__ int slab_lo(int nch, int xcd) { return (nch * xcd) >> 3; }

struct Item {
  int chunk, x0;
  bool in;  // false: the block owns nothing
};
// item j of an XCD; backwards: the timeslices from the last to the first (the
// even-site kernels: they read the odd field the preceding odd-site kernel
// wrote in forward order, whose last timeslices are still in the caches; 3%
// at 24^3x48 with 12 FP32 slots)
__device__ __forceinline__ Item map_item(const SlabMap& m, int T, int xcd, int j, bool backwards) {
  Item it;
  if (m.tmap) {
    const int lo = (T * xcd) >> 3, hi = (T * (xcd + 1)) >> 3;
    const int dt = j % m.tlen;
    it.chunk = j / m.tlen;
    it.in = lo + dt < hi && it.chunk < m.nch;
    it.x0 = backwards ? hi - 1 - dt : lo + dt;
  } else {
    it.x0 = j / m.maxc;
    it.chunk = slab_lo(m.nch, xcd) + (j - it.x0 * m.maxc);
    it.in = it.chunk < slab_lo(m.nch, xcd + 1);
    if (backwards) it.x0 = T - 1 - it.x0;
  }
  return it;
}

__device__ __forceinline__ void locate(const HopArgs& a, const SlabMap& m, int x0, int sp, Site& s) {
  const Geom& g = a.g;
  const int row = div_by(sp, g.L3h, m.mL3h), h = sp - row * g.L3h;
  s.x1 = div_by(row, g.L2, m.mL2);
  s.x2 = row - s.x1 * g.L2;
  const int odd = (a.p + x0 + s.x1 + s.x2) & 1;  // x3 = 2 h + odd
  s.x3 = 2 * h + odd;
  const int i = x0 * g.Vsh + sp, pl = g.L2 * g.L3h;
  s.i = i;
  s.nb[0] = x0 + 1 == g.T ? sp : i + g.Vsh;
  s.nb[1] = x0 == 0 ? i + (g.T - 1) * g.Vsh : i - g.Vsh;
  s.nb[2] = s.x1 + 1 == g.L1 ? i - (g.L1 - 1) * pl : i + pl;
  s.nb[3] = s.x1 == 0 ? i + (g.L1 - 1) * pl : i - pl;
  s.nb[4] = s.x2 + 1 == g.L2 ? i - (g.L2 - 1) * g.L3h : i + g.L3h;
  s.nb[5] = s.x2 == 0 ? i + (g.L2 - 1) * g.L3h : i - g.L3h;
  // x3 + 1 is at the same half index from an even x3, at the next from an odd one
  s.nb[6] = !odd ? i : h + 1 == g.L3h ? i - (g.L3h - 1) : i + 1;
  s.nb[7] = odd ? i : h == 0 ? i + (g.L3h - 1) : i - 1;
}

// The hop for one slot at the thread's site (if valid), the epilogue, and the
// wave's share of the fused reductions, stored as partial `part` of `nparts`.
// Every lane of the wave calls it.  lu, lc: the workgroup's LDS copies of the
// links (LDSL) and of the blocks (LDSB).
template <int P, int EPI, int RED, int PF, bool DAG, bool LDSL, bool LDSB>
__device__ __forceinline__ void slot_work(const HopArgs& a, int slot, const Site& s, int x0, bool valid, int part,
                                          int nparts, const LinkElem<P>* lu, const unsigned* lc, int lane) {
  using R = typename Tr<P>::R;
  const Geom& g = a.g;
  double red[kRedMax];
#pragma unroll
  for (int q = 0; q < kRedMax; ++q) red[q] = 0.0;
  // stores in host order need every lane of the wave; its sites beyond the
  // timeslice are computed as the first one and not stored
  if (valid || EPI == EPI_FULL_HOST) {
    const double* rt = a.slots.ratio + (long)slot * 4 * g.T + (DAG ? 2 * g.T : 0);
    R coef[8] = {(R)rt[x0], (R)rt[g.T + x0], R(1), R(1), R(1), R(1), R(1), R(1)};
    if (a.sratio) {  // uniform over the launch
      const int x[3] = {s.x1, s.x2, s.x3};
      const int Ls[3] = {g.L1, g.L2, g.L3};
      int off = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        coef[2 + 2 * k] = (R)a.sratio[off + (DAG ? 2 * Ls[k] : 0) + x[k]];
        coef[3 + 2 * k] = (R)a.sratio[off + (DAG ? 3 * Ls[k] : Ls[k]) + x[k]];
        off += 4 * Ls[k];
      }
    }
    float one = 1.f;
    if constexpr (P == F16) asm("" : "+s"(one));
    cx<R> acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = cx<R>{R(0), R(0)};
    // opaque here: hoisted out of the caller's slot loop, the offsets would be
    // kept widened to 64 bits and every load would add its base to them
    int i = s.i, nb[8];
    asm volatile("" : "+v"(i));
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      nb[k] = s.nb[k];
      asm volatile("" : "+v"(nb[k]));
    }
    Neighbours<P, PF, DAG, LDSL> n;
    n.template fill<0>(a, slot, i, nb);
    Epilogue<P, EPI, RED, LDSB> epi;
    n.template step<0>(a, slot, i, nb, coef, one, lu, lane, acc, epi);
    epi.finish(a, slot, i, acc, red, lc, lane, x0, s);
  }
  if constexpr (RED != RED_NONE) {
    constexpr int nv = red_values(RED);
    double* pt = a.red.partials + (long)slot * kRedMax * nparts;
    const int v = wave_row_value(lane >> 4);
    const double w = wave_sum4(red[0], red[1], red[2], red[3]);
    if ((lane & 15) == 0 && v < nv) pt[partial_at(nparts, part, v)] = w;
    if constexpr (nv > 4) {
      const double w2 = wave_sum4(red[4], red[5], red[6], red[7]);
      if ((lane & 15) == 0 && 4 + v < nv) pt[partial_at(nparts, part, 4 + v)] = w2;
    }
  }
}

// ------------------------------------------------------------ kernels

// Neighbours in flight (ring depth) and waves per SIMD the registers must
// allow, per precision.  Even / odd sites, us, by depth at the waves below:
//   hop_kernel_slab, one slot, 32^3x64: FP64 1: 510 / 507, 2: 501 / 496, 3: 486 /
//   489, 4: 480 / 484, 6 (spills): 818 / 878; FP32 1: 250 / 231, 2 or 3: 243 / 228, 4
//   (spills): 369 / 326; FP16 1 to 6: 132 .. 134 / 123 .. 127;
//   hop_kernel_shared, 12 slots, 24^3x48, the operator by itself: FP64 1: 682 /
//   679, 2: 679 / 667, 3 (spills): 783 / 790; FP32 1: 330 / 340, 2: 331 / 342, 3:
//   337 / 329, 4: 340 / 340, 6: 337 / 346; FP16 1: 219 / 203, 2: 204 / 204, 3: 203 /
//   207, 4: 207 / 209, 6: 213 / 223.
// Without spills the depth matters little: the kernels are bound by what the L2
// fetches (FP64, FP32) or by instruction issue (FP16).  Fetching the next
// slot's first neighbours during the epilogue was 5-20% slower.
constexpr int slab_pf(int p, int waves) { return p == F64 ? (waves == 1 ? 3 : 2) : p == F32 ? 2 : 4; }
constexpr int slab_min_waves(int p) { return p == F64 ? 1 : 3; }
constexpr int shared_pf(int p) { return p == F32 ? 3 : 2; }
constexpr int shared_threads(int p, bool blk) { return p == F64 && blk ? 384 : 256; }
constexpr int kSharedMinWaves = 2;

constexpr int kCus = 256, kSimds = 4 * kCus;
// Up to so many waves, one per (chunk, timeslice, slot), several slots run as
// one wave each too (FP64 in some cases beyond, see one_wave_per_slot): a
// shared-tile workgroup would leave CUs without work and take its slots one
// after the other.  Even / odd sites, us, one wave per slot
// against shared tile: 768 waves (8^3x16, 12 slots) FP64 14.8 / 15.0 against
// 28.6 / 25.0, FP32 10.6 / 10.4 against 17.9 / 19.2, FP16 9.1 / 9.5 against
// 17.1 / 17.3; 1344 waves (12^3x24, 4 slots) FP64 28.4 / 26.9 against 26.3 / 22.9,
// FP32 14.8 / 14.5 against 15.9 / 15.1; 2880 (36x18x20x14, 2 slots) FP32 28.5 / 28.0
// against 34.7 / 30.6; 4032 (12^3x24, 12 slots) FP32 31.3 / 29.6 against 30.7 /
// 30.8, FP16 21.0 / 20.6 against 26.7 / 26.1; 4096 (16^3x32, 4 slots) FP32 35.4 /
// 32.5 against 33.0 / 28.6, FP16 equal.
constexpr int slab_max_waves(int p) { return p == F64 ? 1024 : p == F32 ? 3072 : 4096; }

// EPI_FULL: the two parities of an item are neighbouring items of an XCD, so
// that a link, the forward one of a site of this parity and a backward one for
// the other parity, is fetched once for both (one FP64 slot, two launches / one:
// 1030 / 745 us at 64x32^3, 315 / 233 at 48x24^3, 18 / 8 at 16x8^3; 12 FP64
// slots, which share their links in LDS: 1620 / 1620 at 48x24^3).  The arguments
// of parity 1 - a.p if `other`.
__device__ __forceinline__ void pick_parity(HopArgs& a, bool other) {
  if (!other) return;
  a.p = 1 - a.p;
  const void* u = a.U_out;
  a.U_out = a.U_in;
  a.U_in = u;
  const SpinorRef f = a.in;
  a.in = a.xin;
  a.xin = f;
  a.out = a.out2;
  a.clov = a.clov2;
}
// the XCD's item of the block
template <int EPI>
__device__ __forceinline__ int xcd_item(HopArgs& a) {
  const int j = blockIdx.x >> 3;
  if constexpr (EPI == site_epi(EPI)) return j;
  pick_parity(a, j & 1);
  return j >> 1;
}

// One wave per (chunk, timeslice, slot), the slots of a chunk in neighbouring
// blocks of the same XCD; W waves per SIMD.
template <int P, int EPIL, int RED, bool DAG, int W>
__global__ void __launch_bounds__(64, W) hop_kernel_slab(HopArgs a, SlabMap m) {
  constexpr int EPI = site_epi(EPIL);
  const int j = xcd_item<EPIL>(a), jj = j / a.nslots, slot = j - jj * a.nslots;
  const Item it = map_item(m, a.g.T, blockIdx.x & 7, jj, EPI == EPI_DIAG);
  if (!it.in || (a.slots.mask && !a.slots.mask[slot])) return;
  const int sp = it.chunk * 64 + threadIdx.x;
  const bool valid = sp < a.g.Vsh;
  Site s;
  locate(a, m, it.x0, valid ? sp : 0, s);
  s.sp0 = it.chunk * 64;
  if constexpr (EPIL == EPI_FULL_HOST) s.odd = __ballot((a.p + it.x0 + s.x1 + s.x2) & 1);
  slot_work<P, EPIL, RED, slab_pf(P, W), DAG, false, false>(a, slot, s, it.x0, valid, it.x0 * m.nch + it.chunk,
                                                        a.g.T * m.nch, nullptr, nullptr, threadIdx.x);
}

// Several slots: one workgroup per (chunk, timeslice), its waves take the
// slots in turn.  The links of the chunk's 64 sites in the 8 hop directions and,
// with BLK, the blocks of the epilogue that are the same for every slot (clover
// blocks of the even sites, A^-1 blocks of the odd ones when all slots share one
// mass) are loaded once into LDS, as stored, instead of once per slot.  Per-slot
// arithmetic and reduction partials are those of the one-slot kernel: bitwise
// the same.  8 waves a CU in two workgroups (FP32, FP16): with 4 or 6 of one
// workgroup the hops of 12 slots at 48x24^3 take 15-80% longer, with 12 of two or
// one 2-30%, since the neighbours of what is in flight have to stay in the L2s.
template <int P>
constexpr size_t shared_tile_bytes(bool blocks) {
  return 8 * 9 * 64 * sizeof(LinkElem<P>) + (blocks ? (blk_units(P) + (P == F16)) * 64 * sizeof(unsigned) : 0);
}

template <int P, int EPIL, int RED, bool DAG, bool BLK>
__global__ void __launch_bounds__(shared_threads(P, BLK), kSharedMinWaves) hop_kernel_shared(HopArgs a, SlabMap m) {
  constexpr int EPI = site_epi(EPIL);
  using E = LinkElem<P>;
  extern __shared__ __align__(16) unsigned char smem[];
  E* lu = reinterpret_cast<E*>(smem);
  unsigned* lc = reinterpret_cast<unsigned*>(smem + 8 * 9 * 64 * sizeof(E));
  const Geom& g = a.g;
  const Item it = map_item(m, g.T, blockIdx.x & 7, xcd_item<EPIL>(a), EPI == EPI_DIAG);
  if (!it.in) return;  // the whole workgroup, before any barrier
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int sp = it.chunk * 64 + lane;
  const bool valid = sp < g.Vsh;
  Site s;
  locate(a, m, it.x0, valid ? sp : 0, s);
  s.sp0 = it.chunk * 64;
  if constexpr (EPIL == EPI_FULL_HOST) s.odd = __ballot((a.p + it.x0 + s.x1 + s.x2) & 1);
  // fill: tasks 0..7 are the link directions, task 8 the blocks; wave w takes
  // tasks w, w + nw, ...  Read once per launch: streamed past L2 (2-3%).
  constexpr bool inv = EPI == EPI_INV || EPI == EPI_INV_SUB;
  if (valid) {
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      if (t % nw != wv || (t == 8 && !BLK)) continue;
      if (t < 8) {
        RawLink<P> u;
        if (t & 1) load_raw_link<P, true>(a.U_in, t >> 1, s.nb[t], g.Vp, u);
        else load_raw_link<P, true>(a.U_out, t >> 1, s.i, g.Vp, u);
#pragma unroll
        for (int k = 0; k < 9; ++k) lu[(t * 9 + k) * 64 + lane] = u.v[k];
      } else if constexpr (BLK) {
        const void* src = inv ? a.slots.ainv_common : a.clov.data;
        if constexpr (P == F64) {
          const double2* q = static_cast<const double2*>(src);
          double2* l = reinterpret_cast<double2*>(lc);
#pragma unroll
          for (int k = 0; k < 36; ++k) l[k * 64 + lane] = vld<true>(at(scalar_base(q + (long)k * g.Vp), s.i));
          continue;
        }
        const uint4* q = static_cast<const uint4*>(src);
#pragma unroll
        for (int k = 0; k < blk_units(P) / 4; ++k) {
          const uint4 v = vld<true>(at(scalar_base(q + (long)k * g.Vp), s.i));
          lc[(4 * k) * 64 + lane] = v.x;
          lc[(4 * k + 1) * 64 + lane] = v.y;
          lc[(4 * k + 2) * 64 + lane] = v.z;
          lc[(4 * k + 3) * 64 + lane] = v.w;
        }
        if constexpr (P == F16) {
          const float* sc = inv ? a.slots.ainv_common_scale : a.clov.scale;
          lc[blk_units(P) * 64 + lane] = __builtin_bit_cast(unsigned, vld<true>(at(sc, s.i)));
        }
      }
    }
  }
  __syncthreads();
  const int part = it.x0 * m.nch + it.chunk, nparts = g.T * m.nch;
#pragma unroll 1
  for (int slot = wv; slot < a.nslots; slot += nw) {
    if (a.slots.mask && !a.slots.mask[slot]) continue;
    // keeps the compiler from hoisting the LDS reads out of this loop into
    // (many) registers
    asm volatile("" ::: "memory");
    slot_work<P, EPIL, RED, shared_pf(P), DAG, true, BLK>(a, slot, s, it.x0, valid, part, nparts, lu, lc, lane);
  }
}

int env_knob(const char* name, int dflt) {
  const char* e = getenv(name);
  return e ? atoi(e) : dflt;
}

unsigned recip32(int d) {
  const unsigned long long m = (1ULL << 32) / (unsigned)d;
  return (unsigned)std::min<unsigned long long>(m, 0xffffffffULL);
}

// The slots of a launch as one wave each, or sharing a tile (see slab_max_waves).
// FP64 launches of one parity beyond that limit: with at most half as many tiles
// as CUs the slots stay waves of their own, and also up to two waves a SIMD
// unless the tiles fill the CUs evenly (512 workgroups run at once, 256 with the
// blocks in LDS).  Schur operator, both kernels, us, waves of their own (two a
// SIMD, see fp64_two_waves) against shared: 64 tiles (2x16^3) 24 slots 45 / 80, 32:
// 56 / 101; 80 (10^4) 16: 46 / 65, 24: 62 / 92; 96 (24x8^3) 32: 77 / 108; 112 (8x12^3)
// 12: 47 / 54, 32: 95 / 115; 128 (4x16^3) 16: 56 / 62, 32: 100 / 111; but 140 (10x12^3)
// 16: 74 / 66.  280 (20x12^3) 4: 43 / 49; 576 (18x16^3) 2: 47 / 62; 768 (24x16^3) 2: 58 /
// 68; 336 (24x12^3) 6: 58 / 64; tiles that fill the CUs: 256 (8x16^3) 6: 47 / 45, 512
// (16^4) 3: 53 / 50.
template <int P, bool FULL>
bool one_wave_per_slot(int items, int nslots) {
  const long waves = (long)items * nslots;
  if (nslots == 1 || waves <= slab_max_waves(P)) return true;
  if (P != F64 || FULL) return false;
  return 2 * items <= kCus || (waves < 2 * kSimds && items % (nslots >= 5 ? kCus : 2 * kCus) != 0);
}

// FP64 waves of their own: registers for two a SIMD (a shorter ring) where one a
// SIMD would need a second, mostly empty round.  Schur operator, us, one / two a
// SIMD: one slot 1080 waves 65.9 / 58.1, 1280 75.0 / 68.7, 1536 86.4 / 82.9, but 1792
// 98.0 / 98.0 and 2048 107 / 116; several slots 1120 50 / 41, 1280 60 / 50, 1792 61 /
// 54 (112 tiles) and 66 / 67 (896), 2016 61 / 58, 2304 73 / 69.  Full operator: one slot
// 1152 waves 32 / 27, 1536 36 / 35; several 1536 28 .. 31 / 23 .. 26.
inline bool fp64_two_waves(long waves, int nslots) {
  return waves > kSimds && (nslots > 1 || 2 * waves <= 3 * kSimds);
}

template <int P, int EPI, int RED, bool DAG>
hipError_t launch_one(const HopArgs& a, hipStream_t st, int* nparts_out) {
  SlabMap m;
  m.nch = (a.g.Vsh + 63) / 64;
  m.maxc = (m.nch + 7) / 8;
  m.tlen = (a.g.T + 7) / 8;
  m.mL3h = recip32(a.g.L3h);
  m.mL2 = recip32(a.g.L2);
  // XCD mapping, chosen per launch: both mappings give bitwise the same
  // results.  The one that spreads the work more evenly, if the XCD with most
  // work has 5% less of it than with the other: slabs give ceil(chunks / 8)
  // chunks to an XCD, timeslice ranges ceil(T / 8) timeslices.  Slabs against
  // ranges, even sites, us: 16x8^3 (4 chunks, half of the XCDs idle) with 12 slots
  // FP64 26.4 / 15.1, FP32 14.4 / 10.7, FP16 12.4 / 9.4; 14x20x18x36 (102 chunks) FP16
  // 65.8 / 72.8, one FP32 slot 21.0 / 21.5.  Otherwise timeslice ranges for one
  // FP32 or FP16 slot (2-6% faster) and for FP16 (12 slots, 24^3x48 and 32^3x64),
  // slabs for several FP32 slots (6%) and FP64 (one slot, both parities, 64x32^3
  // 744 / 850; 12 slots at 48x24^3 1716 / 1788).  DP_HOP_TMAP = 0 / 1 forces one of
  // them.
  static const int tmap_knob = env_knob("DP_HOP_TMAP", -1);
  const double most_slab = 8.0 * m.maxc / m.nch, most_range = 8.0 * m.tlen / a.g.T;
  if (tmap_knob == 0 || tmap_knob == 1) m.tmap = tmap_knob;
  else if (most_slab > 1.05 * most_range) m.tmap = 1;
  else if (most_range > 1.05 * most_slab) m.tmap = 0;
  else m.tmap = P != F64 && (a.nslots == 1 || P == F16) ? 1 : 0;
  const int nblocks = (m.tmap ? 8 * m.tlen * m.nch : 8 * a.g.T * m.maxc) * (EPI == site_epi(EPI) ? 1 : 2);
  *nparts_out = a.g.T * m.nch;
  constexpr bool full = EPI != site_epi(EPI);
  if (!one_wave_per_slot<P, full>(a.g.T * m.nch, a.nslots)) {
    constexpr bool inv = EPI == EPI_INV || EPI == EPI_INV_SUB, diag = site_epi(EPI) == EPI_DIAG;
    // The slots' common blocks in LDS, where there are such.  FP64 blocks fit
    // beside the links (110 KB) only with one workgroup per CU instead of two,
    // of six waves: worth it from so many slots on.  Even sites (C), 48x24^3 /
    // 16^3x32, us without and with: 4 slots 312 / 56.1 and 293 / 58.2, 5: 401 / 73.0
    // and 357 / 72.8, 8: 548 / 107.7 and 500 / 95.8, 12: 775 / 152.8 and 719 / 137.6.
    // Odd sites (A^-1) follow an even-site kernel that has them in LDS; a whole
    // solve, ms without and with: 48x24^3 8 columns 75.9 and 77.1, 10: 94.8 and
    // 95.7, 11: 103.4 and 103.6, 12: 110.1 and 109.4, 14: 126.3 and 124.4, 24: 211.7
    // and 205.9; 36x18x20x14 8: 19.85 and 20.57, 11: 26.7 and 26.8, 12: 28.6 and
    // 28.4, 24: 53.9 and 52.6; 16^3x32 8: 14.0 and 14.3, 12: 19.9 and 20.0, 18: 28.6
    // and 28.2, 24: 37.3 and 36.3.
    const bool blk = (diag || (inv && a.slots.ainv_common)) && (P != F64 || a.nslots >= (diag ? 5 : 12));
    // waves per workgroup: the fewest rounds over the slots
    const int maxw = shared_threads(P, blk) / 64, rounds = (a.nslots + maxw - 1) / maxw;
    const dim3 grid(nblocks), block(64 * ((a.nslots + rounds - 1) / rounds));
    bool done = false;
    if constexpr (inv || diag)
      if (blk) {
        hipLaunchKernelGGL((hop_kernel_shared<P, EPI, RED, DAG, true>), grid, block, shared_tile_bytes<P>(true), st, a, m);
        done = true;
      }
    if constexpr (!diag || P == F64)
      if (!done)
        hipLaunchKernelGGL((hop_kernel_shared<P, EPI, RED, DAG, false>), grid, block, shared_tile_bytes<P>(false), st, a, m);
  } else {
    const dim3 grid(nblocks * a.nslots);
    bool done = false;
    if constexpr (P == F64)
      if (fp64_two_waves((long)a.g.T * m.nch * a.nslots * (full ? 2 : 1), a.nslots)) {
        hipLaunchKernelGGL((hop_kernel_slab<P, EPI, RED, DAG, 2>), grid, dim3(64), 0, st, a, m);
        done = true;
      }
    if (!done) hipLaunchKernelGGL((hop_kernel_slab<P, EPI, RED, DAG, slab_min_waves(P)>), grid, dim3(64), 0, st, a, m);
  }
  return hipGetLastError();
}

template <int P, bool DAG>
hipError_t launch_epi(const HopArgs& a, hipStream_t st, int* np) {
  // fused reductions are only used with the even-site Schur epilogue
  if (a.red.red != RED_NONE && a.epi != EPI_DIAG) return hipErrorInvalidValue;
  switch (a.epi) {
    case EPI_HOP: return launch_one<P, EPI_HOP, RED_NONE, DAG>(a, st, np);
    case EPI_INV: return launch_one<P, EPI_INV, RED_NONE, DAG>(a, st, np);
    case EPI_SUB: return launch_one<P, EPI_SUB, RED_NONE, DAG>(a, st, np);
    case EPI_INV_SUB: return launch_one<P, EPI_INV_SUB, RED_NONE, DAG>(a, st, np);
    case EPI_FULL: return launch_one<P, EPI_FULL, RED_NONE, DAG>(a, st, np);
    case EPI_FULL_HOST:
      if constexpr (P == F64) return launch_one<P, EPI_FULL_HOST, RED_NONE, DAG>(a, st, np);
      else return hipErrorInvalidValue;
    case EPI_DIAG:
      switch (a.red.red) {
        case RED_NONE: return launch_one<P, EPI_DIAG, RED_NONE, DAG>(a, st, np);
        // the reductions with the shadow residual belong to BiCGStab, which
        // never applies the adjoint: those variants are not built
        case RED_DOT_EXT:
          if constexpr (DAG) return hipErrorInvalidValue;
          else return launch_one<P, EPI_DIAG, RED_DOT_EXT, DAG>(a, st, np);
        case RED_TS: return launch_one<P, EPI_DIAG, RED_TS, DAG>(a, st, np);
        case RED_NORM: return launch_one<P, EPI_DIAG, RED_NORM, DAG>(a, st, np);
        case RED_TS4:
          if constexpr (DAG) return hipErrorInvalidValue;
          else return launch_one<P, EPI_DIAG, RED_TS4, DAG>(a, st, np);
        default: return hipErrorInvalidValue;
      }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

}  // namespace dp
