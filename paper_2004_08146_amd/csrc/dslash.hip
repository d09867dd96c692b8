// Wilson(-clover) stencil, eq. (2.5):
//   (D psi)(x) = [(m0+4) + C(x)] psi(x) - 1/2 sum_mu (I - g_mu) U_mu(x) psi(x+mu)
//                                       - 1/2 sum_mu (I + g_mu) U_mu(x-mu)^H psi(x-mu)
// with the shift folded in: mode 0 gives (D - tau Gamma5) psi (eq. (3.7)),
// mode 1 gives (Gamma5 D - tau) psi = (Q - tau) psi (eq. (1.1)).
//
// One thread per site and right-hand side.  Work-groups are mapped to sites
// so that each XCD walks a contiguous slab of the block-major lattice and the
// right-hand sides of one site tile run back to back on the same XCD (their
// shared links then come from that XCD's L2).
#include "qmg_ctx.h"

namespace {

// SI: storage type of the input field (the output, links and clover use S); an
// FP64 apply may read a field stored in FP32 or BF16 with no change in its
// arithmetic, since every such value is exact in FP64.
template <typename S, typename SI = S>
struct DsArgs {
  typename PT<S>::stor* out;
  const typename PT<SI>::stor* in;
  const typename PT<S>::stor* U;
  const typename PT<S>::stor* diag;
  double mass4;
  int64_t fstride;  // complex elements per field
  int nrhs;
  int remap;
  const int* tord;  // block ids in work order
  int per, ngrp;    // k_dslash44l: right-hand sides per work-group, work-groups per block
  int nt_out;       // 1: the output is written with non-temporal stores (streamed past the caches)
  Geom g;
  double tau[QMG_MAXRHS];
};

// the values are formed here: left to itself the compiler defers a direction's sums to the
// end and keeps their terms in registers instead
template <typename C>
__device__ __forceinline__ void pin(Spinor<C>& p) {
#pragma unroll
  for (int i = 0; i < 12; ++i) asm volatile("" : "+v"(p.s[i / 3][i % 3].re), "+v"(p.s[i / 3][i % 3].im));
}

// N rows of 1 << lg elements from element `at` on
template <typename R, int N, typename P>
__device__ __forceinline__ void rows(cpx<R> (&v)[N], const P* f, int64_t at, int lg) {
  const P* q = f + at;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = ldcv<R>(q, (int64_t)i << lg);
}
template <typename R>
__device__ __forceinline__ Half<R> project_rows(const cpx<R> (&v)[12], int mu, bool fwd) {
  Spinor<R> p;
#pragma unroll
  for (int i = 0; i < 12; ++i) p.s[i / 3][i % 3] = v[i];
  return project(p, mu, fwd);
}
template <typename R>
__device__ __forceinline__ Link<R> link_rows(const cpx<R> (&v)[9]) {
  Link<R> u;
#pragma unroll
  for (int i = 0; i < 9; ++i) u.u[i / 3][i % 3] = v[i];
  return u;
}

// hop_pair below with the order of loads and sums left to the compiler
template <typename R, int MU, typename PI, typename P>
__device__ __forceinline__ void hop_pair_free(Spinor<R>& acc, const PI* in, const P* U, const Geom& g, int b, int l) {
  int bn, ln;
  nb_fwd(g, b, l, MU, bn, ln);
  {
    Half<R> h = project(load_spinor<R>(in, g, bn, ln), MU, true);
    accum_recon(acc, umul(load_link<R>(U, g, b, MU, l), h), MU, true);
  }
  nb_bwd(g, b, l, MU, bn, ln);
  {
    Half<R> h = project(load_spinor<R>(in, g, bn, ln), MU, false);
    accum_recon(acc, udagmul(load_link<R>(U, g, bn, MU, ln), h), MU, false);
  }
}

// acc += (I - g_mu) U_mu(x) psi(x+mu) + (I + g_mu) U_mu(x-mu)^H psi(x-mu)
template <typename R, int MU, typename PI, typename P>
__device__ __forceinline__ void hop_pair(Spinor<R>& acc, const PI* in, const P* U, const Geom& g, int b, int l) {
  const int lg = g.bs_log;
  int bn, ln;
  cpx<R> p[12], u[9], q[12], v[9];
  nb_fwd(g, b, l, MU, bn, ln);
  rows(p, in, (((int64_t)bn * 12) << lg) + ln, lg);
  rows(u, U, (((int64_t)b * 36 + 9 * MU) << lg) + l, lg);
  nb_bwd(g, b, l, MU, bn, ln);
  rows(q, in, (((int64_t)bn * 12) << lg) + ln, lg);
  rows(v, U, (((int64_t)bn * 36 + 9 * MU) << lg) + ln, lg);
  accum_recon(acc, umul(link_rows(u), project_rows(p, MU, true)), MU, true);
  accum_recon(acc, udagmul(link_rows(v), project_rows(q, MU, false)), MU, false);
  // FP64: two directions ahead
  if constexpr (sizeof(R) == 4 || MU % 2 == 1) pin(acc);
  if constexpr (sizeof(R) == 4) __builtin_amdgcn_sched_barrier(0);
}

// General blocks.  Bound by the loads of 8 neighbours, whose lines other work-groups share
// through the caches: what counts is how many are in flight.  FREE: the compiler orders loads
// and sums, loads nearly all first and takes 256-330 registers; else one direction (FP64: two)
// at a time, which leaves room for more waves.  The choice is made in launch_t.
template <typename S, bool CLOVER, int MODE, bool UB, typename SI, bool FREE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FREE || std::is_same<S, double>::value ? 1 : 2)))
void k_dslash(DsArgs<S, SI> a) {
  using R = typename PT<S>::real;
  const Geom& g = a.g;
  const int w = blockIdx.x, nw = gridDim.x;
  const int L = (a.remap && (nw & 7) == 0) ? (w & 7) * (nw >> 3) + (w >> 3) : w;
  const int k = L % a.nrhs;
  const int64_t site = (int64_t)(L / a.nrhs) * blockDim.x + threadIdx.x;
  if (site >= g.V) return;
  int b = (int)(site >> g.bs_log);
  if (UB) b = __builtin_amdgcn_readfirstlane(b);
  const int l = (int)(site & ((1 << g.bs_log) - 1));
  const auto* in = a.in + k * a.fstride;
  auto* out = a.out + k * a.fstride;

  Spinor<R> acc;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc.s[s][c] = czero<R>();

  if constexpr (FREE) {
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
      switch (mu) {
        case 0: hop_pair_free<R, 0>(acc, in, a.U, g, b, l); break;
        case 1: hop_pair_free<R, 1>(acc, in, a.U, g, b, l); break;
        case 2: hop_pair_free<R, 2>(acc, in, a.U, g, b, l); break;
        default: hop_pair_free<R, 3>(acc, in, a.U, g, b, l); break;
      }
    }
  } else {
    hop_pair<R, 0>(acc, in, a.U, g, b, l);
    hop_pair<R, 1>(acc, in, a.U, g, b, l);
    hop_pair<R, 2>(acc, in, a.U, g, b, l);
    hop_pair<R, 3>(acc, in, a.U, g, b, l);
  }
  const Spinor<R> self = load_spinor<R>(in, g, b, l);
  Spinor<R> o;
  if (CLOVER) {
    o = apply_diag<R>(a.diag, g, b, l, self);
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) o.s[s][c] = R(a.mass4) * self.s[s][c];
  }
  const R tau = R(a.tau[k]);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      cpx<R> v = o.s[s][c] - R(0.5) * acc.s[s][c];
      if (MODE == 0) {
        // D - tau Gamma5
        v = (s < 2) ? v - tau * self.s[s][c] : v + tau * self.s[s][c];
      } else {
        // Gamma5 D - tau
        v = (s < 2) ? v - tau * self.s[s][c] : -v - tau * self.s[s][c];
      }
      o.s[s][c] = v;
    }
  store_spinor(out, g, b, l, o);
}

// ---- 4^4 blocks: compile-time geometry, 32-bit offsets.
template <typename C, typename P>
__device__ __forceinline__ Spinor<C> ld_spinor44(const P* f, uint32_t b, uint32_t l) {
  Spinor<C> p;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      auto v = cv(ldo(f, ((b * 12u + (uint32_t)(3 * s + c)) << 8) + l));
      p.s[s][c] = cpx<C>{C(v.re), C(v.im)};
    }
  return p;
}
template <typename C, typename P>
__device__ __forceinline__ Link<C> ld_link44(const P* U, uint32_t b, int mu, uint32_t l) {
  Link<C> u;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      auto v = cv(ldo(U, ((b * 36u + (uint32_t)(mu * 9 + 3 * a + c)) << 8) + l));
      u.u[a][c] = cpx<C>{C(v.re), C(v.im)};
    }
  return u;
}

// The arithmetic that the two 4^4 kernels share, with every rounding written out: left to
// itself the compiler fuses one or the other product of a sum, another one in each kernel, and
// a column's last digits would depend on the batch by which the launch picks between them.
template <typename C>
__device__ __forceinline__ cpx<C> mul44(cpx<C> a, cpx<C> b) {
  return {fmar(a.re, b.re, -(a.im * b.im)), fmar(a.re, b.im, a.im * b.re)};
}
template <typename C>
__device__ __forceinline__ cpx<C> mul_conj44(cpx<C> a, cpx<C> b) {
  return {fmar(a.re, b.re, a.im * b.im), fmar(a.re, b.im, -(a.im * b.re))};
}
template <typename C>
__device__ __forceinline__ Half<C> umul44(const Link<C>& U, const Half<C>& h) {
  Half<C> o;
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cpx<C> t = mul44(U.u[a][0], h.h[s][0]);
      cfma(t, U.u[a][1], h.h[s][1]);
      cfma(t, U.u[a][2], h.h[s][2]);
      o.h[s][a] = t;
    }
  return o;
}
template <typename C>
__device__ __forceinline__ Half<C> udagmul44(const Link<C>& U, const Half<C>& h) {
  Half<C> o;
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cpx<C> t = mul_conj44(U.u[0][a], h.h[s][0]);
      cfma_conj(t, U.u[1][a], h.h[s][1]);
      cfma_conj(t, U.u[2][a], h.h[s][2]);
      o.h[s][a] = t;
    }
  return o;
}
// the sum of the two hops of direction MU from their colour-rotated half spinors: both
// kernels add a direction's two hops first, then the directions in order
template <typename C, int MU>
__device__ __forceinline__ Spinor<C> pair44(const Half<C>& f, const Half<C>& b) {
  Spinor<C> p;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    p.s[0][c] = f.h[0][c] + b.h[0][c];
    p.s[1][c] = f.h[1][c] + b.h[1][c];
    const cpx<C> d0 = f.h[0][c] - b.h[0][c], d1 = f.h[1][c] - b.h[1][c];
    if constexpr (MU == 0) p.s[2][c] = d0, p.s[3][c] = d1;
    else if constexpr (MU == 1) p.s[2][c] = tmi(d1), p.s[3][c] = tmi(d0);
    else if constexpr (MU == 2) p.s[2][c] = -d1, p.s[3][c] = d0;
    else p.s[2][c] = tmi(d0), p.s[3][c] = ti(d1);
  }
  return p;
}
// w = one Hermitian 6x6 block (ld(k): its k-th stored entry) times v.  The diagonal is fused
// with a row's first product; MUL: written as a product of its own, which the compiler fuses
// alike but orders the loads otherwise (64x32^3, 16 rhs, bf16 2.24 ms against 2.32 without;
// FP32 3.33 against 3.31, FP64 4 rhs 1.725 against 1.713)
template <typename C, bool MUL, typename F>
__device__ __forceinline__ void block44(cpx<C> (&w)[6], const cpx<C> (&v)[6], F&& ld) {
  C d[6];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const cpx<C> t = ld(k);
    d[2 * k] = t.re;
    d[2 * k + 1] = t.im;
    if constexpr (MUL) w[2 * k] = t.re * v[2 * k], w[2 * k + 1] = t.im * v[2 * k + 1];
  }
  int k = 3;
#pragma unroll
  for (int i = 1; i < 6; ++i)
#pragma unroll
    for (int j = 0; j < i; ++j) {
      const cpx<C> a = ld(k), p = mul44(a, v[j]), q = mul_conj44(a, v[i]);
      ++k;
      w[i] = !MUL && j == 0 ? cpx<C>{fmar(d[i], v[i].re, p.re), fmar(d[i], v[i].im, p.im)} : w[i] + p;
      w[j] = !MUL && i == 1 ? cpx<C>{fmar(d[j], v[j].re, q.re), fmar(d[j], v[j].im, q.im)} : w[j] + q;
    }
}
// (D - tau Gamma5) psi (MODE 0) or (Gamma5 D - tau) psi at one entry of chirality H: o the
// clover part, hops the sum of the hops (half of it is exact)
template <typename C, bool CLOVER, int MODE, int H>
__device__ __forceinline__ cpx<C> tail44(cpx<C> o, C mass4, cpx<C> hops, cpx<C> psi, C tau) {
  const cpx<C> v = CLOVER ? cpx<C>{fmar(C(-0.5), hops.re, o.re), fmar(C(-0.5), hops.im, o.im)}
                          : cpx<C>{fmar(mass4, psi.re, C(-0.5) * hops.re), fmar(mass4, psi.im, C(-0.5) * hops.im)};
  if (H == 0) return {fmar(-tau, psi.re, v.re), fmar(-tau, psi.im, v.im)};
  if (MODE == 0) return {fmar(tau, psi.re, v.re), fmar(tau, psi.im, v.im)};
  return {fmar(-tau, psi.re, -v.re), fmar(-tau, psi.im, -v.im)};
}

// (m0 + 4 + C) psi with the two Hermitian 6x6 blocks of (b, l)
template <typename C, typename P>
__device__ __forceinline__ Spinor<C> diag44(const P* D, uint32_t b, uint32_t l, const Spinor<C>& p) {
  Spinor<C> o;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    cpx<C> v[6], w[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = p.s[2 * h + i / 3][i % 3];
    block44<C, std::is_same<P, uint32_t>::value>(w, v, [&](int k) {
      const auto d = cv(ldo(D, ((b * 36u + (uint32_t)(18 * h + k)) << 8) + l));
      return cpx<C>{C(d.re), C(d.im)};
    });
#pragma unroll
    for (int i = 0; i < 6; ++i) o.s[2 * h + i / 3][i % 3] = w[i];
  }
  return o;
}

// ---- 4^4 blocks, each link loaded once per right-hand side.  A work-group is a block; for one direction at a
// time every site writes to LDS the two half spinors its neighbours need, (1 - gamma) psi
// for the site behind it and U^H (1 + gamma) psi for the site before it, and reads its own
// two.  A site on a face has no reader inside the block for one of them; its place is taken
// by the one that enters from the neighbour block across the same face, so that the reads
// wrap around inside the block.  Wave w forms those of direction w, one lane per face site,
// from the neighbours' spinors before the first direction.  One thread per site gathering
// its 8 neighbours and links, as before, asked L2 for 2.3 KB per site and right-hand side
// in FP32 (here 1.0 KB, 0.7 without the clover term), which is what bounded it; this is
// bound by the lines of the faces and by HBM.  64x32^3 with clover, against the best of
// eleven gathering variants: FP64 1 rhs 0.754 -> 0.670 ms, 16 rhs 8.68 -> 6.22; FP32 1 rhs
// 0.403 -> 0.349, 16 rhs 4.94 -> 3.21; BF16 16 rhs 3.10 -> 2.25.
constexpr int kL44Sh[4] = {6, 4, 2, 0};
template <int MU>
__device__ __forceinline__ uint32_t l44_site(uint32_t j, uint32_t v) {
  if constexpr (MU == 0) return (v << 6) | j;
  else if constexpr (MU == 1) return ((j >> 4) << 6) | (v << 4) | (j & 15u);
  else if constexpr (MU == 2) return ((j >> 2) << 4) | (v << 2) | (j & 3u);
  else return (j << 2) | v;
}

template <typename C, int MU, typename P>
__device__ __forceinline__ void l44_face_link(Link<C>& u, const P* U, const int* nbr, uint32_t b, uint32_t j) {
  u = ld_link44<C>(U, (uint32_t)nbr[b * 8 + 2 * MU + 1], MU, l44_site<MU>(j, 3));
}
// half spinors that enter the block across direction MU at face site j
template <typename C, int MU, typename PI>
__device__ __forceinline__ void l44_face(Half<C>& fh, Half<C>& fw, const PI* in, const Link<C>& u, const int* nbr,
                                         uint32_t b, uint32_t j) {
  const Spinor<C> pf = ld_spinor44<C>(in, (uint32_t)nbr[b * 8 + 2 * MU], l44_site<MU>(j, 0));
  const Spinor<C> pb = ld_spinor44<C>(in, (uint32_t)nbr[b * 8 + 2 * MU + 1], l44_site<MU>(j, 3));
  fh = project(pf, MU, true);
  fw = udagmul44(u, project(pb, MU, false));
}

template <typename C, int MU, bool TWO>
__device__ __forceinline__ void l44_dir(Spinor<C>& acc, const Spinor<C>& psi, const Link<C>& u, const Half<C>& fh,
                                        const Half<C>& fw, cpx<C>* hb, cpx<C>* wb, uint32_t wave, uint32_t lane,
                                        uint32_t l) {
  constexpr int SH = kL44Sh[MU];
  const uint32_t lc = (l >> SH) & 3u;
  if (!TWO) __syncthreads();  // the buffers of the direction before are read
  if (lc != 0u) {
    const Half<C> h = project(psi, MU, true);
#pragma unroll
    for (int i = 0; i < 6; ++i) hb[i * 256 + l] = h.h[i / 3][i % 3];
  }
  {
    const Half<C> w = udagmul44(u, project(psi, MU, false));
    if (lc != 3u)
#pragma unroll
      for (int i = 0; i < 6; ++i) wb[i * 256 + l] = w.h[i / 3][i % 3];
  }
  if (wave == MU) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      hb[i * 256 + l44_site<MU>(lane, 0)] = fh.h[i / 3][i % 3];
      wb[i * 256 + l44_site<MU>(lane, 3)] = fw.h[i / 3][i % 3];
    }
  }
  __syncthreads();
  const uint32_t lf = lc == 3u ? l - (3u << SH) : l + (1u << SH), lb = lc == 0u ? l + (3u << SH) : l - (1u << SH);
  Half<C> h, w;
#pragma unroll
  for (int i = 0; i < 6; ++i) h.h[i / 3][i % 3] = hb[i * 256 + lf];
  h = umul44(u, h);
#pragma unroll
  for (int i = 0; i < 6; ++i) w.h[i / 3][i % 3] = wb[i * 256 + lb];
  const Spinor<C> p = pair44<C, MU>(h, w);
  if constexpr (MU == 0) {
    acc = p;
  } else {
#pragma unroll
    for (int i = 0; i < 12; ++i) acc.s[i / 3][i % 3] = acc.s[i / 3][i % 3] + p.s[i / 3][i % 3];
  }
  pin(acc);
}

// HOLD: the links stay in registers over the work-group's right-hand sides
template <typename S, bool CLOVER, int MODE, typename SI, bool HOLD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_dslash44l(DsArgs<S, SI> a) {
  using C = typename PT<S>::real;
  using P = typename PT<S>::stor;
  using PI = typename PT<SI>::stor;
  constexpr bool TWO = !std::is_same<C, double>::value;  // two buffers: one barrier per direction
  __shared__ cpx<C> buf[(TWO ? 4 : 2) * 6 * 256];
  const int w = blockIdx.x, nw = gridDim.x;
  const int L = (a.remap && (nw & 7) == 0) ? (w & 7) * (nw >> 3) + (w >> 3) : w;
  const int grp = L % a.ngrp;
  const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane(a.tord[L / a.ngrp]);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t l = threadIdx.x;
  const int* nbr = a.g.nbr;
  Link<C> u[HOLD ? 4 : 1], uf;
  auto face_link = [&](uint32_t j) {
    if (wave == 0) l44_face_link<C, 0>(uf, a.U, nbr, b, j);
    else if (wave == 1) l44_face_link<C, 1>(uf, a.U, nbr, b, j);
    else if (wave == 2) l44_face_link<C, 2>(uf, a.U, nbr, b, j);
    else l44_face_link<C, 3>(uf, a.U, nbr, b, j);
  };
  if constexpr (HOLD) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) u[mu] = ld_link44<C>(a.U, b, mu, l);
    face_link(l & 63u);
  }
  const int kend = min(a.nrhs, (grp + 1) * a.per);
#pragma unroll 1
  for (int k = grp * a.per; k < kend; ++k) {
    asm volatile("" : "+v"(l));  // addresses are formed anew, not kept in registers
    const uint32_t lane = l & 63u;
    const PI* in = a.in + (size_t)k * a.fstride;
    const Spinor<C> psi = ld_spinor44<C>(in, b, l);
    Half<C> fh, fw;
    if constexpr (!HOLD) face_link(lane);
    if (wave == 0) l44_face<C, 0>(fh, fw, in, uf, nbr, b, lane);
    else if (wave == 1) l44_face<C, 1>(fh, fw, in, uf, nbr, b, lane);
    else if (wave == 2) l44_face<C, 2>(fh, fw, in, uf, nbr, b, lane);
    else l44_face<C, 3>(fh, fw, in, uf, nbr, b, lane);
    Spinor<C> acc;
    cpx<C>*h0 = buf, *w0 = buf + 6 * 256, *h1 = TWO ? buf + 12 * 256 : h0, *w1 = TWO ? buf + 18 * 256 : w0;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" : "+v"(l));
      if constexpr (!HOLD) u[0] = ld_link44<C>(a.U, b, mu, l);
      switch (mu) {
        case 0: l44_dir<C, 0, TWO>(acc, psi, u[0], fh, fw, h0, w0, wave, lane, l); break;
        case 1: l44_dir<C, 1, TWO>(acc, psi, u[HOLD ? 1 : 0], fh, fw, h1, w1, wave, lane, l); break;
        case 2: l44_dir<C, 2, TWO>(acc, psi, u[HOLD ? 2 : 0], fh, fw, h0, w0, wave, lane, l); break;
        default: l44_dir<C, 3, TWO>(acc, psi, u[HOLD ? 3 : 0], fh, fw, h1, w1, wave, lane, l); break;
      }
    }
    Spinor<C> o;
    if constexpr (CLOVER) o = diag44<C>(a.diag, b, l, psi);
    const C tau = C(a.tau[k]), mass4 = C(a.mass4);
    P* out = a.out + (size_t)k * a.fstride;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        o.s[s][c] = s < 2 ? tail44<C, CLOVER, MODE, 0>(o.s[s][c], mass4, acc.s[s][c], psi.s[s][c], tau)
                          : tail44<C, CLOVER, MODE, 1>(o.s[s][c], mass4, acc.s[s][c], psi.s[s][c], tau);
    if (a.nt_out) {
#pragma unroll
      for (int i = 0; i < 12; ++i) sto_nt(out, ((b * 12u + (uint32_t)i) << 8) + l, vc(o.s[i / 3][i % 3], (P*)nullptr));
    } else {
#pragma unroll
      for (int i = 0; i < 12; ++i) sto(out, ((b * 12u + (uint32_t)i) << 8) + l, vc(o.s[i / 3][i % 3], (P*)nullptr));
    }
    if (TWO && k + 1 < kend) __syncthreads();  // the last direction's reads are done
  }
}

// ---- 4^4 blocks, few of them: a work-group is a quarter of a block (64 sites), wave w
// takes the two hops of direction w, so that a site's 8 hops are one round of loads instead
// of a chain of them, and there are four times as many work-groups.
template <typename C, int MU, typename PI, typename P>
__device__ __forceinline__ Spinor<C> s44_pair(const PI* in, const P* U, const int* nbr, uint32_t b, uint32_t l) {
  constexpr int SH = kL44Sh[MU];
  const uint32_t lc = (l >> SH) & 3u;
  const uint32_t bf = lc == 3u ? (uint32_t)nbr[b * 8 + 2 * MU] : b, bb = lc == 0u ? (uint32_t)nbr[b * 8 + 2 * MU + 1] : b;
  const uint32_t lf = lc == 3u ? l - (3u << SH) : l + (1u << SH), lb = lc == 0u ? l + (3u << SH) : l - (1u << SH);
  const Spinor<C> pf = ld_spinor44<C>(in, bf, lf), pb = ld_spinor44<C>(in, bb, lb);
  const Link<C> uf = ld_link44<C>(U, b, MU, l), ub = ld_link44<C>(U, bb, MU, lb);
  return pair44<C, MU>(umul44(uf, project(pf, MU, true)), udagmul44(ub, project(pb, MU, false)));
}

template <typename S, bool CLOVER, int MODE, typename SI>
__global__ __launch_bounds__(256) void k_dslash44s(DsArgs<S, SI> a) {
  using C = typename PT<S>::real;
  using P = typename PT<S>::stor;
  __shared__ cpx<C> part[4][12][64];
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const uint32_t l = ((blockIdx.x & 3u) << 6) | lane, i = blockIdx.x >> 2;
  const uint32_t b = i / (uint32_t)a.nrhs, k = i - b * (uint32_t)a.nrhs;
  const typename PT<SI>::stor* in = a.in + (size_t)k * a.fstride;
  // waves 0 and 1 finish one chirality each; their site's terms arrive with the neighbours
  cpx<C> v[6], dg[18];
  if (wave < 2) {
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const auto t = cv(ldo(in, ((b * 12u + 6u * wave + (uint32_t)c) << 8) + l));
      v[c] = cpx<C>{C(t.re), C(t.im)};
    }
    if (CLOVER)
#pragma unroll
      for (int c = 0; c < 18; ++c) {
        const auto t = cv(ldo(a.diag, ((b * 36u + 18u * wave + (uint32_t)c) << 8) + l));
        dg[c] = cpx<C>{C(t.re), C(t.im)};
      }
  }
  Spinor<C> acc;
  if (wave == 0) acc = s44_pair<C, 0>(in, a.U, a.g.nbr, b, l);
  else if (wave == 1) acc = s44_pair<C, 1>(in, a.U, a.g.nbr, b, l);
  else if (wave == 2) acc = s44_pair<C, 2>(in, a.U, a.g.nbr, b, l);
  else acc = s44_pair<C, 3>(in, a.U, a.g.nbr, b, l);
#pragma unroll
  for (int c = 0; c < 12; ++c) part[wave][c][lane] = acc.s[c / 3][c % 3];
  __syncthreads();
  const C tau = C(a.tau[k]), mass4 = C(a.mass4);
  typename PT<S>::stor* out = a.out + (size_t)k * a.fstride;
  auto finish = [&](auto hc) {
    constexpr int H = decltype(hc)::value;
    cpx<C> w[6];
    if constexpr (CLOVER) block44<C, std::is_same<P, uint32_t>::value>(w, v, [&](int q) { return dg[q]; });
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const int at = 6 * H + c;
      const cpx<C> hops = ((part[0][at][lane] + part[1][at][lane]) + part[2][at][lane]) + part[3][at][lane];
      const cpx<C> r = tail44<C, CLOVER, MODE, H>(w[c], mass4, hops, v[c], tau);
      sto(out, ((b * 12u + (uint32_t)at) << 8) + l, vc(r, (P*)nullptr));
    }
  };
  if (wave == 0) finish(std::integral_constant<int, 0>{});
  else if (wave == 1) finish(std::integral_constant<int, 1>{});
}

template <typename S, bool CLOVER, int MODE, bool HOLD, typename SI>
void launch44l(DsArgs<S, SI> a, int nb, int per, int nt, hipStream_t s) {
  a.per = per;
  a.ngrp = (a.nrhs + per - 1) / per;
  a.nt_out = nt;
  hipLaunchKernelGGL((k_dslash44l<S, CLOVER, MODE, SI, HOLD>), dim3((unsigned)(nb * a.ngrp)), dim3(256), 0, s, a);
}

template <typename S, bool CLOVER, int MODE, typename SI = S>
void launch_t(const qmg_ctx* c, void* out, const void* in, const double* tau, int nrhs, hipStream_t s,
              int p) {
  using P = typename PT<S>::stor;
  DsArgs<S, SI> a;
  a.out = (P*)out;
  a.in = (const typename PT<SI>::stor*)in;
  a.U = (const P*)c->U[p];
  a.diag = (const P*)c->Dg[p];
  a.mass4 = c->m0 + 4.0;
  a.fstride = (int64_t)field_elems(c);
  a.nrhs = nrhs;
  a.remap = c->tune.dslash_xcd_remap;
  a.tord = c->d_tord;
  a.per = a.ngrp = 1;
  a.nt_out = 0;
  a.g = c->g;
  for (int i = 0; i < QMG_MAXRHS; ++i) a.tau[i] = i < nrhs ? tau[i] : 0.0;
  const int var = c->tune.force_variant >= 0 ? c->tune.force_variant : c->tune.dslash[p][nrhs == 1 ? 0 : 1];
  if (fits44(c, p) && var > 0) {
    // few blocks: the chain of loads of one thread per site is what a launch takes, so
    // four (1 rhs, FP64: 8^4 11.3 -> 5.1 us, 16x16x8x8 12.3 -> 6.7; at 16^4 30 against 22;
    // 8^4 with 16 rhs, FP32: 12.4 -> 10.7, FP64: 20 against 17)
    constexpr int kFew = std::is_same<S, double>::value ? 128 : 256;
    if ((int64_t)c->g.nb * nrhs <= kFew) {
      hipLaunchKernelGGL((k_dslash44s<S, CLOVER, MODE, SI>), dim3(4u * c->g.nb * nrhs), dim3(256), 0, s, a);
      return;
    }
    // an output that half fills the 256 MB Infinity Cache goes past it, and leaves it to the
    // inputs (64x32^3, FP64: 1 rhs 0.705 -> 0.670 ms, 16 rhs 6.55 -> 6.22); a smaller one
    // may still be there when it is read next
    const int nt = (size_t)nrhs * field_elems(c) * cbytes(p) > ((size_t)128 << 20);
    // FP32: links held over several right-hand sides (64x32^3, 16 rhs 3.82 -> 3.21 ms; BF16
    // 2.25 against 2.34; FP64 has no registers for them), as few groups of them as fill the
    // chip: the split with the fewest passes of (links + right-hand sides) over the 512
    // work-groups that run at a time
    if constexpr (std::is_same<S, float>::value) {
      if (nrhs > 1 || c->g.nb > 512) {  // 1 rhs at 16^4: 14.6 us against 14.2
        int per = 1;
        int64_t cost = -1;
        for (int g = 1; g <= nrhs; ++g) {
          const int pg = (nrhs + g - 1) / g;
          const int64_t t = (((int64_t)c->g.nb * g + 511) / 512) * (pg + 1);
          if (cost < 0 || t < cost) { cost = t; per = pg; }
        }
        launch44l<S, CLOVER, MODE, true>(a, c->g.nb, per, nt, s);
        return;
      }
    }
    launch44l<S, CLOVER, MODE, false>(a, c->g.nb, 1, nt, s);
    return;
  }
  const int wg = 256;
  unsigned nwg = (unsigned)((c->g.V + wg - 1) / wg) * (unsigned)nrhs;
  auto go = [&](auto ub, auto free) {
    hipLaunchKernelGGL((k_dslash<S, CLOVER, MODE, decltype(ub)::value, SI, decltype(free)::value>), dim3(nwg), dim3(wg),
                       0, s, a);
  };
  // FREE (all loads early, one or two waves per SIMD) against the fixed order (more waves, less
  // in flight in each): it is the better one where the links are not read again for further
  // right-hand sides or there are too few waves anyway, and where the block, and so every
  // address, is uniform.  FP32, blocks 4x4x4x2: 32x32x16x16, 1 rhs 56.7 against 61.0 us, 3 rhs
  // 162 / 124; 16x8^3, 4 rhs 11.6 / 12.0; 16^4, 2 rhs 26.9 / 21.6, 12 rhs 145 / 108.  Blocks
  // 8x4x4x2, 32x32x16x16, 3 rhs: FP32 121 / 130, FP64 241 / 277, bf16 73 / 60 (1 rhs, 32^3x16:
  // 55.5 / 60.2).  Blocks 4x4x4x2, 16^4, 12 rhs: FP64 228 / 211, bf16 169 / 59; 1 rhs 32x16^3:
  // FP64 59.1 / 57.8, bf16 31.8 / 16.7.
  constexpr bool kF32 = std::is_same<S, float>::value, kBf16 = std::is_same<S, bf16_t>::value;
  if ((1 << c->g.bs_log) >= wg) {
    if constexpr (kBf16)
      if (nrhs > 1) return go(std::true_type{}, std::false_type{});
    go(std::true_type{}, std::true_type{});
  } else {
    if constexpr (kF32)
      if (nrhs == 1 || nwg <= 256) return go(std::false_type{}, std::true_type{});
    go(std::false_type{}, std::false_type{});
  }
}

template <typename S>
void launch_p(const qmg_ctx* c, void* out, const void* in, const double* tau, int nrhs, int mode,
              hipStream_t s, int p) {
  if (c->clover) {
    if (mode == 0) launch_t<S, true, 0>(c, out, in, tau, nrhs, s, p);
    else launch_t<S, true, 1>(c, out, in, tau, nrhs, s, p);
  } else {
    if (mode == 0) launch_t<S, false, 0>(c, out, in, tau, nrhs, s, p);
    else launch_t<S, false, 1>(c, out, in, tau, nrhs, s, p);
  }
}

}  // namespace

hipError_t launch_dslash(const qmg_ctx* c, int p, void* out, const void* in, const double* tau, int nrhs,
                         int mode, hipStream_t s) {
  if (p == QMG_F64) launch_p<double>(c, out, in, tau, nrhs, mode, s, p);
  else if (p == QMG_F32) launch_p<float>(c, out, in, tau, nrhs, mode, s, p);
  else launch_p<bf16_t>(c, out, in, tau, nrhs, mode, s, p);
  return hipGetLastError();
}

hipError_t launch_dslash_d_in(const qmg_ctx* c, void* out, const void* in, int in_prec, const double* tau,
                              int nrhs, hipStream_t s, int mode) {
  if (in_prec == QMG_F64) return launch_dslash(c, QMG_F64, out, in, tau, nrhs, mode, s);
  auto go = [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    if (c->clover) {
      if (in_prec == QMG_F32) launch_t<double, true, M, float>(c, out, in, tau, nrhs, s, QMG_F64);
      else launch_t<double, true, M, bf16_t>(c, out, in, tau, nrhs, s, QMG_F64);
    } else {
      if (in_prec == QMG_F32) launch_t<double, false, M, float>(c, out, in, tau, nrhs, s, QMG_F64);
      else launch_t<double, false, M, bf16_t>(c, out, in, tau, nrhs, s, QMG_F64);
    }
  };
  if (mode == 0) go(std::integral_constant<int, 0>{});
  else go(std::integral_constant<int, 1>{});
  return hipGetLastError();
}
