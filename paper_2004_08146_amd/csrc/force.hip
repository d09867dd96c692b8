// Gauge-field derivative of L = phi^H Q x (Wilson hops of eq. (2.5)).
// L holds each link U_mu(y) linearly in the forward hop at y and conjugated in
// the backward hop at y + mu, so per link
//   G[y,mu]_{ab}    = -1/2 sum_s conj(phi(y)_{s,a})    (g5 (I - g_mu) x(y+mu))_{s,b}
//   Gbar[y,mu]_{ab} = -1/2 sum_s conj(phi(y+mu)_{s,b}) (g5 (I + g_mu) x(y))_{s,a}
// written in canonical order [site][mu][a][b] (complex128).
#include "qmg_ctx.h"

namespace {

// gamma5 (I -/+ gamma_mu) p
template <int MU, bool FWD>
__device__ __forceinline__ Spinor<double> spin_proj_full(const Spinor<double>& p) {
  const Half<double> h = project(p, MU, FWD);
  Spinor<double> o;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) o.s[s][c] = czero<double>();
  accum_recon(o, h, MU, FWD);
#pragma unroll
  for (int s = 2; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) o.s[s][c] = -o.s[s][c];
  return o;
}

// -1/2 sum_s conj(a_{s,i}) b_{s,j} (or its transpose) into row[3 i + j]
template <bool T>
__device__ __forceinline__ void outer(double2* row, const Spinor<double>& a, const Spinor<double>& b) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cpx<double> t = czero<double>();
#pragma unroll
      for (int s = 0; s < 4; ++s) t = t + cmul_conj(a.s[s][T ? j : i], b.s[s][T ? i : j]);
      row[3 * i + j] = make_double2(-0.5 * t.re, -0.5 * t.im);
    }
}

template <int MU>
__device__ __forceinline__ void link_force(double2* row, bool bar, const Geom& g, const double2* phi, const double2* x,
                                           int b, int l) {
  int bn, ln;
  nb_fwd(g, b, l, MU, bn, ln);
  if (!bar)
    outer<false>(row, load_spinor<double>(phi, g, b, l), spin_proj_full<MU, true>(load_spinor<double>(x, g, bn, ln)));
  else
    outer<true>(row, load_spinor<double>(phi, g, bn, ln), spin_proj_full<MU, false>(load_spinor<double>(x, g, b, l)));
}

// 64 sites in block order per work-group, wave = direction; each of G and Gbar is formed in
// LDS and written in runs of sites (a thread writing its link's nine entries put 16 B every
// 576: 99 -> 63 us at 32x16^3)
constexpr int kFTile = 64, kFRow = 37;
__global__ __launch_bounds__(256) void k_force(Geom g, double2* G, double2* Gb, const double2* phi, const double2* x) {
  __shared__ double2 sh[kFTile * kFRow];
  const int64_t s0 = (int64_t)blockIdx.x * kFTile;
  const int ns = (int)min((int64_t)kFTile, g.V - s0);
  const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = threadIdx.x & 63;
  const int b = (int)((s0 + i) >> g.bs_log), l = (int)((s0 + i) & ((1 << g.bs_log) - 1));
#pragma unroll 1
  for (int bar = 0; bar < 2; ++bar) {
    if (i < ns) {
      double2* row = sh + i * kFRow + 9 * mu;
      switch (mu) {
        case 0: link_force<0>(row, bar, g, phi, x, b, l); break;
        case 1: link_force<1>(row, bar, g, phi, x, b, l); break;
        case 2: link_force<2>(row, bar, g, phi, x, b, l); break;
        default: link_force<3>(row, bar, g, phi, x, b, l); break;
      }
    }
    __syncthreads();
    double2* out = bar ? Gb : G;
    for (int e = threadIdx.x; e < 36 * ns; e += 256) {
      const int t = e / 36, c = e - 36 * t;
      const int64_t site = s0 + t;
      out[canon_site(g, (int)(site >> g.bs_log), (int)(site & ((1 << g.bs_log) - 1))) * 36 + c] = sh[t * kFRow + c];
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_force(const qmg_ctx* c, double* dU, double* dUb, const void* phi, const void* x, hipStream_t s) {
  hipLaunchKernelGGL(k_force, dim3((unsigned)((c->g.V + kFTile - 1) / kFTile)), dim3(256), 0, s, c->g, (double2*)dU,
                     (double2*)dUb, (const double2*)phi, (const double2*)x);
  return hipGetLastError();
}
