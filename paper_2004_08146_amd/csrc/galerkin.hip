// Assembly of the Galerkin coarse operator D_c = P^H D P (Sec. 2): the self block and the
// 4 forward blocks of every coarse site, transposed (DcT[b][e][col][row], e = 0 self,
// 1 + mu the block at X + mu).
//
// Column c = (h, j) of P on block b is one chirality half, so D P e_c is read off P itself.
// Its part inside the block (diagonal and the hops that stay inside) is written for a batch
// of columns as spinor fields and restricted by the many-right-hand-side restriction.  The
// hop that leaves block X + mu into X has only the face's sites, and one half spinor there:
// its products with P_X^H (2 ntv x 6 face sites times 6 face sites x 16 columns, per
// direction) are formed on FP64 MFMA straight from P and the links.  Splitting D P into
// five whole spinor fields, as before, wrote and restricted four fields of which three
// quarters were zero, after a prolongation of unit vectors: at 32x16^3 with 24 vectors 7.9 ms,
// now 1.7 (self part 0.63, its restriction 0.47, faces 0.61).
#include "qmg_ctx.h"

namespace {

__device__ __forceinline__ int64_t pcol(const Geom& g, int ntv, int b, int h, int j, int d) {
  return ((((int64_t)b * 2 + h) * ntv + j) * 6 + d) << g.bs_log;
}

// (D inside the block) applied to columns of P in chirality half H; kCols columns share
// every link and clover load.
constexpr int kCols = 2;

template <int H, int MU, bool FWD>
__device__ __forceinline__ void part_hop(Spinor<double> (&q)[kCols], const cpx<double>* sh, const double2* U,
                                         const Geom& g, int b, int l, int bs) {
  const int lc = loc(g, l, MU), st = 1 << g.sh[MU];
  if (FWD ? lc == g.msk[MU] : lc == 0) return;
  const int ln = FWD ? l + st : l - st;
  const Link<double> u = load_link<double>(U, g, b, MU, FWD ? l : ln);
#pragma unroll
  for (int t = 0; t < kCols; ++t) {
    Spinor<double> p;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        p.s[s][c] = s / 2 == H ? sh[(t * 6 + 3 * (s & 1) + c) * bs + ln] : czero<double>();
    Half<double> w = project(p, MU, FWD);
    w = FWD ? umul(u, w) : udagmul(u, w);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) w.h[s][c] = -0.5 * w.h[s][c];
    accum_recon(q[t], w, MU, FWD);
  }
}

template <int H>
__device__ __forceinline__ void self_cols(double2* out, const double2* P, const double2* U, const double2* diag,
                                          const Geom& g, double mass4, int clover, int ntv, int b, int c0, int c,
                                          int ncol, cpx<double>* sh) {
  const int bs = 1 << g.bs_log;
  // not invariant over the columns: the links stay loads (held in registers they leave
  // one wave per SIMD)
  int l = threadIdx.x;
  asm volatile("" : "+v"(l));
  cpx<double> in[kCols][6];
#pragma unroll
  for (int t = 0; t < kCols; ++t)
#pragma unroll
    for (int d = 0; d < 6; ++d) {
      in[t][d] = t < ncol ? ldc(P, pcol(g, ntv, b, H, c + t - H * ntv, d) + l) : czero<double>();
      sh[(t * 6 + d) * bs + l] = in[t][d];
    }
  __syncthreads();
  Spinor<double> q[kCols];
#pragma unroll
  for (int t = 0; t < kCols; ++t)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int k = 0; k < 3; ++k) q[t].s[s][k] = czero<double>();
  part_hop<H, 0, true>(q, sh, U, g, b, l, bs);
  part_hop<H, 0, false>(q, sh, U, g, b, l, bs);
  part_hop<H, 1, true>(q, sh, U, g, b, l, bs);
  part_hop<H, 1, false>(q, sh, U, g, b, l, bs);
  part_hop<H, 2, true>(q, sh, U, g, b, l, bs);
  part_hop<H, 2, false>(q, sh, U, g, b, l, bs);
  part_hop<H, 3, true>(q, sh, U, g, b, l, bs);
  part_hop<H, 3, false>(q, sh, U, g, b, l, bs);
  if (clover) {
    cpx<double> w[kCols][6];
#pragma unroll
    for (int t = 0; t < kCols; ++t)
#pragma unroll
      for (int i = 0; i < 6; ++i) w[t][i] = q[t].s[2 * H + i / 3][i % 3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const cpx<double> d = ldc(diag, didx(g, b, H, k, l));
#pragma unroll
      for (int t = 0; t < kCols; ++t) {
        w[t][2 * k] = w[t][2 * k] + d.re * in[t][2 * k];
        w[t][2 * k + 1] = w[t][2 * k + 1] + d.im * in[t][2 * k + 1];
      }
    }
    int k = 3;
#pragma unroll
    for (int i = 1; i < 6; ++i)
#pragma unroll
      for (int j = 0; j < i; ++j) {
        const cpx<double> a = ldc(diag, didx(g, b, H, k, l));
        ++k;
#pragma unroll
        for (int t = 0; t < kCols; ++t) {
          cfma(w[t][i], a, in[t][j]);
          cfma_conj(w[t][j], a, in[t][i]);
        }
      }
#pragma unroll
    for (int t = 0; t < kCols; ++t)
#pragma unroll
      for (int i = 0; i < 6; ++i) q[t].s[2 * H + i / 3][i % 3] = w[t][i];
  } else {
#pragma unroll
    for (int t = 0; t < kCols; ++t)
#pragma unroll
      for (int i = 0; i < 6; ++i)
        q[t].s[2 * H + i / 3][i % 3] = q[t].s[2 * H + i / 3][i % 3] + mass4 * in[t][i];
  }
  const int64_t fs = g.V * 12;
#pragma unroll
  for (int t = 0; t < kCols; ++t)
    if (t < ncol) store_spinor(out + (c - c0 + t) * fs, g, b, l, q[t]);
  __syncthreads();  // sh is free
}

// blockIdx.x = block, blockIdx.y = share of the columns c0..c0+kb-1; bs threads
__global__ __launch_bounds__(256) void k_self_part(Geom g, double2* out, const double2* P, const double2* U,
                                                   const double2* diag, double mass4, int clover, int ntv, int c0,
                                                   int kb, int per) {
  extern __shared__ unsigned char smem_g[];
  cpx<double>* sh = reinterpret_cast<cpx<double>*>(smem_g);
  const int b = blockIdx.x;
  const int cbeg = c0 + blockIdx.y * per, cend = min(c0 + kb, cbeg + per);
  for (int c = cbeg; c < cend;) {
    // columns of one chirality at a time
    const int lim = c < ntv ? min(cend, ntv) : cend;
    const int n = min(kCols, lim - c);
    if (c < ntv) self_cols<0>(out, P, U, diag, g, mass4, clover, ntv, b, c0, c, n, sh);
    else self_cols<1>(out, P, U, diag, g, mass4, clover, ntv, b, c0, c, n, sh);
    c += n;
  }
}

// DcT[b][0][c0 + kk][i] = part[kk][b][i]
__global__ __launch_bounds__(256) void k_scatter_self(double2* DcT, const double2* part, int nb, int nc, int c0,
                                                      int64_t total) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int i = (int)(idx % nc);
  const int64_t t = idx / nc;
  const int b = (int)(t % nb), kk = (int)(t / nb);
  DcT[(((int64_t)b * 5) * nc + c0 + kk) * nc + i] = part[idx];
}

typedef double gd4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ gd4 gmfma(double a, double b, gd4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// site with face index j in the plane lc_mu = v of a block
__device__ __forceinline__ int face_site(const Geom& g, int mu, int j, int v) {
  const int lo = j & ((1 << g.sh[mu]) - 1);
  return ((j >> g.sh[mu]) * (g.msk[mu] + 1) + v) * (1 << g.sh[mu]) + lo;
}

// One work-group: block b, direction mu, all columns (NT tiles of 16), so that every entry of
// P_b is loaded once.  Four waves, one per (chirality of the row, tile of 16 rows).  The face
// is taken kFace sites at a time; wm[col][3 s + c][site] holds the rotated half spinors
// -1/2 U_mu(x) (1 - gamma_mu) P_{X + mu} e_col.
constexpr int kFace = 16, kW = 6 * kFace + 1;
template <int NT>
__global__ __launch_bounds__(256) void k_face_part(Geom g, double2* DcT, const double2* P, const double2* U, int ntv) {
  __shared__ cpx<double> wm[16 * NT * kW];
  const int b = blockIdx.x >> 2, mu = blockIdx.x & 3, nc = 2 * ntv;
  const int bf = g.nbr[b * 8 + 2 * mu];
  const int fs = (1 << g.bs_log) / (g.msk[mu] + 1);  // sites of the face
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, ln = lane & 15, lk = lane >> 4;
  const int hr = wave >> 1, row = 16 * (wave & 1) + ln;
  // row chirality 1 meets the half spinor through the lower spins of (1 - gamma_mu):
  // spin s' of w is spin sp[s'] of the result times ph[s']
  const int flip = mu == 1 || mu == 2;
  gd4 are[NT], aim[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    are[n] = gd4{0, 0, 0, 0};
    aim[n] = gd4{0, 0, 0, 0};
  }
#pragma unroll 1
  for (int f0 = 0; f0 < fs; f0 += kFace) {
    __syncthreads();
    // 16 columns a pass: a thread keeps its site, so the link is loaded once
    const int fsi = f0 + (int)(threadIdx.x % kFace);
    const bool fon = fsi < fs;
    const int s = threadIdx.x % kFace;
    const int lo0 = face_site(g, mu, fon ? fsi : 0, 0);
    const Link<double> u = load_link<double>(U, g, b, mu, face_site(g, mu, fon ? fsi : 0, g.msk[mu]));
#pragma unroll 1
    for (int cc = threadIdx.x / kFace; cc < 16 * NT; cc += 256 / kFace) {
      Half<double> w;
#pragma unroll
      for (int i = 0; i < 6; ++i) w.h[i / 3][i % 3] = czero<double>();
      if (cc < nc && fon) {
        const int h = cc >= ntv;
        Spinor<double> p;
#pragma unroll
        for (int d = 0; d < 6; ++d) {
          const cpx<double> v = ldc(P, pcol(g, ntv, bf, h, cc - h * ntv, d) + lo0);
          p.s[d / 3][d % 3] = h ? czero<double>() : v;
          p.s[2 + d / 3][d % 3] = h ? v : czero<double>();
        }
        switch (mu) {
          case 0: w = umul(u, project(p, 0, true)); break;
          case 1: w = umul(u, project(p, 1, true)); break;
          case 2: w = umul(u, project(p, 2, true)); break;
          default: w = umul(u, project(p, 3, true)); break;
        }
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) wm[cc * kW + i * kFace + s] = (-0.5) * w.h[i / 3][i % 3];
    }
    __syncthreads();
    // rows of P_b^H at the upper face's sites; four k-slots = four sites of one (spin, colour)
    int fsite[kFace / 4];
#pragma unroll
    for (int q = 0; q < kFace / 4; ++q) fsite[q] = face_site(g, mu, min(f0 + 4 * q + lk, fs - 1), g.msk[mu]);
    cpx<double> a[6][kFace / 4];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const int d = hr == 0 ? i : 3 * (flip ? 1 - i / 3 : i / 3) + i % 3;
#pragma unroll
      for (int q = 0; q < kFace / 4; ++q)
        a[i][q] = ldc(P, pcol(g, ntv, b, hr, min(row, ntv - 1), d) + fsite[q]);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const int sp = i / 3;
#pragma unroll
      for (int q = 0; q < kFace / 4; ++q) {
        // sites past the face meet zeros of wm, rows past ntv are not stored
        cpx<double> av = conj(a[i][q]);
        if (hr == 1) {
          // lower spins rebuilt from w: mu 0: (w0, w1); 1: (-i w1, -i w0); 2: (-w1, w0); 3: (-i w0, i w1)
          if (mu == 1) av = tmi(av);
          else if (mu == 2) av = sp == 1 ? -av : av;
          else if (mu == 3) av = sp == 0 ? tmi(av) : ti(av);
        }
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const cpx<double> bv = wm[(16 * n + ln) * kW + i * kFace + 4 * q + lk];
          are[n] = gmfma(av.re, bv.re, are[n]);
          are[n] = gmfma(-av.im, bv.im, are[n]);
          aim[n] = gmfma(av.re, bv.im, aim[n]);
          aim[n] = gmfma(av.im, bv.re, aim[n]);
        }
      }
    }
  }
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int col = 16 * n + ln;
    if (col < nc)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * (wave & 1) + 4 * r + lk;
        if (i < ntv) DcT[(((int64_t)b * 5 + 1 + mu) * nc + col) * nc + hr * ntv + i] = make_double2(are[n][r], aim[n][r]);
      }
  }
}

}  // namespace

hipError_t launch_self_part(const qmg_ctx* c, void* out, int c0, int kb, hipStream_t s) {
  const Geom& g = c->g;
  const int bs = 1 << g.bs_log;
  // enough work-groups to fill the chip a few times over; the fewer columns a work-group
  // has, the more often a block's links are read from beyond its CU
  int shares = 1;
  while (shares * 4 <= kb && (int64_t)g.nb * shares < 2048) shares *= 2;
  int per = (kb + shares - 1) / shares;
  per += per % kCols;
  hipLaunchKernelGGL(k_self_part, dim3(g.nb, (kb + per - 1) / per), dim3(bs), sizeof(cpx<double>) * 6 * kCols * bs, s,
                     g, (double2*)out, (const double2*)c->P[QMG_F64], (const double2*)c->U[QMG_F64],
                     (const double2*)c->Dg[QMG_F64], c->m0 + 4.0, c->clover ? 1 : 0, c->ntv, c0, kb, per);
  return hipGetLastError();
}

hipError_t launch_scatter_self(const qmg_ctx* c, const void* part, int c0, int kb, hipStream_t s) {
  const int nc = 2 * c->ntv;
  const int64_t total = (int64_t)kb * c->g.nb * nc;
  hipLaunchKernelGGL(k_scatter_self, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                     (double2*)c->Dc[QMG_F64], (const double2*)part, c->g.nb, nc, c0, total);
  return hipGetLastError();
}

hipError_t launch_face_part(const qmg_ctx* c, hipStream_t s) {
  auto go = [&](auto nt) {
    hipLaunchKernelGGL((k_face_part<decltype(nt)::value>), dim3(4u * c->g.nb), dim3(256), 0, s, c->g,
                       (double2*)c->Dc[QMG_F64], (const double2*)c->P[QMG_F64], (const double2*)c->U[QMG_F64], c->ntv);
  };
  switch ((2 * c->ntv + 15) / 16) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    default: go(std::integral_constant<int, 4>{}); break;
  }
  return hipGetLastError();
}
