// Interpolation P from test vectors, restriction y = P^H v and prolongation
// v = P y (Sec. 2: aggregation-based P, R = P^H; Sec. 3.1 on building P).
//
// Aggregates are (lattice block) x (chirality half): spins {0,1} and {2,3},
// so Gamma5 P = P Gamma5^c (text before eq. (2.9)).  P is stored complex
// [nb][2][ntv][6][bs]: column j of aggregate (b, h), entry (spin-in-half,
// colour) d at site l.  Coarse vectors are [nrhs][nb][2*ntv], index h*ntv + j.
// Columns of each aggregate are orthonormalised in column order by modified
// Gram-Schmidt in two rounds over panels of columns.
#include "qmg_ctx.h"
#include "reduce.h"
#include <type_traits>

namespace {

QMG_HD int64_t pidx(const Geom& g, int ntv, int b, int h, int j, int d, int l) {
  return ((((int64_t)b * 2 + h) * ntv + j) * 6 + d) * ((int64_t)1 << g.bs_log) + l;
}

// sums of v[0..NV) over the work-group (whole waves), the same in every thread.  red is
// double buffered by the caller, so one barrier: a half is rewritten after the next sum's
template <int NV>
__device__ __forceinline__ void panel_sum(double (&v)[NV], double* red) {
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  wave_fold<NV>(v, red + wave * NV);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double t = red[i];
    for (int w = 1; w < nw; ++w) t += red[w * NV + i];
    v[i] = t;
  }
}

// One work-group per aggregate (b, h), one thread per site.  Panels of kPanel columns are
// held in registers and orthonormalised in two rounds, each against the columns of the
// earlier panels (read once per round, all columns of the panel against one of them at a
// time) and then among themselves: a column is normalised and at once taken out of those
// after it.  Taken out of a column all together (classical) they left P's columns overlapping where
// six vectors agree to 1e-10 or better (P^H P y off by 4e-7, at 1e-11 by 2.5e-3), since the second
// round begins when all columns of the panel had the first.  Column by column, as before, every earlier column was read four times per
// column from L2: 4.07 ms at 512 blocks of 256 sites and 24 columns, now 0.85 ms, of which
// reading W, writing P in its three storage types and the 72 re-reads of 24 columns take
// about 0.6 at the copy rate.
constexpr int kPanel = 6;
constexpr int kPanelRed = 2 * 4 * 2 * kPanel;  // two halves, up to four waves
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_build_P(Geom g, double2* P, float2* P32, uint32_t* P16, const double2* W,
                                                 int ntv, int* fail) {
  __shared__ double red[kPanelRed];
  __shared__ double norm[kPanel][2];  // of the panel's columns: squared before, left after the rounds so far
  int rb = 0;
  auto half = [&]() {
    double* r = red + rb * (kPanelRed / 2);
    rb ^= 1;
    return r;
  };
  const int b = blockIdx.x >> 1, h = blockIdx.x & 1, l = threadIdx.x;
  const bool on = l < (1 << g.bs_log);  // blocks of fewer than 64 sites leave lanes idle
  const int64_t fs = g.V * 12;
  for (int j0 = 0; j0 < ntv; j0 += kPanel) {
    const int np = ntv - j0 < kPanel ? ntv - j0 : kPanel;
    cpx<double> v[kPanel][6];
    double n0[kPanel];
#pragma unroll
    for (int k = 0; k < kPanel; ++k) {
      n0[k] = 0.0;
#pragma unroll
      for (int d = 0; d < 6; ++d) {
        v[k][d] = on && k < np ? ldc(W + (j0 + k) * fs, sidx(g, b, 6 * h + d, l)) : czero<double>();
        n0[k] += norm2(v[k][d]);
      }
    }
    panel_sum<kPanel>(n0, half());
    if (l == 0)
#pragma unroll
      for (int k = 0; k < kPanel; ++k) {
        norm[k][0] = n0[k];
        norm[k][1] = 1.0;
      }
#pragma unroll 1
    for (int round = 0; round < 2; ++round) {
      cpx<double> p[6];
      auto load = [&](int i) {
#pragma unroll
        for (int d = 0; d < 6; ++d) p[d] = on ? ldc(P, pidx(g, ntv, b, h, i, d, l)) : czero<double>();
      };
      if (j0 > 0) load(0);
#pragma unroll 1
      for (int i = 0; i < j0; ++i) {
        double cf[2 * kPanel];
#pragma unroll
        for (int k = 0; k < kPanel; ++k) {
          cpx<double> a = czero<double>();
#pragma unroll
          for (int d = 0; d < 6; ++d) cfma_conj(a, p[d], v[k][d]);
          cf[2 * k] = a.re;
          cf[2 * k + 1] = a.im;
        }
        cpx<double> pc[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) pc[d] = p[d];
        if (i + 1 < j0) load(i + 1);  // arrives during the sums
        panel_sum<2 * kPanel>(cf, half());
#pragma unroll
        for (int k = 0; k < kPanel; ++k) {
          const cpx<double> c = {-cf[2 * k], -cf[2 * k + 1]};
#pragma unroll
          for (int d = 0; d < 6; ++d) cfma(v[k][d], c, pc[d]);
        }
      }
      auto column = [&](auto kc) {
        constexpr int k = decltype(kc)::value, M = kPanel - 1 - k;
        double n1[1] = {0.0};
#pragma unroll
        for (int d = 0; d < 6; ++d) n1[0] += norm2(v[k][d]);
        panel_sum<1>(n1, half());
        // nn: what is left of the column's norm over both rounds
        const double r = sqrt(n1[0]), nn = norm[k][1] * r;
        const bool bad = k < np && !(nn >= 1e-12 * sqrt(norm[k][0]));
        __syncthreads();
        if (l == 0) {
          norm[k][1] = nn;
          if (bad) fail[0] = 1;
        }
        const double inv = bad || k >= np ? 1.0 : 1.0 / r;
#pragma unroll
        for (int d = 0; d < 6; ++d) v[k][d] = inv * v[k][d];
        if constexpr (M > 0) {
          double cf[2 * M];
#pragma unroll
          for (int i = 0; i < M; ++i) {
            cpx<double> a = czero<double>();
#pragma unroll
            for (int d = 0; d < 6; ++d) cfma_conj(a, v[k][d], v[k + 1 + i][d]);
            cf[2 * i] = a.re;
            cf[2 * i + 1] = a.im;
          }
          panel_sum<2 * M>(cf, half());
#pragma unroll
          for (int i = 0; i < M; ++i) {
            const cpx<double> c = {-cf[2 * i], -cf[2 * i + 1]};
#pragma unroll
            for (int d = 0; d < 6; ++d) cfma(v[k + 1 + i][d], c, v[k][d]);
          }
        }
      };
      column(std::integral_constant<int, 0>{});
      column(std::integral_constant<int, 1>{});
      column(std::integral_constant<int, 2>{});
      column(std::integral_constant<int, 3>{});
      column(std::integral_constant<int, 4>{});
      column(std::integral_constant<int, 5>{});
    }
    if (on) {
#pragma unroll
      for (int k = 0; k < kPanel; ++k)
        if (k < np)
#pragma unroll
          for (int d = 0; d < 6; ++d) {
            const int64_t o = pidx(g, ntv, b, h, j0 + k, d, l);
            stc(P, o, v[k][d]);
            const cpx<float> f = {float(v[k][d].re), float(v[k][d].im)};
            stc(P32, o, f);
            stc(P16, o, f);
          }
    }
  }
}

// y[k][b][o] = sum_{l,d} conj(P[b][h][j][d][l]) v[k][b][6h+d][l], o = h*ntv + j, for few
// right-hand sides or small blocks: one work-group per (block, chirality, NR right-hand
// sides), one thread per site, four columns of P in flight at a time, shared by the
// right-hand sides; the sums over the sites run in FP64.  With the columns summed eight at a
// time by shuffles and both chiralities in turn, 256 blocks (16^4, ntv 24, FP64, 1 rhs) took
// 83 us; now 58, against 54 for reading P at the copy rate.
template <typename S, typename C, int NR>
__global__ __launch_bounds__(256) void k_restrict(Geom g, typename PT<C>::stor* y, const typename PT<S>::stor* P,
                                                  const typename PT<S>::stor* v, int ntv, int nrhs, int64_t fstride) {
  using R = typename PT<S>::real;
  using RC = typename PT<C>::real;
  constexpr int NJ = 4, NV = 2 * NJ * NR;
  __shared__ double red[2][4 * NV];
  const int ng = (nrhs + NR - 1) / NR;
  const int b = blockIdx.x / (2 * ng), q = blockIdx.x - b * 2 * ng, h = q & 1, k0 = (q >> 1) * NR;
  const int l = threadIdx.x, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  // blocks of fewer than 64 sites leave lanes idle: those load site 0 and add nothing (a load
  // behind a branch waited for the one before in BF16: 256 blocks, ntv 24, 1 rhs 49 us, now 14)
  const bool on = l < (1 << g.bs_log);
  const int ls = on ? l : 0;
  const int nr = min(NR, nrhs - k0), nc = 2 * ntv;
  cpx<R> vv[NR][6];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int d = 0; d < 6; ++d)
      vv[r][d] = ldcv<R>(v + (int64_t)(k0 + min(r, nr - 1)) * fstride, sidx(g, b, 6 * h + d, ls));
  int rb = 0;
  for (int j0 = 0; j0 < ntv; j0 += NJ) {
    double acc[NV];
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
      // columns past the last are read as the last and not stored
      const int j = min(j0 + t, ntv - 1);
      cpx<R> p[6];
#pragma unroll
      for (int d = 0; d < 6; ++d) p[d] = ldcv<R>(P, pidx(g, ntv, b, h, j, d, ls));
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        cpx<R> s = czero<R>();
#pragma unroll
        for (int d = 0; d < 6; ++d) cfma_conj(s, p[d], vv[r][d]);
        acc[2 * (r * NJ + t)] = on ? double(s.re) : 0.0;
        acc[2 * (r * NJ + t) + 1] = on ? double(s.im) : 0.0;
      }
    }
    double* rd = red[rb];
    rb ^= 1;
    wave_fold<NV>(acc, rd + wave * NV);
    __syncthreads();
    if (l < NV / 2) {
      double re = rd[2 * l], im = rd[2 * l + 1];
      for (int w = 1; w < nw; ++w) {
        re += rd[w * NV + 2 * l];
        im += rd[w * NV + 2 * l + 1];
      }
      const int r = l / NJ, j = j0 + l % NJ;
      if (r < nr && j < ntv)
        stcv(y + ((int64_t)(k0 + r) * g.nb + b) * nc, h * ntv + j, cpx<RC>{RC(re), RC(im)});
    }
  }
}

// v[k][b][6h+d][l] = sum_j P[b][h][j][d][l] y[k][b][h*ntv+j], U columns in flight at a time
template <typename S, typename C, int U>
__global__ __launch_bounds__(256) void k_prolong(Geom g, typename PT<S>::stor* v, const typename PT<S>::stor* P,
                                                 const typename PT<C>::stor* y, int ntv, int nrhs,
                                                 int64_t fstride) {
  using R = typename PT<S>::real;
  __shared__ cpx<R> ys[32];
  // one work-group per (block, chirality, right-hand side)
  const int b = blockIdx.x / (2 * nrhs), q = blockIdx.x - b * 2 * nrhs, h = q & 1, k = q >> 1, l = threadIdx.x;
  const auto* yi = y + ((int64_t)k * g.nb + b) * 2 * ntv + h * ntv;
  for (int o = l; o < ntv; o += blockDim.x) ys[o] = ldcv<R>(yi, o);
  __syncthreads();
#pragma unroll 2
  for (int d = 0; d < 6; ++d) {
    cpx<R> s = czero<R>();
#pragma unroll U
    for (int j = 0; j < ntv; ++j) s = s + ldcv<R>(P, pidx(g, ntv, b, h, j, d, l)) * ys[j];
    stcv(v + k * fstride, sidx(g, b, 6 * h + d, l), s);
  }
}

// ---- many right-hand sides
// P read once per site for every rhs: the coarse inputs of the block live in LDS
template <typename S, typename C>
__global__ __launch_bounds__(256) void k_prolong_mr(Geom g, typename PT<S>::stor* v, const typename PT<S>::stor* P,
                                                    const typename PT<C>::stor* y, int ntv, int nrhs, int64_t fstride) {
  using R = typename PT<S>::real;
  __shared__ cpx<R> ys[QMG_MAXRHS * 64];
  const int b = blockIdx.x, l = threadIdx.x;
  const int nc = 2 * ntv;
  for (int o = l; o < nrhs * nc; o += blockDim.x) {
    const int k = o / nc, i = o % nc;
    ys[k * 64 + i] = ldcv<R>(y + ((int64_t)k * g.nb + b) * nc, i);
  }
  __syncthreads();
  for (int h = 0; h < 2; ++h)
    for (int d = 0; d < 6; ++d) {
      cpx<R> pc[32];
#pragma unroll
      for (int j = 0; j < 32; ++j) pc[j] = j < ntv ? ldcv<R>(P, pidx(g, ntv, b, h, j, d, l)) : czero<R>();
      for (int k = 0; k < nrhs; ++k) {
        cpx<R> s = czero<R>();
#pragma unroll
        for (int j = 0; j < 32; ++j)
          if (j < ntv) s = s + pc[j] * ys[k * 64 + h * ntv + j];
        stcv(v + (int64_t)k * fstride, sidx(g, b, 6 * h + d, l), s);
      }
    }
}

// ---- restriction on MFMA: per block and chirality h, Y_h (ntv x 16 rhs) =
// P_h^H (ntv x K) V_h (K x 16), K = 6 * 256 (spin-in-half, colour, site),
// as four real 16x16x4 products per k-step.  One wave per chirality; the 4 k
// values of a step are 4 sites (stride 4) with the same (spin, colour).
typedef float tf4 __attribute__((ext_vector_type(4)));
typedef double td4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ tf4 tmfma(float a, float b, tf4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ td4 tmfma(double a, double b, td4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
template <typename R> struct TAcc;
template <> struct TAcc<float> { using T = tf4; };
template <> struct TAcc<double> { using T = td4; };
template <typename R> __device__ __forceinline__ int trow(int l, int r);
template <> __device__ __forceinline__ int trow<float>(int l, int r) { return 4 * (l >> 4) + r; }
template <> __device__ __forceinline__ int trow<double>(int l, int r) { return 4 * r + (l >> 4); }

template <typename S, typename C, int MT>
__global__ __launch_bounds__(128) void k_restrict_mfma(Geom g, typename PT<C>::stor* y, const typename PT<S>::stor* P,
                                                       const typename PT<S>::stor* v, int ntv, int nrhs, int64_t fstride) {
  using R = typename PT<S>::real;
  using AT = typename TAcc<R>::T;
  const int b = blockIdx.x, n0 = blockIdx.y * 16;
  const int h = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int ln = lane & 15, lk = lane >> 4;
  const int n = n0 + ln;
  const bool nok = n < nrhs;
  const auto* vn = v + (int64_t)(nok ? n : 0) * fstride;
  AT acc_re[MT], acc_im[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    acc_re[t] = AT{0, 0, 0, 0};
    acc_im[t] = AT{0, 0, 0, 0};
  }
  // each (spin, colour) row of 256 sites is summed in a fresh accumulator and
  // then added to the total: accumulation depth 64 + 6 instead of 384
#pragma unroll 1
  for (int d = 0; d < 6; ++d) {
    AT part_re[MT], part_im[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      part_re[t] = AT{0, 0, 0, 0};
      part_im[t] = AT{0, 0, 0, 0};
    }
    // 16 sites per step: lane (ln, lk) loads sites l0 + 4 lk .. l0 + 4 lk + 3 of
    // its P row and rhs with two wide loads; MFMA q takes site l0 + 4 lk + q in
    // k-slot lk (the same site order in A and B, so the sum is unchanged)
#pragma unroll 2
    for (int l0 = 0; l0 < 256; l0 += 16) {
      const int l = l0 + 4 * lk;
      cpx<R> bv[4];
      ld4c(vn + sidx(g, b, 6 * h + d, l), bv);
      if (!nok)
#pragma unroll
        for (int q = 0; q < 4; ++q) bv[q] = czero<R>();
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const int i = 16 * t + ln;
        cpx<R> p[4];
        if (i < ntv) ld4c(P + pidx(g, ntv, b, h, i, d, l), p);
        else
#pragma unroll
          for (int q = 0; q < 4; ++q) p[q] = czero<R>();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // A = conj(P): (p.re, -p.im)
          part_re[t] = tmfma(p[q].re, bv[q].re, part_re[t]);
          part_re[t] = tmfma(p[q].im, bv[q].im, part_re[t]);
          part_im[t] = tmfma(p[q].re, bv[q].im, part_im[t]);
          part_im[t] = tmfma(-p[q].im, bv[q].re, part_im[t]);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      acc_re[t] += part_re[t];
      acc_im[t] += part_im[t];
    }
  }
  if (!nok) return;
  const int nc = 2 * ntv;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * t + trow<R>(lane, r);
      if (i < ntv) stcv(y + ((int64_t)n * g.nb + b) * nc, h * ntv + i, cpx<R>{acc_re[t][r], acc_im[t][r]});
    }
}

// ---- prolongation on MFMA: per block b, chirality h and spin-colour row d,
// the tile v[n0..n0+15][6h+d][16 sites] = Y^T (16 rhs x ntv) P_hd (ntv x 16
// sites); Y^T stays in registers for the 96 tiles of (b, h), four waves share them.
template <typename S, typename C>
__global__ __launch_bounds__(256) void k_prolong_mfma(Geom g, typename PT<S>::stor* v, const typename PT<S>::stor* P,
                                                      const typename PT<C>::stor* y, int ntv, int nrhs,
                                                      int64_t fstride) {
  using R = typename PT<S>::real;
  using AT = typename TAcc<R>::T;
  const int b = blockIdx.x, h = blockIdx.y, n0 = blockIdx.z * 16;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int ln = lane & 15, lk = lane >> 4;
  const int nc = 2 * ntv, nks = (ntv + 3) >> 2;
  const bool nok = n0 + ln < nrhs;
  cpx<R> ya[8];
#pragma unroll
  for (int st = 0; st < 8; ++st) {
    const int j = 4 * st + lk;
    ya[st] = (st < nks && nok && j < ntv) ? ldcv<R>(y, ((int64_t)(n0 + ln) * g.nb + b) * nc + h * ntv + j)
                                          : czero<R>();
  }
#pragma unroll 1
  for (int tile = wave; tile < 96; tile += 4) {
    const int d = tile >> 4, s0 = (tile & 15) << 4;
    AT cre = AT{0, 0, 0, 0}, cim = AT{0, 0, 0, 0};
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      if (st < nks) {
        const int j = 4 * st + lk;
        const cpx<R> pb = j < ntv ? ldcv<R>(P, pidx(g, ntv, b, h, j, d, s0 + ln)) : czero<R>();
        cre = tmfma(ya[st].re, pb.re, cre);
        cre = tmfma(-ya[st].im, pb.im, cre);
        cim = tmfma(ya[st].re, pb.im, cim);
        cim = tmfma(ya[st].im, pb.re, cim);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = n0 + trow<R>(lane, r);
      if (n < nrhs) stcv(v + (int64_t)n * fstride, sidx(g, b, 6 * h + d, s0 + ln), cpx<R>{cre[r], cim[r]});
    }
  }
}

template <typename S>
void restrict_t(const qmg_ctx* c, void* yc, const void* v, int nrhs, hipStream_t s, int p) {
  using P = typename PT<S>::stor;
  const int bs = 1 << c->g.bs_log;
  if (nrhs >= c->tune.restrict_mfma_min_rhs && bs == 256 && c->ntv <= 32) {
    dim3 grid(c->g.nb, (nrhs + 15) / 16);
    const int mt = (c->ntv + 15) / 16;
    auto go = [&](auto mtc) {
      constexpr int MT = decltype(mtc)::value;
      if (p == QMG_F64)
        hipLaunchKernelGGL((k_restrict_mfma<S, double, MT>), grid, dim3(128), 0, s, c->g, (double2*)yc,
                           (const P*)c->P[p], (const P*)v, c->ntv, nrhs, (int64_t)field_elems(c));
      else
        hipLaunchKernelGGL((k_restrict_mfma<S, float, MT>), grid, dim3(128), 0, s, c->g, (float2*)yc,
                           (const P*)c->P[p], (const P*)v, c->ntv, nrhs, (int64_t)field_elems(c));
    };
    if (mt == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 2>{});
    return;
  }
  auto go = [&](auto nrc) {
    constexpr int NR = decltype(nrc)::value;
    const dim3 grid((unsigned)(c->g.nb * 2 * ((nrhs + NR - 1) / NR))), blk((unsigned)std::max(bs, 64));
    using C = typename PT<S>::real;  // coarse vectors: double for FP64, else float
    hipLaunchKernelGGL((k_restrict<S, C, NR>), grid, blk, 0, s, c->g, (typename PT<C>::stor*)yc, (const P*)c->P[p],
                       (const P*)v, c->ntv, nrhs, (int64_t)field_elems(c));
  };
  if (nrhs == 1) go(std::integral_constant<int, 1>{});
  else if (nrhs == 2 || std::is_same<S, double>::value) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, std::is_same<S, double>::value ? 2 : 4>{});
}

template <typename S>
void prolong_t(const qmg_ctx* c, void* v, const void* yc, int nrhs, hipStream_t s, int p) {
  using P = typename PT<S>::stor;
  const int bs = 1 << c->g.bs_log;
  if (nrhs >= c->tune.restrict_mfma_min_rhs && bs == 256 && c->ntv <= 32) {
    dim3 grid(c->g.nb, 2, (nrhs + 15) / 16);
    if (p == QMG_F64)
      hipLaunchKernelGGL((k_prolong_mfma<S, double>), grid, dim3(256), 0, s, c->g, (P*)v, (const P*)c->P[p],
                         (const double2*)yc, c->ntv, nrhs, (int64_t)field_elems(c));
    else
      hipLaunchKernelGGL((k_prolong_mfma<S, float>), grid, dim3(256), 0, s, c->g, (P*)v, (const P*)c->P[p],
                         (const float2*)yc, c->ntv, nrhs, (int64_t)field_elems(c));
    return;
  }
  if (nrhs > 1) {
    if (p == QMG_F64)
      hipLaunchKernelGGL((k_prolong_mr<S, double>), dim3(c->g.nb), dim3(bs), 0, s, c->g, (P*)v, (const P*)c->P[p],
                         (const double2*)yc, c->ntv, nrhs, (int64_t)field_elems(c));
    else
      hipLaunchKernelGGL((k_prolong_mr<S, float>), dim3(c->g.nb), dim3(bs), 0, s, c->g, (P*)v, (const P*)c->P[p],
                         (const float2*)yc, c->ntv, nrhs, (int64_t)field_elems(c));
    return;
  }
  auto go = [&](auto uc) {
    using C = typename PT<S>::real;  // coarse vectors: double for FP64, else float
    hipLaunchKernelGGL((k_prolong<S, C, decltype(uc)::value>), dim3(c->g.nb * 2 * nrhs), dim3(bs), 0, s, c->g, (P*)v,
                       (const P*)c->P[p], (const typename PT<C>::stor*)yc, c->ntv, nrhs, (int64_t)field_elems(c));
  };
  // eight columns at a time unless that leaves a rest, which goes one by one (2^4 blocks on 24^4, ntv 12, bf16
  // eight 70.8 us, four 55; 4^4 blocks on 16^4, ntv 24, bf16 eight 12.8, four 17.9)
  if (c->ntv % 8 == 0) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 4>{});
}

}  // namespace

hipError_t launch_build_P(const qmg_ctx* c, const void* W, int ntv, int* d_fail, hipStream_t s) {
  const int bs = 1 << c->g.bs_log;
  hipLaunchKernelGGL(k_build_P, dim3(2 * c->g.nb), dim3(std::max(64, bs)), 0, s, c->g, (double2*)c->P[QMG_F64],
                     (float2*)c->P[QMG_F32], (uint32_t*)c->P[QMG_BF16], (const double2*)W, ntv, d_fail);
  return hipGetLastError();
}

hipError_t launch_restrict(const qmg_ctx* c, int p, void* yc, const void* v, int nrhs, hipStream_t s) {
  if (p == QMG_F64) restrict_t<double>(c, yc, v, nrhs, s, p);
  else if (p == QMG_F32) restrict_t<float>(c, yc, v, nrhs, s, p);
  else restrict_t<bf16_t>(c, yc, v, nrhs, s, p);
  return hipGetLastError();
}

hipError_t launch_prolong(const qmg_ctx* c, int p, void* v, const void* yc, int nrhs, hipStream_t s) {
  if (p == QMG_F64) prolong_t<double>(c, v, yc, nrhs, s, p);
  else if (p == QMG_F32) prolong_t<float>(c, v, yc, nrhs, s, p);
  else prolong_t<bf16_t>(c, v, yc, nrhs, s, p);
  return hipGetLastError();
}
