// Application of the Galerkin coarse operator D_c = P^H D P (Sec. 2):
// out_k = (D_c - tau_k Gamma5^c) in_k.
//
// D_c couples each coarse site (lattice block) b to itself and to its 8
// neighbouring blocks.  Only the self block and the 4 forward blocks are
// stored: D is Gamma5-Hermitian and Gamma5 P = P Gamma5^c (text before
// eq. (2.9)), so Gamma5^c D_c Gamma5^c = D_c^H and, hop type by hop type, the
// block coupling b to X - mu is Gamma5^c (the block coupling X - mu to b)^H
// Gamma5^c.  The apply kernels rebuild those backward blocks on the fly.
// Blocks are stored transposed, DcT[b][e][j][i] = D_c[b][e]_{ij}, e = 0 self, 1 + mu for
// the block at X + mu (kept apart from the -mu coupling even when the two
// neighbours coincide).  In the 9-entry stencil numbering used by the kernels,
// d = 0 is self, d = 1 + 2 mu the block at X + mu, d = 2 + 2 mu the one at
// X - mu.  The apply kernels serve every coarse level: they take the level's
// neighbour table, site count and blocks.
#include "qmg_ctx.h"

namespace {

// coarse vectors are held in FP64 with FP64 blocks, in FP32 otherwise
template <typename S> using CT = typename PT<S>::real;

struct TauArr {
  double t[QMG_MAXRHS];
  int qform;  // 1: Gamma5^c (D_c - tau Gamma5^c) = Gamma5^c D_c - tau, the Galerkin P^H (Q - tau) P
};

// Few right-hand sides: one work-group per coarse site, wave d takes stencil entry d (the
// nine are summed through LDS), lane i row i.  One wave doing the nine in turn left a
// launch waiting for its loads: 41 us for 256 sites (ntv 24, FP64, 1 rhs), now 20, bound by
// the row-wise reads of the four backward blocks.
template <typename S, typename C, int T>
__global__ __launch_bounds__(576) void k_coarse_apply(const int* nbr, int nb, typename PT<C>::stor* out,
                                                      const typename PT<S>::stor* DcT, const typename PT<C>::stor* in,
                                                      int nc, int nrhs, TauArr tau) {
  using R = typename PT<C>::real;
  __shared__ cpx<R> xin[9][T][64];
  const int b = blockIdx.x, k0 = blockIdx.y * T;
  const int d = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = threadIdx.x & 63;
  const int nbk = d == 0 ? b : nbr[b * 8 + d - 1];
  cpx<R> acc[T], self[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int k = k0 + t;
    self[t] = i < nc && k < nrhs ? ldcv<R>(in, ((int64_t)k * nb + nbk) * nc + i) : czero<R>();
    xin[d][t][i] = self[t];
    acc[t] = czero<R>();
  }
  __syncthreads();
  const R g5 = i < nc / 2 ? R(1) : R(-1);
  if (i < nc) {
    if (d == 0 || (d & 1)) {
      // self (e = 0) or forward block e = 1 + mu of this site: row j of the transposed block
      const auto* Dd = DcT + ((int64_t)b * 5 + (d + 1) / 2) * nc * nc + i;
#pragma unroll 8
      for (int j = 0; j < nc; ++j) {
        const cpx<R> a = ldcv<R>(Dd, (int64_t)j * nc);
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = acc[t] + a * xin[d][t][j];
      }
    } else {
      // backward block: D_c[b][X - mu]_{ij} = g_i g_j conj(F_{ji}), F the forward block of
      // the site at X - mu, whose transposed storage holds F_{ji} at i * nc + j
      const auto* Fd = DcT + ((int64_t)nbk * 5 + d / 2) * nc * nc + (int64_t)i * nc;
#pragma unroll 8
      for (int j = 0; j < nc; ++j) {
        const cpx<R> f = ldcv<R>(Fd, j);
        const R gg = j < nc / 2 ? g5 : -g5;
        const cpx<R> a = {gg * f.re, -gg * f.im};
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = acc[t] + a * xin[d][t][j];
      }
    }
  }
  // each wave has read its own row of xin only
#pragma unroll
  for (int t = 0; t < T; ++t) xin[d][t][i] = acc[t];
  __syncthreads();
  if (d > 0 || i >= nc) return;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int k = k0 + t;
    if (k >= nrhs) break;
    cpx<R> v = xin[0][t][i];
#pragma unroll
    for (int q = 1; q < 9; ++q) v = v + xin[q][t][i];
    v = v - (R(tau.t[k]) * g5) * self[t];
    stcv(out, ((int64_t)k * nb + b) * nc + i, tau.qform ? g5 * v : v);
  }
}

// The same on many coarse sites: one wave per site takes the nine entries in turn.  There a
// launch is bound by what all its waves issue and load, of which nine of them spend more (the
// sum through LDS, nine times the idle lanes): 4096 sites, FP64, ntv 20, 1 rhs 276 us against 138.
template <typename S, typename C, int T>
__global__ __launch_bounds__(64) void k_coarse_apply1(const int* nbr, int nb, typename PT<C>::stor* out,
                                                      const typename PT<S>::stor* DcT, const typename PT<C>::stor* in,
                                                      int nc, int nrhs, TauArr tau) {
  using R = typename PT<C>::real;
  __shared__ cpx<R> xin[9][T][64];
  const int b = blockIdx.x, k0 = blockIdx.y * T, i = threadIdx.x;
  // all lanes load, also where rows are short (ntv 5, 4 rhs a lane's row each: 1.2 times slower)
  for (int e = i; e < 9 * T * nc; e += 64) {
    const int d = e / (T * nc), t = e / nc % T, j = e % nc;
    const int nbk = d == 0 ? b : nbr[b * 8 + d - 1];
    xin[d][t][j] = k0 + t < nrhs ? ldcv<R>(in, ((int64_t)(k0 + t) * nb + nbk) * nc + j) : czero<R>();
  }
  __syncthreads();
  if (i >= nc) return;
  cpx<R> acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = czero<R>();
  const R g5 = i < nc / 2 ? R(1) : R(-1);
  for (int d = 0; d < 9; ++d) {
    if (d == 0 || (d & 1)) {
      const auto* Dd = DcT + ((int64_t)b * 5 + (d + 1) / 2) * nc * nc + i;
      for (int j = 0; j < nc; ++j) {
        const cpx<R> a = ldcv<R>(Dd, (int64_t)j * nc);
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = acc[t] + a * xin[d][t][j];
      }
    } else {
      const auto* Fd = DcT + ((int64_t)nbr[b * 8 + d - 1] * 5 + d / 2) * nc * nc + (int64_t)i * nc;
      for (int j = 0; j < nc; ++j) {
        const cpx<R> f = ldcv<R>(Fd, j);
        const R gg = j < nc / 2 ? g5 : -g5;
        const cpx<R> a = {gg * f.re, -gg * f.im};
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = acc[t] + a * xin[d][t][j];
      }
    }
  }
#pragma unroll
  for (int t = 0; t < T; ++t)
    if (k0 + t < nrhs) {
      const cpx<R> v = acc[t] - (R(tau.t[k0 + t]) * g5) * xin[0][t][i];
      stcv(out, ((int64_t)(k0 + t) * nb + b) * nc + i, tau.qform ? g5 * v : v);
    }
}

// ---- MFMA coarse apply: per coarse site b and tile of 16 columns, Out (2ntv x 16) =
// sum_d D_c[b][d] (2ntv x 2ntv) In_{nbr(b,d)} (2ntv x 16).
typedef float mf4 __attribute__((ext_vector_type(4)));
typedef double md4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ mf4 mfma(float a, float b, mf4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ md4 mfma(double a, double b, md4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

template <typename R> struct MAcc;
template <> struct MAcc<float> { using T = mf4; };
template <> struct MAcc<double> { using T = md4; };

// row of output register r of lane l inside a 16x16 tile
template <typename R> __device__ __forceinline__ int mrow(int l, int r);
template <> __device__ __forceinline__ int mrow<float>(int l, int r) { return 4 * (l >> 4) + r; }
template <> __device__ __forceinline__ int mrow<double>(int l, int r) { return 4 * r + (l >> 4); }

// four consecutive stored entries, as wide loads
__device__ __forceinline__ void ld4s(const double2* p, double2* f) {
#pragma unroll
  for (int q = 0; q < 4; ++q) f[q] = p[q];
}
__device__ __forceinline__ void ld4s(const float2* p, float2* f) {
  const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  f[0] = {a.x, a.y}, f[1] = {a.z, a.w}, f[2] = {b.x, b.y}, f[3] = {b.z, b.w};
}
__device__ __forceinline__ void ld4s(const uint32_t* p, uint32_t* f) {
  const uint4 a = reinterpret_cast<const uint4*>(p)[0];
  f[0] = a.x, f[1] = a.y, f[2] = a.z, f[3] = a.w;
}

// One wave per 16-row tile t, the waves share the staged inputs.  PACK: up to 8 right-hand
// sides, columns 0-7 their real parts and 8-15 their imaginary parts, two real products per
// step of 4 (the staged pair is (re, -im) or (im, re)); else 16 right-hand sides per tile and
// four products.
// Backward blocks: sum_j g_i g_j conj(F_ji) y_j = g_i conj(sum_j F_ji conj(g_j y_j)), so the
// staged input takes g_j and the conjugation and the sum, kept apart, the rest.
// Each run of 16 contraction indices goes in the order j = jb + 4 lk + q (step q): a lane's
// four inputs, and its four entries of a backward block, are consecutive.  The blocks and
// inputs of the next entry are loaded while this one is multiplied.  Inputs staged with the
// right-hand side fastest, so that all writes of a wave met in one LDS bank, no loads ahead
// and four products for any batch took, 32^4 (4096 sites), ntv 24: FP32 8 rhs 138 us, 11 rhs
// 142; FP64 8 rhs 252; bf16 8 rhs 119; 16^4 FP32 8 rhs 23.7.  Now 100, 121, 197, 64 and 12.0.
// Bound: the nine blocks per site, 7 TB/s through the fabric (a forward block that another
// XCD reads as a backward one is read twice); with 9-16 rhs also the FP32 matrix rate (69 us).
// Three groups of waves on three entries each gained nothing: 8 rhs FP32 159 us.
template <typename S, int NT, bool PACK>
__global__ __launch_bounds__(64 * NT) void k_coarse_mfma(const int* nbr, const int* ord, int nb,
                                                         typename PT<CT<S>>::stor* out,
                                                         const typename PT<S>::stor* DcT,
                                                         const typename PT<CT<S>>::stor* in, int nrhs, TauArr tau) {
  using R = CT<S>;
  using AT = typename MAcc<R>::T;
  constexpr int NC = 16 * NT;               // 2 ntv
  constexpr int NR = PACK ? 8 : 16;         // right-hand sides of a work-group
  constexpr int LD = NC + (sizeof(R) == 8 ? 1 : 2);  // row stride: no bank shared by 16 lanes' 16 bytes
  constexpr int NA = PACK ? 1 : 2;          // accumulators: (re | im), or re and im
  __shared__ cpx<R> Bs[2][16][LD];
  // each XCD walks a contiguous share of the sites in lexicographic order, so that a forward
  // block is still in its L2 when the neighbour reads it as a backward block (in colour order
  // that neighbour ran half a launch later: 32^4, FP32, 8 rhs 153 -> 140 us)
  const int L = (nb & 7) == 0 ? (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  const int b = ord ? ord[L] : L, n0 = blockIdx.y * NR;
  const int tid = threadIdx.x, t = tid >> 6, l = tid & 63;
  const int ln = l & 15, lk = l >> 4;
  const int irow = 16 * t + ln;
  const int sj = tid % NC, sn = tid / NC;  // staging: entry sj of rhs sn + 4 e
  const R gj = sj < NC / 2 ? R(1) : R(-1);

  AT af[NA], ab[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) af[k] = ab[k] = AT{0, 0, 0, 0};
  typename PT<S>::stor ar[NC / 4], an[NC / 4];
  cpx<R> br[NR / 4];

  auto load = [&](int d, typename PT<S>::stor (&f)[NC / 4]) {
    const int nbk = d == 0 ? b : nbr[b * 8 + d - 1];
#pragma unroll
    for (int e = 0; e < NR / 4; ++e) {
      const int n = n0 + sn + 4 * e;
      br[e] = n < nrhs ? ldcv<R>(in, ((int64_t)n * nb + nbk) * NC + sj) : czero<R>();
    }
    if (d == 0 || (d & 1)) {
      // self or forward block: A_ij at row j of the transposed block
      const auto* Dd = DcT + ((int64_t)b * 5 + (d + 1) / 2) * NC * NC + (4 * lk) * NC + irow;
#pragma unroll
      for (int j = 0; j < NC / 4; ++j) f[j] = Dd[((j >> 2) * 16 + (j & 3)) * NC];
    } else {
      // forward block F of the site at X - mu: F_ji at row i
      const auto* Fd = DcT + ((int64_t)nbk * 5 + d / 2) * NC * NC + irow * NC + 4 * lk;
#pragma unroll
      for (int j = 0; j < NC / 4; j += 4) ld4s(Fd + 4 * j, f + j);
    }
  };
  auto stage = [&](int d, int buf) {
    const bool fwd = d == 0 || (d & 1);
#pragma unroll
    for (int e = 0; e < NR / 4; ++e) {
      const int n = sn + 4 * e;
      const cpx<R> v = fwd ? br[e] : cpx<R>{gj * br[e].re, -gj * br[e].im};
      if constexpr (PACK) {
        Bs[buf][n][sj] = {v.re, -v.im};
        Bs[buf][n + 8][sj] = {v.im, v.re};
      } else {
        Bs[buf][n][sj] = v;
      }
    }
  };
  auto mult = [&](int buf, AT (&acc)[NA]) {
#pragma unroll
    for (int j = 0; j < NC / 4; ++j) {
      const cpx<R> a = ldcv<R>(ar, j);
      const cpx<R> v = Bs[buf][ln][(j >> 2) * 16 + 4 * lk + (j & 3)];
      if constexpr (PACK) {
        acc[0] = mfma(a.re, v.re, acc[0]);
        acc[0] = mfma(a.im, v.im, acc[0]);
      } else {
        acc[0] = mfma(a.re, v.re, acc[0]);
        acc[1] = mfma(a.re, v.im, acc[1]);
        acc[0] = mfma(a.im, -v.im, acc[0]);
        acc[1] = mfma(a.im, v.re, acc[1]);
      }
    }
  };

  load(1, ar);
  stage(1, 0);
#pragma unroll
  for (int s = 0; s < 9; ++s) {
    const int d = (s + 1) % 9, dn = (s + 2) % 9;  // the site itself last
    __syncthreads();
    if (s < 8) load(dn, an);
    if (d == 0 || (d & 1)) mult(s & 1, af);
    else mult(s & 1, ab);
    if (s < 8) {
      stage(dn, (s + 1) & 1);
#pragma unroll
      for (int j = 0; j < NC / 4; ++j) ar[j] = an[j];
    }
  }

  const int n = PACK ? n0 + (ln & 7) : n0 + ln;
  const R tn = n < nrhs ? R(tau.t[n]) : R(0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * t + mrow<R>(l, r);
    const R g5 = i < NC / 2 ? R(1) : R(-1);
    cpx<R> v, self = Bs[0][PACK ? ln & 7 : ln][i];
    if constexpr (PACK) {
      const R x = af[0][r] + (ln < 8 ? g5 : -g5) * ab[0][r], o = __shfl_xor(x, 8);
      v = ln < 8 ? cpx<R>{x, o} : cpx<R>{o, x};
      self.im = -self.im;
    } else {
      v = {af[0][r] + g5 * ab[0][r], af[1][r] - g5 * ab[1][r]};
    }
    v = {v.re - tn * g5 * self.re, v.im - tn * g5 * self.im};
    if (tau.qform) v = g5 * v;
    // packed: the two lanes of an entry store two of the four rows each
    if (n < nrhs && (!PACK || (ln >> 3) == (r >> 1))) stcv(out, ((int64_t)n * nb + b) * NC + i, v);
  }
}

// one coarse level's stencil: nb sites, 2 ntv components each, blocks D
// (storage precision S) and the neighbour table
struct CLevel {
  const int* nbr;
  const int* ord;  // site ids in lexicographic order (null: they are)
  int nb, ntv;
  const void* D;
};

template <typename S, int NT>
void capply_mfma(const CLevel& lv, void* out, const void* in, const TauArr& tau, int nrhs, hipStream_t s) {
  using P = typename PT<CT<S>>::stor;
  const auto* D = (const typename PT<S>::stor*)lv.D;
  if (nrhs <= 8)
    hipLaunchKernelGGL((k_coarse_mfma<S, NT, true>), dim3(lv.nb), dim3(64 * NT), 0, s, lv.nbr, lv.ord, lv.nb, (P*)out, D,
                       (const P*)in, nrhs, tau);
  else
    hipLaunchKernelGGL((k_coarse_mfma<S, NT, false>), dim3(lv.nb, (nrhs + 15) / 16), dim3(64 * NT), 0, s, lv.nbr, lv.ord,
                       lv.nb, (P*)out, D, (const P*)in, nrhs, tau);
}

template <typename S, int T>
void capply_t(const CLevel& lv, bool one, void* out, const void* in, const TauArr& tau, int nrhs, hipStream_t s) {
  using P = typename PT<CT<S>>::stor;
  const int nc = 2 * lv.ntv;
  const dim3 grid(lv.nb, (nrhs + T - 1) / T);
  const auto* D = (const typename PT<S>::stor*)lv.D;
  if (one)
    hipLaunchKernelGGL((k_coarse_apply1<S, CT<S>, T>), grid, dim3(64), 0, s, lv.nbr, lv.nb, (P*)out, D, (const P*)in, nc,
                       nrhs, tau);
  else
    hipLaunchKernelGGL((k_coarse_apply<S, CT<S>, T>), grid, dim3(576), 0, s, lv.nbr, lv.nb, (P*)out, D, (const P*)in, nc,
                       nrhs, tau);
}

template <typename S>
void capply_s(const qmg_ctx* c, const CLevel& lv, void* out, const void* in, const double* htau, int nrhs,
              hipStream_t s, int qform) {
  TauArr t;
  for (int i = 0; i < QMG_MAXRHS; ++i) t.t[i] = i < nrhs ? htau[i] : 0.0;
  t.qform = qform;
  // The matrix-core kernel takes rows in whole tiles of 16 (ntv = 8, 16, 24).  It has the
  // blocks of the next entry in flight and wins wherever the launch is bound by reading them;
  // with one or two right-hand sides and few sites one wave per entry has the shorter chain.
  // 1 rhs, ntv 24, the other kernel against it: FP64 16 sites (3 MB of blocks) 10.5 / 13.5 us,
  // 128 sites (24 MB) 16.7 / 14.0; FP32 512 sites (47 MB) 12.5 / 13.9, 1024 sites (94 MB)
  // 25.2 / 22.6; bf16 1024 sites (47 MB) 14.6 / 17.5, 2048 sites (94 MB) 31.1 / 31.1.
  // 3 rhs, 16 sites: FP64 15.6 / 14.2, FP32 12.5 / 10.3.
  const int64_t bytes = (int64_t)lv.nb * 5 * 4 * lv.ntv * lv.ntv * sizeof(typename PT<S>::stor);
  const bool many = nrhs >= 3 || bytes > (std::is_same<S, double>::value ? 16 : 64) * (int64_t(1) << 20);
  if (c->tune.coarse_mfma && many) {
    if (lv.ntv == 24) return capply_mfma<S, 3>(lv, out, in, t, nrhs, s);
    if (lv.ntv == 16) return capply_mfma<S, 2>(lv, out, in, t, nrhs, s);
    if (lv.ntv == 8) return capply_mfma<S, 1>(lv, out, in, t, nrhs, s);
  }
  // One wave per site or nine.  From 4 rhs on by the rounds that the work-groups of 4 rhs take:
  // 256 (FP64) or 512 of nine waves run at a time, four times as many of one wave, and a round
  // of those takes 3.4 times as long (nine / one, FP64 512 sites: 4 rhs 0.6, 8 rhs 1.15, 12 rhs
  // 0.9; FP32 1024 sites: 4 rhs 0.8, 8 rhs 1.3, 12 rhs 1.0; 2048 and more: 1.0-1.3 everywhere).
  // Fewer rhs: FP64 512 sites 0.6-1.1, 1024 1.2-1.5, more 1.3-2.3; FP32 and bf16, 1 or 2 rhs,
  // are better with nine (0.2-1.0) but for short rows on 4096 sites and more (ntv 5 and 12:
  // 1.0-1.6; bf16, 1 rhs, from 8192), 3 rhs from 1024 sites on 1.0-2.2.  3 rhs are three times one rhs where the rows
  // are short or the blocks stay in the caches (2048 sites, ntv 28, FP32 0.75 against 1.1).
  constexpr bool f64 = std::is_same<S, double>::value;
  bool one;
  if (nrhs >= 4) {
    constexpr int64_t kRun = f64 ? 256 : 512;
    const int64_t wgs = (int64_t)lv.nb * ((nrhs + 3) / 4);
    one = 10 * ((wgs + kRun - 1) / kRun) >= 34 * ((wgs + 4 * kRun - 1) / (4 * kRun));
  } else {
    const int few = std::is_same<S, bf16_t>::value && nrhs == 1 ? 8192 : 4096;
    one = nrhs == 3 || f64 ? lv.nb >= 1024 : lv.nb >= few && lv.ntv <= 12;
  }
  const bool three = nrhs == 3 && one && (lv.ntv <= 20 || bytes <= 128 * (int64_t(1) << 20));
  if (nrhs >= 3 && !three) capply_t<S, 4>(lv, one, out, in, t, nrhs, s);
  else if (nrhs == 2) capply_t<S, 2>(lv, one, out, in, t, nrhs, s);
  else capply_t<S, 1>(lv, one, out, in, t, nrhs, s);
}

}  // namespace

// tau: host array of nrhs shifts
hipError_t launch_coarse_apply(const qmg_ctx* c, int p, void* out, const void* in, const double* dtau, int nrhs,
                               hipStream_t s, int qform) {
  const CLevel lv{c->g.nbr, c->g.lexord, c->g.nb, c->ntv, c->Dc[p]};
  if (p == QMG_F64) capply_s<double>(c, lv, out, in, dtau, nrhs, s, qform);
  else if (p == QMG_F32) capply_s<float>(c, lv, out, in, dtau, nrhs, s, qform);
  else capply_s<bf16_t>(c, lv, out, in, dtau, nrhs, s, qform);
  return hipGetLastError();
}

// level-3 operator A3(tau) = D3 - tau Gamma5^cc (D3 stored in the coarse precision of p)
hipError_t launch_apply_l3(const qmg_ctx* c, int p, void* out, const void* in, const double* dtau, int nrhs,
                           hipStream_t s, int qform) {
  const int sp = p == QMG_F64 ? 0 : 1;
  const CLevel lv{c->l3.nbr3, nullptr, c->l3.n3, c->l3.ntv2, c->l3.D3[sp]};
  if (p == QMG_F64) capply_s<double>(c, lv, out, in, dtau, nrhs, s, qform);
  else capply_s<float>(c, lv, out, in, dtau, nrhs, s, qform);
  return hipGetLastError();
}
