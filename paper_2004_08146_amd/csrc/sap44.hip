// SAP on 4^4 blocks with the hops between blocks carried in a halo field.
//
// A half-sweep needs r = f - A x on every block of its colour.  The hops that enter the
// block come from blocks of the other colour, whose x the previous half-sweep wrote, so
// that half-sweep also writes them: halo[block][hop][6][64] holds, for each of the 8 hops
// that enter the block, the colour-rotated half spinors -1/2 U (1 -+ gamma) x at the 64
// sites of that face (as many numbers as a spinor field).  r is then f, the hops inside
// the block (from LDS, as in the minimal-residual steps) and the halo: x, f and the halo
// are read, x and the halo written, all in full cache lines, where gathering the
// neighbours' x touched five times the block's own lines in faces across directions 2, 3
// and waited for eight dependent rounds of loads.  Same terms as the gather, other order.
// The four applications of the block operator (x, three minimal-residual steps) are bound
// by vector instructions: 0.54 ms each of a half-sweep's 3.2 ms at 64x32^3, FP32, 16
// right-hand sides.  Measured against the gather, clover, MR(3) blocks:
//   three sweeps, 64x32^3, FP32, 16 right-hand sides   29.2 -> 20.3 ms
//   three sweeps, 48x24^3, BF16, 2 right-hand sides    1.32 -> 0.96 ms
//   four sweeps, 24x16^3, FP64, 24 right-hand sides    7.35 -> 4.42 ms
#include "qmg_ctx.h"
#include "reduce.h"

namespace {

constexpr int kSh[4] = {6, 4, 2, 0};  // bit position of local coordinate mu in l

template <typename S>
struct Sap44Args {
  using R = typename PT<S>::real;
  using P = typename PT<S>::stor;
  P* x;
  const P* f;
  cpx<R>* halo;
  const P* U;
  const P* diag;
  R mass4;
  int64_t fstride;  // complex elements per field (x, f and halo alike)
  int nrhs;
  int per;          // right-hand sides per work-group
  int first_block;
  int nblk;
  int n_mr;
  int solve;        // 0: only write the halo of x
  int halo_out;     // another half-sweep follows
  const int* nbr;
  R tau[QMG_MAXRHS];
};

// keeps values derived from v from being computed once outside a loop and held in registers
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}
template <typename R>
__device__ __forceinline__ cpx<R> ldx(const cpx<R>* base, uint32_t elem) {
  return *reinterpret_cast<const cpx<R>*>(reinterpret_cast<const char*>(base) + (size_t)(elem * (uint32_t)sizeof(cpx<R>)));
}
template <typename R>
__device__ __forceinline__ void stx(cpx<R>* base, uint32_t elem, cpx<R> v) {
  *reinterpret_cast<cpx<R>*>(reinterpret_cast<char*>(base) + (size_t)(elem * (uint32_t)sizeof(cpx<R>))) = v;
}

// index of site l within its face across direction mu (the other three coordinates)
template <int MU>
__device__ __forceinline__ uint32_t face_of(uint32_t l) {
  if constexpr (MU == 0) return l & 63u;
  else if constexpr (MU == 1) return ((l >> 6) << 4) | (l & 15u);
  else if constexpr (MU == 2) return ((l >> 4) << 2) | (l & 3u);
  else return l >> 2;
}
// site with face index j and coordinate v in direction mu
template <int MU>
__device__ __forceinline__ uint32_t site_of(uint32_t j, uint32_t v) {
  if constexpr (MU == 0) return (v << 6) | j;
  else if constexpr (MU == 1) return ((j >> 4) << 6) | (v << 4) | (j & 15u);
  else if constexpr (MU == 2) return ((j >> 2) << 4) | (v << 2) | (j & 3u);
  else return (j << 2) | v;
}

// LDS of a work-group: -1/2 U of directions 1..3 and the vector that the block operator
// is applied to.  Direction 0 couples whole waves (local coordinate 0 is the wave), so a
// lane keeps the two links of its own hops there in registers.  In FP32 that is 80 KB, so
// two work-groups share a CU and one's loads run under the other's arithmetic (with all
// four directions and two right-hand sides in one work-group the same kernel waited for
// its loads: 3.9 ms a half-sweep at 64x32^3 and 16 right-hand sides).  In FP64 it is 160 KB.
// A lane whose neighbour lies outside the block reads one of the zeros that pad each row
// (in FP32 16 of them, so that it reads at its neighbour's banks).
template <typename R>
struct Lds44 {
  static constexpr int kPad = std::is_same<R, double>::value ? 1 : 16, kStride = 256 + kPad;
  __device__ static uint32_t outside(uint32_t ln) { return 256u + (ln & (kPad - 1)); }
};

template <typename R>
__device__ __forceinline__ Spinor<R> row_spinor(const cpx<R>* rh, uint32_t l) {
  Spinor<R> p;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) p.s[s][c] = rh[(3 * s + c) * Lds44<R>::kStride + l];
  return p;
}
template <typename R>
__device__ __forceinline__ Link<R> row_link(const cpx<R>* Ul, int mu, uint32_t l) {
  Link<R> u;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) u.u[a][c] = Ul[(mu * 9 + 3 * a + c) * 256 + l];
  return u;
}
// -1/2 U from global memory
template <typename R, typename P>
__device__ __forceinline__ Link<R> half_link(const P* U, uint32_t b, int mu, uint32_t l) {
  Link<R> u;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const auto v = cv(ldo(U, ((b * 36u + (uint32_t)(mu * 9 + 3 * a + c)) << 8) + l));
      u.u[a][c] = cpx<R>{R(-0.5) * R(v.re), R(-0.5) * R(v.im)};
    }
  return u;
}

// q += (-1/2 hop) of the vector in rh, hops that leave the block dropped
template <typename R, int HOP>
__device__ __forceinline__ void block_hop(Spinor<R>& q, const cpx<R>* rh, const cpx<R>* Ul, uint32_t l) {
  constexpr int MU = HOP / 2;
  constexpr bool FWD = HOP % 2 == 0;
  const uint32_t lc = (l >> kSh[MU]) & 3u;
  const bool in = FWD ? lc < 3u : lc > 0u;
  const uint32_t ln = FWD ? l + (1u << kSh[MU]) : l - (1u << kSh[MU]);
  const Half<R> h = project(row_spinor(rh, in ? ln : Lds44<R>::outside(ln)), MU, FWD);
  const Link<R> u = row_link(Ul, MU - 1, FWD ? l : (ln & 255u));
  accum_recon(q, FWD ? umul(u, h) : udagmul(u, h), MU, FWD);
}

// acc += (-1/2 hop) that enters the block through hop HOP; w: the six halo values
template <typename R, int HOP>
__device__ __forceinline__ void halo_add(Spinor<R>& acc, const cpx<R> (&w)[6], uint32_t l) {
  constexpr int MU = HOP / 2;
  constexpr bool FWD = HOP % 2 == 0;
  const uint32_t lc = (l >> kSh[MU]) & 3u;
  const bool on = FWD ? lc == 3u : lc == 0u;
  Half<R> h;
  if constexpr (std::is_same<R, double>::value) {
    // one wave per SIMD: no branch, so that all loads of the halo are in flight together
#pragma unroll
    for (int i = 0; i < 6; ++i) h.h[i / 3][i % 3] = on ? w[i] : czero<R>();
    accum_recon(acc, h, MU, FWD);
  } else if (on) {
#pragma unroll
    for (int i = 0; i < 6; ++i) h.h[i / 3][i % 3] = w[i];
    accum_recon(acc, h, MU, FWD);
  }
}

template <typename R, int MU>
__device__ __forceinline__ void load_halo(cpx<R> (&w)[2][6], const cpx<R>* halo, uint32_t b, uint32_t l) {
  const uint32_t j = face_of<MU>(l);
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int i = 0; i < 6; ++i) w[d][i] = ldx(halo, ((b * 8u + 2u * MU + d) * 6u + i) * 64u + j);
}

// x's hops that leave the block in direction mu, one lane per face site:
// upper face to the block at X + mu, lower face to the block at X - mu
template <typename R, int MU>
__device__ __forceinline__ void send_halo(cpx<R>* halo, const cpx<R>* rh, const Link<R>& up, const Link<R>& lo,
                                          const int* nbr, uint32_t b, uint32_t j) {
  const Half<R> hu = udagmul(up, project(row_spinor(rh, site_of<MU>(j, 3)), MU, false));
  const Half<R> hl = umul(lo, project(row_spinor(rh, site_of<MU>(j, 0)), MU, true));
  const uint32_t bu = (uint32_t)nbr[b * 8 + 2 * MU], bl = (uint32_t)nbr[b * 8 + 2 * MU + 1];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    stx(halo, ((bu * 8u + 2u * MU + 1u) * 6u + i) * 64u + j, hu.h[i / 3][i % 3]);
    stx(halo, ((bl * 8u + 2u * MU) * 6u + i) * 64u + j, hl.h[i / 3][i % 3]);
  }
}

// o += (m0 + 4 + C - tau Gamma5) v
template <typename R, bool CLOVER>
__device__ __forceinline__ void diag_add(Spinor<R>& o, const cpx<R> (&dg)[2][18], R mass4, const Spinor<R>& v, R tau) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const R t = h == 0 ? -tau : tau;
    if (CLOVER) {
      cpx<R> in[6], w[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        in[i] = v.s[2 * h + i / 3][i % 3];
        w[i] = o.s[2 * h + i / 3][i % 3];
      }
      int k = 3;
#pragma unroll
      for (int i = 1; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) {
          cfma(w[i], dg[h][k], in[j]);
          cfma_conj(w[j], dg[h][k], in[i]);
          ++k;
        }
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        const R d = (i % 2 == 0 ? dg[h][i / 2].re : dg[h][i / 2].im) + t;
        o.s[2 * h + i / 3][i % 3] = cpx<R>{fmar(d, in[i].re, w[i].re), fmar(d, in[i].im, w[i].im)};
      }
    } else {
#pragma unroll
      for (int s = 2 * h; s < 2 * h + 2; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c)
          o.s[s][c] = cpx<R>{fmar(mass4 + t, v.s[s][c].re, o.s[s][c].re), fmar(mass4 + t, v.s[s][c].im, o.s[s][c].im)};
    }
  }
}

// A_block of the vector in rh (v: its value at this lane's site)
template <typename R, bool CLOVER, bool QF>
__device__ __forceinline__ Spinor<R> block_op(const cpx<R> (&dg)[2][18], R mass4, const Spinor<R>& v, R tau,
                                              const cpx<R>* rh, const cpx<R>* Ul, const Link<R>& u0f,
                                              const Link<R>& u0b, uint32_t x0, uint32_t l) {
  // the hops first: the diagonal, the largest term, joins the sum last
  Spinor<R> q;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) q.s[s][c] = czero<R>();
  block_hop<R, 2>(q, rh, Ul, l);
  __builtin_amdgcn_sched_barrier(0);
  block_hop<R, 3>(q, rh, Ul, l);
  __builtin_amdgcn_sched_barrier(0);
  block_hop<R, 4>(q, rh, Ul, l);
  __builtin_amdgcn_sched_barrier(0);
  block_hop<R, 5>(q, rh, Ul, l);
  __builtin_amdgcn_sched_barrier(0);
  block_hop<R, 6>(q, rh, Ul, l);
  __builtin_amdgcn_sched_barrier(0);
  block_hop<R, 7>(q, rh, Ul, l);
  __builtin_amdgcn_sched_barrier(0);
  // a wave skips the hop that leaves the block in direction 0
  if (x0 < 3u) accum_recon(q, umul(u0f, project(row_spinor(rh, l + 64u), 0, true)), 0, true);
  if (x0 > 0u) accum_recon(q, udagmul(u0b, project(row_spinor(rh, l - 64u), 0, false)), 0, false);
  __builtin_amdgcn_sched_barrier(0);
  diag_add<R, CLOVER>(q, dg, mass4, v, tau);
  __builtin_amdgcn_sched_barrier(0);
  if (QF) {
#pragma unroll
    for (int s = 2; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) q.s[s][c] = -q.s[s][c];
  }
  return q;
}

// One colour's half-sweep; one work-group per block and `per` right-hand sides.
template <typename S, bool CLOVER, bool QF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(std::is_same<S, double>::value ? 1 : 2)))
void k_sap44h(Sap44Args<S> a) {
  using R = typename PT<S>::real;
  using P = typename PT<S>::stor;
  constexpr int kStride = Lds44<R>::kStride, kPad = Lds44<R>::kPad;
  __shared__ cpx<R> Ul[27 * 256];
  __shared__ cpx<R> rh[12 * kStride];
  __shared__ R red[2][4 * 3];
  int rb = 0;
  const int w = blockIdx.x, nw = gridDim.x;
  const int L = ((nw & 7) == 0) ? (w & 7) * (nw >> 3) + (w >> 3) : w;
  const int grp = L / a.nblk;
  const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane(a.first_block + (L - grp * a.nblk));
  const uint32_t x0 = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t l = threadIdx.x;
  const int* nbr = a.nbr;
  for (int i = (int)threadIdx.x; i < 12 * kPad; i += 256) rh[(i / kPad) * kStride + 256 + i % kPad] = czero<R>();
#pragma unroll 9
  for (int i = 0; i < 27; ++i) {
    const auto v = cv(ldo(a.U, ((b * 36u + (uint32_t)(9 + i)) << 8) + l));
    Ul[i * 256 + l] = cpx<R>{R(-0.5) * R(v.re), R(-0.5) * R(v.im)};
  }
  const Link<R> u0f = half_link<R>(a.U, b, 0, l), u0b = half_link<R>(a.U, b, 0, x0 > 0 ? l - 64u : l);
  cpx<R> dg[2][18];
  // the launch that only forms the halo has no use for it (32x16^3, FP32, 2 rhs, one sweep
  // 92.6 -> 87.1 us)
  if (CLOVER && a.solve) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int k = 0; k < 18; ++k) {
        const auto v = cv(ldo(a.diag, ((b * 36u + (uint32_t)(h * 18 + k)) << 8) + l));
        dg[h][k] = cpx<R>{R(v.re), R(v.im)};
      }
  }
  const int kend = min(a.nrhs, (grp + 1) * a.per);
#pragma unroll 1
  for (int k = grp * a.per; k < kend; ++k) {
    l = opaque(l);
    P* x = a.x + (size_t)k * a.fstride;
    cpx<R>* halo = a.halo + (size_t)k * a.fstride;
    const R tau = a.tau[k];
    Spinor<R> cur;  // the vector that the block operator is applied to next: x, then the residual
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      const auto v = cv(ldo(x, ((b * 12u + (uint32_t)i) << 8) + l));
      cur.s[i / 3][i % 3] = cpx<R>{R(v.re), R(v.im)};
    }
    if (a.solve) {
      const P* f = a.f + (size_t)k * a.fstride;
      Spinor<R> oth;  // -f + the entering hops of D (Q form: of Gamma5 times that), then x
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        const auto v = cv(ldo(f, ((b * 12u + (uint32_t)i) << 8) + l));
        oth.s[i / 3][i % 3] = QF && i >= 6 ? cpx<R>{R(v.re), R(v.im)} : cpx<R>{-R(v.re), -R(v.im)};
      }
      {
        cpx<R> h0[2][6], h1[2][6];
        load_halo<R, 0>(h0, halo, b, l);
        load_halo<R, 1>(h1, halo, b, l);
        halo_add<R, 0>(oth, h0[0], l);
        halo_add<R, 1>(oth, h0[1], l);
        load_halo<R, 2>(h0, halo, b, l);
        halo_add<R, 2>(oth, h1[0], l);
        halo_add<R, 3>(oth, h1[1], l);
        load_halo<R, 3>(h1, halo, b, l);
        halo_add<R, 4>(oth, h0[0], l);
        halo_add<R, 5>(oth, h0[1], l);
        halo_add<R, 6>(oth, h1[0], l);
        halo_add<R, 7>(oth, h1[1], l);
      }
      // it < 0: r = (f - hops that enter) - A_block x; then minimal-residual steps on r
#pragma unroll 1
      for (int it = -1; it < a.n_mr; ++it) {
        l = opaque(l);
#pragma unroll
        for (int i = 0; i < 12; ++i) rh[i * kStride + l] = cur.s[i / 3][i % 3];
        __syncthreads();
        const Spinor<R> q = block_op<R, CLOVER, QF>(dg, a.mass4, cur, tau, rh, Ul, u0f, u0b, x0, l);
        if (it < 0) {
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const cpx<R> xv = cur.s[s][c];
              cur.s[s][c] = (QF && s >= 2 ? oth.s[s][c] : -oth.s[s][c]) - q.s[s][c];
              oth.s[s][c] = xv;
            }
          __syncthreads();  // the hops of x are read
          continue;
        }
        R v[3] = {R(0), R(0), R(0)};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const cpx<R> p = q.s[s][c], y = cur.s[s][c];
            v[0] = fmar(p.im, y.im, fmar(p.re, y.re, v[0]));
            v[1] = fmar(-p.im, y.re, fmar(p.re, y.im, v[1]));
            v[2] = fmar(p.im, p.im, fmar(p.re, p.re, v[2]));
          }
        // sums over the block; red is double buffered: a half is rewritten two steps later,
        // after every thread has passed the barriers in between
        R* rd = red[rb];
        rb ^= 1;
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = wave_sum63(v[i]);
        if (lane == 63u)
#pragma unroll
          for (int i = 0; i < 3; ++i) rd[x0 * 3 + i] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = ((rd[i] + rd[3 + i]) + rd[6 + i]) + rd[9 + i];
        cpx<R> alpha = czero<R>();
        if (v[2] > R(0)) alpha = cpx<R>{v[0] / v[2], v[1] / v[2]};
        const cpx<R> malpha = {-alpha.re, -alpha.im};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            cfma(oth.s[s][c], alpha, cur.s[s][c]);
            cfma(cur.s[s][c], malpha, q.s[s][c]);
          }
      }
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        // the halo is formed from x as stored
        const P xo = vc(oth.s[i / 3][i % 3], (P*)nullptr);
        sto(x, ((b * 12u + (uint32_t)i) << 8) + l, xo);
        const auto v = cv(xo);
        cur.s[i / 3][i % 3] = cpx<R>{R(v.re), R(v.im)};
      }
    }
    if (a.halo_out) {
#pragma unroll
      for (int i = 0; i < 12; ++i) rh[i * kStride + l] = cur.s[i / 3][i % 3];
      __syncthreads();
      // direction 0 goes to the wave that holds its upper links
      const uint32_t j = opaque(threadIdx.x & 63u);
      const uint32_t mu = (x0 + 1u) & 3u;
      const uint32_t bl = (uint32_t)nbr[b * 8 + 2 * mu + 1];
      if (mu == 0) send_halo<R, 0>(halo, rh, u0f, half_link<R>(a.U, bl, 0, site_of<0>(j, 3)), nbr, b, j);
      else if (mu == 1) send_halo<R, 1>(halo, rh, row_link(Ul, 0, site_of<1>(j, 3)), half_link<R>(a.U, bl, 1, site_of<1>(j, 3)), nbr, b, j);
      else if (mu == 2) send_halo<R, 2>(halo, rh, row_link(Ul, 1, site_of<2>(j, 3)), half_link<R>(a.U, bl, 2, site_of<2>(j, 3)), nbr, b, j);
      else send_halo<R, 3>(halo, rh, row_link(Ul, 2, site_of<3>(j, 3)), half_link<R>(a.U, bl, 3, site_of<3>(j, 3)), nbr, b, j);
    }
    __syncthreads();  // rh is free
  }
}

constexpr size_t kHaloMax = (size_t)8 << 30;  // halo bytes of the right-hand sides smoothed together

template <typename S>
hipError_t sweeps(qmg_ctx* c, int p, void* x, const void* f, const double* tau, int nrhs, int nsweep, int n_mr,
                  hipStream_t s, int qform, bool* done) {
  using R = typename PT<S>::real;
  using P = typename PT<S>::stor;
  const size_t n = field_elems(c);
  const int group = (int)std::max<size_t>(1, std::min<size_t>((size_t)nrhs, kHaloMax / (n * sizeof(cpx<R>))));
  void* halo = ws_try(c, kHaloName, n * group * sizeof(cpx<R>), s);
  *done = halo != nullptr;
  if (!*done) return hipSuccess;
  const bool own_capture = c->cap_stream && s == c->cap_stream;
  hipError_t e = own_capture ? hipSuccess : scratch_acquire(c, s);
  const int ncol[2] = {c->g.ncol0, c->g.nb - c->g.ncol0};
  for (int k0 = 0; k0 < nrhs && e == hipSuccess; k0 += group) {
    Sap44Args<S> a;
    a.x = (P*)x + (size_t)k0 * n;
    a.f = (const P*)f + (size_t)k0 * n;
    a.halo = (cpx<R>*)halo;
    a.U = (const P*)c->U[p];
    a.diag = (const P*)c->Dg[p];
    a.mass4 = R(c->m0 + 4.0);
    a.fstride = (int64_t)n;
    a.nrhs = std::min(group, nrhs - k0);
    a.n_mr = n_mr;
    a.nbr = c->g.nbr;
    for (int i = 0; i < QMG_MAXRHS; ++i) a.tau[i] = i < a.nrhs ? R(tau[k0 + i]) : R(0);
    auto half = [&](int col, bool solve, bool halo_out) {
      a.first_block = col == 0 ? 0 : c->g.ncol0;
      a.nblk = ncol[col];
      a.solve = solve;
      a.halo_out = halo_out;
      // Split of the batch over work-groups: a work-group first loads its block's links and
      // clover term, which takes about as long as one right-hand side, so as few groups as
      // fill the chip: the split with the fewest passes of (setup + right-hand sides) over
      // the work-groups that run at a time.
      const int slots = 256 * (std::is_same<S, double>::value ? 1 : 2);
      int best = 1;
      int64_t cost = -1;
      for (int g = 1; g <= a.nrhs; ++g) {
        const int per = (a.nrhs + g - 1) / g;
        const int64_t t = (int64_t)((a.nblk * g + slots - 1) / slots) * (per + 1);
        if (cost < 0 || t < cost) { cost = t; best = g; }
      }
      a.per = (a.nrhs + best - 1) / best;
      const dim3 grid((unsigned)(a.nblk * ((a.nrhs + a.per - 1) / a.per))), blk(256);
      if (qform) {
        if (c->clover) hipLaunchKernelGGL((k_sap44h<S, true, true>), grid, blk, 0, s, a);
        else hipLaunchKernelGGL((k_sap44h<S, false, true>), grid, blk, 0, s, a);
      } else {
        if (c->clover) hipLaunchKernelGGL((k_sap44h<S, true, false>), grid, blk, 0, s, a);
        else hipLaunchKernelGGL((k_sap44h<S, false, false>), grid, blk, 0, s, a);
      }
    };
    half(1, false, true);  // the hops from colour 1's initial x
    for (int sw = 0; sw < nsweep; ++sw) {
      half(0, true, true);
      half(1, true, sw + 1 < nsweep);
    }
    e = hipGetLastError();
  }
  return e != hipSuccess || own_capture ? e : scratch_release(c, s);
}

}  // namespace

hipError_t launch_sap44(qmg_ctx* c, int p, void* x, const void* f, const double* tau, int nrhs, int nsweep, int n_mr,
                        hipStream_t s, int qform, bool* done) {
  if (p == QMG_F64) return sweeps<double>(c, p, x, f, tau, nrhs, nsweep, n_mr, s, qform, done);
  if (p == QMG_F32) return sweeps<float>(c, p, x, f, tau, nrhs, nsweep, n_mr, s, qform, done);
  return sweeps<bf16_t>(c, p, x, f, tau, nrhs, nsweep, n_mr, s, qform, done);
}
