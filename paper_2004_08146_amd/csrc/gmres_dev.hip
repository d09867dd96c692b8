// Device-resident GMRES scalars (Hessenberg column, Givens rotations,
// back-substitution) so a fixed-step coarse GMRES -- and with it the whole
// V-cycle -- runs without host round trips and can be captured in a HIP graph.
// The same driver runs the GMRES smoother on the fine level and, with a third
// level, the level-3 GMRES and the level-2 flexible GMRES (K-cycle).
// Being part of the preconditioner, this coarse GMRES makes a single classical
// Gram-Schmidt pass per step (no data-dependent second pass).  The basis is
// stored unnormalised after its first vector (v_j = sig_j W_j, W_j the stored
// vector): each product is orthogonalised in place in the next basis slot, so
// no scaling pass is needed, and the last step, whose new vector is never used,
// takes ||w_new||^2 = ||w||^2 - sum_i |v_i^H w|^2 from its dot pass instead of
// an update pass.  The update also gives its result a power of two near sig_j, so that
// ||W_{j+1}|| stays near h_{j+1,j} for any number of steps.
// One thread per right-hand side; the rotations follow the same convention as
// the host solver: [[c, s], [-conj(s), c]] [a; b] = [r; 0], c real.
#include <functional>
#include <string>

#include "qmg_ctx.h"
#include "reduce.h"

namespace {

struct GmState {
  double* H;     // [nrhs][m+1][m] complex (row-major: (i, j) at i*m + j)
  double* g;     // [nrhs][m+1] complex
  double* cs;    // [nrhs][m]
  double* sn;    // [nrhs][m] complex
  double* beta;  // [nrhs]
  double* sig;   // [nrhs][m+1]: v_j = sig_j W_j
  int m;
};

__device__ inline cpx<double> ldz(const double* p, int64_t i) { return {p[2 * i], p[2 * i + 1]}; }
__device__ inline void stz(double* p, int64_t i, cpx<double> v) { p[2 * i] = v.re; p[2 * i + 1] = v.im; }

// beta = ||r||, a = 1/beta (0 if beta == 0), g = (beta, 0, ...), H = 0
__global__ void k_gm_init(GmState st, const double* norms, double* a, int nrhs) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nrhs) return;
  const double b = sqrt(fmax(norms[2 * k], 0.0));
  st.beta[k] = b;
  a[2 * k] = b > 0 ? 1.0 / b : 0.0;
  a[2 * k + 1] = 0.0;
  const int m = st.m;
  for (int i = 0; i <= m; ++i) stz(st.g, (int64_t)k * (m + 1) + i, cpx<double>{i == 0 ? b : 0.0, 0.0});
  for (int i = 0; i < (m + 1) * m; ++i) stz(st.H, (int64_t)k * (m + 1) * m + i, czero<double>());
  for (int i = 0; i <= m; ++i) st.sig[(int64_t)k * (m + 1) + i] = i == 0 ? 1.0 : 0.0;
}

constexpr int kGmWG = 256;
// sums of the nchunk partial results (pairs) of value j, in every thread's out[j], j < J
__device__ void gm_sums(const double* partial, int J, int nchunk, double (*out)[2]) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int j = wave; j < J; j += kGmWG / 64) {
    double re = 0.0, im = 0.0;
    for (int c = lane; c < nchunk; c += 64) {
      re += partial[((int64_t)j * nchunk + c) * 2];
      im += partial[((int64_t)j * nchunk + c) * 2 + 1];
    }
    re = wave_sum63(re);
    im = wave_sum63(im);
    if (lane == 63) {
      out[j][0] = re;
      out[j][1] = im;
    }
  }
  __syncthreads();
}

// close column j: h_{j+1,j} = sig_j ||w_new|| / scale (w_new = the projected A W_j times
// scale, stored as W_{j+1}, so sig_{j+1} = 1 / ||w_new||), rotate, update g; one thread,
// hc: the column's entries 0..j
__device__ void gm_close(const GmState& st, int k, int j, double norm2w, double scale, double (*hc)[2]) {
  const int m = st.m;
  double* H = st.H + (int64_t)k * (m + 1) * m * 2;
  double* g = st.g + (int64_t)k * (m + 1) * 2;
  double* cs = st.cs + (int64_t)k * m;
  double* sn = st.sn + (int64_t)k * m * 2;
  double* sg = st.sig + (int64_t)k * (m + 1);
  const double wn = sqrt(fmax(norm2w, 0.0));
  const double hn = scale > 0 ? sg[j] / scale * wn : 0.0;
  sg[j + 1] = wn > 0 ? 1.0 / wn : 0.0;
  cpx<double> cur = {hc[0][0], hc[0][1]};
  for (int i = 0; i < j; ++i) {
    const cpx<double> hi1 = {hc[i + 1][0], hc[i + 1][1]};
    const double c = cs[i];
    const cpx<double> s = ldz(sn, i);
    stz(H, (int64_t)i * m + j, c * cur + s * hi1);
    cur = c * hi1 - conj(s) * cur;
  }
  const cpx<double> h1 = {hn, 0.0};
  double c;
  cpx<double> s;
  const double na = sqrt(norm2(cur)), nb = hn;
  if (nb == 0.0) { c = 1.0; s = czero<double>(); }
  else if (na == 0.0) { c = 0.0; s = cpx<double>{1.0, 0.0}; }
  else {
    const double rho = sqrt(na * na + nb * nb);
    c = na / rho;
    s = (1.0 / (na * rho)) * (cur * conj(h1));
  }
  cs[j] = c;
  stz(sn, j, s);
  stz(H, (int64_t)j * m + j, c * cur + s * h1);
  const cpx<double> gj = ldz(g, j);
  stz(g, j + 1, -(conj(s) * gj));
  stz(g, j, c * gj);
}

// One classical Gram-Schmidt pass for w = A W_j, d_i = W_i^H w summed here from the chunk
// sums: H[i][j] = sig_i sig_j d_i, coef_i = -sig_i^2 d_i (w -= (v_i^H w) v_i).
// last: the sums also hold ||w||^2 (at index J); the squared norm of the projected w,
// ||w||^2 - sum_i sig_i^2 |d_i|^2, takes the place of the update pass and the column is
// closed at once.  One work-group per right-hand side, which also closes the column where
// five launches of a few waves did (16 of 32 us a step at 32^4, 8 rhs, now 11).
// longcol: work-group k's column in memory, for more steps than fit in LDS (else null).
__global__ __launch_bounds__(kGmWG) void k_gm_coef(GmState st, const double* partial, int nchunk, double* coef, int j,
                                                   int last, double* longcol) {
  extern __shared__ double gsh[];
  const int k = blockIdx.x;
  double(*d)[2] = reinterpret_cast<double(*)[2]>(longcol ? longcol + (int64_t)k * 2 * (st.m + 2) : gsh);
  const int J = j + 1, m = st.m, ld = J + (last ? 1 : 0);
  gm_sums(partial + (int64_t)k * ld * nchunk * 2, ld, nchunk, d);
  const double* sg = st.sig + (int64_t)k * (m + 1);
  if (!last) {
    for (int i = threadIdx.x; i < J; i += kGmWG) {
      const cpx<double> di = {d[i][0], d[i][1]};
      stz(coef, (int64_t)k * J + i, -(sg[i] * sg[i]) * di);
      stz(st.H, (int64_t)k * (m + 1) * m + (int64_t)i * m + j, (sg[i] * sg[j]) * di);
    }
  } else if (threadIdx.x == 0) {  // scales d in place: no other thread reads it here
    double proj = 0.0;
    for (int i = 0; i < J; ++i) {
      const double s2 = sg[i] * sg[i];
      proj += s2 * (d[i][0] * d[i][0] + d[i][1] * d[i][1]);
      d[i][0] *= sg[i] * sg[j];
      d[i][1] *= sg[i] * sg[j];
    }
    gm_close(st, k, j, fmax(d[J][0] - proj, 0.0), 1.0, d);
  }
}

// closes column j from the chunk sums of ||w_new||^2
__global__ __launch_bounds__(kGmWG) void k_gm_col(GmState st, const double* partial, int nchunk, int j,
                                                  double* longcol) {
  extern __shared__ double gsh[];
  __shared__ double nrm[1][2];
  const int k = blockIdx.x, m = st.m;
  double(*hc)[2] = reinterpret_cast<double(*)[2]>(longcol ? longcol + (int64_t)k * 2 * (m + 2) : gsh);
  for (int i = threadIdx.x; i <= j; i += kGmWG) {
    const cpx<double> h = ldz(st.H, (int64_t)k * (m + 1) * m + (int64_t)i * m + j);
    hc[i][0] = h.re;
    hc[i][1] = h.im;
  }
  gm_sums(partial + (int64_t)k * nchunk * 2, 1, nchunk, nrm);
  if (threadIdx.x == 0) gm_close(st, k, j, nrm[0][0], basis_scale(st.sig[(int64_t)k * (m + 1) + j]), hc);
}

// y = R^{-1} g (R: the rotated Hessenberg, kk columns) -> coef[k][0..kk)
__global__ void k_gm_solve(GmState st, double* coef, int kk, int nrhs) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nrhs) return;
  const int m = st.m;
  const double* H = st.H + (int64_t)k * (m + 1) * m * 2;
  const double* g = st.g + (int64_t)k * (m + 1) * 2;
  for (int i = kk - 1; i >= 0; --i) {
    cpx<double> t = ldz(g, i);
    for (int l = i + 1; l < kk; ++l) t = t - ldz(H, (int64_t)i * m + l) * ldz(coef, (int64_t)k * kk + l);
    const cpx<double> d = ldz(H, (int64_t)i * m + i);
    const double dd = norm2(d);
    // a zero pivot only follows an exact breakdown; that column adds nothing
    stz(coef, (int64_t)k * kk + i, dd > 0 ? cpx<double>{(t.re * d.re + t.im * d.im) / dd, (t.im * d.re - t.re * d.im) / dd}
                                         : czero<double>());
  }
  // y_i multiplies v_i = sig_i W_i (or M v_i = sig_i Z_i): coefficients of the stored vectors
  const double* sg = st.sig + (int64_t)k * (m + 1);
  for (int i = 0; i < kk; ++i) stz(coef, (int64_t)k * kk + i, sg[i] * ldz(coef, (int64_t)k * kk + i));
}

}  // namespace

// The operator of a device GMRES run: n complex elements per right-hand side
// in storage precision cp; prec set: flexible GMRES, right-preconditioned by
// prec (the preconditioned directions are kept and form the update).
struct DevOp {
  int64_t n;
  int cp;
  std::string tag;  // workspace name prefix (nested runs need distinct tags)
  std::function<hipError_t(void* out, const void* in)> apply;
  std::function<qmg_status(void* z, const void* v)> prec;
};

// Fixed-step (F)GMRES from zero with every scalar on the device
// (graph-capturable).  Work buffers come from ws (allocate them before a
// capture with the same sizes).
static qmg_status gmres_device(qmg_ctx* c, const DevOp& op, void* y, const void* r, int nrhs, int iters,
                               hipStream_t s) {
  const int cp = op.cp;
  const int64_t n = op.n;
  const size_t vb = (size_t)n * cbytes(cp);
  const size_t bb = vb * nrhs;
  const int m = iters;
  const std::string& tag = op.tag;
  const bool flex = (bool)op.prec;
  void* V = ws_get(c, tag + "_V", bb * (m + 1));
  void* Z = flex ? ws_get(c, tag + "_Z", bb * m) : nullptr;
  double* part = (double*)ws_get(c, tag + "_part", sizeof(double) * multidot_partial_doubles(n, m + 2, nrhs));
  double* coef = (double*)ws_get(c, tag + "_coef", sizeof(double) * 2 * (m + 1) * nrhs);
  double* a = (double*)ws_get(c, tag + "_a", sizeof(double) * 2 * nrhs);
  double* nrm = (double*)ws_get(c, tag + "_nrm", sizeof(double) * 2 * nrhs);
  GmState st;
  st.m = m;
  st.H = (double*)ws_get(c, tag + "_H", sizeof(double) * 2 * (m + 1) * m * nrhs);
  st.g = (double*)ws_get(c, tag + "_g", sizeof(double) * 2 * (m + 1) * nrhs);
  st.cs = (double*)ws_get(c, tag + "_cs", sizeof(double) * m * nrhs);
  st.sn = (double*)ws_get(c, tag + "_sn", sizeof(double) * 2 * m * nrhs);
  st.beta = (double*)ws_get(c, tag + "_beta", sizeof(double) * nrhs);
  st.sig = (double*)ws_get(c, tag + "_sig", sizeof(double) * (m + 1) * nrhs);
  if (!V || (flex && !Z) || !part || !coef || !a || !nrm || !st.H || !st.g || !st.cs || !st.sn ||
      !st.beta || !st.sig)
    return set_err(c, QMG_E_NOMEM, "out of device memory (device GMRES)");
  const dim3 g1((nrhs + 63) / 64), b1(64);
  const int64_t vs = n * nrhs;
  const int nchunk = dot_chunks(n);
  const bool big = m > 2000;
  double* longcol = big ? (double*)ws_get(c, tag + "_dots", sizeof(double) * 2 * (m + 2) * nrhs) : nullptr;
  if (big && !longcol) return set_err(c, QMG_E_NOMEM, "out of device memory (device GMRES)");
  hipError_t e = launch_multidot(cp, nrm, r, 0, 0, r, n, n, nrhs, part, s, 1);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_gm_init, g1, b1, 0, s, st, nrm, a, nrhs);
    e = launch_scale(cp, V, r, a, n, n, nrhs, s);
  }
  for (int j = 0; j < m && e == hipSuccess; ++j) {
    char* Vj = (char*)V + (size_t)j * bb;
    char* w = Vj + bb;  // the product is orthogonalised in place in slot j + 1
    const int last = j + 1 == m ? 1 : 0;
    if (flex) {
      char* Zj = (char*)Z + (size_t)j * bb;
      qmg_status ps = op.prec(Zj, Vj);
      if (ps != QMG_OK) return ps;
      e = op.apply(w, Zj);
    } else {
      e = op.apply(w, Vj);
    }
    const size_t lds = longcol ? 0 : sizeof(double) * 2 * (j + 2);
    if (e == hipSuccess) e = launch_dot_partials(cp, V, vs, j + 1, w, n, n, nrhs, part, s, last);
    if (e == hipSuccess) {
      hipLaunchKernelGGL(k_gm_coef, dim3(nrhs), dim3(kGmWG), lds, s, st, part, nchunk, coef, j, last, longcol);
      if (!last) {
        e = launch_axpy_partials(cp, w, V, vs, j + 1, coef, n, n, nrhs, part, s, nullptr, QMG_F64, st.sig, m + 1, j);
        if (e == hipSuccess) hipLaunchKernelGGL(k_gm_col, dim3(nrhs), dim3(kGmWG), lds, s, st, part, nchunk, j, longcol);
      }
      if (e == hipSuccess) e = hipGetLastError();
    }
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_gm_solve, g1, b1, 0, s, st, coef, m, nrhs);
    e = launch_fill_zero(y, bb, s);
  }
  if (e == hipSuccess) e = launch_multiaxpy(cp, y, flex ? Z : V, vs, m, coef, n, n, nrhs, s);
  if (e != hipSuccess) return hip_err(c, e, "device GMRES");
  return QMG_OK;
}

// GMRES on the coarse operator (coarse precision of p); shares its basis
// buffers with the host-driven coarse GMRES (never live at the same time)
qmg_status coarse_gmres_device(qmg_ctx* c, int p, void* y, const void* r, const double* tau, int nrhs, int iters,
                               hipStream_t s, int qform) {
  DevOp op{(int64_t)coarse_elems(c), coarse_prec(p), "cg",
           [=](void* out, const void* in) { return launch_coarse_apply(c, p, out, in, tau, nrhs, s, qform); }, {}};
  return gmres_device(c, op, y, r, nrhs, iters, s);
}

// GMRES on the fine stencil in precision p (the smoother of Sec. 2's GMRES option)
qmg_status fine_gmres_device(qmg_ctx* c, int p, void* y, const void* r, const double* tau, int nrhs, int iters,
                             hipStream_t s, int qform) {
  DevOp op{(int64_t)field_elems(c), p, "fs",
           [=](void* out, const void* in) { return launch_dslash(c, p, out, in, tau, nrhs, qform ? 1 : 0, s); }, {}};
  return gmres_device(c, op, y, r, nrhs, iters, s);
}

// ---- third level.  M2 r2 = z: P2 y3 with y3 from k3 GMRES steps on
// A3(tau) y3 = P2^H r2, then s2 GMRES steps from zero on A_c e = r2 - A_c z
// and z + e.  Level-2 and level-3 vectors are in the coarse precision of p.
qmg_status level2_cycle(qmg_ctx* c, int p, void* z, const void* r, const double* tau, int nrhs, int k3, int s2,
                        hipStream_t s, int qform) {
  const int cp = coarse_prec(p);
  const int64_t n2 = (int64_t)coarse_elems(c), n3 = (int64_t)l3_elems(c);
  void* r3 = ws_get(c, "l3_r", (size_t)n3 * nrhs * cbytes(cp));
  void* y3 = ws_get(c, "l3_y", (size_t)n3 * nrhs * cbytes(cp));
  if (!r3 || !y3) return set_err(c, QMG_E_NOMEM, "out of device memory (level-2 cycle)");
  hipError_t e = launch_restrict_l3(c, p, r3, r, nrhs, s);
  if (e != hipSuccess) return hip_err(c, e, "restrict to level 3");
  DevOp op3{n3, cp, "l3g",
            [=](void* out, const void* in) { return launch_apply_l3(c, p, out, in, tau, nrhs, s, qform); }, {}};
  qmg_status st = gmres_device(c, op3, y3, r3, nrhs, k3, s);
  if (st != QMG_OK) return st;
  e = launch_prolong_l3(c, p, z, y3, nrhs, s);
  if (e != hipSuccess) return hip_err(c, e, "prolong from level 3");
  if (s2 > 0) {
    void* az = ws_get(c, "l2_az", (size_t)n2 * nrhs * cbytes(cp));
    void* ez = ws_get(c, "l2_ez", (size_t)n2 * nrhs * cbytes(cp));
    if (!az || !ez) return set_err(c, QMG_E_NOMEM, "out of device memory (level-2 smoothing)");
    e = launch_coarse_apply(c, p, az, z, tau, nrhs, s, qform);
    if (e == hipSuccess) e = launch_xmy(cp, az, r, n2, n2, nrhs, s);
    if (e != hipSuccess) return hip_err(c, e, "level-2 smoothing residual");
    st = coarse_gmres_device(c, p, ez, az, tau, nrhs, s2, s, qform);
    if (st != QMG_OK) return st;
    e = launch_add(cp, z, ez, n2, n2, nrhs, s);
    if (e != hipSuccess) return hip_err(c, e, "level-2 smoothing update");
  }
  return QMG_OK;
}

// k2 FGMRES steps from zero on A_c(tau) y = r, right-preconditioned by M2
// (a K-cycle on level 2)
qmg_status level2_kcycle(qmg_ctx* c, int p, void* y, const void* r, const double* tau, int nrhs, int k2, int k3,
                         int s2, hipStream_t s, int qform) {
  DevOp op{(int64_t)coarse_elems(c), coarse_prec(p), "kc",
           [=](void* out, const void* in) { return launch_coarse_apply(c, p, out, in, tau, nrhs, s, qform); },
           [=](void* z, const void* v) { return level2_cycle(c, p, z, v, tau, nrhs, k3, s2, s, qform); }};
  return gmres_device(c, op, y, r, nrhs, k2, s);
}
