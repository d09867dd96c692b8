// Vector kernels for the Krylov solvers: batched dot products (two stages,
// fixed summation order, results bitwise reproducible), batched axpy, scaling.
// A batch is nrhs vectors of n complex numbers, vector k at offset k*stride;
// a basis V_j (j < J) is at offset j*vstride.  Dot products accumulate in
// double whatever the storage precision.
#include <type_traits>

#include "qmg_ctx.h"
#include "reduce.h"

namespace {

constexpr int kDotWG = 256;
constexpr int kDotPerThread = 8;
constexpr int64_t kChunk = (int64_t)kDotWG * kDotPerThread;

// partial[(k*J + j)*nchunk + chunk] = sum over the chunk of conj(V_j,k) w_k.  Four basis
// vectors at a time, without branches inside the vector: their loads are in flight together
// and one barrier serves their sums, where each vector waited for the sum before it (coarse
// vectors of 32^4 against 10 of the basis on average, FP32: 8 rhs 55 -> 24 us, 11 rhs
// 61 -> 41; the basis of 11 leaves the Infinity Cache).
constexpr int kDotGroup = 4;
template <typename S>
__global__ __launch_bounds__(kDotWG) void k_dot_stage1(double* partial, const typename PT<S>::stor* V, int64_t vstride,
                                                      int J, const typename PT<S>::stor* w, int64_t n,
                                                      int64_t stride, int nchunk, int with_self,
                                                      int64_t vkstride) {
  constexpr int NV = 2 * kDotGroup, NW = kDotWG / 64;
  __shared__ double red[2][NW * NV];
  const int chunk = blockIdx.x, k = blockIdx.y;
  const int64_t i0 = chunk * kChunk + threadIdx.x;
  const auto* wk = w + k * stride;
  const int JT = J + with_self;
  auto body = [&](auto fullc) {
    constexpr bool kFull = decltype(fullc)::value;
    auto get = [&](const typename PT<S>::stor* p, int t) {
      const int64_t i = i0 + (int64_t)t * kDotWG;
      return kFull || i < n ? ldcv<double>(p, i) : czero<double>();
    };
    cpx<double> wl[kDotPerThread];
#pragma unroll
    for (int t = 0; t < kDotPerThread; ++t) wl[t] = get(wk, t);
    int rb = 0;
    for (int j0 = 0; j0 < JT; j0 += kDotGroup) {
      double acc[NV];
#pragma unroll
      for (int q = 0; q < kDotGroup; ++q) {
        acc[2 * q] = acc[2 * q + 1] = 0.0;
        const int j = j0 + q;
        if (j < J) {
          const auto* vj = V + j * vstride + k * vkstride;
#pragma unroll
          for (int t = 0; t < kDotPerThread; ++t) {
            const cpx<double> p = cmul_conj(get(vj, t), wl[t]);
            acc[2 * q] += p.re;
            acc[2 * q + 1] += p.im;
          }
        } else if (j < JT) {
#pragma unroll
          for (int t = 0; t < kDotPerThread; ++t) acc[2 * q] += norm2(wl[t]);
        }
      }
      double* rd = red[rb];
      rb ^= 1;
      wave_fold<NV>(acc, rd + (threadIdx.x >> 6) * NV);
      __syncthreads();
      const int v = threadIdx.x;
      if (v < NV && j0 + v / 2 < JT) {
        double t = rd[v];
#pragma unroll
        for (int g = 1; g < NW; ++g) t += rd[g * NV + v];
        partial[(((int64_t)k * JT + j0 + v / 2) * nchunk + chunk) * 2 + (v & 1)] = t;
      }
    }
  };
  // a chunk inside the vector has no bounds to check: its loads need no branches
  if ((int64_t)(chunk + 1) * kChunk <= n) body(std::true_type{});
  else body(std::false_type{});
}

// The loads of eight entries of one or two basis vectors are in flight together (8 coarse
// vectors of 32^4, FP32, 10 basis vectors: 32 -> 23 us).
// w_k = scale_k (w_k + sum_j coef[k*J+j] V_j,k) over one chunk, and partial[k][chunk] =
// ||new w_k||^2 there; scale_k = basis_scale(sig[k*ldsig + aj]), or 1 without sig.  (The
// scale on w itself made the basis wait for w: 16^4 FP64 solve 11.38 -> 11.47 ms.)
// With a copy type C (FP32 or BF16 storage), the new w is also written to cp in
// that storage, rounded through FP32 exactly as the conversion kernel rounds it.
template <typename S, typename C = void>
__global__ __launch_bounds__(kDotWG) void k_axpy_norm(typename PT<S>::stor* w, const typename PT<S>::stor* V,
                                                     int64_t vstride, int J, const double* coef, const double* sig,
                                                     int ldsig, int aj, int64_t n, int64_t stride, int nchunk,
                                                     double* partial, C* cp) {
  using R = typename PT<S>::real;
  __shared__ double red[2 * (kDotWG / 64)];
  const int chunk = blockIdx.x, k = blockIdx.y;
  const int64_t i0 = chunk * kChunk + threadIdx.x;
  auto* wk = w + k * stride;
  const double al = sig ? basis_scale(sig[(int64_t)k * ldsig + aj]) : 1.0;
  double acc[2] = {0.0, 0.0};
  auto body = [&](auto fullc) {
    constexpr bool kFull = decltype(fullc)::value;
    auto get = [&](const typename PT<S>::stor* p, int t) {
      const int64_t i = i0 + (int64_t)t * kDotWG;
      return kFull || i < n ? ldcv<double>(p, i) : czero<double>();
    };
    cpx<double> v[kDotPerThread];
#pragma unroll
    for (int t = 0; t < kDotPerThread; ++t) v[t] = get(wk, t);
#pragma unroll 2
    for (int j = 0; j < J; ++j) {
      const cpx<double> c = {coef[((int64_t)k * J + j) * 2], coef[((int64_t)k * J + j) * 2 + 1]};
      const auto* vj = V + j * vstride + k * stride;
#pragma unroll
      for (int t = 0; t < kDotPerThread; ++t) v[t] = v[t] + c * get(vj, t);
    }
#pragma unroll
    for (int t = 0; t < kDotPerThread; ++t) {
      const int64_t i = i0 + (int64_t)t * kDotWG;
      if (kFull || i < n) {
        const cpx<R> vr = {R(al * v[t].re), R(al * v[t].im)};
        const auto st = vc(vr, (typename PT<S>::stor*)nullptr);
        wk[i] = st;
        if constexpr (!std::is_void<C>::value) stcv(cp + k * stride, i, cpx<float>{float(vr.re), float(vr.im)});
        const auto sv = cv(st);  // the norm is that of the vector as stored
        acc[0] += norm2(cpx<double>{double(sv.re), double(sv.im)});
      }
    }
  };
  if ((int64_t)(chunk + 1) * kChunk <= n) body(std::true_type{});
  else body(std::false_type{});
  wg_sum<double, 2>(acc, red);
  if (threadIdx.x == 0) {
    partial[((int64_t)k * nchunk + chunk) * 2] = acc[0];
    partial[((int64_t)k * nchunk + chunk) * 2 + 1] = 0.0;
  }
}

// dots[k*J + j] = ordered tree sum of the partials
__global__ __launch_bounds__(256) void k_dot_stage2(double* dots, const double* partial, int J, int nchunk) {
  __shared__ double red[2 * 4];
  const int j = blockIdx.x, k = blockIdx.y;
  const double* p = partial + ((int64_t)k * J + j) * nchunk * 2;
  double acc[2] = {0.0, 0.0};
  for (int c = threadIdx.x; c < nchunk; c += blockDim.x) {
    acc[0] += p[2 * c];
    acc[1] += p[2 * c + 1];
  }
  wg_sum<double, 2>(acc, red);
  if (threadIdx.x == 0) {
    dots[((int64_t)k * J + j) * 2] = acc[0];
    dots[((int64_t)k * J + j) * 2 + 1] = acc[1];
  }
}

// As k_dot_stage2 for the projections of one Gram-Schmidt pass: dots as it, and for j < J
// also the update's coefficients coef[k*J + j] = -sig_j^2 dots (basis v_j = sig_j W_j)
__global__ __launch_bounds__(256) void k_project_stage2(double* dots, double* coef, const double* partial,
                                                        const double* sig, int ldsig, int J, int JT, int nchunk) {
  __shared__ double red[2 * 4];
  const int j = blockIdx.x, k = blockIdx.y;
  const double s = sig[(int64_t)k * ldsig + min(j, J - 1)];  // before the sums, not after
  const double* p = partial + ((int64_t)k * JT + j) * nchunk * 2;
  double acc[2] = {0.0, 0.0};
  for (int c = threadIdx.x; c < nchunk; c += blockDim.x) {
    acc[0] += p[2 * c];
    acc[1] += p[2 * c + 1];
  }
  wg_sum<double, 2>(acc, red);
  if (threadIdx.x == 0) {
    dots[((int64_t)k * JT + j) * 2] = acc[0];
    dots[((int64_t)k * JT + j) * 2 + 1] = acc[1];
    if (j < J) {
      const double s2 = -s * s;
      coef[((int64_t)k * J + j) * 2] = s2 * acc[0];
      coef[((int64_t)k * J + j) * 2 + 1] = s2 * acc[1];
    }
  }
}

// norms[2k] = ||w_k||^2, norms[2k + 1] = basis_scale(sig_aj) (1 for aj < 0), and the scale of
// w_k as basis vector `at`: sig = 1 / ||w_k||
__global__ __launch_bounds__(256) void k_norm_stage2(double* norms, const double* partial, double* sig, int ldsig,
                                                     int aj, int at, int nchunk) {
  __shared__ double red[2 * 4];
  const int k = blockIdx.x;
  const double scale = aj < 0 ? 1.0 : basis_scale(sig[(int64_t)k * ldsig + aj]);
  const double* p = partial + (int64_t)k * nchunk * 2;
  double acc[2] = {0.0, 0.0};
  for (int c = threadIdx.x; c < nchunk; c += blockDim.x) acc[0] += p[2 * c];
  wg_sum<double, 2>(acc, red);
  if (threadIdx.x == 0) {
    norms[2 * k] = acc[0];
    norms[2 * k + 1] = scale;
    const double h = sqrt(fmax(acc[0], 0.0));
    sig[(int64_t)k * ldsig + at] = h > 0.0 && isfinite(h) ? 1.0 / h : 0.0;
  }
}

__global__ void k_sig_init(double* sig, int ldsig, int nrhs) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ldsig * nrhs) sig[i] = i % ldsig == 0 ? 1.0 : 0.0;
}

// sig_at = 0 for the right-hand sides in mask
__global__ void k_sig_drop(double* sig, int ldsig, int at, uint64_t mask, int nrhs) {
  const int k = threadIdx.x;
  if (k < nrhs && (mask >> k & 1)) sig[(int64_t)k * ldsig + at] = 0.0;
}

template <typename S, typename SV = S>
__global__ __launch_bounds__(256) void k_multiaxpy(typename PT<S>::stor* w, const typename PT<SV>::stor* V,
                                                   int64_t vstride, int J, const double* coef, int64_t n,
                                                   int64_t stride) {
  using R = typename PT<S>::real;
  const int k = blockIdx.y;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  auto* wk = w + k * stride;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
    cpx<double> acc = ldcv<double>(wk, i);
    for (int j = 0; j < J; ++j) {
      cpx<double> c = {coef[((int64_t)k * J + j) * 2], coef[((int64_t)k * J + j) * 2 + 1]};
      acc = acc + c * ldcv<double>(V + j * vstride + k * stride, i);
    }
    stcv(wk, i, cpx<R>{R(acc.re), R(acc.im)});
  }
}

// y_k = a_k x_k; with a copy type C (FP32 or BF16 storage) the result is also
// written to cp, rounded through FP32 as the conversion kernel rounds it
template <typename S, typename C = void>
__global__ __launch_bounds__(256) void k_scale(typename PT<S>::stor* y, const typename PT<S>::stor* x, const double* a,
                                               int64_t n, int64_t stride, C* cp) {
  using R = typename PT<S>::real;
  const int k = blockIdx.y;
  const cpx<double> ak = {a[2 * k], a[2 * k + 1]};
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
    cpx<double> v = ak * ldcv<double>(x + k * stride, i);
    const cpx<R> vr = {R(v.re), R(v.im)};
    stcv(y + k * stride, i, vr);
    if constexpr (!std::is_void<C>::value) stcv(cp + k * stride, i, cpx<float>{float(vr.re), float(vr.im)});
  }
}

template <typename S>
__global__ __launch_bounds__(256) void k_xmy(typename PT<S>::stor* y, const typename PT<S>::stor* x, int64_t n,
                                             int64_t stride) {
  using R = typename PT<S>::real;
  const int k = blockIdx.y;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
    cpx<R> v = ldcv<R>(x + k * stride, i) - ldcv<R>(y + k * stride, i);
    stcv(y + k * stride, i, v);
  }
}

// y = Gamma5 x on fine fields (spins 2, 3 change sign); n = total complex elements
template <typename S>
__global__ __launch_bounds__(256) void k_gamma5(typename PT<S>::stor* y, const typename PT<S>::stor* x, int64_t n,
                                                int bs_log) {
  using R = typename PT<S>::real;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
    const int comp = (int)((i >> bs_log) % 12);
    cpx<R> v = ldcv<R>(x, i);
    stcv(y, i, comp >= 6 ? -v : v);
  }
}

// plain streaming copy, 16 B per lane per step (bandwidth probe)
__global__ __launch_bounds__(256) void k_stream_copy(uint4* dst, const uint4* src, int64_t n) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) dst[i] = src[i];
}

__global__ void k_zero(uint32_t* p, int64_t n) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) p[i] = 0u;
}

unsigned ew_grid(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192)); }

template <typename F>
void by_prec(int p, F&& f) {
  if (p == QMG_F64) f(double{});
  else if (p == QMG_F32) f(float{});
  else f(bf16_t{});
}

}  // namespace

int dot_chunks(int64_t n) { return (int)((n + kChunk - 1) / kChunk); }

hipError_t launch_dot_partials(int p, const void* V, int64_t vstride, int J, const void* w, int64_t n, int64_t stride,
                               int nrhs, double* partial, hipStream_t s, int with_self) {
  const int nchunk = dot_chunks(n);
  by_prec(p, [&](auto tag) {
    using S = decltype(tag);
    using P = typename PT<S>::stor;
    hipLaunchKernelGGL(k_dot_stage1<S>, dim3(nchunk, nrhs), dim3(kDotWG), 0, s, partial, (const P*)V, vstride, J,
                       (const P*)w, n, stride, nchunk, with_self, stride);
  });
  return hipGetLastError();
}

hipError_t launch_multidot(int p, double* dots, const void* V, int64_t vstride, int J, const void* w, int64_t n,
                           int64_t stride, int nrhs, double* partial, hipStream_t s, int with_self) {
  const hipError_t e = launch_dot_partials(p, V, vstride, J, w, n, stride, nrhs, partial, s, with_self);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dot_stage2, dim3(J + with_self, nrhs), dim3(256), 0, s, dots, partial, J + with_self,
                     dot_chunks(n));
  return hipGetLastError();
}

// dots[(k*J + j)*2] = <V_j, w_k> for nw vectors w_k (offset k*wstride) against
// one shared basis: the work-groups of all w_k read a basis chunk together
hipError_t launch_multidot_shared(int p, double* dots, const void* V, int64_t vstride, int J, const void* w,
                                  int64_t wstride, int nw, int64_t n, double* partial, hipStream_t s) {
  const int nchunk = (int)((n + kChunk - 1) / kChunk);
  by_prec(p, [&](auto tag) {
    using S = decltype(tag);
    using P = typename PT<S>::stor;
    hipLaunchKernelGGL(k_dot_stage1<S>, dim3(nchunk, nw), dim3(kDotWG), 0, s, partial, (const P*)V, vstride, J,
                       (const P*)w, n, wstride, nchunk, 0, (int64_t)0);
  });
  hipLaunchKernelGGL(k_dot_stage2, dim3(J, nw), dim3(256), 0, s, dots, partial, J, nchunk);
  return hipGetLastError();
}

// w_k = scale_k (w_k + sum_j coef V_j,k); partial[k][chunk] = ||w_k||^2 over the chunk afterwards
hipError_t launch_axpy_partials(int p, void* w, const void* V, int64_t vstride, int J, const double* coef, int64_t n,
                                int64_t stride, int nrhs, double* partial, hipStream_t s, void* copy, int copy_prec,
                                const double* sig, int ldsig, int aj) {
  const int nchunk = dot_chunks(n);
  const dim3 grid(nchunk, nrhs), blk(kDotWG);
  if (copy && p == QMG_F64 && copy_prec == QMG_F32) {
    hipLaunchKernelGGL((k_axpy_norm<double, float2>), grid, blk, 0, s, (double2*)w, (const double2*)V, vstride, J,
                       coef, sig, ldsig, aj, n, stride, nchunk, partial, (float2*)copy);
  } else if (copy && p == QMG_F64 && copy_prec == QMG_BF16) {
    hipLaunchKernelGGL((k_axpy_norm<double, uint32_t>), grid, blk, 0, s, (double2*)w, (const double2*)V, vstride, J,
                       coef, sig, ldsig, aj, n, stride, nchunk, partial, (uint32_t*)copy);
  } else {
    if (copy) return hipErrorInvalidValue;  // only FP64 vectors are copied to FP32 / BF16
    by_prec(p, [&](auto tag) {
      using S = decltype(tag);
      using P = typename PT<S>::stor;
      hipLaunchKernelGGL((k_axpy_norm<S, void>), grid, blk, 0, s, (P*)w, (const P*)V, vstride, J, coef, sig, ldsig,
                         aj, n, stride, nchunk, partial, (void*)nullptr);
    });
  }
  return hipGetLastError();
}

hipError_t launch_project(int p, double* dots, double* coef, const double* sig, int ldsig, const void* V,
                          int64_t vstride, int J, const void* w, int64_t n, int64_t stride, int nrhs, double* partial,
                          hipStream_t s, int with_self) {
  const hipError_t e = launch_dot_partials(p, V, vstride, J, w, n, stride, nrhs, partial, s, with_self);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_project_stage2, dim3(J + with_self, nrhs), dim3(256), 0, s, dots, coef, partial, sig, ldsig, J,
                     J + with_self, dot_chunks(n));
  return hipGetLastError();
}

hipError_t launch_axpy_sig(int p, void* w, const void* V, int64_t vstride, int J, const double* coef, int64_t n,
                           int64_t stride, int nrhs, double* norms, double* sig, int ldsig, int aj, int at,
                           double* partial, hipStream_t s, void* copy, int copy_prec) {
  const hipError_t e = launch_axpy_partials(p, w, V, vstride, J, coef, n, stride, nrhs, partial, s, copy, copy_prec,
                                            aj < 0 ? nullptr : sig, ldsig, aj);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_norm_stage2, dim3(nrhs), dim3(256), 0, s, norms, partial, sig, ldsig, aj, at, dot_chunks(n));
  return hipGetLastError();
}

hipError_t launch_sig_drop(double* sig, int ldsig, int at, uint64_t mask, int nrhs, hipStream_t s) {
  static_assert(QMG_MAXRHS <= 64, "one bit per right-hand side");
  hipLaunchKernelGGL(k_sig_drop, dim3(1), dim3(64), 0, s, sig, ldsig, at, mask, nrhs);
  return hipGetLastError();
}

hipError_t launch_sig_init(double* sig, int ldsig, int nrhs, hipStream_t s) {
  hipLaunchKernelGGL(k_sig_init, dim3((ldsig * nrhs + 255) / 256), dim3(256), 0, s, sig, ldsig, nrhs);
  return hipGetLastError();
}

// scratch needed by launch_multidot, launch_dot_partials and launch_axpy_partials: doubles
size_t multidot_partial_doubles(int64_t n, int J, int nrhs) {
  return (size_t)((n + kChunk - 1) / kChunk) * (J + 1) * nrhs * 2;
}

hipError_t launch_multiaxpy(int p, void* w, const void* V, int64_t vstride, int J, const double* coef, int64_t n,
                            int64_t stride, int nrhs, hipStream_t s) {
  by_prec(p, [&](auto tag) {
    using S = decltype(tag);
    using P = typename PT<S>::stor;
    hipLaunchKernelGGL(k_multiaxpy<S>, dim3(ew_grid(n), nrhs), dim3(256), 0, s, (P*)w, (const P*)V, vstride, J,
                       coef, n, stride);
  });
  return hipGetLastError();
}

hipError_t launch_multiaxpy_d(void* w, const void* V, int vprec, int64_t vstride, int J, const double* coef,
                              int64_t n, int64_t stride, int nrhs, hipStream_t s) {
  by_prec(vprec, [&](auto tag) {
    using SV = decltype(tag);
    using PV = typename PT<SV>::stor;
    hipLaunchKernelGGL((k_multiaxpy<double, SV>), dim3(ew_grid(n), nrhs), dim3(256), 0, s, (double2*)w, (const PV*)V,
                       vstride, J, coef, n, stride);
  });
  return hipGetLastError();
}

hipError_t launch_scale(int p, void* y, const void* x, const double* a, int64_t n, int64_t stride, int nrhs,
                        hipStream_t s, void* copy, int copy_prec) {
  const dim3 grid(ew_grid(n), nrhs), blk(256);
  if (copy && p == QMG_F64 && copy_prec == QMG_F32) {
    hipLaunchKernelGGL((k_scale<double, float2>), grid, blk, 0, s, (double2*)y, (const double2*)x, a, n, stride,
                       (float2*)copy);
  } else if (copy && p == QMG_F64 && copy_prec == QMG_BF16) {
    hipLaunchKernelGGL((k_scale<double, uint32_t>), grid, blk, 0, s, (double2*)y, (const double2*)x, a, n, stride,
                       (uint32_t*)copy);
  } else {
    if (copy) return hipErrorInvalidValue;  // only FP64 vectors are copied to FP32 / BF16
    by_prec(p, [&](auto tag) {
      using S = decltype(tag);
      using P = typename PT<S>::stor;
      hipLaunchKernelGGL((k_scale<S, void>), grid, blk, 0, s, (P*)y, (const P*)x, a, n, stride, (void*)nullptr);
    });
  }
  return hipGetLastError();
}

template <typename S>
__global__ __launch_bounds__(256) void k_add(typename PT<S>::stor* y, const typename PT<S>::stor* x, int64_t n,
                                             int64_t stride) {
  using R = typename PT<S>::real;
  const int k = blockIdx.y;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
    const cpx<R> v = ldcv<R>(y + k * stride, i) + ldcv<R>(x + k * stride, i);
    stcv(y + k * stride, i, v);
  }
}

hipError_t launch_add(int p, void* y, const void* x, int64_t n, int64_t stride, int nrhs, hipStream_t s) {
  by_prec(p, [&](auto tag) {
    using S = decltype(tag);
    using P = typename PT<S>::stor;
    hipLaunchKernelGGL(k_add<S>, dim3(ew_grid(n), nrhs), dim3(256), 0, s, (P*)y, (const P*)x, n, stride);
  });
  return hipGetLastError();
}

hipError_t launch_xmy(int p, void* y, const void* x, int64_t n, int64_t stride, int nrhs, hipStream_t s) {
  by_prec(p, [&](auto tag) {
    using S = decltype(tag);
    using P = typename PT<S>::stor;
    hipLaunchKernelGGL(k_xmy<S>, dim3(ew_grid(n), nrhs), dim3(256), 0, s, (P*)y, (const P*)x, n, stride);
  });
  return hipGetLastError();
}

hipError_t launch_gamma5_bs(int p, void* y, const void* x, int64_t n, int bs_log, hipStream_t s) {
  by_prec(p, [&](auto tag) {
    using S = decltype(tag);
    using P = typename PT<S>::stor;
    hipLaunchKernelGGL(k_gamma5<S>, dim3(ew_grid(n)), dim3(256), 0, s, (P*)y, (const P*)x, n, bs_log);
  });
  return hipGetLastError();
}

hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 16);
  // 4 work-groups per CU of 256 threads: enough loads in flight to saturate HBM
  // with each lane streaming a long contiguous range of 16-B chunks
  if (n > 0) hipLaunchKernelGGL(k_stream_copy, dim3(1024), dim3(256), 0, s, (uint4*)dst, (const uint4*)src, n);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* y, size_t bytes, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 4);
  if (n > 0) hipLaunchKernelGGL(k_zero, dim3(ew_grid(n)), dim3(256), 0, s, (uint32_t*)y, n);
  return hipGetLastError();
}
