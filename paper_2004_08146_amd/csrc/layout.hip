// Canonical <-> block-major field layout and precision conversion.
#include "qmg_ctx.h"

namespace {

// 256 sites in block order per work-group, transposed through LDS: the canonical side is
// read and written in runs of a block's last direction (768 B for 4^4 blocks), the internal
// side in rows of sites.  With one thread walking its site's 192 B the canonical accesses
// were 16 B apart by 192: 32x16^3 FP64 pack 16.8 -> 15.1 us, unpack 21.5 -> 10.6.
constexpr int kTile = 256, kRow = kTile + 1;

template <typename S>
__global__ __launch_bounds__(256) void k_pack(Geom g, typename PT<S>::stor* out, const double2* canon) {
  __shared__ double2 sh[12 * kRow];
  const int64_t s0 = (int64_t)blockIdx.x * kTile;
  const int ns = (int)min((int64_t)kTile, g.V - s0);
  const double2* src = canon + (int64_t)blockIdx.y * g.V * 12;
  auto* dst = out + (int64_t)blockIdx.y * g.V * 12;
  double2 v[12];  // all loads in flight together
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const int e = min((int)threadIdx.x + 256 * k, 12 * ns - 1), c = e % 12;
    const int64_t site = s0 + e / 12;
    v[k] = src[canon_site(g, (int)(site >> g.bs_log), (int)(site & ((1 << g.bs_log) - 1))) * 12 + c];
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const int e = min((int)threadIdx.x + 256 * k, 12 * ns - 1);
    sh[(e % 12) * kRow + e / 12] = v[k];
  }
  __syncthreads();
  const int i = threadIdx.x;
  if (i >= ns) return;
  const int b = (int)((s0 + i) >> g.bs_log), l = (int)((s0 + i) & ((1 << g.bs_log) - 1));
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const double2 v = sh[c * kRow + i];
    stcv(dst, sidx(g, b, c, l), cpx<double>{v.x, v.y});
  }
}

template <typename S>
__global__ __launch_bounds__(256) void k_unpack(Geom g, double2* canon, const typename PT<S>::stor* in) {
  __shared__ double2 sh[12 * kRow];
  const int64_t s0 = (int64_t)blockIdx.x * kTile;
  const int ns = (int)min((int64_t)kTile, g.V - s0);
  double2* dst = canon + (int64_t)blockIdx.y * g.V * 12;
  const auto* src = in + (int64_t)blockIdx.y * g.V * 12;
  const int t = threadIdx.x;
  if (t < ns) {
    const int b = (int)((s0 + t) >> g.bs_log), l = (int)((s0 + t) & ((1 << g.bs_log) - 1));
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const cpx<double> v = ldcv<double>(src, sidx(g, b, c, l));
      sh[c * kRow + t] = make_double2(v.re, v.im);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 12 * ns; e += 256) {
    const int i = e / 12, c = e - 12 * i;
    const int64_t site = s0 + i;
    dst[canon_site(g, (int)(site >> g.bs_log), (int)(site & ((1 << g.bs_log) - 1))) * 12 + c] = sh[c * kRow + i];
  }
}

template <typename D, typename S>
__global__ __launch_bounds__(256) void k_convert(typename PT<D>::stor* dst, const typename PT<S>::stor* src,
                                                 int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += step) {
    if constexpr (std::is_same<D, double>::value) stcv(dst, i, ldcv<double>(src, i));
    else stcv(dst, i, ldcv<float>(src, i));
  }
}

dim3 site_grid(const Geom& g, int nrhs) { return dim3((unsigned)((g.V + 255) / 256), (unsigned)nrhs); }

}  // namespace

hipError_t launch_pack(const Geom& g, void* out, int p, const double* canon, int nrhs, hipStream_t s) {
  auto c = reinterpret_cast<const double2*>(canon);
  if (p == QMG_F64) hipLaunchKernelGGL(k_pack<double>, site_grid(g, nrhs), dim3(256), 0, s, g, (double2*)out, c);
  else if (p == QMG_F32) hipLaunchKernelGGL(k_pack<float>, site_grid(g, nrhs), dim3(256), 0, s, g, (float2*)out, c);
  else hipLaunchKernelGGL(k_pack<bf16_t>, site_grid(g, nrhs), dim3(256), 0, s, g, (uint32_t*)out, c);
  return hipGetLastError();
}

hipError_t launch_unpack(const Geom& g, double* canon, const void* in, int p, int nrhs, hipStream_t s) {
  auto c = reinterpret_cast<double2*>(canon);
  if (p == QMG_F64) hipLaunchKernelGGL(k_unpack<double>, site_grid(g, nrhs), dim3(256), 0, s, g, c, (const double2*)in);
  else if (p == QMG_F32) hipLaunchKernelGGL(k_unpack<float>, site_grid(g, nrhs), dim3(256), 0, s, g, c, (const float2*)in);
  else hipLaunchKernelGGL(k_unpack<bf16_t>, site_grid(g, nrhs), dim3(256), 0, s, g, c, (const uint32_t*)in);
  return hipGetLastError();
}

template <typename D>
static void conv_from(void* dst, const void* src, int ps, int64_t n, hipStream_t s) {
  using DS = typename PT<D>::stor;
  unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, 65536);
  if (grid == 0) return;
  if (ps == QMG_F64) hipLaunchKernelGGL((k_convert<D, double>), dim3(grid), dim3(256), 0, s, (DS*)dst, (const double2*)src, n);
  else if (ps == QMG_F32) hipLaunchKernelGGL((k_convert<D, float>), dim3(grid), dim3(256), 0, s, (DS*)dst, (const float2*)src, n);
  else hipLaunchKernelGGL((k_convert<D, bf16_t>), dim3(grid), dim3(256), 0, s, (DS*)dst, (const uint32_t*)src, n);
}

hipError_t launch_convert(void* dst, int pd, const void* src, int ps, int64_t n, hipStream_t s) {
  if (pd == QMG_F64) conv_from<double>(dst, src, ps, n, s);
  else if (pd == QMG_F32) conv_from<float>(dst, src, ps, n, s);
  else conv_from<bf16_t>(dst, src, ps, n, s);
  return hipGetLastError();
}
