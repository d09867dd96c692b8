// Work-group reductions with a fixed summation order.
#pragma once
#include "qmg_device.h"

// sum of NV values over the work-group (power-of-two size), same result in
// every thread.  red: LDS scratch of at least NV * max(blockDim.x/64, blockDim.x) (for
// blockDim.x < 64) elements.  Ends with a barrier so red can be reused.
template <typename R, int NV>
__device__ __forceinline__ void wg_sum(R (&v)[NV], R* red) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (nt >= 64) {
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
    if (lane == 0)
#pragma unroll
      for (int i = 0; i < NV; ++i) red[wave * NV + i] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      R s = red[i];
      for (int w = 1; w < nw; ++w) s += red[w * NV + i];
      v[i] = s;
    }
  } else {
#pragma unroll
    for (int i = 0; i < NV; ++i) red[i * nt + tid] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      R s = red[i * nt];
      for (int t = 1; t < nt; ++t) s += red[i * nt + t];
      v[i] = s;
    }
  }
  __syncthreads();
}

// v plus the value DPP control CTRL brings, in the rows of ROWS (others, and lanes with no
// source, add zero)
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, ROWS, 0xf, true));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)u, CTRL, ROWS, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
  return v + __longlong_as_double(((uint64_t)hi << 32) | lo);
}
// sum over the lanes of each row of 16, in the row's last lane (fixed order)
template <typename R>
__device__ __forceinline__ R row_sum15(R v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  return dpp_add<0x118, 0xf>(v);
}
// sum over the 64 lanes, in lane 63 (row shifts, then row broadcasts: fixed order)
template <typename R>
__device__ __forceinline__ R wave_sum63(R v) {
  v = row_sum15(v);
  v = dpp_add<0x142, 0xa>(v);
  return dpp_add<0x143, 0xc>(v);
}

// Sums of v[0..NV) over the wave, written to red[0..NV).  Two registers are added after
// exchanging their halves (then rows), so that each addition serves twice (four times) as
// many values: 5 instructions a value where summing each over 64 lanes takes 18.
template <int NV>
__device__ __forceinline__ void wave_fold(const double (&v)[NV], double* red) {
  constexpr int N1 = (NV + 1) / 2, N2 = (N1 + 1) / 2;
  double h[N1 + 1], q[N2];
#pragma unroll
  for (int i = 0; i < N1; ++i) {
    const uint64_t a = __double_as_longlong(v[2 * i]), b = 2 * i + 1 < NV ? __double_as_longlong(v[2 * i + 1]) : 0;
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    // lanes 0..31 add the halves of v[2i], lanes 32..63 those of v[2i + 1]
    h[i] = __longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) + __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]);
  }
  h[N1] = 0.0;
#pragma unroll
  for (int i = 0; i < N2; ++i) {
    const uint64_t a = __double_as_longlong(h[2 * i]), b = __double_as_longlong(h[2 * i + 1 < N1 ? 2 * i + 1 : N1]);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    // rows 0..3 hold v[4i], v[4i + 2], v[4i + 1], v[4i + 3]
    q[i] = row_sum15(__longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) +
                     __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]));
  }
  const int lane = threadIdx.x & 63;
  if ((lane & 15) == 15) {
    const int r = lane >> 4, at = r == 1 ? 2 : r == 2 ? 1 : r;
#pragma unroll
    for (int i = 0; i < N2; ++i)
      if (4 * i + at < NV) red[4 * i + at] = q[i];
  }
}
