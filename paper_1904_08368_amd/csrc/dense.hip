// dense + bias + activation:  y[m,j] = sum_i x[m,i] * w[j,i] + b[j]   (one fused
// primitive function, paper Section 4.1).  At inference batch sizes this op only streams
// the weight matrix once (weight-bandwidth bound), so a wave owns one output unit j,
// its lanes stride along the reduction axis with 16-byte loads, and the same weight
// vector feeds MB rows of x before a cross-lane sum.  WPO = 4: one output unit per workgroup, the reduction
// split over its waves (a long reduction over few rows: 3136 -> 512 at m = 1 3.7 us, 4.7 with one wave
// per unit -- seven loads one behind the other on 128 workgroups).
#include "kernels.hpp"

namespace relay {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

// UNROLL: two rounds of the reduction at a time.  Where few rows of x are in use (fp32, one row, 3136 -> 512: 5.4 -> 4.0 us); with
// eight rows and more the doubled live vectors cost more than the overlap gives (fp32, 32 rows, 3136 -> 4096: 72 us without, 115 with).
template <bool IS_F16, int MB, int WPO = 1, bool UNROLL = false>
__global__ __launch_bounds__(256) void dense_kernel(int M, int N, int K, const void* xv, const void* wv,
                                                    const float* bias, int act, void* yv) {
  constexpr int VE = IS_F16 ? 8 : 4;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int j = WPO == 1 ? blockIdx.x * 4 + wave : (int)blockIdx.x;
  if (j >= N) return;  // whole wave leaves together
  for (int m0 = 0; m0 < M; m0 += MB) {
    float acc[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[i] = 0.f;
    auto round = [&](int k0) {
      float wf[VE];
      if constexpr (IS_F16) {
        const half8 t = *reinterpret_cast<const half8*>(static_cast<const _Float16*>(wv) + (long)j * K + k0);
#pragma unroll
        for (int e = 0; e < VE; ++e) wf[e] = (float)t[e];
      } else {
        const float4 t = *reinterpret_cast<const float4*>(static_cast<const float*>(wv) + (long)j * K + k0);
        wf[0] = t.x; wf[1] = t.y; wf[2] = t.z; wf[3] = t.w;
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int m = m0 + i;
        if (m >= M) break;
        if constexpr (IS_F16) {
          const half8 t = *reinterpret_cast<const half8*>(static_cast<const _Float16*>(xv) + (long)m * K + k0);
#pragma unroll
          for (int e = 0; e < VE; ++e) acc[i] = fmaf((float)t[e], wf[e], acc[i]);
        } else {
          const float4 t = *reinterpret_cast<const float4*>(static_cast<const float*>(xv) + (long)m * K + k0);
          acc[i] = fmaf(t.x, wf[0], acc[i]);
          acc[i] = fmaf(t.y, wf[1], acc[i]);
          acc[i] = fmaf(t.z, wf[2], acc[i]);
          acc[i] = fmaf(t.w, wf[3], acc[i]);
        }
      }
    };
    const int first = (WPO == 1 ? lane : (int)threadIdx.x) * VE;
    if constexpr (UNROLL) {
#pragma unroll 2
      for (int k0 = first; k0 < K; k0 += 64 * WPO * VE) round(k0);
    } else {
      for (int k0 = first; k0 < K; k0 += 64 * WPO * VE) round(k0);
    }
    __shared__ float part[WPO][MB];
    // (all rows are summed before the first is stored: their lane exchanges overlap)
#pragma unroll
    for (int i = 0; i < MB; ++i) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) acc[i] += __shfl_xor(acc[i], o, 64);
      if (WPO > 1 && lane == 0) part[wave][i] = acc[i];
    }
    if constexpr (WPO > 1) __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      float v = acc[i];
      if constexpr (WPO > 1) {
        v = 0.f;
#pragma unroll
        for (int u = 0; u < WPO; ++u) v += part[u][i];
      }
      const int m = m0 + i;
      if ((WPO == 1 ? lane : (int)threadIdx.x) == 0 && m < M) {
        if (bias) v += bias[j];
        if (act == 1) v = v > 0.f ? v : 0.f;
        if constexpr (IS_F16)
          static_cast<_Float16*>(yv)[(long)m * N + j] = (_Float16)v;
        else
          static_cast<float*>(yv)[(long)m * N + j] = v;
      }
    }
    if constexpr (WPO > 1) __syncthreads();  // (the next rows reuse the partial sums)
  }
}

}  // namespace

// fp16: a workgroup per output unit, for a long reduction over few rows and units.  The other side is the small-tile matrix kernel,
// which reads the filters once for all rows but takes whole multiples of 32 of the reduction; where it cannot go, a
// wave per unit.  Measured, this kernel / the other side, us: against small tiles, k = 4096: m = 1, 512 units 3.7 / 4.5, 1500 4.8 / 5.0;
// m = 2, 1000 units 4.5 / 4.5; m = 4, 512 units 4.7 / 4.5, 4096 12.3 / 5.4; k = 2048, 4096 units 7.6 / 4.2; k = 9216: m = 1, 2048 units
// 8.1 / 8.5, m = 3, 1000 units 6.5 / 7.2, m = 4, 1500 units 9.3 / 7.3.  Against a wave per unit, k = 3000: m = 1, 512 units
// 3.7 / 4.6, 2048 5.2 / 4.9, m = 4, 1500 units 5.8 / 6.8, 2048 6.4 / 6.9, 4096 12.2 / 9.6.
bool dense_splits_units(int m, int n, int k) {
  if (m > 4 || k < 2048) return false;
  if (k % 32) return n <= 2048;
  return (m <= 2 && n <= 1024) || (k >= 8192 && (long)m * n <= 3072);
}

hipError_t launch_dense(int m, int n, int k, bool is_f16, const void* x, const void* w, const float* bias, int act,
                        void* y, hipStream_t st) {
  // a wave keeps MB rows of x against one weight row: 32 when the batch has that many, so the
  // weights are read once and one round of loads covers the whole reduction of a typical layer
  dim3 block(256), grid((unsigned)((n + 3) / 4));
  if (is_f16) {
    if (dense_splits_units(m, n, k))
      hipLaunchKernelGGL((dense_kernel<true, 4, 4, true>), dim3((unsigned)n), block, 0, st, m, n, k, x, w, bias, act, y);
    else if (m == 1)
      hipLaunchKernelGGL((dense_kernel<true, 8, 1, true>), grid, block, 0, st, m, n, k, x, w, bias, act, y);
    else if (m > 8)
      hipLaunchKernelGGL((dense_kernel<true, 32>), grid, block, 0, st, m, n, k, x, w, bias, act, y);
    else
      hipLaunchKernelGGL((dense_kernel<true, 8>), grid, block, 0, st, m, n, k, x, w, bias, act, y);
  } else if (m == 1) {
    hipLaunchKernelGGL((dense_kernel<false, 8, 1, true>), grid, block, 0, st, m, n, k, x, w, bias, act, y);
  } else {
    hipLaunchKernelGGL((dense_kernel<false, 8>), grid, block, 0, st, m, n, k, x, w, bias, act, y);
  }
  return hipGetLastError();
}

}  // namespace relay
