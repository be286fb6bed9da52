// Global average pool + dense + bias + activation in one launch: the head of an image classifier (one fused function, paper
// Section 4.1).  Apart, both are mostly launch: at batch 1, 49 positions of 512 channels and 1000 units 3.9 + 2.9 us inside a network,
// for 50 KB of activations and 1 MB of filters.  Here every workgroup pools the image whose outputs it makes -- once for each
// group of units, which re-reads the activations from L2 but saves the trip through memory and the launch -- with its
// filters already on the way.
#include "kernels.hpp"

namespace relay {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

struct HeadArgs {
  int N, C, HW, units, act;
  int cvt_log2;   // threads of a position: a power of two of at least C / 8
  const half8* x;
  const half8* w;
  const float* bias;
  _Float16* pooled;
  _Float16* y;
};

constexpr int kThreads = 512, kWaves = kThreads / 64;

// A wave makes one output.  KI: reduction vectors of a lane, C <= 512 KI.  DEPTH: positions a thread has in flight.
template <int KI, int DEPTH>
__global__ __launch_bounds__(kThreads) void avgpool_dense_kernel(const int N, const int C, const int HW, const int units, const int cvt_log2_act,
                                                                  const half8* x, const half8* w_units, _Float16* y, const float* bias,
                                                                  _Float16* pooled) {
  const HeadArgs a{N, C, HW, units, cvt_log2_act >> 8, cvt_log2_act & 255, x, w_units, bias, pooled, y};
  __shared__ float part[kThreads * 8];
  __shared__ half8 pl[KI * 64];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = (int)blockIdx.x % a.N, ug = (int)blockIdx.x / a.N;
  const int CV = a.C >> 3, CVT = 1 << a.cvt_log2, parts = kThreads >> a.cvt_log2;
  const int j = ug * kWaves + wave;
  half8 w[KI];
#pragma unroll
  for (int k = 0; k < KI; ++k) {
    const int kv = k * 64 + lane;
    w[k] = kv < CV ? a.w[(size_t)min(j, a.units - 1) * CV + kv] : half8{0, 0, 0, 0, 0, 0, 0, 0};
  }
  const int v = tid & (CVT - 1), p = tid >> a.cvt_log2;
  float sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (v < CV) {
    const half8* xp = a.x + (size_t)n * a.HW * CV + v;
    for (int q0 = p; q0 < a.HW; q0 += parts * DEPTH) {
      half8 t[DEPTH];
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) t[d] = xp[(size_t)min(q0 + d * parts, a.HW - 1) * CV];
#pragma unroll
      for (int d = 0; d < DEPTH; ++d)
        if (q0 + d * parts < a.HW)
#pragma unroll
          for (int e = 0; e < 8; ++e) sum[e] += (float)t[d][e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[(p * 8 + e) * CVT + v] = sum[e];
  __syncthreads();
  const float inv = 1.0f / (float)a.HW;
  for (int c = tid; c < 8 * CVT; c += kThreads) {   // (channel vector c % CVT, element c / CVT)
    const int cv = c & (CVT - 1), e = c >> a.cvt_log2;
    float s = 0.f;
    for (int q = 0; q < parts; ++q) s += part[(q * 8 + e) * CVT + cv];
    if (cv < CV) reinterpret_cast<_Float16*>(&pl[cv])[e] = (_Float16)(s * inv);
  }
  __syncthreads();
  if (ug == 0 && tid < CV) reinterpret_cast<half8*>(a.pooled)[(size_t)n * CV + tid] = pl[tid];
  float acc = 0.f;
#pragma unroll
  for (int k = 0; k < KI; ++k)
    if (k * 64 + lane < CV) {
      const half8 xv = pl[k * 64 + lane];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf((float)xv[e], (float)w[k][e], acc);
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0 && j < a.units) {
    float r = acc + (a.bias ? a.bias[j] : 0.f);
    if (a.act == 1) r = r > 0.f ? r : 0.f;
    a.y[(size_t)n * a.units + j] = (_Float16)r;
  }
}

template <int KI>
hipError_t launch_head(const HeadArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)(a.N * ((a.units + kWaves - 1) / kWaves))), block(kThreads);
  // (apart, and in this order, because fourteen words of leading scalars are in registers when a wave starts: all but `pooled`)
  const int mode = a.act << 8 | a.cvt_log2;
  if (a.HW <= 8 * (kThreads >> a.cvt_log2))
    hipLaunchKernelGGL((avgpool_dense_kernel<KI, 8>), grid, block, 0, st, a.N, a.C, a.HW, a.units, mode, a.x, a.w, a.y, a.bias, a.pooled);
  else
    hipLaunchKernelGGL((avgpool_dense_kernel<KI, 16>), grid, block, 0, st, a.N, a.C, a.HW, a.units, mode, a.x, a.w, a.y, a.bias, a.pooled);   // (two rounds of 8 behind each other otherwise)
  return hipGetLastError();
}

}  // namespace

bool avgpool_dense_supported(int n, int c, int hw, int units) { return c % 8 == 0 && c <= 2048; }

// (a launch holds fewer than 2^32 threads)
bool avgpool_dense_fits(int n, int units) { return (long)n * ((units + kWaves - 1) / kWaves) * kThreads < (1L << 32); }

// While its workgroups fit the CUs at once and an image is quickly read by each of them.  Two launches / this one, us, one behind the
// other: one image and 1000 units, 49 positions of 512 channels 5.6 / 4.0, 100 of 512 5.9 / 4.8, 144 of 512 5.5 / 6.0, 49 of 1024 5.7 /
// 5.2, 16 of 2048 6.1 / 4.8, 49 of 2048 6.4 / 7.2; two images of 49 x 512 5.6 / 4.2; 100 units, 784 x 64, 16 images 6.5 / 5.5.
// More images, with four units or four images to a workgroup: 8 of 49 x 512 5.7 / 4.7 (no gain inside a network), 16 5.7 / 6.7, 32
// 5.8 / 10.4; 4 of 49 x 1024 5.9 / 5.9.
bool avgpool_dense_pays(int n, int c, int hw, int units) {
  return avgpool_dense_supported(n, c, hw, units) && (long)n * ((units + kWaves - 1) / kWaves) <= 256 && (long)hw * c <= 57344;
}

hipError_t launch_avgpool_dense(int n, int c, int hw, int units, const void* x, const void* w, const float* bias, int act, void* pooled,
                                void* y, hipStream_t st) {
  HeadArgs a;
  a.N = n; a.C = c; a.HW = hw; a.units = units; a.act = act;
  a.cvt_log2 = 3;
  while ((8 << a.cvt_log2) < c) ++a.cvt_log2;
  a.x = static_cast<const half8*>(x); a.w = static_cast<const half8*>(w); a.bias = bias;
  a.pooled = static_cast<_Float16*>(pooled); a.y = static_cast<_Float16*>(y);
  return c <= 512 ? launch_head<1>(a, st) : c <= 1024 ? launch_head<2>(a, st) : launch_head<4>(a, st);
}

}  // namespace relay
