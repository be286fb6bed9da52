// Small kernels around the fused primitive functions: filter packing and the NCHW->NHWC
// conversion (compile-time layout alteration in the paper's terms, Section 5.3), and the
// two pools that chain ResNet / MobileNet layer shapes.
#include "kernels.hpp"
#include "lds_dma.hpp"
#include "maxpool_tile.hpp"

namespace relay {
namespace {

// OIHW [K][Csrc][R][S] -> [K][Kp] with reduction index (r, s, c), c < C, zero elsewhere.
template <typename T>
__global__ __launch_bounds__(256) void pack_filters_kernel(const T* w, T* out, int K, int Csrc, int C, int R, int S,
                                                           int Kp) {
  const long total = (long)K * Kp;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int kk = (int)(idx % Kp);
  const int k = (int)(idx / Kp);
  T v = 0;
  if (kk < R * S * C) {
    const int tap = kk / C, c = kk - tap * C;
    const int r = tap / S, s = tap - r * S;
    if (c < Csrc) v = w[(((long)k * Csrc + c) * R + r) * S + s];
  }
  out[idx] = v;
}

// depthwise filters [C][RS] -> [RS][C]
__global__ __launch_bounds__(256) void pack_dw_kernel(const uint16_t* w, uint16_t* out, int C, int RS) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= C * RS) return;
  const int c = idx % C, t = idx / C;
  out[idx] = w[c * RS + t];
}

template <typename T>
__global__ __launch_bounds__(256) void nchw_to_nhwc_kernel(const T* x, T* y, int N, int C, int H, int W, int Cpad) {
  const long total = (long)N * H * W * Cpad;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int c = (int)(idx % Cpad);
  long t = idx / Cpad;
  const int w_ = (int)(t % W);
  t /= W;
  const int h = (int)(t % H);
  const int n = (int)(t / H);
  y[idx] = c < C ? x[(((long)n * C + c) * H + h) * W + w_] : (T)0;
}

// The same conversion for 2- and 1-byte types in 16-byte pieces: a thread takes PX consecutive pixels of VE
// channels (8 x 8 halves; 4 x 16 bytes), one vector load per channel, transposes them in registers -- an output
// word is a byte permute of the words of two (four) channels -- and stores 16 bytes per pixel.  Lanes run along
// the pixels first (4 lanes: 64 bytes of a channel row), then along the channels.  Bound by memory: 256 channels at
// 28 x 28, batch 32: 32.0 -> 5.9 us for 25.7 MB (one element per thread read 2 bytes of a line each).
template <typename T>
__global__ __launch_bounds__(64) void nchw_to_nhwc_vec_kernel(const T* x, T* y, int C, int HW, int Cpad, int pgroups, int cgroups, int tiles) {
  constexpr int VE = 16 / (int)sizeof(T), PX = sizeof(T) == 2 ? 8 : 4;
  constexpr int NV = PX * (int)sizeof(T) / 4;  // words of a channel's piece
  const int tile = xcd_remap((int)blockIdx.x, tiles);   // (image, pixel block, channel block); the XCD of the conv that reads it
  const int per_n = pgroups * cgroups;
  const int n = tile / per_n, rem = tile - n * per_n;
  const int pb = rem / cgroups, cb = rem - pb * cgroups;
  const int lane = threadIdx.x;
  int p0 = (pb * 8 + (lane & 3) + 4 * (lane >> 5)) * PX;
  const int c0 = (cb * 8 + ((lane >> 2) & 7)) * VE;
  if (p0 >= HW || c0 >= Cpad) return;
  p0 = min(p0, HW - PX);  // the last piece of an image ends with it: a few pixels are written twice, alike
  const T* xp = x + ((long)n * C + c0) * HW + p0;
  unsigned in[VE][NV];
#pragma unroll
  for (int c = 0; c < VE; ++c) {
#pragma unroll
    for (int v = 0; v < NV; ++v) in[c][v] = 0u;
    if (c0 + c < C) __builtin_memcpy(in[c], xp + (long)c * HW, PX * sizeof(T));
  }
  T* yp = y + ((long)n * HW + p0) * Cpad + c0;
#pragma unroll
  for (int i = 0; i < PX; ++i) {
    unsigned o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (sizeof(T) == 2) {
        // halves i & 1 of word i / 2 of channels 2q and 2q + 1
        o[q] = __builtin_amdgcn_perm(in[2 * q + 1][i / 2], in[2 * q][i / 2], (i & 1) ? 0x07060302u : 0x05040100u);
      } else {
        // byte i of channels 4q .. 4q + 3
        const unsigned sel = (unsigned)(i | ((4 + i) << 8)) | 0x0c0c0000u;
        const unsigned lo = __builtin_amdgcn_perm(in[4 * q + 1][0], in[4 * q][0], sel);
        const unsigned hi = __builtin_amdgcn_perm(in[4 * q + 3][0], in[4 * q + 2][0], sel);
        o[q] = lo | (hi << 16);
      }
    }
    *reinterpret_cast<uint4*>(yp + (long)i * Cpad) = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// [N][C<=4][H][W] -> [N][H+2ph][Wp][4], zeros in the border, in the slack columns and in the channels past C: one thread
// per PX neighbouring output pixels (Wp is a multiple of 8).  Memory-bound in principle; the two software divisions per
// pixel cost more than the traffic: fp16, 3 x 224 x 224, batch 32 (9.6 MB in, 13.7 MB out) 7.3 -> 6.2 us with the host's constants,
// 6.05 with two pixels and 16 bytes stored per thread.
template <typename T, int PX>
__global__ __launch_bounds__(256) void pack_input_nhwc4_kernel(const T* x, T* y, int C, int H, int W, int ph, int pw, int Hp, int Wp,
                                                               unsigned total, FastDiv fd_w, FastDiv fd_h) {
  // (32-bit index arithmetic: the padded tensor has fewer than 2^31 bytes, checked by the entry point)
  const unsigned idx = blockIdx.x * 256u + threadIdx.x;
  if (idx >= total) return;
  const unsigned t = fast_div(idx, fd_w);
  const int w0 = (int)(idx - t * (unsigned)(Wp / PX)) * PX - pw;
  const int n = (int)fast_div(t, fd_h);
  const int h = (int)t - n * Hp - ph;
  // (a pixel outside the image loads the nearest one inside instead of branching: all loads in flight at once)
  const bool row_ok = (unsigned)h < (unsigned)H;
  const int hc = min(max(h, 0), H - 1);
  T v[PX][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const T* row = x + ((size_t)(unsigned)(n * C + (c < C ? c : 0)) * H + hc) * W;
#pragma unroll
    for (int i = 0; i < PX; ++i) v[i][c] = c < C ? row[min(max(w0 + i, 0), W - 1)] : (T)0;   // (uniform condition)
  }
#pragma unroll
  for (int i = 0; i < PX; ++i)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (!row_ok || (unsigned)(w0 + i) >= (unsigned)W) v[i][c] = 0;
  struct alignas(PX * 4 * sizeof(T) < 16 ? PX * 4 * sizeof(T) : 16) Out {
    T e[PX * 4];
  } o;
#pragma unroll
  for (int i = 0; i < PX; ++i)
#pragma unroll
    for (int c = 0; c < 4; ++c) o.e[i * 4 + c] = v[i][c];
  reinterpret_cast<Out*>(y)[idx] = o;
}

// OIHW [K][Csrc][R][S] -> [K][Kp], reduction index r*ck + s*4 + c (one filter row per chunk)
template <typename T>
__global__ __launch_bounds__(256) void pack_filters_rows_kernel(const T* w, T* out, int K, int Csrc, int R, int S,
                                                                int ck, int Kp) {
  const long total = (long)K * Kp;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int kk = (int)(idx % Kp);
  const int k = (int)(idx / Kp);
  T v = 0;
  const int r = kk / ck, in_row = kk - r * ck;
  const int s = in_row >> 2, c = in_row & 3;
  if (r < R && s < S && c < Csrc) v = w[(((long)k * Csrc + c) * R + r) * S + s];
  out[idx] = v;
}

// max pool, NHWC, one 16-byte channel vector per thread; padding taps are skipped.
template <typename V, int VE>
__global__ __launch_bounds__(256) void maxpool_kernel(const V* x, V* y, int N, int CV, int H, int W, int R, int stride,
                                                      int pad, int Ho, int Wo) {
  const long total = (long)N * Ho * Wo * CV;
  long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int cv = (int)(idx % CV);
  long t = idx / CV;
  const int q = (int)(t % Wo);
  t /= Wo;
  const int p = (int)(t % Ho);
  const int n = (int)(t / Ho);
  V best;
  bool have = false;
  for (int r = 0; r < R; ++r) {
    const int ih = p * stride - pad + r;
    if ((unsigned)ih >= (unsigned)H) continue;
    for (int s = 0; s < R; ++s) {
      const int iw = q * stride - pad + s;
      if ((unsigned)iw >= (unsigned)W) continue;
      const V v = x[(((long)n * H + ih) * W + iw) * CV + cv];
      if (!have) {
        best = v;
        have = true;
      } else {
#pragma unroll
        for (int e = 0; e < VE; ++e) best[e] = v[e] > best[e] ? v[e] : best[e];
      }
    }
  }
  if (!have) {
#pragma unroll
    for (int e = 0; e < VE; ++e) best[e] = 0;
  }
  y[idx] = best;
}

template <typename V, int VE, int R, int STRIDE, int OUT>
__global__ __launch_bounds__(256) void maxpool_fixed_kernel(const V* x, V* y, const PoolGeom g) {
  maxpool_fixed_tile<V, VE, R, STRIDE, OUT>(x, y, g, (int)blockIdx.x);
}

// global average pool, NHWC fp16 -> [N][C] fp16, fp32 sum.  One workgroup per image and CVB channel vectors; 256 / CVB
// thread groups share the positions, their sums meet by lane exchanges and once in LDS.  Bound by
// latency: 49 positions of 512 channels took 3.6 us at batch 1 and 4.0 at batch 32 with one workgroup per image whose
// four thread groups read 13 positions each in turn, 2.4 and 2.6 with CVB = 8.
template <int CVB>
__global__ __launch_bounds__(256) void avgpool_f16_kernel(const half8* x, half8* y, int N, int CV, int HW, int groups) {
  constexpr int PARTS = 256 / CVB;
  __shared__ float part[3][CVB][8];
  const int n = blockIdx.x / groups, g = blockIdx.x - n * groups;
  const int cvl = threadIdx.x & (CVB - 1), pi = threadIdx.x / CVB, wave = threadIdx.x >> 6;
  const int cv = g * CVB + cvl;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (cv < CV) {
    const half8* xp = x + (long)n * HW * CV + cv;
#pragma unroll 4
    for (int i = pi; i < HW; i += PARTS) {
      const half8 v = xp[(long)i * CV];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += (float)v[e];
    }
  }
#pragma unroll
  for (int o = 32; o >= CVB; o >>= 1)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
  if (wave > 0 && (threadIdx.x & 63) < CVB)
#pragma unroll
    for (int e = 0; e < 8; ++e) part[wave - 1][cvl][e] = acc[e];
  __syncthreads();
  if (threadIdx.x < CVB && cv < CV) {
    half8 o;
    const float inv = 1.0f / (float)HW;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      o[e] = (_Float16)((acc[e] + part[0][cvl][e] + part[1][cvl][e] + part[2][cvl][e]) * inv);
    y[(long)n * CV + cv] = o;
  }
}

inline unsigned blocks_for(long total) { return (unsigned)((total + 255) / 256); }

}  // namespace

hipError_t launch_pack_filters(const void* w, void* out, int K, int Csrc, int C, int R, int S, int Kp, int esize,
                               hipStream_t st) {
  const long total = (long)K * Kp;
  dim3 grid(blocks_for(total)), block(256);
  if (esize == 1)
    hipLaunchKernelGGL((pack_filters_kernel<int8_t>), grid, block, 0, st, (const int8_t*)w, (int8_t*)out, K, Csrc, C,
                       R, S, Kp);
  else if (esize == 2)
    hipLaunchKernelGGL((pack_filters_kernel<uint16_t>), grid, block, 0, st, (const uint16_t*)w, (uint16_t*)out, K,
                       Csrc, C, R, S, Kp);
  else
    hipLaunchKernelGGL((pack_filters_kernel<uint32_t>), grid, block, 0, st, (const uint32_t*)w, (uint32_t*)out, K,
                       Csrc, C, R, S, Kp);
  return hipGetLastError();
}

hipError_t launch_pack_dw_filters(const void* w, void* out, int C, int RS, hipStream_t st) {
  hipLaunchKernelGGL(pack_dw_kernel, dim3(blocks_for((long)C * RS)), dim3(256), 0, st, (const uint16_t*)w,
                     (uint16_t*)out, C, RS);
  return hipGetLastError();
}

namespace {
typedef _Float16 half8v __attribute__((ext_vector_type(8)));

// One unfused elementwise operator over an fp16 NHWC tensor: what a framework without operator
// fusion launches behind a convolution (paper Section 5.2 measures fusion against exactly this).
// Every operator reads its input tensor and writes a new one, rounded to fp16.
//   OP 0 bias add: x + p0[c];  1 scale/shift: x*p0[c] + p1[c];  2 add: x + other;  3 relu
template <int OP>
__global__ __launch_bounds__(256) void elementwise_f16_kernel(long nvec, int cvecs, const half8v* x, const float* p0,
                                                              const float* p1, const half8v* other, half8v* y) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= nvec) return;
  const int c = (int)(i % cvecs) * 8;
  const half8v v = x[i];
  half8v o;
  if constexpr (OP == 2) {
    const half8v r = other[i];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (_Float16)((float)v[e] + (float)r[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = (float)v[e];
      float u;
      if constexpr (OP == 0) u = t + p0[c + e];
      else if constexpr (OP == 1) u = t * p0[c + e] + p1[c + e];
      else u = t > 0.f ? t : 0.f;
      o[e] = (_Float16)u;
    }
  }
  y[i] = o;
}
}  // namespace

hipError_t launch_elementwise_f16(int op, long npix, int c, const void* x, const float* p0, const float* p1,
                                  const void* other, void* y, hipStream_t st) {
  const long nvec = npix * (c / 8);
  const dim3 grid((unsigned)((nvec + 255) / 256)), block(256);
  const half8v* xv = static_cast<const half8v*>(x);
  const half8v* ov = static_cast<const half8v*>(other);
  half8v* yv = static_cast<half8v*>(y);
  switch (op) {
    case 0: hipLaunchKernelGGL((elementwise_f16_kernel<0>), grid, block, 0, st, nvec, c / 8, xv, p0, p1, ov, yv); break;
    case 1: hipLaunchKernelGGL((elementwise_f16_kernel<1>), grid, block, 0, st, nvec, c / 8, xv, p0, p1, ov, yv); break;
    case 2: hipLaunchKernelGGL((elementwise_f16_kernel<2>), grid, block, 0, st, nvec, c / 8, xv, p0, p1, ov, yv); break;
    default: hipLaunchKernelGGL((elementwise_f16_kernel<3>), grid, block, 0, st, nvec, c / 8, xv, p0, p1, ov, yv); break;
  }
  return hipGetLastError();
}

namespace {
// Axis scale folding (paper Section 4.4): the per-channel factor next to a convolution is
// multiplied into the OIHW filters once, ahead of time.  The product of a filter value and an
// fp32 factor is exact in fp64, so the result is rounded exactly once, to the filter type.
template <typename T>
__global__ __launch_bounds__(256) void fold_scale_axis_kernel(long n, int C, int RS, bool axis_in, const T* w,
                                                              const float* scale, T* out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const long kc = i / RS;  // k*C + c
  const int ch = axis_in ? (int)(kc % C) : (int)(kc / C);
  out[i] = (T)((double)w[i] * (double)scale[ch]);
}

__global__ __launch_bounds__(256) void fold_bias_kernel(int K, const float* bias, const float* scale,
                                                        const float* shift, float* out) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= K) return;
  const double b = bias ? (double)bias[k] : 0.0;
  out[k] = (float)__dadd_rn(__dmul_rn(b, (double)scale[k]), (double)shift[k]);  // product rounded, then the sum: no fma
}
}  // namespace

hipError_t launch_fold_scale_axis(bool is_f16, int K, int C, int RS, bool axis_in, const void* w, const float* scale,
                                  void* w_out, hipStream_t st) {
  const long n = (long)K * C * RS;
  if (is_f16)
    hipLaunchKernelGGL((fold_scale_axis_kernel<_Float16>), dim3(blocks_for(n)), dim3(256), 0, st, n, C, RS, axis_in,
                       (const _Float16*)w, scale, (_Float16*)w_out);
  else
    hipLaunchKernelGGL((fold_scale_axis_kernel<float>), dim3(blocks_for(n)), dim3(256), 0, st, n, C, RS, axis_in,
                       (const float*)w, scale, (float*)w_out);
  return hipGetLastError();
}

hipError_t launch_fold_bias(int K, const float* bias, const float* scale, const float* shift, float* out,
                            hipStream_t st) {
  hipLaunchKernelGGL(fold_bias_kernel, dim3(blocks_for(K)), dim3(256), 0, st, K, bias, scale, shift, out);
  return hipGetLastError();
}

template <typename V, int VE>
hipError_t launch_maxpool3(int N, int CV, int H, int W, int stride, int pad, int Ho, int Wo, const void* x, void* y, hipStream_t st) {
  const int out = pool_outputs(N, CV, stride, Ho, Wo);
  const PoolGeom g = pool_geom(N, CV, H, W, stride, pad, Ho, Wo, out);
  const dim3 grid(blocks_for(g.total)), block(256);
  if (out == 2) hipLaunchKernelGGL((maxpool_fixed_kernel<V, VE, 3, 1, 2>), grid, block, 0, st, (const V*)x, (V*)y, g);
  else hipLaunchKernelGGL((maxpool_fixed_kernel<V, VE, 3, 0, 1>), grid, block, 0, st, (const V*)x, (V*)y, g);
  return hipGetLastError();
}

hipError_t launch_maxpool(bool is_i8, int N, int C, int H, int W, int R, int stride, int pad, int Ho, int Wo,
                          const void* x, void* y, hipStream_t st) {
  if (R == 3)   // (tensors below 2^31 elements, checked by the entry point)
    return is_i8 ? launch_maxpool3<char16, 16>(N, C / 16, H, W, stride, pad, Ho, Wo, x, y, st)
                 : launch_maxpool3<half8, 8>(N, C / 8, H, W, stride, pad, Ho, Wo, x, y, st);
  if (is_i8) {
    const int cv = C / 16;
    hipLaunchKernelGGL((maxpool_kernel<char16, 16>), dim3(blocks_for((long)N * Ho * Wo * cv)), dim3(256), 0, st,
                       (const char16*)x, (char16*)y, N, cv, H, W, R, stride, pad, Ho, Wo);
  } else {
    const int cv = C / 8;
    hipLaunchKernelGGL((maxpool_kernel<half8, 8>), dim3(blocks_for((long)N * Ho * Wo * cv)), dim3(256), 0, st,
                       (const half8*)x, (half8*)y, N, cv, H, W, R, stride, pad, Ho, Wo);
  }
  return hipGetLastError();
}

hipError_t launch_avgpool_f16(int N, int C, int HW, const void* x, void* y, hipStream_t st) {
  const int cv = C / 8;
  // 8 channel vectors (128 bytes of a pixel) a workgroup; more where that leaves thread groups without a position (2048
  // channels, batch 32: 4 positions 3.0 us with 8, 2.1 with 64, 25 positions 3.3 with 8, 2.7 with 16); fewer where there are fewer
  // and the positions go round more than once (8 channels, 3136 positions: 13.6 us with 8, 3.1 with 1).
  int cvb = 8;
  while (cvb < 64 && 256 / cvb > HW) cvb *= 2;
  while (cvb > 1 && cvb / 2 >= cv && 256 / cvb < HW) cvb /= 2;
  const int groups = (cv + cvb - 1) / cvb;
  const dim3 grid((unsigned)(N * groups)), block(256);
  switch (cvb) {
#define RELAY_AVGPOOL_CASE(b) \
  case b: hipLaunchKernelGGL((avgpool_f16_kernel<b>), grid, block, 0, st, (const half8*)x, (half8*)y, N, cv, HW, groups); break;
    RELAY_AVGPOOL_CASE(1) RELAY_AVGPOOL_CASE(2) RELAY_AVGPOOL_CASE(4) RELAY_AVGPOOL_CASE(8)
    RELAY_AVGPOOL_CASE(16) RELAY_AVGPOOL_CASE(32) RELAY_AVGPOOL_CASE(64)
#undef RELAY_AVGPOOL_CASE
  }
  return hipGetLastError();
}

hipError_t launch_pack_input_nhwc4(int esize, int N, int C, int H, int W, int ph, int pw, int Wp, const void* x,
                                   void* y, hipStream_t st) {
  const int Hp = H + 2 * ph;
  // Two pixels per thread pay on large fp16 images only (4 channels, 1.7 M pixels 7.5 -> 6.7 us; 8640 pixels 2.06 against 2.10);
  // int8, whose stores are half as wide, is faster with one at all sizes but the largest of one channel (3 channels, 26 K pixels 2.03 us
  // against 2.36 with two and 2.25 with four, 1.7 M pixels 5.1 against 5.7 and 5.3).
  const int px = esize == 2 && (long)N * Hp * Wp >= 200 * 1000 ? 2 : 1;
  const unsigned total = (unsigned)((long)N * Hp * (Wp / px));
  const FastDiv fd_w = make_fastdiv((uint32_t)(Wp / px)), fd_h = make_fastdiv((uint32_t)Hp);
  const dim3 grid(blocks_for(total)), block(256);
  if (esize == 1)
    hipLaunchKernelGGL((pack_input_nhwc4_kernel<int8_t, 1>), grid, block, 0, st, (const int8_t*)x, (int8_t*)y, C, H, W, ph, pw, Hp, Wp, total,
                       fd_w, fd_h);
  else if (px == 1)
    hipLaunchKernelGGL((pack_input_nhwc4_kernel<uint16_t, 1>), grid, block, 0, st, (const uint16_t*)x, (uint16_t*)y, C, H, W, ph, pw, Hp, Wp,
                       total, fd_w, fd_h);
  else
    hipLaunchKernelGGL((pack_input_nhwc4_kernel<uint16_t, 2>), grid, block, 0, st, (const uint16_t*)x, (uint16_t*)y, C, H, W, ph, pw, Hp, Wp,
                       total, fd_w, fd_h);
  return hipGetLastError();
}

hipError_t launch_pack_filters_rows(const void* w, void* out, int K, int Csrc, int R, int S, int ck, int Kp,
                                    int esize, hipStream_t st) {
  dim3 grid(blocks_for((long)K * Kp)), block(256);
  if (esize == 1)
    hipLaunchKernelGGL((pack_filters_rows_kernel<int8_t>), grid, block, 0, st, (const int8_t*)w, (int8_t*)out, K, Csrc,
                       R, S, ck, Kp);
  else
    hipLaunchKernelGGL((pack_filters_rows_kernel<uint16_t>), grid, block, 0, st, (const uint16_t*)w, (uint16_t*)out,
                       K, Csrc, R, S, ck, Kp);
  return hipGetLastError();
}

hipError_t launch_nchw_to_nhwc(int esize, int N, int C, int H, int W, int Cpad, const void* x, void* y,
                               hipStream_t st) {
  const long total = (long)N * H * W * Cpad;
  dim3 grid(blocks_for(total)), block(256);
  const int ve = 16 / esize, px = esize == 2 ? 8 : 4;
  // (int8: from 200 K elements on.  20 -> 32 channels: 12800 elements 2.24 us in pieces, 2.05 an element per
  // thread, 100 K 2.30 and 2.12, 200 K 2.36 and 2.43, 400 K 2.53 and 2.93; fp16 is never slower in pieces)
  if ((esize == 2 || (esize == 1 && total >= 200 * 1000)) && Cpad % ve == 0 && H * W >= px && (reinterpret_cast<uintptr_t>(y) & 15) == 0) {
    const int pg = (H * W + 8 * px - 1) / (8 * px), cg = (Cpad + 8 * ve - 1) / (8 * ve);
    if ((long)N * pg * cg <= 0x7fffffffL) {
      const dim3 tiles((unsigned)(N * pg * cg)), wave(64);
      if (esize == 1)
        hipLaunchKernelGGL((nchw_to_nhwc_vec_kernel<int8_t>), tiles, wave, 0, st, (const int8_t*)x, (int8_t*)y, C, H * W, Cpad, pg, cg, N * pg * cg);
      else
        hipLaunchKernelGGL((nchw_to_nhwc_vec_kernel<uint16_t>), tiles, wave, 0, st, (const uint16_t*)x, (uint16_t*)y, C, H * W, Cpad,
                           pg, cg, N * pg * cg);
      return hipGetLastError();
    }
  }
  if (esize == 1)
    hipLaunchKernelGGL((nchw_to_nhwc_kernel<int8_t>), grid, block, 0, st, (const int8_t*)x, (int8_t*)y, N, C, H, W,
                       Cpad);
  else if (esize == 2)
    hipLaunchKernelGGL((nchw_to_nhwc_kernel<uint16_t>), grid, block, 0, st, (const uint16_t*)x, (uint16_t*)y, N, C, H,
                       W, Cpad);
  else
    hipLaunchKernelGGL((nchw_to_nhwc_kernel<uint32_t>), grid, block, 0, st, (const uint32_t*)x, (uint32_t*)y, N, C, H,
                       W, Cpad);
  return hipGetLastError();
}

}  // namespace relay
