// The body of the max pool with a compile-time window, for the kernels that run it.
#pragma once

#include "fastdiv.hpp"
#include "lds_dma.hpp"

namespace relay {

struct PoolGeom {
  int CV, H, W, stride, pad, Ho, Wo, rows;   // rows: ceil(Ho / OUT)
  unsigned total;                            // N * rows * Wo * CV
  FastDiv fd_cv, fd_wo, fd_rows;
};

// The geometry of a 3 x 3 pool whose threads produce `out` outputs below each other.
inline PoolGeom pool_geom(int N, int CV, int H, int W, int stride, int pad, int Ho, int Wo, int out) {
  const int rows = (Ho + out - 1) / out;
  return PoolGeom{CV, H, W, stride, pad, Ho, Wo, rows, (unsigned)((long)N * rows * Wo * CV), make_fastdiv((uint32_t)CV), make_fastdiv((uint32_t)Wo),
                  make_fastdiv((uint32_t)rows)};
}
// (two outputs per thread once that still leaves the chip several workgroups per CU: one image of 256 x 28 x 28 2.7 against 3.2 us)
inline int pool_outputs(int N, int CV, int stride, int Ho, int Wo) { return stride == 1 && (long)N * Ho * Wo * CV >= 512 * 1024 ? 2 : 1; }

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef signed char char16 __attribute__((ext_vector_type(16)));

// max of one more tap.  fp16: packed maxima, which pass over a NaN; the sequential "larger than the best so far" also keeps a
// NaN that the window begins with, so that one is put back at the end (keep_first).
__device__ __forceinline__ void take_max(char16& best, const char16& v) { best = v > best ? v : best; }
__device__ __forceinline__ void take_max(half8& best, const half8& v) { best = __builtin_elementwise_max(best, v); }
__device__ __forceinline__ void keep_first(char16&, const char16&) {}
__device__ __forceinline__ void keep_first(half8& best, const half8& first) { best = first == first ? best : first; }

// max pool, NHWC, one 16-byte channel vector per thread, for a compile-time window R x R: every tap is loaded, with its coordinates clamped
// into the image.  A clamped tap repeats an element that the window already holds (the window
// of a valid output overlaps the image in both directions), so the maximum is unchanged, and
// with no branches all R*R loads are in flight at once.  Workgroups are renumbered so that an
// XCD works through a contiguous range of output rows: rows that two windows share are then
// fetched into one L2.
// A thread produces OUT outputs below each other from the rows under all of them (stride 1: 2 outputs from 4 rows of taps,
// not 6).  32-bit indices and the host's division constants: three 64-bit software divisions per thread were most of
// its instructions.  256 channels at 28 x 28, batch 32, 3x3 / stride 1: 10.7 -> 7.0 us.
// place: the workgroup's place among the pool's
template <typename V, int VE, int R, int STRIDE, int OUT>
__device__ __forceinline__ void maxpool_fixed_tile(const V* x, V* y, const PoolGeom& g, int place) {
  static_assert(OUT == 1 || STRIDE == 1, "outputs below each other share rows at stride 1");
  // (place passes through: arithmetic on it stays behind the loads of all arguments)
  asm volatile("" : "+s"(place) : "s"(g.CV), "s"(g.H), "s"(g.W), "s"(g.stride), "s"(g.pad), "s"(g.Ho), "s"(g.Wo), "s"(g.rows), "s"(g.total),
               "s"(g.fd_cv.mul), "s"(g.fd_cv.shift), "s"(g.fd_wo.mul), "s"(g.fd_wo.shift), "s"(g.fd_rows.mul), "s"(g.fd_rows.shift));
  const unsigned idx = (unsigned)xcd_remap(place, (int)((g.total + 255u) / 256u)) * 256u + threadIdx.x;
  if (idx >= g.total) return;
  const unsigned t1 = fast_div(idx, g.fd_cv), t2 = fast_div(t1, g.fd_wo);
  const int cv = (int)(idx - t1 * (unsigned)g.CV), q = (int)(t1 - t2 * (unsigned)g.Wo);
  const int n = (int)fast_div(t2, g.fd_rows), p0 = ((int)t2 - n * g.rows) * OUT;
  const int stride = STRIDE ? STRIDE : g.stride;
  const V* xn = x + (size_t)((unsigned)n * (unsigned)(g.H * g.W)) * g.CV + cv;
  V v[R + OUT - 1][R];
#pragma unroll
  for (int r = 0; r < R + OUT - 1; ++r) {
    const int ih = min(max(p0 * stride - g.pad + r, 0), g.H - 1);
#pragma unroll
    for (int s = 0; s < R; ++s) {
      const int iw = min(max(q * stride - g.pad + s, 0), g.W - 1);
      v[r][s] = xn[(unsigned)((ih * g.W + iw) * g.CV)];
    }
  }
#pragma unroll
  for (int o = 0; o < OUT; ++o) {
    // (a later output below the image takes clamped rows and is not stored)
    V best = v[o][0];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int s = 0; s < R; ++s)
        if (r + s) take_max(best, v[o + r][s]);
    keep_first(best, v[o][0]);
    if (p0 + o < g.Ho) y[((size_t)(unsigned)(n * g.Ho + p0 + o) * g.Wo + q) * g.CV + cv] = best;
  }
}

}  // namespace
}  // namespace relay
