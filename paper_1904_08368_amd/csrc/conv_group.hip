// Convs that read different tensors, none the other's output, as ONE launch: a 3x3 conv on the 3x3 kernel's 128 x 64 tiles and up to
// two convs on the implicit GEMM's (paper Section 4.4, for the members of an Inception block that cannot share an input).
//
// One after the other each of them ends with the chip half empty: the 128 -> 192 3x3 conv of a block of 32 images of 28 x 28 is 633
// tiles on 512 workgroup slots (19.4 us), the 32 -> 96 5x5 one 392 tiles of 25 short steps in a row, each waiting at a barrier
// (13.9 us), the 256 -> 64 1x1 one 196 tiles that are mostly first loads and stores (6.6 us).  Sharing a grid, the tiles of one fill
// the slots and the waits that the others leave.  A workgroup's number says whose tile it runs; each runs the code, and sums in the order, of
// the conv's own launch.  What a tile needs of LDS and registers is the most of the three: two workgroups fit a CU, as by themselves.
// The longest tiles come first, the shortest last, so that the last round is short.
// Measured, 32 images of 28 x 28: these three 37.9 -> 27.1 us (graph-timed; 36.1 -> 25.4 on another card), the whole block, called one after another, 65.5 ->
// 53.3; the order 5x5, 3x3, 1x1 takes 12.9 us off a block of 64.9, 3x3 first 8.1, 1x1 before 3x3 11.7.  The rule that chooses is api.cpp's.
#include <atomic>

#include "conv_halo_tile.hpp"
#include "igemm_dma_tile.hpp"
#include "maxpool_tile.hpp"

namespace relay {
namespace {

// The numbers of workgroups come first, in preloaded registers: whose tile it is is known before the first argument is fetched.
__global__ __launch_bounds__(256, 2) void conv_group_kernel(const int tiles1, const int tiles3, const int tiles2, const ConvArgs a1, const HaloArgs a3,
                                                            const ConvArgs a2) {
  extern __shared__ uint4 lds[];
  const int wg = (int)blockIdx.x, first3 = tiles1, first2 = tiles1 + tiles3;
  if (wg < first3) igemm_dma_tile<false, 2, 2, 2, 1, 4, 1, 1, false, true, false>(a1, xcd_remap(wg, tiles1), lds);
  else if (wg < first2) conv3x3_halo_tile<false, 2, 2, 2, 1, 2, 1, false, 1, true, false>(a3, xcd_remap(wg - first3, tiles3), wg - first3, tiles3);
  else igemm_dma_tile<false, 2, 2, 2, 1, 3, 2, 1, false, true, false>(a2, xcd_remap(wg - first2, tiles2), lds);
}

constexpr int kBM = 128, kBN = 64;

// A conv and a 3x3 max pool that do not read each other's outputs: the 1x1 members of an Inception block on its input and the block's pool.  The
// conv's tiles wait for their few loads and the pool for memory; both pass over the same tensor, which one of them by itself leaves behind
// for the other in HBM.  So workgroups of the two alternate, eight at a time (one to an XCD), in the proportion of their numbers: an XCD works
// through both in the same order, and reads the tensor once for the two.  Measured: 256 -> 288 and the 3 x 3 / stride 1 pool on 32 images of 28 x 28, in a
// block of three launches instead of four, 53.3 -> 48.7 us; the two alone at the rule that chooses (api.cpp).
// The proportion holds in every fourth of an XCD's workgroups by itself, because its four shader engines take workgroups in turn: with the
// two alternating one by one, or one to three, the convs were all on two engines, or on one (32 images of 56 x 56, 256 -> 512 92.4 us against
// 74.3 for two launches, 192 -> 96 38.1 against 31.3; now 74.5 and 28.6).
// mul: (groups of eight of the conv << 32) / all groups, rounded up; there are four groups or a multiple.
template <int STRIDE, int OUT>
__global__ __launch_bounds__(256, 4) void conv_pool_kernel(const unsigned mul, const int tiles, const int pooled, const ConvArgs a, const PoolGeom g, const half8* x,
                                                           half8* y) {
  extern __shared__ uint4 lds[];
  const unsigned number = blockIdx.x >> 3, round = number >> 2, engine = number & 3;
  auto convs_of = [&](unsigned e, unsigned rounds) { return (unsigned)(((unsigned long long)rounds * mul + ((unsigned long long)e << 30)) >> 32); };
  const bool conv = convs_of(engine, round + 1) > convs_of(engine, round);
  unsigned convs = 0;
  for (unsigned e = 0; e < 4; ++e) convs += convs_of(e, round + (e < engine));
  const int place = (int)((conv ? convs : number - convs) * 8 + (blockIdx.x & 7));
  if (place >= (conv ? tiles : pooled)) return;   // (the last eight of either)
  if (conv) igemm_dma_tile<false, 2, 2, 2, 1, 3, 1, 1, false, true, false>(a, xcd_remap(place, tiles), lds);
  else maxpool_fixed_tile<half8, 8, 3, STRIDE, OUT>(x, y, g, place);
}

template <int STRIDE, int OUT>
hipError_t launch_pool_with(const ConvArgs& a, int tiles, const PoolGeom& g, const void* x, void* y, hipStream_t st) {
  const int pooled = (int)((g.total + 255u) / 256u), groups = ((tiles + 7) / 8 + (pooled + 7) / 8 + 3) & ~3;
  const unsigned mul = (unsigned)((((unsigned long long)((tiles + 7) / 8) << 32) + (unsigned)groups - 1) / (unsigned)groups);
  const size_t lds_bytes = igemm_dma_slots<false, 2, 2, 2, 1, 3, 1, false>() * 16;
  hipLaunchKernelGGL((conv_pool_kernel<STRIDE, OUT>), dim3((unsigned)groups * 8u), dim3(256), lds_bytes, st, mul, tiles, pooled, a, g,
                     static_cast<const half8*>(x), static_cast<half8*>(y));
  return hipGetLastError();
}

}  // namespace

// The 3x3 kernel's variant 0 with 128-byte chunks and LDS for two workgroups a CU; its sums are those of every variant with such
// chunks (a chunk's nine taps one after another) but the one that splits them (6).
bool conv_group_takes_3x3(const ConvArgs& a) {
  HaloArgs h;
  size_t lds_bytes;
  return a.nseg && conv_halo_group_args(a, h, lds_bytes) && lds_bytes <= 80 * 1024 - 64;
}

long conv_group_tiles(const ConvArgs& a, bool is_c3) {
  HaloArgs h;
  size_t lds_bytes;
  const long rows = is_c3 && conv_halo_group_args(a, h, lds_bytes) ? h.g.Mflat : a.M;
  return (rows + kBM - 1) / kBM * ((a.K + kBN - 1) / kBN);
}

hipError_t launch_conv_group(const ConvArgs* c3, const ConvArgs* c1, const ConvArgs* c2, hipStream_t st) {
  HaloArgs h{};
  ConvArgs m[2] = {};
  int tiles[3] = {0, 0, 0};
  size_t lds_bytes = 0;
  if (c3) {
    if (!conv_group_takes_3x3(*c3) || !conv_halo_group_args(*c3, h, lds_bytes)) return hipErrorInvalidValue;
    const int tiles_m = (h.g.Mflat + kBM - 1) / kBM, tiles_n = (c3->K + kBN - 1) / kBN;
    h.g.fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
    h.g.fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
    tiles[0] = tiles_m * tiles_n;
  }
  const ConvArgs* c[2] = {c1, c2};
  const size_t ring[2] = {igemm_dma_slots<false, 2, 2, 2, 1, 4, 1, false>() * 16, igemm_dma_slots<false, 2, 2, 2, 1, 3, 2, false>() * 16};
  for (int i = 0; i < 2; ++i) {
    if (!c[i]) continue;
    m[i] = *c[i];
    if (!igemm_dma_supported(m[i], false) || (i == 1 && m[i].C % (2 * BKV * 8))) return hipErrorInvalidValue;
    const int tiles_m = (m[i].M + kBM - 1) / kBM, tiles_n = (m[i].K + kBN - 1) / kBN;
    m[i].split = 1;
    m[i].fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
    m[i].fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
    tiles[1 + i] = tiles_m * tiles_n;
    lds_bytes = lds_bytes > ring[i] ? lds_bytes : ring[i];
  }
  static std::atomic<bool> raised{false};  // dynamic LDS above the default limit has to be asked for once per kernel
  if (!raised.load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_group_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
    if (e != hipSuccess) return e;
    raised.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(conv_group_kernel, dim3(tiles[0] + tiles[1] + tiles[2]), dim3(256), lds_bytes, st, tiles[1], tiles[0], tiles[2], m[0], h, m[1]);
  return hipGetLastError();
}

// The conv runs on the small-ring 128 x 64 tiles that it takes by itself, four to a CU.
hipError_t launch_conv_pool(const ConvArgs& conv, int N, int C, int H, int W, int stride, int pad, int Ho, int Wo, const void* x, void* y, hipStream_t st) {
  const int out = pool_outputs(N, C / 8, stride, Ho, Wo);
  if (!igemm_dma_small_ring(conv) || C % 8) return hipErrorInvalidValue;
  ConvArgs a = conv;
  const int tiles_m = (a.M + kBM - 1) / kBM, tiles_n = (a.K + kBN - 1) / kBN;
  a.split = 1;
  a.fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
  a.fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
  const PoolGeom g = pool_geom(N, C / 8, H, W, stride, pad, Ho, Wo, out);
  const int tiles = tiles_m * tiles_n;
  return out == 2 ? launch_pool_with<1, 2>(a, tiles, g, x, y, st) : launch_pool_with<0, 1>(a, tiles, g, x, y, st);
}

}  // namespace relay
