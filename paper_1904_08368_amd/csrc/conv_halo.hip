// 3x3 / stride 1 / pad 1 conv2d for gfx950 that stages the activations ONCE per channel chunk
// (paper Section 4.1 / 4.2: same fused primitive function as conv_igemm_dma.hip, other schedule).
//
// The implicit-GEMM kernel re-fetches the activation tile for each of the nine filter taps: its
// L2->LDS traffic is what bounds the 3x3 layers of the workloads.  Here the pixels are numbered in
// a "padded-flat" coordinate in which a filter tap is a constant shift:
//     o = n*F + p*P + q,   P = W + 1,  F = (H + 1)*P
// (one shared zero column between image rows, one shared zero row between images: the left
// padding of a row is the right padding of the row before it).  Output position o reads input
// position o + r*P + s for tap (r, s), where input position g holds pixel (row - 1, col - 1) of
// image g / F with (row, col) = divmod(g % F, P), and zero when row == 0 or col == 0.  A
// workgroup owns BM consecutive positions (positions with q == W or p == H are computed and
// dropped: 3-15 % of the work on these images) x BN channels.  Per chunk of CK input channels it
// needs the BM + 2P + 2 input positions from its first one on -- the halo -- which it loads once
// into LDS with global->LDS loads (zero fill by out-of-range offset, as in the other kernel);
// the nine taps then read the same buffer at row offsets r*P + s.  The LDS swizzle is keyed on
// row >> 2 and any 16 consecutive rows cover all banks, so the shifted reads stay conflict-free.  (16 x 16 tiles read two runs of
// 16 rows that start 18 apart: 30 % of their LDS clocks are conflicts, 7 % of the flat 256 x 64 tile's.)
// Filters go through a 3-stage ring, one tap x chunk per stage, exactly as before.
//
// Pipeline: a "step" is one (chunk, tap).  Step i multiplies operands that step i-1 read from LDS and reads those of step
// i+1 behind its own MFMAs, so that LDS and matrix cores work at the same time; behind them a wave also issues the filter
// loads of step i+3 and its share of the NEXT chunk's halo (spread over the first 7 taps).  Nine steps per chunk and three
// ring stages make the stage of a step, and how many loads may be pending at its barrier, compile-time constants.
// What bounds it: layers of one or two tiles per CU spend about 5 us on launch, first loads and stores (256 -> 256 at 14 x 14, batch
// 32: 11.1 us of which the MFMAs take 4.2); large ones the L2-to-LDS loads and the clock that the card holds under the matrix
// cores' load (512 -> 512 at 28 x 28, batch 32, over four seconds: 1030 to 1080 TFLOP/s at 1.73 to 1.77 GHz on random data, 1523 at 2.40
// GHz on zeros; a library's best 8192^3 product 1550 at 1.70 GHz on random data).
#include <cstdio>

#include <atomic>
#include <type_traits>

#include "conv_halo_tile.hpp"

namespace relay {
namespace {

template <bool IS_I8, int WAVES_M, int WAVES_N, int TM, int TN, int KP, int HB = 1, bool SQUARE = false, int SK = 1, bool EXT = false,
          bool POOL = false>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * SK, 2) void conv3x3_halo_kernel(const int workgroups, const HaloArgs block) {
  conv3x3_halo_tile<IS_I8, WAVES_M, WAVES_N, TM, TN, KP, HB, SQUARE, SK, EXT, POOL>(block, xcd_remap((int)blockIdx.x, workgroups), (int)blockIdx.x, workgroups);
}

struct HaloTile {
  int waves_m, waves_n, tm, tn, hb;
  bool square;
  int sk;
  constexpr int waves() const { return waves_m * waves_n * sk; }
  constexpr int bm() const { return waves_m * tm * 32; }
  constexpr int bn() const { return waves_n * tn * 32; }
};
// must match launch_halo_typed (int8: 0, 1 and 6 only)
constexpr HaloTile kHalo[] = {
    {2, 2, 2, 1, 1, false, 1},   // 0: 128 x 64
    {2, 2, 1, 1, 1, false, 1},   // 1: 64 x 64
    {4, 1, 2, 2, 2, false, 1},   // 2: 256 x 64, four waves of 64 x 64
    {4, 2, 2, 2, 1, false, 1},   // 3: 256 x 128, eight waves of 64 x 64
    {4, 1, 2, 2, 2, false, 1},   // 4: 256 x 64 with 64-byte chunks: two workgroups per CU also on wide images
    {4, 1, 2, 2, 2, true, 1},    // 5: 256 x 64 as 16 x 16 outputs of one image
    {1, 1, 2, 2, 1, false, 4},   // 6: 64 x 64, four waves that each run a quarter of the k-steps of the whole tile
};
constexpr int kNumHalo = 7;

// 64-byte planes of a chunk, 0 where the variant has no form for the channel count
int chunk_planes(const ConvArgs& a, bool is_i8, int v) {
  const int ve = is_i8 ? 16 : 8;
  const bool two = a.C % (2 * BKV * ve) == 0, four = a.C % (4 * BKV * ve) == 0;
  // the 64 x 64 tiles take 256-byte chunks (half the barriers per product) where the channel count allows and
  // the halo still fits the load slots
  const HaloTile& t = kHalo[v];
  if ((v == 1 || v == 6) && four && 4 * ((t.bm() + 2 * (a.W + 1) + 2 + 15) / 16) <= XPW * t.hb * t.waves()) return 4;
  if (v == 6) return 0;
  if (v == 4) return 1;
  if (v == 5) return a.C == 2 * BKV * ve ? 2 : 1;   // (one chunk: the halo needs one buffer only)
  return two ? 2 : 1;
}

bool make_geom(const ConvArgs& a, bool is_i8, int v, HaloGeom& g, size_t& lds_bytes) {
  const int kp = chunk_planes(a, is_i8, v), ve = is_i8 ? 16 : 8;
  if (kp == 0) return false;
  if (kHalo[v].square) {
    g.P = (a.W + SQ - 1) / SQ;                       // tiles of a row
    g.F = ((a.H + SQ - 1) / SQ) * g.P;               // ... of an image
    if ((long)a.N * g.F * SQ * SQ > 0x3fffffffL) return false;
    g.Mflat = a.N * g.F * SQ * SQ;
    g.fd_row = make_fastdiv((uint32_t)g.P);
    g.rcp_p = g.rcp_f = 0.f;
  } else {
    g.P = a.W + 1;
    g.F = (a.H + 1) * g.P;
    if ((long)a.N * g.F > 0x3fffffffL || g.F >= (1 << 21)) return false;
    g.Mflat = a.N * g.F;
    g.rcp_p = 1.0f / (float)g.P;
    g.rcp_f = 1.0f / (float)g.F;
    g.fd_row = make_fastdiv(1u);
  }
  const int rows = kHalo[v].square ? SQP * SQP : kHalo[v].bm() + 2 * g.P + 2;
  g.xblk = (rows + 15) / 16;
  g.ncc = a.C / (kp * BKV * ve);
  g.nxbuf = g.ncc > 1 ? 2 : 1;
  g.fd_f = make_fastdiv((uint32_t)g.F);
  if (kp * g.xblk > XPW * kHalo[v].hb * kHalo[v].waves()) return false;  // a halo must fit the waves' load slots
  const size_t ring = (size_t)g.nxbuf * kp * g.xblk * 64 + (size_t)NSW * kp * kHalo[v].bn() * BKV + 64;
  const HaloTile& t = kHalo[v];
  const int own = t.tm * t.tn / t.sk;   // blocks a wave finishes
  const size_t epi = (size_t)t.waves() * ((t.sk > 1 ? (t.tm * t.tn - own) * 4 * 64 : 0) + 32 * ((t.sk == 4 ? 1 : t.tn) * 8 + 1));
  g.tab_slot = (int)(ring > epi ? ring : epi);
  lds_bytes = ((size_t)g.tab_slot + (size_t)g.xblk * 4) * 16;  // + 4 bytes per halo position
  return lds_bytes <= 160 * 1024;
}

template <bool EXT, bool IS_I8, int WM, int WN, int TM, int TN, int KP, int HB, bool SQUARE, int SK, bool POOL = false>
hipError_t launch_halo_store(const ConvArgs& a, const HaloGeom& g, size_t lds_bytes, hipStream_t st) {
  auto kern = conv3x3_halo_kernel<IS_I8, WM, WN, TM, TN, KP, HB, SQUARE, SK, EXT, POOL>;
  static std::atomic<bool> raised{false};  // dynamic LDS above the default limit has to be asked for once per kernel
  if (!raised.load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                             160 * 1024);
    if (e != hipSuccess) return e;
    raised.store(true, std::memory_order_release);
  }
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  const int tiles_m = (g.Mflat + BM - 1) / BM, tiles_n = (a.K + BN - 1) / BN;
  HaloArgs block{g, a};
  block.g.fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
  block.g.fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(64 * WM * WN * SK), lds_bytes, st, tiles_m * tiles_n, block);
  return hipGetLastError();
}

// (output channel segments take an instantiation of their own, as in the implicit GEMM)
template <bool IS_I8, int WM, int WN, int TM, int TN, int KP, int HB = 1, bool SQUARE = false, int SK = 1>
hipError_t launch_halo_one(const ConvArgs& a, const HaloGeom& g, size_t lds_bytes, hipStream_t st) {
  return a.nseg ? launch_halo_store<true, IS_I8, WM, WN, TM, TN, KP, HB, SQUARE, SK>(a, g, lds_bytes, st)
                : launch_halo_store<false, IS_I8, WM, WN, TM, TN, KP, HB, SQUARE, SK>(a, g, lds_bytes, st);
}

template <bool IS_I8>
hipError_t launch_halo_typed(const ConvArgs& a, const HaloGeom& g, size_t lds_bytes, int v, int kp, hipStream_t st) {
  if (v == 0) return kp == 2 ? launch_halo_one<IS_I8, 2, 2, 2, 1, 2>(a, g, lds_bytes, st)
                             : launch_halo_one<IS_I8, 2, 2, 2, 1, 1>(a, g, lds_bytes, st);
  if constexpr (!IS_I8) {
    if (v == 2) return kp == 2 ? launch_halo_one<IS_I8, 4, 1, 2, 2, 2, 2>(a, g, lds_bytes, st)
                               : launch_halo_one<IS_I8, 4, 1, 2, 2, 1, 2>(a, g, lds_bytes, st);
    if (v == 3) return kp == 2 ? launch_halo_one<IS_I8, 4, 2, 2, 2, 2>(a, g, lds_bytes, st)
                               : launch_halo_one<IS_I8, 4, 2, 2, 2, 1>(a, g, lds_bytes, st);
    if (v == 4) return launch_halo_one<IS_I8, 4, 1, 2, 2, 1, 2>(a, g, lds_bytes, st);
    if (v == 5) return kp == 2 ? launch_halo_one<IS_I8, 4, 1, 2, 2, 2, 2, true>(a, g, lds_bytes, st)
                               : launch_halo_one<IS_I8, 4, 1, 2, 2, 1, 2, true>(a, g, lds_bytes, st);
  }
  if (v == 6) return launch_halo_one<IS_I8, 1, 1, 2, 2, 4, 1, false, 4>(a, g, lds_bytes, st);
  if (kp == 4) return launch_halo_one<IS_I8, 2, 2, 1, 1, 4>(a, g, lds_bytes, st);
  return kp == 2 ? launch_halo_one<IS_I8, 2, 2, 1, 1, 2>(a, g, lds_bytes, st)
                 : launch_halo_one<IS_I8, 2, 2, 1, 1, 1>(a, g, lds_bytes, st);
}

}  // namespace

int conv_halo_variant_count() { return kNumHalo; }

namespace {
// 3x3, stride 1, pad 1, plain NHWC, whole chunks of channels, deterministic rounding.
bool conv_halo_shape(const ConvArgs& a, bool is_i8) {
  const int es = is_i8 ? 1 : 2, ve = is_i8 ? 16 : 8;
  if (a.R != 3 || a.S != 3 || a.sh != 1 || a.sw != 1 || a.ph != 1 || a.pw != 1) return false;
  if (a.xs_w != a.C || a.xs_h != a.W * a.C || a.xs_n != a.H * a.W * a.C) return false;
  if (a.C % (BKV * ve) != 0 || a.round_mode == ROUND_STOCHASTIC) return false;
  // Output channel segments, as long as they share the window and hold whole vectors of 8 channels: the 128 -> 192 conv of an Inception
  // block at 32 x 28 x 28 into 192 of 480 channels 21.3 us by the implicit GEMM, 16.9 here (20.0 against 24.1 behind the block's
  // other launches, its operands no longer in L2).
  if (a.nseg && (a.seg_centre || (a.K & 7) || (a.flags & F_RES))) return false;   // (segments of the whole window, in vectors of 8 channels)
  if ((size_t)a.N * a.xs_n * es > 0x7fffffffu || (size_t)a.K * a.Kp * es > 0x7fffffffu) return false;
  return true;
}

bool halo_fits(const ConvArgs& a, bool is_i8, int v, size_t most_lds = 160 * 1024) {
  HaloGeom g;
  size_t lds_bytes;
  return make_geom(a, is_i8, v, g, lds_bytes) && lds_bytes <= most_lds;
}
}  // namespace

bool conv_halo_supported(const ConvArgs& a, bool is_i8, int v) {
  return v >= 0 && v < kNumHalo && !(is_i8 && v >= 2 && v <= 5) && conv_halo_shape(a, is_i8) && halo_fits(a, is_i8, v);
}

namespace {
// What a variant is estimated to take: a + b n + c n s + e x s microseconds, with s the steps of a tile, x the tiles per CU and
// n the tiles of the CU that has most.  Fitted to about 1500 random layers (32 to 1024 channels, 32 to 512 filters, 5 to 250
// pixels a side, 1 to 64 images; rms error 3 to 8 %), separately for chunks of one and of several reductions (a tile of one
// chunk needs one halo buffer, so that two or three workgroups fit a CU).
struct HaloCost {
  int v, kp;
  bool one;    // the channels are a single chunk
  int most;    // not for more tiles than this: beyond, several rounds of a tile made for few of them (0: any number)
  float a, b, c, e;
};
constexpr HaloCost kCostF16[] = {
    {0, 1, false, 0, 3.23f, 1.23f, 0.092f, 0.037f},
    {0, 2, false, 0, 2.44f, 1.81f, 0.155f, 0.068f},
    {0, 2, true, 0, 3.58f, 0.00f, 0.232f, 0.106f},
    {1, 2, true, 512, 3.16f, 0.00f, 0.183f, 0.045f},
    {1, 4, false, 512, 0.83f, 2.88f, 0.213f, 0.070f},
    {1, 4, true, 512, 2.53f, 0.00f, 0.352f, 0.051f},
    {3, 2, false, 0, 0.00f, 6.75f, 0.429f, 0.337f},
    {4, 1, false, 0, 2.73f, 3.32f, 0.134f, 0.081f},
    {5, 1, false, 0, 3.87f, 2.13f, 0.145f, 0.045f},
    {5, 2, true, 0, 4.03f, 0.00f, 0.485f, 0.174f},
    {6, 4, false, 512, 0.86f, 3.16f, 0.155f, 0.100f},
    {6, 4, true, 512, 2.51f, 0.00f, 0.362f, 0.052f},
};
constexpr HaloCost kCostI8[] = {
    {0, 1, false, 0, 3.60f, 1.01f, 0.110f, 0.017f},
    {0, 1, true, 0, 4.32f, 0.00f, 0.158f, 0.046f},
    {0, 2, false, 0, 2.15f, 2.86f, 0.157f, 0.038f},
    {0, 2, true, 0, 3.77f, 0.00f, 0.295f, 0.012f},
    {1, 1, true, 1024, 3.81f, 0.00f, 0.090f, 0.040f},
    {1, 2, true, 1024, 3.68f, 0.00f, 0.177f, 0.002f},
    {1, 4, false, 512, 0.85f, 0.00f, 0.406f, 0.036f},
    {1, 4, true, 512, 3.16f, 0.00f, 0.322f, 0.047f},
    {6, 4, false, 512, 1.07f, 0.00f, 0.364f, 0.056f},
    {6, 4, true, 512, 3.07f, 0.00f, 0.347f, 0.045f},
};
}  // namespace

// Layers that a caller's forced split of the reduction (n > 1) leaves whole.  Their 128 x 64 tiles give every CU one or fill the
// 512 workgroup slots up to twice over (256 channels and more, 64 -> 64 in fp16: any number), so that there is nothing to gain
// from partial sums and these would be large: 206 MB for 256 -> 256 at 56 x 56, batch 32 in two runs.  Outside this range a
// forced split is the implicit GEMM's, also of a layer that conv_halo_pick would take (512 -> 512 at 14 x 14, batch 8).
bool conv_halo_keeps_whole(const ConvArgs& a, bool is_i8) {
  if (a.R != 3 || a.S != 3 || a.C < 64 || a.nseg || !conv_halo_shape(a, is_i8)) return false;
  const long flat = (long)a.N * (a.H + 1) * (a.W + 1), tiles_n = (a.K + 63) / 64;
  if (!is_i8 && a.C >= 512 && a.W <= 7 && chunk_planes(a, is_i8, 1) == 4 && halo_fits(a, is_i8, 1)) {
    const long t64 = ((flat + 63) / 64) * tiles_n;
    if (t64 >= 190 && t64 <= 512) return true;
  }
  const bool thin = !is_i8 && a.C == 64 && a.K <= 64;
  if ((a.W > 56 && !thin) || !halo_fits(a, is_i8, 0)) return false;
  const long t128 = ((flat + 127) / 128) * tiles_n;
  if (!is_i8 && (a.C >= 256 || thin)) return t128 >= 190;
  return t128 >= 190 && t128 <= (!is_i8 && a.C == 64 ? 1024 : 512);
}

// The variant the heuristic takes, or -1 to leave the layer to the other kernels: the least of the estimates above,
// where it is below those of the implicit GEMM and of the small-tile kernel.
//  * Below 80 tiles of 64 x 64 the small-tile kernel is the better one always (the search is not even begun: it costs
//    an eager call about 0.2 us).
//  * fp16, a layer the small-tile kernel would take: only variant 6, which sums in four runs as that kernel does.  The others sum
//    in one, which is less exact.
//  * fp16 with a max pool behind it in mind: not variant 6.  The pooled launch promises the bits of the two calls and follows the
//    order of one run of sums, not the exchange of four.
//  * 256 x 64 tiles with 64-byte chunks: only two to a CU, by their number and by their LDS (alone they wait at every barrier:
//    12 x 20 x 18, 512 -> 512 38.6 us against 32.4 as 128 x 64).
//  * 64 -> 64 channels in fp16, 128-position tiles for between one and about three rounds of the chip's 512 workgroup slots: the
//    256-position tile halves the rounds (56 x 56 at batch 32: 13.9 against 14.9 us).
//    But while the implicit GEMM's 128 pixels a tile, without the pad positions, are still one round of those slots, that one is left the layer
//    (31 x 57 x 37, 511 tiles there and 534 here: 10.0 us against 12.0; 20 x 56 x 59, 517 and 535: 13.9 against 12.1).
//    Two of its workgroups have to fit a CU's LDS (images up to 86 wide): 34 x 23 x 121, 64 -> 56 13.9 us by the implicit GEMM, 17.0.
//  * Layers that 128 x 64 tiles suit (conv_halo_keeps_whole) leave them only for a clear gain, since the estimates err by 10 %: for
//    the implicit GEMM where it is estimated at 0.9 of their time (0.82 with its 64-byte chunks, whose estimates are low), for 16 x 16
//    tiles at 0.95 (0.9).  Of 492 and 141 random layers that the plain minimum took away 42 % and 20 % became slower, by up to 24 %
//    (int8 42 x 27 x 13, 576 -> 80 17.8 us, implicit GEMM 22.5); with the margins 0.4 % and 2 %.
//  * int8, a single chunk, 64 x 64 tiles on images wider than 62, whose halos are three times the tile and more: only where all tiles
//    fit the LDS of the chip at once (44 x 18 x 72, 128 -> 64 in 1026 tiles 10.9 us, implicit GEMM 9.2; 3 x 175 x 68, 128 -> 32 in 570
//    7.0 and 8.1).
//  * int8 that gives the 256 x 128 tile of the implicit GEMM its 384 tiles stays there (512 -> 512 at 33 x 55, batch 18: 94
//    against 110 us).
// Fp16 at batch 32, graph-timed, before this kernel overlapped its operand reads with the matrix instructions and had the wider
// tiles / now: 64 -> 64 at 224 x 224 208 (implicit GEMM) / 148 us, 64 -> 128 at 112 x 112 84 / 72, 128 -> 128 147 / 125, 128 -> 256 at
// 56 x 56 81 / 67, 256 -> 256 127 / 120, 256 -> 512 at 28 x 28 66.6 / 60.4, 512 -> 512 126.5 / 109.6; 64 -> 64 at 56 x 56 14.5 / 13.9,
// 128 -> 128 at 28 x 28 11.3 / 11.1, 512 -> 512 at 7 x 7 14.1 / 13.1.
int conv_halo_pick(const ConvArgs& a, bool is_i8) {
  if (a.R != 3 || a.S != 3 || a.C < 64) return -1;
  const long flat = (long)a.N * (a.H + 1) * (a.W + 1), tiles_n = (a.K + 63) / 64;
  if (((flat + 63) / 64) * tiles_n < 80 || !conv_halo_shape(a, is_i8)) return -1;
  const long t128 = ((flat + 127) / 128) * tiles_n;
  if (!is_i8 && a.C == 64 && a.K <= 64 && t128 > 512 && t128 <= 1700 && halo_fits(a, is_i8, 2, 80 * 1024)) return (a.M + 127) / 128 <= 512 ? -1 : 2;
  if (is_i8 && igemm_dma_wide(a)) return -1;
  const float staged = igemm_dma_estimate(a, is_i8), small = conv_small_estimate(a, is_i8);
  const int ve = is_i8 ? 16 : 8;
  const bool whole = conv_halo_keeps_whole(a, is_i8);
  float best = whole ? staged * (a.C % (2 * BKV * ve) ? 1.f / 0.82f : 1.f / 0.9f) : 0.98f * staged;
  if (best > 0.98f * small) best = 0.98f * small;
  int pick = -1;
  const bool pooled = !is_i8 && igemm_dma_pool_supported(a, false);
  const int rows = is_i8 ? (int)(sizeof(kCostI8) / sizeof(HaloCost)) : (int)(sizeof(kCostF16) / sizeof(HaloCost));
  for (int i = 0; i < rows; ++i) {
    const HaloCost& h = is_i8 ? kCostI8[i] : kCostF16[i];
    const HaloTile& t = kHalo[h.v];
    const int chunk = h.kp * BKV * ve;
    if ((a.C == chunk) != h.one || a.C % chunk != 0 || (!is_i8 && small < staged && h.v != 6) || (pooled && h.v == 6)) continue;
    const long tm = t.square ? (long)a.N * ((a.H + SQ - 1) / SQ) * ((a.W + SQ - 1) / SQ) : (flat + t.bm() - 1) / t.bm();
    const long tiles = tm * ((a.K + t.bn() - 1) / t.bn());
    if ((h.most && tiles > h.most) || ((h.v == 4 || h.v == 5) && tiles <= 256)) continue;
    const float n = (float)((tiles + 255) / 256), x = (float)tiles * (1.f / 256.f), s = 9.f * (float)(a.C / chunk);
    const float us = (h.a + n * (h.b + h.c * s) + h.e * x * s) * (whole && h.v == 5 ? (a.C % (2 * BKV * ve) ? 1.f / 0.9f : 1.f / 0.95f) : 1.f);
    const size_t most_lds = 160 * 1024 / (h.v == 4 ? 2 : is_i8 && h.v == 1 && h.one && a.W > 62 ? (tiles + 255) / 256 : 1);
    if (us < best && chunk_planes(a, is_i8, h.v) == h.kp && halo_fits(a, is_i8, h.v, most_lds)) {
      best = us;
      pick = h.v;
    }
  }
  return pick;
}

bool conv_halo_group_args(const ConvArgs& a, HaloArgs& block, size_t& lds_bytes) {
  if (!conv_halo_supported(a, false, 0) || chunk_planes(a, false, 0) != 2 || !make_geom(a, false, 0, block.g, lds_bytes)) return false;
  block.a = a;
  return true;
}

int conv_halo_chunk(const ConvArgs& a, bool is_i8, int v) { return chunk_planes(a, is_i8, v) * BKV * (is_i8 ? 16 : 8); }

void conv_halo_kernel_name(const ConvArgs& a, bool is_i8, int v, char* buf, size_t len) {
  const HaloTile& t = kHalo[v];
  // (trailing template arguments at their defaults are left out, though a trace prints all eleven)
  char tail[40] = "";
  if (a.nseg) snprintf(tail, sizeof(tail), ", %s, %d, true", t.square ? "true" : "false", t.sk);
  else if (t.sk > 1) snprintf(tail, sizeof(tail), ", %s, %d", t.square ? "true" : "false", t.sk);
  else if (t.square) snprintf(tail, sizeof(tail), ", true");
  snprintf(buf, len, "conv3x3_halo_kernel<%s, %d, %d, %d, %d, %d, %d%s>", is_i8 ? "true" : "false", t.waves_m, t.waves_n, t.tm, t.tn,
           chunk_planes(a, is_i8, v), t.hb, tail);
}

// 2x2 / stride 2 max pool behind the conv, on 16 x 16 tiles: fp16, whole vectors of channels, whole windows, and a relu (no NaN left
// to order).  The pool's read of the conv outputs and its launch go: of 64 -> 64 at batch 32 of 224 x 224 155 + 42 us as two launches,
// of 128 -> 128 at 112 x 112 120 + 21 us; 168 and 127 as one each.  (The whole network
// gains 24 of 1170 us: the convs behind take 5 % longer than with the pools between them, the card's clock being what its load allows.)
bool conv_halo_pool2_supported(const ConvArgs& a) {
  return conv_halo_supported(a, false, 5) && !a.nseg && (a.flags & F_RELU) && !(a.flags & F_RES) && !((a.H | a.W) & 1) && !(a.K & 7) &&
         (long)a.M * 2 <= 0x7fffffffL;
}

hipError_t launch_conv_halo_pool2(const ConvArgs& a, void* y_pooled, hipStream_t st) {
  HaloGeom g;
  size_t lds_bytes;
  if (!conv_halo_pool2_supported(a) || !make_geom(a, false, 5, g, lds_bytes)) return hipErrorInvalidValue;
  g.y_pooled = y_pooled;
  g.fd_w = make_fastdiv((uint32_t)a.W);
  return chunk_planes(a, false, 5) == 2 ? launch_halo_store<false, false, 4, 1, 2, 2, 2, 2, true, 1, true>(a, g, lds_bytes, st)
                                        : launch_halo_store<false, false, 4, 1, 2, 2, 1, 2, true, 1, true>(a, g, lds_bytes, st);
}

hipError_t launch_conv_halo(const ConvArgs& a, bool is_i8, int v, hipStream_t st) {
  HaloGeom g;
  size_t lds_bytes;
  if (!make_geom(a, is_i8, v, g, lds_bytes)) return hipErrorInvalidValue;
  const int kp = chunk_planes(a, is_i8, v);
  return is_i8 ? launch_halo_typed<true>(a, g, lds_bytes, v, kp, st) : launch_halo_typed<false>(a, g, lds_bytes, v, kp, st);
}

}  // namespace relay
