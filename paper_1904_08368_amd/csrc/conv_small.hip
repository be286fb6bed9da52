// Implicit-GEMM conv2d for gfx950 where a layer has few output tiles (small batches, deep layers): the
// waves of a workgroup split the REDUCTION of one small tile between them.
//
// The staged kernels (conv_igemm_dma.hip, conv_halo.hip) give a 64 x 64 tile to a workgroup, so a
// batch-1 layer of ResNet-18 has 8 to 50 workgroups for 256 compute units, each of which walks its
// 9 to 36 reduction chunks one after another behind a barrier per chunk: bound by that serial chain, not by any
// unit.  Here a tile is TM x TN blocks of 16 pixels x 16 channels (16 x 16 up to 32 x 64) and wave w
// takes the w-th run of the reduction's units (U steps of 64 bytes of one filter tap).  Each wave brings its
// operands into a ring in LDS that is its own -- global->LDS loads, 16 tile rows x 64 bytes each, as in
// the staged kernels -- so nothing in the loop is a barrier and a wave waits for its own loads only.
// (Loading the MFMA operands straight into registers was measured first: a wave's load then has its lanes
// along the tile rows, the texture addresser takes one lane per clock, 36 KB/us per CU against 75 to
// 100 with four lanes along each row; 256 -> 256 at 14 x 14 took 6.3 us instead of 3.9.)
// Padding taps, ragged rows and channels get an out-of-range buffer offset and read zeros.  The partial
// tiles meet once in LDS and are added in wave order (the result does not depend on timing; int8 is
// exact in any order), then the fused tail runs as in the other kernels.
//
// Bound: the launch with its chain of argument fetch, first loads and store (2.6 us), then the bytes a CU
// draws for its tile (about 125 KB/us): each goes into LDS and out again once, which keeps LDS as busy as the one wave a SIMD has
// issues instructions (a 16 x 16 tile of 512 channels: 1.9 K clocks to the last of the first requests, 4.5 K in nine units, 1.4 K for the tail).
// An input patch shared by the waves (fewer bytes, but a barrier and a wait in front of the loop; 512 channels, seven images 8.3 -> 8.0 us, one image
// 5.5 -> 5.9), eight waves (5.5 -> 5.9) and deeper rings (1 to 4 % slower with operands from beyond the L2) were no better.  Graph-timed at batch 1, staged kernels -> this one: fp16 64 -> 64 at
// 56 x 56 5.1 -> 3.8 us, 128 at 28 x 28 5.9 -> 3.7, 256 at 14 x 14 8.2 -> 3.9, 512 at 7 x 7 9.5 -> 4.7; int8 5.0 -> 3.5,
// 5.3 -> 3.5, 5.8 -> 3.3, 9.0 -> 3.9.
#include <cmath>
#include <cstdio>
#include <type_traits>

#include "dma_common.hpp"

namespace relay {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

template <bool IS_I8>
struct Mma16;
template <>
struct Mma16<false> {
  typedef floatx4 acc_t;
  static __device__ __forceinline__ acc_t mma(const uint4& a, const uint4& b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  }
};
template <>
struct Mma16<true> {
  typedef intx4 acc_t;
  static __device__ __forceinline__ acc_t mma(const uint4& a, const uint4& b, acc_t c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(intx4, a), __builtin_bit_cast(intx4, b), c, 0, 0, 0);
  }
};

// A filter offset that stays out of range whatever reduction position (or kOob) is added to it: no packed
// filter tensor reaches it (its size is a multiple of 128 below 2^31).
constexpr unsigned kDeadRow = 0x7ffffff0u;

// n / d by the host's constants without a branch: (uniform) the divisor 1 has no multiplier
__device__ __forceinline__ uint32_t div_by(uint32_t n, FastDiv f) { return (__umulhi(n, f.mul) >> f.shift) | (n & (f.mul ? 0u : ~0u)); }

// What the host works out for a launch, so that no wave divides or multiplies for it.
struct SmallGeom {
  int tiles_m, tiles_n;
  int per_tap, per_wave, units;  // units of a filter tap, of a wave's run, of the reduction
  FastDiv fd_per_tap, fd_s;      // division by per_tap and by S
};

// EXT: the instantiation that stores output channel segments.  NA: accumulators per block of a tile, used in turn (see small_runs).
// tile: the workgroup's place among the tiles of this conv (xcd_remap).
template <bool IS_I8, int TM, int TN, int W, int U, int NS, bool EXT, int NA>
__device__ __forceinline__ void small_tile(const ConvArgs& a, const SmallGeom& g, int tile) {
  constexpr int VE = IS_I8 ? 16 : 8;
  constexpr int ES = IS_I8 ? 1 : 2;
  constexpr int CU = U * BKV * VE;  // channels per unit: U steps of 64 bytes
  constexpr int BM = TM * 16, BN = TN * 16;
  constexpr int ITEMS = TM * TN * 32;               // (pixel, 8 channels) pieces of the tile
  constexpr int IPT = (ITEMS + 64 * W - 1) / (64 * W);
  constexpr int LPU = (TM + TN) * U;                // loads (and KiB of LDS) per unit
  constexpr int RING = NS * LPU * 64;               // 16-byte slots of a wave's ring
  static_assert(TM * TN * 64 <= RING, "a wave's partial tile reuses its ring");
  static_assert((NS - 1) * LPU <= 63, "vmcnt is a 6-bit counter");
  typedef typename Mma16<IS_I8>::acc_t acc_t;

  __shared__ uint4 ring[W * RING];
  __shared__ float cst[2 * BN];

  // Every argument is asked for at the top, so that the scalar loads leave as one batch with one wait.  The workgroup's number passes through
  // the same statement: arithmetic on it that needs only some of the arguments was moved ahead of the others' loads, and two batches one
  // behind the other are two latencies of 480 to 1100 clocks (the host has just written that memory, no cache has it yet).  With the
  // other kernels', whose prologues had two or three batches, and the copied blocks of the pairs: ResNet-18 at batch 1 81.9 -> 75.5 us, int8 66.8
  // -> 61.4, at batch 7 131.8 -> 126.2, at batch 32 264.2 -> 260.9, deep Q-network 18.0 -> 17.3, MobileNet-v1 of 11 images 130.9 -> 129.4.
#define RELAY_ASKED                                                                                                                      \
  "s"(a.x), "s"(a.w), "s"(a.y), "s"(a.res), "s"(a.bias), "s"(a.scale), "s"(a.shift), "s"(a.qbias), "s"(a.N), "s"(a.H), "s"(a.W), "s"(a.C), \
      "s"(a.K), "s"(a.R), "s"(a.S), "s"(a.sh), "s"(a.sw), "s"(a.ph), "s"(a.pw), "s"(a.Ho), "s"(a.Wo), "s"(a.xs_n), "s"(a.xs_h),           \
      "s"(a.xs_w), "s"(a.tap_spread), "s"(a.n_major), "s"(a.M), "s"(a.Kred), "s"(a.Kp), "s"(a.flags), "s"(a.fd_wo.mul), "s"(a.fd_wo.shift), \
      "s"(a.fd_howo.mul), "s"(a.fd_howo.shift), "s"(a.fd_tiles_m.mul), "s"(a.fd_tiles_m.shift), "s"(a.fd_tiles_n.mul),                    \
      "s"(a.fd_tiles_n.shift), "s"(g.tiles_m), "s"(g.tiles_n), "s"(g.per_tap), "s"(g.per_wave), "s"(g.units), \
      "s"(g.fd_per_tap.mul), "s"(g.fd_per_tap.shift), "s"(g.fd_s.mul), "s"(g.fd_s.shift)
  if constexpr (IS_I8)
    asm volatile("" : "+s"(tile) : RELAY_ASKED, "s"(a.lshift), "s"(a.rshift), "s"(a.round_add), "s"(a.qmode), "s"(a.clip_lo), "s"(a.clip_hi), "s"(a.qmult),
                 "s"(a.qshift));
  else
    asm volatile("" : "+s"(tile) : RELAY_ASKED);
#undef RELAY_ASKED

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile_q = (int)div_by((uint32_t)tile, a.n_major ? a.fd_tiles_m : a.fd_tiles_n);
  const int tile_n = a.n_major ? tile_q : tile - tile_q * g.tiles_n;
  const int tile_m = a.n_major ? tile - tile_q * g.tiles_m : tile_q;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  // staging role of this lane: row lr of a block of 16 tile rows, and the k-vector that belongs in its slot
  const int lr = lane >> 2, lk = (lane & 3) ^ lds_swizzle(lr);
  const intx4 rs_x = make_rsrc(a.x, (unsigned)((size_t)a.N * a.xs_n * ES));
  const intx4 rs_w = make_rsrc(a.w, (unsigned)((size_t)a.K * a.Kp * ES));
  uint4* my = ring + wave * RING;
  const unsigned my_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint4*)(&ring[0]) + (unsigned)(wave * RING) * 16u;

  // ---- this wave's run of the reduction's units (filter tap x CU channels) and where it starts
  const int ubeg = wave * g.per_wave;
  int left = min(g.units - ubeg, g.per_wave);
  int is_tap = (int)div_by((uint32_t)ubeg, g.fd_per_tap), is_c = ubeg - is_tap * g.per_tap;
  int is_r = (int)div_by((uint32_t)is_tap, g.fd_s), is_s = is_tap - is_r * a.S;
  unsigned is_w = (unsigned)(ubeg * (CU * ES));

  unsigned w_off[TN];
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const int ch = n0 + t * 16 + lr;
    w_off[t] = ch < a.K ? (unsigned)((ch * a.Kp + lk * VE) * ES) : kDeadRow;
  }
  // the filters of a unit need no decoding: those of the first one leave before the pixels are worked out
  auto request_filters = [&](int st) {
    const unsigned dst = my_base + (unsigned)(st * LPU) * 1024u;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int u = 0; u < U; ++u) lds_dma16(rs_w, dst + (unsigned)(t * U + u) * 1024u, w_off[t] + is_w + u * 64);
    is_w += CU * ES;
  };
  if (left > 0) request_filters(0);
  int x_off[TM];        // byte offset of tap (0, 0) of the lane's pixel
  // Is a tap inside the image?  One pixel block: a bit of a mask worked out once (two instructions fewer in a loop that issues one every five
  // clocks: 512 channels at 7 x 7 5.4 us, 5.7 with comparisons).  Two: two comparisons, which start the first loads earlier (at 7 x 8, seven
  // images, 8.6 -> 8.1 us together with the early operands below, 16 images 11.6 -> 10.5, int8 7.7 -> 7.3).
  constexpr bool MASKS = TM == 1;
  unsigned x_taps[TM];         // MASKS: bit t: tap t lies inside the image
  int x_row[TM], x_col[TM];    // else: input row and column of tap (0, 0)
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int m = m0 + t * 16 + lr;
    const int n = (int)div_by((uint32_t)m, a.fd_howo), rem = m - n * (a.Ho * a.Wo);
    const int p = (int)div_by((uint32_t)rem, a.fd_wo), q = rem - p * a.Wo;
    const int ih0 = p * a.sh - a.ph, iw0 = q * a.sw - a.pw;
    x_off[t] = (n * a.xs_n + ih0 * a.xs_h + iw0 * a.xs_w + lk * VE) * ES;
    x_row[t] = m < a.M ? ih0 : -0x10000000;   // (rows past the end lie in no image)
    x_col[t] = iw0;
    if constexpr (!MASKS) continue;
    // the run of valid filter columns, replicated at every valid filter row
    const int rlo = max(0, -ih0), rhi = min(a.R, a.H - ih0);
    const int clo = max(0, -iw0), chi = min(a.S, a.W - iw0);
    const unsigned colbits = (unsigned)((1ull << max(chi, 0)) - 1ull) & ~(unsigned)((1ull << clo) - 1ull);
    const unsigned rows = a.tap_spread & (unsigned)((1ull << (max(rhi, 0) * a.S)) - 1ull) & ~(unsigned)((1ull << (rlo * a.S)) - 1ull);
    x_taps[t] = (m < a.M && rhi > rlo && chi > clo) ? colbits * rows : 0u;
  }

  auto request_pixels = [&](int st) {
    const unsigned tapbit = 1u << is_tap;
    const unsigned dx = (unsigned)((is_r * a.xs_h + is_s * a.xs_w + is_c * CU) * ES);
    const unsigned dst = my_base + (unsigned)(st * LPU + TN * U) * 1024u;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const bool in = MASKS ? (x_taps[t] & tapbit) != 0u : (unsigned)(x_row[t] + is_r) < (unsigned)a.H && (unsigned)(x_col[t] + is_s) < (unsigned)a.W;
      const unsigned off = in ? (unsigned)x_off[t] + dx : kOob;
#pragma unroll
      for (int u = 0; u < U; ++u) lds_dma16(rs_x, dst + (unsigned)(t * U + u) * 1024u, off + u * 64);
    }
    if (++is_c == g.per_tap) {
      is_c = 0;
      ++is_tap;
      if (++is_s == a.S) {
        is_s = 0;
        ++is_r;
      }
    }
  };
  if (left > 0) request_pixels(0);
#pragma unroll
  for (int st = 1; st < NS; ++st)
    if (st < left) {
      request_filters(st);
      request_pixels(st);
    }

  acc_t acc[NA][TN][TM];   // step u of a unit adds to accumulator (phase * U + u) % NA of its block
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][tn][tm][v] = 0;
  // MFMA operand of lane l: row l % 16, k-vector l / 16 of a block's 64-byte step
  const int slot = lds_slot(lane & 15, lane >> 4);
  using std::integral_constant;
  auto mma_unit = [&](int st, auto phase) {
    const uint4* at = my + st * (LPU * 64) + slot;
    uint4 f[TN + TM][U];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < TN + TM; ++t) f[t][u] = at[(t * U + u) * 64];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
          acc_t& c = acc[(decltype(phase)::value * U + u) % NA][tn][tm];
          c = Mma16<IS_I8>::mma(f[tn][u], f[TN + tm][u], c);
        }
  };

  // The constants of the tile's channels and the residual operand are asked for here, behind the first operands: neither latency then
  // stands behind the reduction.
  float k0 = 1.f, k1 = 0.f, k2 = 0.f;
  if (tid < BN) {
    const int c = n0 + tid < a.K ? n0 + tid : a.K - 1;
    if constexpr (IS_I8) {
      k0 = __builtin_bit_cast(float, (a.flags & F_BIAS) ? a.qbias[c] : 0);
    } else {
      if (a.flags & F_BN) k0 = a.scale[c], k1 = a.shift[c];
      if (a.flags & F_BIAS) k2 = a.bias[c];
    }
  }
  const bool vec_ok = (a.K & 7) == 0;
  const bool pre_res = (a.flags & F_RES) && vec_ok;
  uint4 resv[IPT];
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    const int item = it * (64 * W) + tid, m_out = m0 + item / (TN * 2), ech = n0 + item % (TN * 2) * 8;
    resv[it] = make_uint4(0u, 0u, 0u, 0u);
    if (pre_res && item < ITEMS && m_out < a.M && ech < a.K) resv[it] = load_residual8<IS_I8>(a, m_out, ech);
  }

  // NS units are in flight.  The ring is the wave's own: no barrier, only its own loads are waited for.
  int st = 0;
  auto step = [&](auto phase) {  // one unit multiplied, another requested in its place
    wait_loads<(NS - 1) * LPU>();
    mma_unit(st, phase);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    request_filters(st);
    request_pixels(st);
    st = st + 1 == NS ? 0 : st + 1;
    --left;
  };
  constexpr int TURN = NA > U ? NA / U : 1;  // units that go round the accumulators
  static_assert(NA % U == 0 || U % NA == 0, "a turn is a whole number of units");
  while (left > NS + TURN - 1) {
    step(integral_constant<int, 0>{});
    if constexpr (TURN > 1) step(integral_constant<int, 1>{});
    if constexpr (TURN > 2) {
      step(integral_constant<int, 2>{});
      step(integral_constant<int, 3>{});
    }
  }
  if constexpr (TURN > 1)
    if (left > NS) step(integral_constant<int, 0>{});
  if constexpr (TURN > 2) {
    if (left > NS) step(integral_constant<int, 1>{});
    if (left > NS) step(integral_constant<int, 2>{});
  }
  // the last NS (or fewer) units: the loads in flight run out
  if constexpr (TURN == 1) {
    for (; left > 0; --left) {
      if (NS > 3 && left > 3) wait_loads<(NS > 3 ? 3 : 0) * LPU>();
      else if (NS > 2 && left == 3) wait_loads<(NS > 2 ? 2 : 0) * LPU>();
      else if (left == 2) wait_loads<LPU>();
      else wait_loads<0>();
      mma_unit(st, integral_constant<int, 0>{});
      st = st + 1 == NS ? 0 : st + 1;
    }
  } else {
    auto last = [&](auto l) {
      if (left >= decltype(l)::value) {
        wait_loads<(decltype(l)::value - 1) * LPU>();
        mma_unit(st, l);
        st = st + 1 == NS ? 0 : st + 1;
      }
    };
    if constexpr (NS > 3) last(integral_constant<int, 4>{});
    if constexpr (NS > 2) last(integral_constant<int, 3>{});
    last(integral_constant<int, 2>{});
    last(integral_constant<int, 1>{});
  }
#pragma unroll
  for (int n = NA / 2; n > 0; n /= 2)
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[i][tn][tm] += acc[i + n][tn][tm];
  if (tid < BN) {
    cst[tid] = k0;
    if constexpr (!IS_I8) cst[BN + tid] = k2 * k0 + k1;  // (acc + b)*sc + sf
  }

  // ---- partial tiles to LDS.  Lane l of a block holds channels 4 (l / 16) .. + 3 of pixel l % 16.
#pragma unroll
  for (int tn = 0; tn < TN; ++tn)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
      my[(tm * TN + tn) * 64 + lane] =
          make_uint4(as_u32(acc[0][tn][tm][0]), as_u32(acc[0][tn][tm][1]), as_u32(acc[0][tn][tm][2]), as_u32(acc[0][tn][tm][3]));
  __syncthreads();
  typedef typename std::conditional<IS_I8, int, float>::type sum_t;
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    // a piece: consecutive threads hold consecutive channels of a pixel
    const int item = it * (64 * W) + tid;
    const int it_c = item % (TN * 2), it_p = item / (TN * 2);
    const int m_out = m0 + it_p, ech = n0 + it_c * 8;
    if (item >= ITEMS || m_out >= a.M || ech >= a.K) continue;
    // block (it_p / 16, it_c / 2), pixel it_p % 16, channels 8 (it_c % 2) .. + 7
    const uint4* src = ring + ((it_p >> 4) * TN + (it_c >> 1)) * 64 + (it_p & 15) + 32 * (it_c & 1);
    sum_t sum[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const uint4 lo = src[w * RING], hi = src[w * RING + 16];
      const unsigned r[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) sum[e] += __builtin_bit_cast(sum_t, r[e]);
    }
    unsigned raw[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) raw[e] = as_u32(sum[e]);
    LaneParams lp;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (IS_I8) {
        lp.ibias[e] = __builtin_bit_cast(int, cst[it_c * 8 + e]);
      } else {
        lp.mul[e] = cst[it_c * 8 + e];
        lp.add[e] = cst[BN + it_c * 8 + e];
      }
    }
    const OutLoc ol = EXT ? locate_output(a, ech) : OutLoc{nullptr, 0, 0, 0};
    finish_store8<IS_I8, false, EXT>(a, raw, m_out, ech, lp, ol, vec_ok, pre_res, resv[it]);
  }
}

struct SmallArgs {
  SmallGeom g;
  ConvArgs a;
};
template <bool IS_I8, int TM, int TN, int W, int U, int NS, bool EXT, int NA>
__global__ __launch_bounds__(64 * W) void igemm_small_kernel(const int tiles, const SmallArgs c) {
  small_tile<IS_I8, TM, TN, W, U, NS, EXT, NA>(c.a, c.g, xcd_remap((int)blockIdx.x, tiles));
}

// Two convs that do not read each other's output, in one launch: the first `tiles` workgroups run the first, the others the
// second.  The argument block is picked by a uniform index and copied whole: read field by field through that index its loads were 40 to
// 57 of one word each, and the arguments there after 2600 to 3200 clocks where a single conv's are after 700.
struct SmallPair {
  SmallArgs c[2];
};
template <bool IS_I8, int TM, int TN, int W, int U, int NS>
__global__ __launch_bounds__(64 * W) void igemm_small_pair_kernel(const int tiles, const int others, const SmallPair p) {
  const int second = (int)blockIdx.x >= tiles ? 1 : 0;
  const SmallArgs c = p.c[second];
  small_tile<IS_I8, TM, TN, W, U, NS, false, 1>(c.a, c.g, xcd_remap((int)blockIdx.x - (second ? tiles : 0), second ? others : tiles));
}

struct SmallTile {
  int tm, tn, w;
};
#define RELAY_SMALL_TILES(X) \
  X(0, 1, 1, 2) X(1, 1, 1, 4) X(2, 1, 2, 2) X(3, 1, 2, 4) X(4, 2, 2, 4) X(5, 2, 4, 4)
#define RELAY_SMALL_ENTRY(i, tm, tn, w) {tm, tn, w},
constexpr SmallTile kSmall[] = {RELAY_SMALL_TILES(RELAY_SMALL_ENTRY)};
constexpr int kNumSmall = sizeof(kSmall) / sizeof(kSmall[0]);

constexpr bool unit_fits(int u, int tm, int tn, int w) { return 2 * (tm + tn) * u * w <= 156; }   // two stages in LDS
constexpr int stages(int u, int tm, int tn, int w) {
  return (tm + tn) * u * w * 4 <= 64 ? 4 : (tm + tn) * u * w * 3 <= 80 ? 3 : 2;
}

// blocks of a tile that can have more than one accumulator (the 32 x 64 tile takes no layers from kernels of more runs)
constexpr int kMostBlocks = 4;

// Bytes of a reduction chunk of the staged kernels: the most that divide the channels of a tap.
int staged_chunk(const ConvArgs& a, bool is_i8) {
  const int per_tap = a.C * (is_i8 ? 1 : 2);
  return per_tap % 256 == 0 ? 256 : per_tap % 128 == 0 ? 128 : 64;
}

// Accumulators per block of a tile, fp16: in how many runs a wave sums.  A run's rounding error grows with its length and a matrix
// instruction rounds about four times, so four waves with one accumulator each are less exact than the kernels they
// took the layer from where those sum in more runs: a reduction split over 5 to 16 workgroups (at most 32 tiles of 64 x 64, a
// run for every 6 staged chunks), and a dense layer (lane by lane, in 64).  Rms error of the fp32 sums against 64 bits in 1e-7, the
// other kernel / one accumulator / as chosen here: 512 channels 3 x 3 1.80 / 2.19 / 1.60, 1024 1.97 / 3.15 / 1.77, 192 channels 5 x 5 1.48 /
// 2.21 / 1.30; dense, k = 1024 0.89 / 1.10 / 0.86, 4096 1.43 / 2.12 / 1.10, 9216 2.14 / 3.04 / 1.66.  Not split and not dense, one is
// more exact than the kernel before (256 channels 3 x 3 2.36 / 1.55).
// Two cost nothing measurable on a 16-pixel tile; four 0.3 to 0.6 us of a layer of 6 to 8.
int small_runs(const ConvArgs& a, bool is_i8, int v, bool dense) {
  if (is_i8 || kSmall[v].tm * kSmall[v].tn > kMostBlocks) return 1;
  if (dense) return a.M >= 16 && a.Kred % 64 == 0 ? 1 : a.Kred <= 2048 ? 2 : 4;   // (of 16 rows and whole chunks: from the staged kernel)
  const int chunks = a.Kred * 2 / staged_chunk(a, false);
  const long tiles64 = (long)((a.M + 63) / 64) * ((a.K + 63) / 64);
  return tiles64 > 32 || chunks < 30 ? 1 : chunks < 48 ? 2 : 4;
}

// steps per unit: the most that divide the channels of a tap
int small_unit(const ConvArgs& a, bool is_i8, int v) {
  const int per = a.C / (BKV * (is_i8 ? 16 : 8));
  const SmallTile& t = kSmall[v];
  if (per % 4 == 0 && unit_fits(4, t.tm, t.tn, t.w)) return 4;
  return per % 2 == 0 && unit_fits(2, t.tm, t.tn, t.w) ? 2 : 1;
}

template <bool IS_I8, int TM, int TN, int W, int U>
SmallGeom small_geom(const ConvArgs& a, ConvArgs& b) {
  SmallGeom g;
  g.tiles_m = (a.M + TM * 16 - 1) / (TM * 16);
  g.tiles_n = (a.K + TN * 16 - 1) / (TN * 16);
  g.per_tap = a.C / (U * BKV * (IS_I8 ? 16 : 8));
  g.units = a.R * a.S * g.per_tap;
  g.per_wave = (g.units + W - 1) / W;
  g.fd_per_tap = make_fastdiv((uint32_t)g.per_tap);
  g.fd_s = make_fastdiv((uint32_t)a.S);
  b = a;
  b.fd_tiles_m = make_fastdiv((uint32_t)g.tiles_m);
  b.fd_tiles_n = make_fastdiv((uint32_t)g.tiles_n);
  return g;
}

template <bool IS_I8, int TM, int TN, int W, int U, int NA>
hipError_t launch_small_alone(const ConvArgs& a, hipStream_t st) {
  constexpr int NS = stages(U, TM, TN, W);
  SmallArgs c;
  c.g = small_geom<IS_I8, TM, TN, W, U>(a, c.a);
  const int tiles = c.g.tiles_m * c.g.tiles_n;
  if (a.nseg)
    hipLaunchKernelGGL((igemm_small_kernel<IS_I8, TM, TN, W, U, NS, true, NA>), dim3(tiles), dim3(64 * W), 0, st, tiles, c);
  else
    hipLaunchKernelGGL((igemm_small_kernel<IS_I8, TM, TN, W, U, NS, false, NA>), dim3(tiles), dim3(64 * W), 0, st, tiles, c);
  return hipGetLastError();
}

// second: NULL, or the conv that shares the launch
template <bool IS_I8, int TM, int TN, int W, int U>
hipError_t launch_small_one(const ConvArgs& a, const ConvArgs* second, int runs, hipStream_t st) {
  constexpr int NS = stages(U, TM, TN, W);
  if (second) {
    SmallPair p;
    p.c[0].g = small_geom<IS_I8, TM, TN, W, U>(a, p.c[0].a);
    p.c[1].g = small_geom<IS_I8, TM, TN, W, U>(*second, p.c[1].a);
    const int tiles = p.c[0].g.tiles_m * p.c[0].g.tiles_n;
    const int others = p.c[1].g.tiles_m * p.c[1].g.tiles_n;
    hipLaunchKernelGGL((igemm_small_pair_kernel<IS_I8, TM, TN, W, U, NS>), dim3(tiles + others), dim3(64 * W), 0, st, tiles, others, p);
    return hipGetLastError();
  }
  if constexpr (!IS_I8 && TM * TN <= kMostBlocks) {
    if (runs == 4) return launch_small_alone<IS_I8, TM, TN, W, U, 4>(a, st);
    if (runs == 2) return launch_small_alone<IS_I8, TM, TN, W, U, 2>(a, st);
  }
  return launch_small_alone<IS_I8, TM, TN, W, U, 1>(a, st);
}

template <bool IS_I8, int TM, int TN, int W>
hipError_t launch_small_units(const ConvArgs& a, const ConvArgs* second, int u, int runs, hipStream_t st) {
  if constexpr (unit_fits(4, TM, TN, W))
    if (u == 4) return launch_small_one<IS_I8, TM, TN, W, 4>(a, second, runs, st);
  if constexpr (unit_fits(2, TM, TN, W))
    if (u == 2) return launch_small_one<IS_I8, TM, TN, W, 2>(a, second, runs, st);
  return launch_small_one<IS_I8, TM, TN, W, 1>(a, second, runs, st);
}

template <bool IS_I8>
hipError_t launch_small_typed(const ConvArgs& a, const ConvArgs* second, int v, int runs, hipStream_t st) {
  const int u = small_unit(a, IS_I8, v);
  switch (v) {
#define RELAY_SMALL_CASE(i, tm, tn, w) \
  case i: return launch_small_units<IS_I8, tm, tn, w>(a, second, u, runs, st);
    RELAY_SMALL_TILES(RELAY_SMALL_CASE)
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int conv_small_variant_count() { return kNumSmall; }

bool conv_small_supported(const ConvArgs& a, bool is_i8, int v) {
  if (v < 0 || v >= kNumSmall || a.seg_centre || a.pool || a.round_mode == ROUND_STOCHASTIC) return false;
  // (tiles are counted, and pixels decoded, in 31 bits)
  return igemm_dma_supported(a, is_i8) && (size_t)a.M + 64 < (1u << 31);
}

// The variant the heuristic takes, or -1 to leave the layer to the staged kernels.  Both sides are estimated in
// microseconds from measurements on the ResNet-18 / MobileNet-v1 layers at batch 1 to 32 (graph-timed):
//   here    2.65 for a launch with its prologue and tail, 0.1 per block of tile side, the operand bytes of a
//           tile at 125 KB/us (what a CU draws through its texture addresser), 0.6 for every further
//           round of tiles over the 256 CUs (l3 at batch 1, 208 tiles of 147 KB: 3.9 measured; at batch 2
//           5.5 with the same tile, 4.5 with the next larger one)
//   staged  2.7 and 0.26 per reduction chunk (0.32 for a chunk of 256 bytes) while every CU holds at most one
//           64 x 64 tile: 512 -> 512 at 7 x 7, batch 8: 14.0 us against 7.5 here; 256 -> 256 at 14 x 14, batch 8: 8.4
//           against 7.0, batch 16: 8.8 against 12.6
// A layer of more than 256 such tiles goes to the tall tiles of the staged kernels, which this one does not reach.
namespace {
int small_best(const ConvArgs& a, bool is_i8, bool regroup, float* us_out) {
  const int row = a.Kred * (is_i8 ? 1 : 2);  // reduction bytes of a tile row
  // fp16: splitting a reduction groups its sums anew.  The convs that other entry points run as part of a larger
  // launch with a promise of the same bits keep the staged kernels' order: a 1x1 conv (behind a depthwise conv),
  // a conv with a max pool behind it, and a strided conv whose window is centred on a 1x1 shortcut conv's (merged with it:
  // such a launch is always the staged kernel's).  At batch 1 that costs 128 -> 256 at 28 x 28 / 2 4.4 us instead
  // of 3.5 and 256 -> 512 at 14 x 14 / 2 5.7 instead of 4.0 (on that kernel's 32 x 32 tiles; 5.8 and 8.4 on its others).
  const bool centred = (a.sh > 1 || a.sw > 1) && (a.R & 1) && (a.S & 1) && a.ph == a.R / 2 && a.pw == a.S / 2;
  if (!is_i8 && !regroup && (a.R * a.S == 1 || centred || igemm_dma_pool_supported(a, false))) return -1;
  const int chunk = staged_chunk(a, is_i8);
  float best = 0.98f * (2.7f + (chunk == 256 ? 0.32f : 0.26f) * (float)(row / chunk));
  int pick = -1;
  for (int v = 0; v < kNumSmall; ++v) {
    const SmallTile& t = kSmall[v];
    if (regroup && a.M <= 16 && t.tm > 1) continue;   // (rows that no pixel fills)
    if ((t.w == 2) != (row <= 512) && t.tm + t.tn <= 3) continue;  // two waves where there is little to split (2.7 against 2.8 us)
    const long tiles = (long)((a.M + t.tm * 16 - 1) / (t.tm * 16)) * ((a.K + t.tn * 16 - 1) / (t.tn * 16));
    const int rounds = (int)((tiles + 255) / 256);
    const float kb = (float)((t.tm + t.tn) * 16) * (float)row * (1.f / 1024.f);
    const float us = 2.65f + 0.1f * (float)(t.tm + t.tn - 2) + (float)rounds * kb * (1.f / 125.f) + 0.6f * (float)(rounds - 1);
    if (us < best) {
      best = us;
      pick = v;
    }
  }
  *us_out = best;
  return pick;
}

bool small_considered(const ConvArgs& a, bool is_i8) {
  return conv_small_supported(a, is_i8, 0) && (long)((a.M + 63) / 64) * ((a.K + 63) / 64) <= 256;
}
}  // namespace

int conv_small_pick(const ConvArgs& a, bool is_i8, bool regroup) {
  float us;
  if (!small_considered(a, is_i8) || conv_halo_pick(a, is_i8) >= 0) return -1;
  return small_best(a, is_i8, regroup, &us);
}

float conv_small_estimate(const ConvArgs& a, bool is_i8) {
  float us;
  return small_considered(a, is_i8) && small_best(a, is_i8, false, &us) >= 0 ? us : INFINITY;
}

bool conv_small_sums_by_taps(const ConvArgs& a, int v) {
  return a.R * a.S == 9 && a.C == 64 && kSmall[v].w == 4 && small_unit(a, false, v) == 2 && small_runs(a, false, v, false) == 1;
}

int conv_small_sums(const ConvArgs& a, int v) { return kSmall[v].w * small_runs(a, false, v, false); }

void conv_small_kernel_name(const ConvArgs& a, bool is_i8, int v, char* buf, size_t len) {
  const SmallTile& t = kSmall[v];
  const int u = small_unit(a, is_i8, v);
  snprintf(buf, len, "igemm_small_kernel<%s, %d, %d, %d, %d, %d, %s, %d>", is_i8 ? "true" : "false", t.tm, t.tn, t.w, u,
           stages(u, t.tm, t.tn, t.w), a.nseg ? "true" : "false", small_runs(a, is_i8, v, false));
}

hipError_t launch_conv_small(const ConvArgs& a, bool is_i8, int v, hipStream_t st, bool dense) {
  const int runs = small_runs(a, is_i8, v, dense);
  return is_i8 ? launch_small_typed<true>(a, nullptr, v, runs, st) : launch_small_typed<false>(a, nullptr, v, runs, st);
}

// Two convs share a launch where their tiles fit the chip at once, as many to a CU as its LDS takes.  ResNet-18's first convs
// and shortcuts of a stage in int8, graph-timed together against one after the other: at batch 1, 416 tiles of 128 -> 256, two to a
// CU, 4.8 us against 5.7, 256 -> 512 4.4 against 5.8; at batch 16 400 tiles, one to a CU, 10.6 against 10.4.
// fp16: only with the groups of sums of the second conv's own launch (own: the variant it takes by itself, or -1), so
// that both results are those of the separate launches bit for bit; the first conv runs its own variant.
bool conv_small_pair_supported(const ConvArgs& a, const ConvArgs& b, bool is_i8, int v, int own) {
  if (!conv_small_supported(a, is_i8, v) || !conv_small_supported(b, is_i8, v) || a.nseg || b.nseg) return false;
  if (!is_i8 && (own < 0 || kSmall[own].w != kSmall[v].w || small_unit(b, false, own) != small_unit(b, false, v) ||
                 small_runs(a, false, v, false) > 1 || small_runs(b, false, own, false) > 1))   // (the paired kernel has one accumulator)
    return false;
  const int u = small_unit(a, is_i8, v);
  if (small_unit(b, is_i8, v) != u) return false;
  const SmallTile& t = kSmall[v];
  const long lds = (long)t.w * stages(u, t.tm, t.tn, t.w) * (t.tm + t.tn) * u * 1024 + 2 * t.tn * 16 * 4;
  long tiles = 0;
  for (const ConvArgs* c : {&a, &b}) tiles += (long)((c->M + t.tm * 16 - 1) / (t.tm * 16)) * ((c->K + t.tn * 16 - 1) / (t.tn * 16));
  return tiles <= 256 * (160 * 1024 / lds);
}

hipError_t launch_conv_small_pair(const ConvArgs& a, const ConvArgs& b, bool is_i8, int v, hipStream_t st) {
  return is_i8 ? launch_small_typed<true>(a, &b, v, 1, st) : launch_small_typed<false>(a, &b, v, 1, st);
}

}  // namespace relay
