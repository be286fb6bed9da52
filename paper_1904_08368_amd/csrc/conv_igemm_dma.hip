// Implicit-GEMM conv2d for gfx950: MFMA main loop fed by direct global->LDS loads through a
// multi-stage LDS ring, fused epilogue (paper Section 4.1 / 4.2).
//
// GEMM view: rows m = (image, p, q) output pixels, columns = output channels, reduction
// kk = (r, s, c).  NHWC activations and [k][r][s][c] filters are both contiguous along the
// reduction axis and move as 16-byte k-vectors.  A workgroup owns BM pixels x BN channels;
// a wave owns TM x TN MFMA blocks of 32x32 (filters are the A operand).
//
// Staging: per 64-byte reduction chunk every wave issues `buffer_load_dwordx4 ... lds`
// instructions, each moving 16 tile rows x 64 B straight into LDS (lane i writes 16 bytes
// at base + 16*i), no VGPRs involved.  The LDS bank swizzle is applied on the global side:
// lane i fetches the k-vector that belongs in its fixed LDS slot.  Filter taps that fall in
// the padding, rows past the end of the tensor and channels past Cout get a buffer offset
// beyond num_records; the buffer unit then writes zeros (checked on hardware), so the MFMA
// loop has no special cases.  NS ring stages keep NS-1 chunks in flight behind one barrier
// per chunk.  The loads are inline asm on purpose: the compiler, not seeing LDS written,
// does not drain the memory pipeline before every LDS read; ordering is by the explicit
// vmcnt waits and barriers below.  The texture addresser takes 64 B/clk per CU, about as
// long per chunk as the MFMAs of a 256x128 tile take, so the loads of chunk kc+NS-1 are
// issued one at a time between the MFMAs of chunk kc instead of in a burst after the
// barrier, where all waves would queue for the addresser while the matrix pipe idles.
//
// Epilogue: accumulators go through LDS once (wave-private, 32 pixels at a time) so that a
// lane ends up with 8 consecutive channels of one pixel: per-channel constants are then the
// same for every pixel a lane handles, the residual is one 16-byte load and the result one
// 16-byte (fp16) or 8-byte (int8) store in full NHWC rows.
//
// Needs C to be a whole number of chunks (32 halves / 64 int8) and R*S <= 32; other shapes
// go to the register-staged kernel in conv_igemm.hip.
#include <cstdio>
#include <type_traits>

#include "igemm_dma_tile.hpp"

namespace relay {
namespace {

template <bool IS_I8, int WAVES_M, int WAVES_N, int TM, int TN, int NS, int KP, int SK, bool STOCH, bool EXT,
          bool POOL = false>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * SK,
                             // two workgroups per CU where their LDS rings fit side by side
                             (NS * KP * (WAVES_M * TM + WAVES_N * TN) * 32 * 64 <= 80 * 1024 ? 2 : 1))
    void igemm_dma_kernel(const int workgroups, const ConvArgs a) {
  __shared__ uint4 ring[igemm_dma_slots<IS_I8, WAVES_M, WAVES_N, TM, TN, NS, KP, POOL>()];
  igemm_dma_tile<IS_I8, WAVES_M, WAVES_N, TM, TN, NS, KP, SK, STOCH, EXT, POOL>(a, xcd_remap((int)blockIdx.x, workgroups), ring);
}

// The tile for fp16 layers of few pixels whose sums other launches promise to the bit (strided convs centred on a shortcut's,
// 1x1 convs): every output is still one accumulator fed in the order of the tiles above, but a workgroup owns 32 x 32
// outputs, so that four times as many CUs take part, and its waves have one job each: four load (16 rows of one operand), the
// fifth multiplies.  The fifth reads chunk kc from LDS while it multiplies chunk kc - 1, so a chunk takes the longest of its
// loads (KP KB per wave), its LDS reads and its MFMAs (64 KP clocks) instead of their sum behind a barrier.
template <int KP>
__device__ __forceinline__ void igemm_dma_narrow_tile(const ConvArgs& a, int wg) {
  constexpr int VE = 8, ES = 2, CK = KP * BKV * VE, BM = 32, BN = 32, NS = KP == 4 ? 4 : (KP == 2 ? 6 : 8);
  constexpr int PLANE = (BM + BN) * BKV, STAGE = KP * PLANE, KSTEPS = KP * 2;
  constexpr int EP = BN / 4 + 1;
  __shared__ uint4 ring[NS * STAGE + 32 * EP];
  asm volatile("" : "+s"(wg) : RELAY_ASKED, "s"(a.res), "s"(a.y));
#undef RELAY_ASKED
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.K + BN - 1) / BN;
  const int tile = wg;
  const int tile_q = (int)fast_div((uint32_t)tile, a.n_major ? a.fd_tiles_m : a.fd_tiles_n);
  const int tile_n = a.n_major ? tile_q : tile - tile_q * tiles_n;
  const int tile_m = a.n_major ? tile - tile_q * tiles_m : tile_q;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int nchunks = a.Kred / CK;

  if (wave < 4) {  // (uniform) a loader: rows 16 (wave % 2) ... of the activations (waves 0, 1) or of the filters
    const int srow = lane >> 2, row = (wave & 1) * 16 + srow, kvl = (lane & 3) ^ lds_swizzle(row);
    const bool filters = wave >= 2;
    unsigned off, taps;
    intx4 rs = filters ? make_rsrc(a.w, (unsigned)((size_t)a.K * a.Kp * ES)) : make_rsrc(a.x, (unsigned)((size_t)a.N * a.xs_n * ES));
#pragma unroll
    for (int i = 0; i < 4; ++i) rs[i] = __builtin_amdgcn_readfirstlane(rs[i]);   // (in scalar registers, as the loads want it)
    if (filters) {
      off = (unsigned)(((n0 + row) * a.Kp + kvl * VE) * ES);
      taps = n0 + row < a.K ? ~0u : 0u;
    } else {
      const int n_0 = (int)fast_div((uint32_t)m0, a.fd_howo), rem_0 = m0 - n_0 * (a.Ho * a.Wo);
      const int p_0 = (int)fast_div((uint32_t)rem_0, a.fd_wo), q_0 = rem_0 - p_0 * a.Wo;
      int dp, q, dn, p;
      small_divmod(q_0 + row, a.Wo, a.rcp_wo, dp, q);
      small_divmod(p_0 + dp, a.Ho, a.rcp_ho, dn, p);
      const int ih0 = p * a.sh - a.ph, iw0 = q * a.sw - a.pw;
      const int rlo = max(0, -ih0), rhi = min(a.R, a.H - ih0), clo = max(0, -iw0), chi = min(a.S, a.W - iw0);
      const unsigned colbits = (unsigned)((1ull << max(chi, 0)) - 1ull) & ~(unsigned)((1ull << clo) - 1ull);
      const unsigned rows = a.tap_spread & (unsigned)((1ull << (max(rhi, 0) * a.S)) - 1ull) & ~(unsigned)((1ull << (rlo * a.S)) - 1ull);
      taps = m0 + row < a.M && rhi > rlo && chi > clo ? colbits * rows : 0u;   // (the column run at every valid row)
      off = (unsigned)(((n_0 + dn) * a.xs_n + ih0 * a.xs_h + iw0 * a.xs_w + kvl * VE) * ES);
    }
    const unsigned base = (unsigned)(size_t)(__attribute__((address_space(3))) uint4*)(&ring[0]) + (unsigned)wave * 1024u;
    int tap = 0, r = 0, s = 0, c = 0, stage = 0;
    auto issue = [&](int kc) {  // chunk kc (past the end: zeros nobody reads, so that the wait counts stay constants)
      const unsigned delta = (unsigned)((filters ? kc * CK : r * a.xs_h + s * a.xs_w + c) * ES);
      const bool live = kc < nchunks && ((taps >> (filters ? 0 : tap)) & 1u);
#pragma unroll
      for (int pl = 0; pl < KP; ++pl)
        lds_dma16(rs, base + (unsigned)(stage * STAGE + pl * PLANE) * 16u, live ? off + delta + (unsigned)(pl * 64) : kOob);
      stage = stage + 1 == NS ? 0 : stage + 1;
      c += CK;
      if (c == a.C) {
        c = 0;
        ++tap;
        if (++s == a.S) {
          s = 0;
          ++r;
        }
      }
    };
    for (int kc = 0; kc < NS - 1; ++kc) issue(kc);
    for (int kc = 0; kc < nchunks; ++kc) {
      wait_loads<(NS - 2) * KP>();   // chunk kc has landed
      __builtin_amdgcn_s_barrier();  // the multiplying wave has read chunk kc - 1, whose stage is filled next
      issue(kc + NS - 1);
    }
    wait_loads<0>();   // (LDS is given back only when nothing writes to it any more)
    return;
  }

  // ---- the multiplying wave.  Its constants and residuals come while the first chunks do.
  constexpr int CG = BN / 8, PPI = 64 / CG, ITS = 32 / PPI;
  const int ech = n0 + (lane % CG) * 8, epix = lane / CG;
  const bool vec_ok = (a.K & 7) == 0, pre_res = (a.flags & F_RES) && vec_ok;
  RawLaneParams rawp;
  fetch_lane_params<false>(a, ech, rawp);
  uint4 resv[ITS];
  if (pre_res) {
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int m = m0 + it * PPI + epix;
      resv[it] = m < a.M && ech < a.K ? load_residual8<false>(a, m, ech) : make_uint4(0u, 0u, 0u, 0u);
    }
  }
  typedef typename Mma<false>::acc_t acc_t;
  acc_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0;
  const int lrow = lane & 31, lhalf = lane >> 5;
  const int slot = lds_slot(lrow, lhalf);   // (the other k-vectors of a plane: ^ 2)
  uint4 wf[2][KSTEPS], xf[2][KSTEPS];
  int stage = 0;
  auto read = [&](int set) {
    const uint4* st = ring + stage * STAGE;
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k) {
      xf[set][k] = st[(k >> 1) * PLANE + (slot ^ (2 * (k & 1)))];
      wf[set][k] = st[(k >> 1) * PLANE + BM * BKV + (slot ^ (2 * (k & 1)))];
    }
    stage = stage + 1 == NS ? 0 : stage + 1;
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k) acc = Mma<false>::mma(wf[set][k], xf[set][k], acc);
    asm volatile("" : "+v"(acc));   // (not sunk below the next barrier)
  };
  auto meet = [&]() {  // everything read so far has arrived, the next chunk has landed
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  meet();
  read(0);
  int kc = 1;
  for (; kc + 1 < nchunks; kc += 2) {
    meet();
    read(1);
    multiply(0);
    meet();
    read(0);
    multiply(1);
  }
  if (kc < nchunks) {
    meet();
    read(1);
    multiply(0);
    multiply(1);
  } else {
    multiply(0);
  }
  LaneParams lp;
  finish_lane_params<false>(rawp, lp);
  uint4* stg = ring + NS * STAGE;
#pragma unroll
  for (int g = 0; g < 4; ++g)
    stg[lrow * EP + 2 * g + lhalf] = make_uint4(as_u32(acc[4 * g]), as_u32(acc[4 * g + 1]), as_u32(acc[4 * g + 2]), as_u32(acc[4 * g + 3]));
  const OutLoc ol{nullptr, 0, 0, 0};
#pragma unroll
  for (int it = 0; it < ITS; ++it) {
    const int pix = it * PPI + epix, m = m0 + pix;
    const uint4 lo = stg[pix * EP + (lane % CG) * 2], hi = stg[pix * EP + (lane % CG) * 2 + 1];
    const unsigned raw[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    if (m < a.M && ech < a.K) finish_store8<false, false>(a, raw, m, ech, lp, ol, vec_ok, pre_res, resv[it]);
  }
}

template <int KP>
__global__ __launch_bounds__(320) void igemm_dma_kernel_narrow(const int workgroups, const ConvArgs a) {
  igemm_dma_narrow_tile<KP>(a, xcd_remap((int)blockIdx.x, workgroups));
}

// Two convs that do not read each other's output, in one launch: the first `tiles` workgroups run the first, the others the
// second (see igemm_small_pair_kernel).
struct DmaPair {
  ConvArgs a[2];
};
template <bool IS_I8, int WAVES_M, int WAVES_N, int TM, int TN, int NS, int KP>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, (NS * KP * (WAVES_M * TM + WAVES_N * TN) * 32 * 64 <= 80 * 1024 ? 2 : 1))
    void igemm_dma_pair_kernel(const int tiles, const int others, const DmaPair p) {
  const int second = (int)blockIdx.x >= tiles ? 1 : 0;
  const ConvArgs a = p.a[second];
  __shared__ uint4 ring[igemm_dma_slots<IS_I8, WAVES_M, WAVES_N, TM, TN, NS, KP, false>()];
  igemm_dma_tile<IS_I8, WAVES_M, WAVES_N, TM, TN, NS, KP, 1, false, false, false>(a, xcd_remap((int)blockIdx.x - (second ? tiles : 0), second ? others : tiles), ring);
}

template <int KP>
__global__ __launch_bounds__(320) void igemm_dma_pair_kernel_narrow(const int tiles, const int others, const DmaPair p) {
  const int second = (int)blockIdx.x >= tiles ? 1 : 0;
  const ConvArgs a = p.a[second];
  igemm_dma_narrow_tile<KP>(a, xcd_remap((int)blockIdx.x - (second ? tiles : 0), second ? others : tiles));
}

struct DmaTile {
  int waves_m, waves_n, tm, tn, ns, kp, sk;
  constexpr int bm() const { return waves_m * tm * 32; }
  constexpr int bn() const { return waves_n * tn * 32; }
};
// largest first; must match launch_typed
constexpr DmaTile kTiles[] = {
    {2, 2, 4, 2, 3, 1, 1},  // 256 x 128
    {4, 1, 4, 2, 3, 1, 1},  // 512 x 64
    {2, 1, 4, 2, 3, 1, 1},  // 256 x 64, two waves
    {2, 2, 2, 2, 3, 1, 1},  // 128 x 128
    {2, 2, 2, 1, 4, 1, 1},  // 128 x 64
    {2, 2, 1, 1, 4, 1, 1},  // 64 x 64
    // 128-byte chunks (need C % 64 == 0 for fp16, C % 128 == 0 for int8)
    {2, 2, 4, 2, 3, 2, 1},  // 256 x 128
    {2, 2, 4, 2, 2, 2, 1},  // 256 x 128, two stages
    {2, 2, 2, 2, 3, 2, 1},  // 128 x 128
    {2, 2, 2, 1, 3, 2, 1},  // 128 x 64
    {2, 2, 1, 1, 3, 2, 1},  // 64 x 64
    {2, 1, 4, 2, 3, 2, 1},  // 256 x 64, two waves
    // k-split wave pairs
    {2, 1, 2, 2, 3, 2, 2},  // 128 x 64, four waves of 64 x 64
    {1, 1, 2, 2, 3, 2, 2},  // 64 x 64, two waves of 64 x 64
    // tall tiles for layers with few output channels
    {4, 1, 2, 2, 3, 1, 1},  // 256 x 64, four waves of 64 x 64
    // 256-byte chunks: half as many barriers for the long reductions of the 512-channel layers
    {2, 2, 1, 1, 3, 4, 1},  // 64 x 64
    // short reductions over very many pixels (the first layer): a small ring, four workgroups per CU
    {2, 2, 2, 1, 3, 1, 1},  // 128 x 64
    // layers with at most 32 output channels over very many pixels (MobileNet's first layer): two waves, no
    // matrix work or epilogue lanes spent on channels that do not exist
    {2, 1, 2, 1, 3, 1, 1},  // 128 x 32
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

template <bool IS_I8, bool STOCH, int WAVES_M, int WAVES_N, int TM, int TN, int NS, int KP, int SK = 1>
hipError_t launch_one(const ConvArgs& a, hipStream_t st) {
  constexpr int BM = WAVES_M * TM * 32, BN = WAVES_N * TN * 32;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.K + BN - 1) / BN;
  const int tiles = tiles_m * tiles_n * (a.split > 1 ? a.split : 1);
  ConvArgs b = a;
  b.fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
  b.fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
  if (STOCH || a.nseg || a.split > 1)
    hipLaunchKernelGGL((igemm_dma_kernel<IS_I8, WAVES_M, WAVES_N, TM, TN, NS, KP, SK, STOCH, true>), dim3(tiles),
                       dim3(64 * WAVES_M * WAVES_N * SK), 0, st, tiles, b);
  else
    hipLaunchKernelGGL((igemm_dma_kernel<IS_I8, WAVES_M, WAVES_N, TM, TN, NS, KP, SK, false, false>), dim3(tiles),
                       dim3(64 * WAVES_M * WAVES_N * SK), 0, st, tiles, b);
  return hipGetLastError();
}

// second: NULL, or the conv that shares the launch
template <int KP>
hipError_t launch_narrow_one(const ConvArgs& a, const ConvArgs* second, hipStream_t st) {
  DmaPair p;
  p.a[0] = a;
  if (second) p.a[1] = *second;
  int tiles[2] = {0, 0};
  for (int i = 0; i < (second ? 2 : 1); ++i) {
    const int tiles_m = (p.a[i].M + 31) / 32, tiles_n = (p.a[i].K + 31) / 32;
    tiles[i] = tiles_m * tiles_n;
    p.a[i].fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
    p.a[i].fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
  }
  if (second) hipLaunchKernelGGL(igemm_dma_pair_kernel_narrow<KP>, dim3(tiles[0] + tiles[1]), dim3(320), 0, st, tiles[0], tiles[1], p);
  else hipLaunchKernelGGL(igemm_dma_kernel_narrow<KP>, dim3(tiles[0]), dim3(320), 0, st, tiles[0], p.a[0]);
  return hipGetLastError();
}

int narrow_planes(const ConvArgs& a) { return a.C % 128 == 0 ? 4 : a.C % 64 == 0 ? 2 : 1; }

hipError_t launch_narrow(const ConvArgs& a, const ConvArgs* second, hipStream_t st) {
  const int kp = narrow_planes(a);
  return kp == 4 ? launch_narrow_one<4>(a, second, st) : kp == 2 ? launch_narrow_one<2>(a, second, st) : launch_narrow_one<1>(a, second, st);
}

template <bool IS_I8, int WAVES_M, int WAVES_N, int TM, int TN, int NS, int KP>
hipError_t launch_pair_one(const ConvArgs& a, const ConvArgs& b, hipStream_t st) {
  constexpr int BM = WAVES_M * TM * 32, BN = WAVES_N * TN * 32;
  DmaPair p;
  p.a[0] = a;
  p.a[1] = b;
  int tiles[2];
  for (int i = 0; i < 2; ++i) {
    const int tiles_m = (p.a[i].M + BM - 1) / BM, tiles_n = (p.a[i].K + BN - 1) / BN;
    tiles[i] = tiles_m * tiles_n;
    p.a[i].split = 1;
    p.a[i].fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
    p.a[i].fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
  }
  hipLaunchKernelGGL((igemm_dma_pair_kernel<IS_I8, WAVES_M, WAVES_N, TM, TN, NS, KP>), dim3(tiles[0] + tiles[1]), dim3(64 * WAVES_M * WAVES_N), 0, st, tiles[0], tiles[1], p);
  return hipGetLastError();
}

// the tiles the short strided convs take
template <bool IS_I8>
hipError_t launch_pair_typed(const ConvArgs& a, const ConvArgs& b, int tile, hipStream_t st) {
  switch (tile) {
    case 4: return launch_pair_one<IS_I8, 2, 2, 2, 1, 4, 1>(a, b, st);
    case 5: return launch_pair_one<IS_I8, 2, 2, 1, 1, 4, 1>(a, b, st);
    case 9: return launch_pair_one<IS_I8, 2, 2, 2, 1, 3, 2>(a, b, st);
    case 10: return launch_pair_one<IS_I8, 2, 2, 1, 1, 3, 2>(a, b, st);
    default: return launch_pair_one<IS_I8, 2, 2, 1, 1, 3, 4>(a, b, st);
  }
}

template <bool IS_I8, bool STOCH>
hipError_t launch_typed(const ConvArgs& a, int tile, hipStream_t st) {
  switch (tile) {
    case 0: return launch_one<IS_I8, STOCH, 2, 2, 4, 2, 3, 1>(a, st);
    case 1: return launch_one<IS_I8, STOCH, 4, 1, 4, 2, 3, 1>(a, st);
    case 2: return launch_one<IS_I8, STOCH, 2, 1, 4, 2, 3, 1>(a, st);
    case 3: return launch_one<IS_I8, STOCH, 2, 2, 2, 2, 3, 1>(a, st);
    case 4: return launch_one<IS_I8, STOCH, 2, 2, 2, 1, 4, 1>(a, st);
    case 5: return launch_one<IS_I8, STOCH, 2, 2, 1, 1, 4, 1>(a, st);
    case 6: return launch_one<IS_I8, STOCH, 2, 2, 4, 2, 3, 2>(a, st);
    case 7: return launch_one<IS_I8, STOCH, 2, 2, 4, 2, 2, 2>(a, st);
    case 8: return launch_one<IS_I8, STOCH, 2, 2, 2, 2, 3, 2>(a, st);
    case 9: return launch_one<IS_I8, STOCH, 2, 2, 2, 1, 3, 2>(a, st);
    case 10: return launch_one<IS_I8, STOCH, 2, 2, 1, 1, 3, 2>(a, st);
    case 11: return launch_one<IS_I8, STOCH, 2, 1, 4, 2, 3, 2>(a, st);
    case 12: return launch_one<IS_I8, STOCH, 2, 1, 2, 2, 3, 2, 2>(a, st);
    case 13: return launch_one<IS_I8, STOCH, 1, 1, 2, 2, 3, 2, 2>(a, st);
    case 14: return launch_one<IS_I8, STOCH, 4, 1, 2, 2, 3, 1, 1>(a, st);
    case 15: return launch_one<IS_I8, STOCH, 2, 2, 1, 1, 3, 4, 1>(a, st);
    case 16: return launch_one<IS_I8, STOCH, 2, 2, 2, 1, 3, 1, 1>(a, st);
    default: return launch_one<IS_I8, STOCH, 2, 1, 2, 1, 3, 1, 1>(a, st);
  }
}

long tiles_of(const ConvArgs& a, const DmaTile& t) {
  return (long)((a.M + t.bm() - 1) / t.bm()) * ((a.K + t.bn() - 1) / t.bn());
}

constexpr int kNarrow = kNumTiles;   // the number of the 32 x 32 tile behind those of the list

bool narrow_fits(const ConvArgs& a, bool is_i8) { return !is_i8 && !a.nseg && !a.pool && a.split <= 1 && a.Kred >= BKV * 8; }

// can tile t run this layer?  (its chunk must divide the channel count)
bool tile_fits(const ConvArgs& a, bool is_i8, int t) {
  if (t == kNarrow) return narrow_fits(a, is_i8);
  return t >= 0 && t < kNumTiles && a.C % (kTiles[t].kp * BKV * (is_i8 ? 16 : 8)) == 0;
}

// Tile choice from measured sweeps over the ResNet / MobileNet layer shapes: the 256x128
// tile once it gives every CU two workgroups, else 128x64, else 64x64 (small-M layers need
// the workgroup count more than the per-tile intensity); the longest chunks C and LDS allow.
int pick_tile(const ConvArgs& a, bool is_i8) {
  const bool kp2 = a.C % (2 * BKV * (is_i8 ? 16 : 8)) == 0;
  // short reductions over many pixels (the row-packed first layer, the early pointwise layers): a tile
  // lives for a handful of chunks, mostly the latency of its first loads and its stores; many
  // small-ring workgroups per CU overlap those
  // at most 32 output channels over very many pixels: the two-wave 128 x 32 tile (MobileNet's first layer at batch 32: 16.3 against 18.9 us)
  if (a.K <= 32 && a.Kred <= 8 * BKV * (is_i8 ? 16 : 8) && tiles_of(a, kTiles[17]) >= 1024) return 17;
  if (a.Kred <= 8 * BKV * (is_i8 ? 16 : 8) && tiles_of(a, kTiles[16]) >= 512) return 16;
  // 64 output channels over very many pixels in int8 (layer 1): tall tiles of 64 x 64 per wave
  if (a.K <= 64 && is_i8 && tiles_of(a, kTiles[14]) >= 384) return 14;
  if (a.K > 64 && tiles_of(a, kTiles[0]) >= 384) return 0;  // (measured down to 392 tiles: 737 vs 613 TFLOP/s on 512 -> 512 at 28 x 28)
  const int mid = kp2 ? 9 : 4;
  if (tiles_of(a, kTiles[mid]) >= 190) return mid;
  // a layer that gives each CU at most one 64 x 64 workgroup can afford the 96 KiB ring of 256-byte chunks
  if (a.C % (4 * BKV * (is_i8 ? 16 : 8)) == 0 && tiles_of(a, kTiles[15]) <= 256) return 15;
  return kp2 ? 10 : 5;
}

// What the tile pick_tile takes is estimated to cost a 3 x 3 layer, a + b n + c n k + e x k microseconds with k the chunks of the
// reduction, x the tiles per CU and n the tiles of the CU that has most (fitted as the 3 x 3 kernel's estimates are); fp16, int8.
struct DmaCost {
  int tile;
  float f[4], q[4];
};
constexpr DmaCost kCost[] = {
    {0, {7.26f, 1.97f, 0.261f, 0.304f}, {3.71f, 5.50f, 0.348f, 0.188f}},
    {4, {3.49f, 0.36f, 0.043f, 0.213f}, {4.89f, 0.00f, 0.056f, 0.187f}},
    {5, {5.82f, 0.00f, 0.076f, 0.000f}, {4.10f, 0.00f, 0.121f, 0.000f}},
    {9, {2.63f, 0.83f, 0.124f, 0.246f}, {3.43f, 0.34f, 0.137f, 0.246f}},
    {10, {3.95f, 0.00f, 0.160f, 0.000f}, {4.26f, 0.00f, 0.133f, 0.015f}},
    {14, {0.00f, 0.67f, 0.363f, 0.146f}, {0.00f, 0.67f, 0.363f, 0.146f}},   // (int8 only)
    {15, {3.27f, 0.00f, 0.287f, 0.057f}, {3.69f, 0.00f, 0.280f, 0.036f}},
};

// The 32 x 32 tile where each CU gets at most one and the reduction is long enough for its loaders to run ahead (graph-timed, the
// 64 x 64 tile / this one, stride 2: 256 -> 512 at 14 x 14 8.36 / 5.68 us, its 1x1 shortcut 3.62 / 3.21, 128 -> 256 at 28 x 28 5.77 /
// 4.36, 64 -> 128 at 56 x 56 5.06 / 4.13, its shortcut of a single chunk 3.10 / 3.16; 1x1 1024 -> 1024 at 7 x 7 5.41 / 4.16; two
// tiles to a CU 5.8 / 6.9).
long narrow_tiles(const ConvArgs& a) { return (long)((a.M + 31) / 32) * ((a.K + 31) / 32); }
bool narrow_better(const ConvArgs& a, bool is_i8) {
  if (!narrow_fits(a, is_i8) || narrow_tiles(a) > 256) return false;
  return a.C % 128 == 0 || (a.C % 64 == 0 && a.Kred / 64 >= 8);
}

// The same of two convs in one launch.  Together they may give a CU two tiles where one kind is short: it then runs beside the
// other's, whose own loads leave it room (graph-timed pairs, 64 x 64 tiles / these: 3x3 / 2 and 1x1 / 2, 448 tiles of 512 -> 512 15.97 / 12.0
// us, 304 of 128 -> 128 7.08 / 5.41, 512 of 256 -> 512 10.2 / 8.8; two 1x1 / 2, 256 of 512 -> 512 5.18 / 4.29, but 272 of 128 -> 256 4.11 /
// 5.24, 352 of 512 -> 512 5.22 / 6.33).
bool narrow_pair(const ConvArgs& a, const ConvArgs& b, bool is_i8) {
  if (!narrow_better(a, is_i8) || !narrow_fits(b, is_i8) || narrow_tiles(b) > 256 || narrow_planes(a) != narrow_planes(b)) return false;
  return narrow_tiles(a) + narrow_tiles(b) <= 256 || a.Kred >= 4 * b.Kred || b.Kred >= 4 * a.Kred;
}

int resolve_tile(const ConvArgs& a, bool is_i8, int tile) {
  if (tile_fits(a, is_i8, tile)) return tile;
  return narrow_better(a, is_i8) ? kNarrow : pick_tile(a, is_i8);
}

}  // namespace

bool igemm_dma_supported(const ConvArgs& a, bool is_i8) {
  const int es = is_i8 ? 1 : 2;
  const int ck = BKV * 16 / es;
  const size_t lim = 0x7fffffffu;  // buffer offsets are 32-bit and 0x80000000 marks "out of range"
  // tile rows are decoded as small offsets from the tile's first pixel (float reciprocal, < 2^22)
  return (a.C % ck) == 0 && a.R * a.S <= 32 && (size_t)a.N * a.xs_n * es <= lim &&
         (size_t)a.K * a.Kp * es <= lim && a.Wo < (1 << 20) && a.Ho < (1 << 20);
}

// Two convs share a launch where both take the same of these tiles by themselves (the sums are then grouped as in their own
// launches), and the one whose ring leaves room for a single workgroup per CU only where that is one round.  ResNet-18's
// first convs and shortcuts of a stage at batch 32, together against one after the other: 784 tiles of 128 x 64 14.8 us
// against 11.7 + 5.5, 392 12.4 against 10.5 + 5.2; int8 at batch 16 9.9 against 7.8 + 4.4, 64 x 64 tiles 8.2 against 6.3 + 3.7.
// fp16 at batch 1: 32 tiles of 128 -> 256 7.0 against 8.5 for both, 256 -> 512 9.8 against 11.5.
int igemm_dma_pair_tile(const ConvArgs& a, const ConvArgs& b, bool is_i8) {
  if (!igemm_dma_supported(a, is_i8) || !igemm_dma_supported(b, is_i8) || a.nseg || b.nseg || a.pool || b.pool ||
      a.round_mode == ROUND_STOCHASTIC || b.round_mode == ROUND_STOCHASTIC)
    return -1;
  const int t = pick_tile(a, is_i8);
  if (t != pick_tile(b, is_i8)) return -1;
  if (t == 15) return tiles_of(a, kTiles[t]) + tiles_of(b, kTiles[t]) <= 256 ? t : -1;
  return t == 4 || t == 5 || t == 9 || t == 10 ? t : -1;
}

hipError_t launch_conv_igemm_dma_pair(const ConvArgs& a, const ConvArgs& b, bool is_i8, int tile, hipStream_t st) {
  // (same sums, whatever the tile)
  if (narrow_pair(a, b, is_i8)) return launch_narrow(a, &b, st);
  return is_i8 ? launch_pair_typed<true>(a, b, tile, st) : launch_pair_typed<false>(a, b, tile, st);
}

bool igemm_dma_pool_supported(const ConvArgs& a, bool is_i8) {
  // whole 7 x 8 blocks of pooled outputs, vector stores, the plain fused tail
  return igemm_dma_supported(a, is_i8) && a.Ho % 14 == 0 && a.Wo % 16 == 0 && (a.K & 7) == 0 && !(a.flags & F_RES) &&
         a.round_mode != ROUND_STOCHASTIC && a.nseg == 0;
}

void fill_pool_args(ConvArgs& a) {
  a.pool = 1;
  a.pool_block = a.C;
  a.pool_tiles_row = (a.Wo / 2) / 8;
  a.pool_tiles_img = ((a.Ho / 2) / 7) * a.pool_tiles_row;
  a.fd_pool_row = make_fastdiv((uint32_t)a.pool_tiles_row);
  a.fd_pool_img = make_fastdiv((uint32_t)a.pool_tiles_img);
}

// 256 x 64 tiles of four 64 x 64 waves with a two-stage ring: 41 KB of LDS, three workgroups per CU.
// A workgroup's life is mostly latency (first loads, epilogue, pooling), so the third resident
// workgroup buys more than a third ring stage (measured on the 7x7 first layer of ResNet-18).
namespace {
// The row-packed view of an NHWC4 image, one chunk per filter row, at stride 2: the form that stages the input patch once.
// 7x7 / 2, 64 channels, 224 x 224: fp16 batch 32 26.0 -> 22.4 us, batch 1 6.9 -> 6.1; int8 batch 16 16.0 -> 13.8, batch 1 7.4 -> 6.1
// (the reduction with its loads 7.5 K -> 4.5 K cycles of a workgroup; the two-stage ring with more stages was slower, its
// loads are bound by the addresser, not by latency).  The pooling behind it (4.5 K cycles) is the larger part now.
bool pool_stem(const ConvArgs& a, bool is_i8) {
  return a.xs_w == 4 && a.C == BKV * (is_i8 ? 16 : 8) && a.S == 1 && a.sh == 2 && a.sw == 2 && a.R <= 7 && a.ph == 0 && a.pw == 0;
}

template <bool IS_I8>
hipError_t launch_pool_one(const ConvArgs& a, int tiles, hipStream_t st) {
  if (pool_stem(a, IS_I8))
    hipLaunchKernelGGL((igemm_dma_kernel<IS_I8, 4, 1, 2, 2, 1, 1, 1, false, false, true>), dim3(tiles), dim3(256), 0, st, tiles, a);
  else
    hipLaunchKernelGGL((igemm_dma_kernel<IS_I8, 4, 1, 2, 2, 2, 1, 1, false, false, true>), dim3(tiles), dim3(256), 0, st, tiles, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_conv_igemm_dma_pool(const ConvArgs& a, bool is_i8, hipStream_t st) {
  constexpr int BN = 64;
  const int tiles_m = a.N * a.pool_tiles_img, tiles_n = (a.K + BN - 1) / BN;
  ConvArgs b = a;
  b.fd_tiles_m = make_fastdiv((uint32_t)tiles_m);
  b.fd_tiles_n = make_fastdiv((uint32_t)tiles_n);
  b.split = 1;
  return is_i8 ? launch_pool_one<true>(b, tiles_m * tiles_n, st) : launch_pool_one<false>(b, tiles_m * tiles_n, st);
}

void igemm_dma_pool_kernel_name(const ConvArgs& a, bool is_i8, char* buf, size_t len) {
  snprintf(buf, len, "igemm_dma_kernel<%s, 4, 1, 2, 2, %d, 1, 1, false, false, true>", is_i8 ? "true" : "false", pool_stem(a, is_i8) ? 1 : 2);
}

// a layer with the 256 x 128 tile's 384 tiles or more
bool igemm_dma_wide(const ConvArgs& a) { return a.K > 64 && tiles_of(a, kTiles[0]) >= 384; }

DmaChoice igemm_dma_choice(const ConvArgs& a) {
  const int tile = pick_tile(a, false);
  return {kTiles[tile].bm(), kTiles[tile].bn(), tiles_of(a, kTiles[tile]), tile == 16};
}

float igemm_dma_estimate(const ConvArgs& a, bool is_i8) {
  const int tile = pick_tile(a, is_i8);
  const DmaTile& t = kTiles[tile];
  const long tiles = tiles_of(a, t);
  const float n = (float)((tiles + 255) / 256), x = (float)tiles * (1.f / 256.f);
  const float k = (float)(a.Kred / (t.kp * BKV * (is_i8 ? 16 : 8)));
  for (const DmaCost& c : kCost)
    if (c.tile == tile) {
      const float(&p)[4] = is_i8 ? c.q : c.f;
      return p[0] + n * (p[1] + p[2] * k) + p[3] * x * k;
    }
  return 0.f;   // (a tile no 3 x 3 layer of 64 channels takes: nothing is faster)
}

bool igemm_dma_small_ring(const ConvArgs& a) { return resolve_tile(a, false, -1) == 16; }

int igemm_dma_tile_count() { return kNumTiles + 1; }

int igemm_dma_plan_split(const ConvArgs& a, bool is_i8, int tile, int want, size_t* counter_bytes,
                         size_t* total_bytes) {
  // (the 32 x 32 tile is for layers that are not split: what the other tiles would do stays the answer)
  const DmaTile& t = kTiles[tile != kNarrow && tile_fits(a, is_i8, tile) ? tile : pick_tile(a, is_i8)];
  const int tiles = (int)tiles_of(a, t);
  const int chunks = a.Kred / (t.kp * BKV * (is_i8 ? 16 : 8));
  int split = want;
  if (split <= 0) {
    // Few tiles and a long reduction (the deep layers at small batch): the reduction is what can
    // still be spread over the idle CUs.  Handing a tile over costs about as much as six chunks of
    // the main loop and grows with the number of workgroups (measured on 7x7 and 14x14 layers of
    // 256 and 512 channels at batch 1 to 16): at least six chunks per workgroup, at most 128
    // workgroups, and only layers of at most 32 tiles and at least 24 chunks (int8: 12).
    split = 1;
    // (fp16, 18 chunks, 16 tiles -- 256 channels at 14 x 14, batch 1: 8.5 us unsplit, 9.3 us in three)
    if (tiles <= 32 && chunks >= (is_i8 ? 12 : 24)) {
      split = 128 / tiles;
      if (split > chunks / 6) split = chunks / 6;
      if (split > 16) split = 16;
    }
  }
  if (split > chunks) split = chunks;
  if (split < 1) split = 1;
  const int per = (chunks + split - 1) / split;
  split = (chunks + per - 1) / per;  // every workgroup gets at least one chunk
  *counter_bytes = (size_t)tiles * kCntStride * sizeof(unsigned);
  *total_bytes = split > 1 ? *counter_bytes + (size_t)tiles * split * t.bm() * t.bn() * 4 : 0;
  return split;
}

void igemm_dma_kernel_name(const ConvArgs& a, bool is_i8, int tile, char* buf, size_t len) {
  tile = resolve_tile(a, is_i8, tile);
  if (tile == kNarrow) {
    snprintf(buf, len, "igemm_dma_kernel_narrow<%d>", narrow_planes(a));
    return;
  }
  const DmaTile& t = kTiles[tile];
  const bool stoch = is_i8 && a.round_mode == ROUND_STOCHASTIC;
  snprintf(buf, len, "igemm_dma_kernel<%s, %d, %d, %d, %d, %d, %d, %d, %s, %s, false>", is_i8 ? "true" : "false", t.waves_m,
           t.waves_n, t.tm, t.tn, t.ns, t.kp, t.sk, stoch ? "true" : "false",
           (stoch || a.nseg || a.split > 1) ? "true" : "false");
}

hipError_t launch_conv_igemm_dma(const ConvArgs& a, bool is_i8, int tile, hipStream_t st) {
  tile = resolve_tile(a, is_i8, tile);
  if (tile == kNarrow) return launch_narrow(a, nullptr, st);
  if (!is_i8) return launch_typed<false, false>(a, tile, st);
  return a.round_mode == ROUND_STOCHASTIC ? launch_typed<true, true>(a, tile, st) : launch_typed<true, false>(a, tile, st);
}

}  // namespace relay
