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

#include "dma_common.hpp"

namespace relay {
namespace {

struct HaloGeom {
  int P, F;           // row pitch W + 1 and image pitch (H + 1) * P of the flat coordinate; square tiles: F tiles per image
  int Mflat;          // N * F flat output positions; square tiles: 256 positions for each tile
  float rcp_p, rcp_f;
  int xblk;           // 16-row blocks per plane of a halo buffer
  int nxbuf;          // halo buffers: 2 when there are several channel chunks, else 1
  int ncc;            // channel chunks, C / CK
  int tab_slot;       // 16-byte slot of LDS where the pixel table starts (behind the ring and the epilogue staging)
  FastDiv fd_f, fd_row;             // division by F and (square tiles) by the tiles of a row
  FastDiv fd_tiles_m, fd_tiles_n;   // ... by the tile counts of the launched variant
  // the 2x2 / stride 2 maxima of the outputs [N][H/2][W/2][K], and division by W (square tiles with POOL)
  void* y_pooled;
  FastDiv fd_w;
};

struct HaloArgs {
  HaloGeom g;
  ConvArgs a;
};

constexpr int NSW = 3;         // filter ring stages (9 taps per chunk keep step % NSW compile-time)
constexpr int XPW = 8;         // halo blocks a wave loads per chunk, times HB
constexpr unsigned kNoBlock = ~0u;

// The loads behind step t of a chunk that has a successor: lw filter loads, then a wave's share of the xn halo blocks of
// the next chunk, spread over the first seven steps.  (It is read from the end of the ninth on.)
constexpr int halo_first(int t, int xn) { return t >= 7 ? xn : t * (xn / 7) + (t < xn % 7 ? t : xn % 7); }
constexpr int loads_behind(int t, int lw, int xn) { return lw + halo_first(t + 1, xn) - halo_first(t, xn); }

constexpr int SQ = 16, SQP = SQ + 2;   // square tiles: 16 x 16 outputs, 18 x 18 halo positions

// HB: a halo holds at most XPW * HB * waves blocks of 16 positions
// SQUARE: the tile is 16 x 16 outputs of one image instead of 256 consecutive flat positions; its halo is 324 rows whatever
// the image's width
// SK: waves that share a tile of sums and split the k-steps of every step between them (their sums meet in LDS before the
// epilogue, where each finishes 1 / SK of the tile).  A wave then owns an SK times larger tile for the same workgroup
// tile, so each matrix instruction needs fewer operand reads -- what the small tiles are bound by.
template <bool IS_I8, int WAVES_M, int WAVES_N, int TM, int TN, int KP, int HB = 1, bool SQUARE = false, int SK = 1, bool EXT = false,
          bool POOL = false>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * SK, 2) void conv3x3_halo_kernel(const int workgroups, const HaloArgs block) {
  const HaloGeom& g = block.g;
  const ConvArgs& a = block.a;
  constexpr int NW = WAVES_M * WAVES_N * SK;
  constexpr int VE = IS_I8 ? 16 : 8;
  constexpr int ES = IS_I8 ? 1 : 2;
  constexpr int CK = KP * BKV * VE;
  constexpr int BM = WAVES_M * TM * 32, BN = WAVES_N * TN * 32;
  constexpr int WTM = TM * 32, WTN = TN * 32;
  constexpr int WB = BN / 16;            // filter staging blocks of a plane: 16 rows x 64 B
  static_assert(KP * WB % NW == 0, "filter staging blocks must divide over the waves");
  constexpr int LW = KP * WB / NW;       // filter loads per step per wave: blocks i * NW + wave, plane by plane
  constexpr int XN = XPW * HB;           // halo blocks (of 16 positions x 64 bytes) per wave,
  constexpr int XJ = XN / KP;            // ... of a plane
  static_assert(XN % KP == 0, "whole blocks of all planes");
  constexpr int KSTEPS = KP * (BKV / 2);
  constexpr int KSW = KSTEPS / SK;       // ... of which this wave runs KSW
  constexpr int NM = KSW * TN * TM;      // MFMAs of a step
  constexpr int NR = KSW * (TN + TM);    // operand reads of a step
  static_assert(SK == 1 || (SK == 2 && TM == 2) || (SK == 4 && TM == 2 && TN == 2), "a wave finishes a row of blocks, or a block");
  static_assert(XN + NSW * LW + 8 <= 63, "vmcnt is a 6-bit counter");
  static_assert(9 % NSW == 0, "the ring stage of a step has to be a compile-time constant");
  constexpr int WPLANE = BN * BKV;       // 16-byte slots of one filter plane
  constexpr int WSTAGE = KP * WPLANE;
  constexpr int TM_E = SK > 1 ? 1 : TM, TN_E = SK == 4 ? 1 : TN;   // blocks a wave finishes
  constexpr int EP = TN_E * 8 + 1;
  static_assert(!SQUARE || BM == SQ * SQ, "a square tile is 256 positions");
  const int P = SQUARE ? SQP : g.P;
  typedef typename Mma<IS_I8>::acc_t acc_t;

  extern __shared__ uint4 lds[];
  const int xplane = g.xblk * 64;                   // slots of one halo plane
  const int xbuf_slots = KP * xplane;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint4*)(&lds[0]);
  const unsigned wring_base = lds_base + (unsigned)(g.nxbuf * xbuf_slots) * 16u;
  const unsigned dump_base = wring_base + (unsigned)(NSW * WSTAGE) * 16u;
  const uint4* wring = lds + g.nxbuf * xbuf_slots;

  // Every argument the kernel uses is asked for here, so that their scalar loads leave as one batch with one
  // wait; left to itself the compiler loads them where they are first used, and the prologue then waits
  // for five scalar-load round trips one after another.  (The workgroup's number passes through the same statement: arithmetic on it that
  // needs only some of them would otherwise be placed ahead of the others' loads.)
  int tile = xcd_remap((int)blockIdx.x, workgroups);
  const void* ptr_x = a.x;   // (through it too, like the operands' addresses: their copies into a descriptor wait for nothing ahead of it)
  const void* ptr_w = a.w;
#define RELAY_ASKED                                                                                                                     \
  "s"(a.y), "s"(a.res), "s"(a.bias), "s"(a.scale), "s"(a.shift), "s"(a.qbias), "s"(a.N), "s"(a.H), "s"(a.W), "s"(a.C), \
      "s"(a.K), "s"(a.Kp), "s"(a.flags), "s"(a.param_vec), "s"(a.n_major), "s"(a.xs_n), "s"(g.P), "s"(g.F), "s"(g.Mflat), "s"(g.rcp_p),  \
      "s"(g.rcp_f), "s"(g.xblk), "s"(g.nxbuf), "s"(g.ncc), "s"(g.tab_slot), "s"(g.fd_f.mul), "s"(g.fd_f.shift), "s"(g.fd_tiles_m.mul),   \
      "s"(g.fd_tiles_m.shift), "s"(g.fd_tiles_n.mul), "s"(g.fd_tiles_n.shift)
  if constexpr (IS_I8)   // (the quantized tail's own arguments too)
    asm volatile("" : "+s"(tile), "+s"(ptr_x), "+s"(ptr_w) : RELAY_ASKED, "s"(a.lshift), "s"(a.rshift), "s"(a.round_add), "s"(a.qmode), "s"(a.clip_lo), "s"(a.clip_hi),
                 "s"(a.qmult), "s"(a.qshift));
  else
    asm volatile("" : "+s"(tile), "+s"(ptr_x), "+s"(ptr_w) : RELAY_ASKED);
#undef RELAY_ASKED
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (WAVES_M * WAVES_N), wsub = wave % (WAVES_M * WAVES_N);
  const int wm = wsub % WAVES_M, wn = wsub / WAVES_M;
  const int tiles_m = (g.Mflat + BM - 1) / BM, tiles_n = (a.K + BN - 1) / BN;
  const int tile_q = (int)fast_div((uint32_t)tile, a.n_major ? g.fd_tiles_m : g.fd_tiles_n);
  const int tile_n = a.n_major ? tile_q : tile - tile_q * tiles_n;
  const int tile_m = a.n_major ? tile - tile_q * tiles_m : tile_q;
  const int o0 = tile_m * BM, n0 = tile_n * BN;
  // (uniform) image and in-image position of the tile's first position; square tiles: image and tile of it
  const int n_0 = (int)fast_div((uint32_t)(SQUARE ? tile_m : o0), g.fd_f);
  const int rem_0 = (SQUARE ? tile_m : o0) - n_0 * g.F;

  // ---- first loads out as early as possible: the epilogue constants (oldest, so that nothing ever waits for
  //      them longer than for a ring load), then the filters of step 0, which need no decoding.  What the waits count on is
  //      this order: constants, filters of step 0 (LW loads), the halo of chunk 0 (XN; a dump load stands in for a block that is
  //      none), the filters of steps 1 and 2, up to four touches; from then on, behind step t of a chunk, the filters of step
  //      t + 3 and that step's share of the next chunk's halo (loads_behind), in the last chunk only what filters are left.
  const int srow = lane >> 2, sphys = lane & 3;
  constexpr int CG = TN_E * 4;  // lanes per pixel row in the epilogue
  const int tm_lo = SK == 1 ? 0 : (SK == 2 ? wk : wk >> 1), tn_lo = SK == 4 ? wk & 1 : 0;   // the first block this wave finishes
  const int ech = n0 + wn * WTN + tn_lo * 32 + (lane % CG) * 8;
  RawLaneParams rawp;
  fetch_lane_params<IS_I8>(a, ech, rawp);
  unsigned w_off[LW];
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int b = i * NW + wave, row = (b % WB) * 16 + srow;
    const int kvl = sphys ^ lds_swizzle(row);
    const int ch = n0 + row;
    w_off[i] = ch < a.K ? (unsigned)((ch * a.Kp + (b / WB) * (BKV * VE) + kvl * VE) * ES) : kOob;
  }
  const intx4 rs_x = make_rsrc(ptr_x, (unsigned)((size_t)a.N * a.xs_n * ES));
  const intx4 rs_w = make_rsrc(ptr_w, (unsigned)((size_t)a.K * a.Kp * ES));
  auto issue_filters = [&](int s) {  // the filters of step (0, s), s < NSW
#pragma unroll
    for (int i = 0; i < LW; ++i)
      lds_dma16(rs_w, wring_base + (unsigned)(s * WSTAGE + (i * NW + wave) * 64) * 16u, w_off[i] + (unsigned)(s * a.C * ES));
  };
  issue_filters(0);

  // ---- pixel table: for each of the halo's xblk * 16 flat positions the index (n * H + row) * W + col of
  //      the input pixel there, or ~0 where the position is padding.  One decode per thread (or two)
  //      instead of one per load and per stored pixel: the halo loads below look their rows up here, and so
  //      does the epilogue, because the output pixel of flat position o is the input pixel of o + P + 1.
  unsigned* ptab = reinterpret_cast<unsigned*>(lds + g.tab_slot);
  if constexpr (SQUARE) {
    const int ty = (int)fast_div((uint32_t)rem_0, g.fd_row), tx = rem_0 - ty * g.P;
    for (int r = tid; r < g.xblk * 16; r += NW * 64) {
      const int hy = r / SQP, rowi = ty * SQ - 1 + hy, coli = tx * SQ - 1 + (r - hy * SQP);
      ptab[r] = ((unsigned)rowi < (unsigned)a.H && (unsigned)coli < (unsigned)a.W && hy < SQP)
                    ? (unsigned)((n_0 * a.H + rowi) * a.W + coli) : ~0u;
    }
  } else {
    for (int r = tid; r < g.xblk * 16; r += NW * 64) {
      int dn, r1, rowi, coli;
      small_divmod(rem_0 + r, g.F, g.rcp_f, dn, r1);
      small_divmod(r1, g.P, g.rcp_p, rowi, coli);
      const int n = n_0 + dn;
      ptab[r] = (n < a.N && rowi >= 1 && coli >= 1) ? (unsigned)((n * a.H + rowi - 1) * a.W + coli - 1) : ~0u;
    }
  }
  // (the table is LDS traffic only: the loads already in flight are not waited for here)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();

  // ---- this lane's part of a halo: of each plane the blocks j * NW + wave, j < XJ, so that a position is looked up once for all
  //      planes.  Branch-free: the loads of a wave are XN whatever the halo's size (a dump load for a block that is none), and few
  //      instructions, because a wave that has its SIMD to itself issues one every four to five clocks.  (Counted block by block over all
  //      planes, with a division, two branches and a look-up each, this stretch was 1.75 K of a 64 x 64 tile's 12 K clocks: 128 -> 128 at
  //      25 x 25, 12 images 7.0 -> 6.7 us, 64 -> 64 at 56 x 56, 32 images 16.6 -> 15.9, operands from beyond the L2.)
  unsigned x_off[XJ];    // byte offset of the 16 bytes this lane fetches (chunk 0, plane 0), or out of range
  unsigned x_dst[XJ];    // (uniform) where their plane 0 goes in a halo buffer; the dump's place for a block that is none
  unsigned x_px[XJ];     // (all table reads first: one wait for all of them)
  const int kvl_x = sphys ^ lds_swizzle(srow);   // (the swizzle repeats every 16 rows)
#pragma unroll
  for (int j = 0; j < XJ; ++j) x_px[j] = ptab[min(j * NW + wave, g.xblk - 1) * 16 + srow];
#pragma unroll
  for (int j = 0; j < XJ; ++j) {
    const bool some = j * NW + wave < g.xblk;   // (uniform)
    unsigned off = x_px[j] * (unsigned)(a.C * ES) + (unsigned)(kvl_x * VE * ES);
    asm volatile("" : "+v"(off));
    x_off[j] = some && x_px[j] != ~0u ? off : kOob;
    x_dst[j] = some ? (unsigned)(j * NW + wave) * 1024u : kNoBlock;
  }
  // load xt of a wave's XN: plane xt % KP of its block xt / KP, of the chunk `at` bytes into a pixel, to the halo buffer at `buf`
  auto issue_halo = [&](int xt, unsigned buf, unsigned at) {
    const unsigned dst = x_dst[xt / KP];
    lds_dma16(rs_x, dst != kNoBlock ? buf + dst + (unsigned)(xt % KP * xplane) * 16u : dump_base, x_off[xt / KP] + (unsigned)(xt % KP * 64) + at);
  };
#pragma unroll
  for (int t = 0; t < XN; ++t) issue_halo(t, lds_base, 0u);
#pragma unroll
  for (int s = 1; s < NSW; ++s) issue_filters(s);

  // ---- the filters this XCD is going to read, towards its L2 (see touch_filters): with n_major the channel tiles of
  //      its run of tiles, else all of them.  (These loads are younger than those the first two steps wait for, and
  //      older than all others.)  Only in short launches (measured up to 912 tiles x chunks): in longer ones the first
  //      use of the filters is a small part of the time and the extra wait costs as much (VGG-16 0.7 %).
  const int nb = workgroups, xcd_idx = (int)blockIdx.x >> 3;
  int touched = 0;
  if (nb * g.ncc <= 1024 && xcd_idx < 64) {
    const int per = nb >> 3, wgs = min(per + 1, 64);  // (two workgroups on each of the XCD's 32 CUs)
    unsigned first = 0, bytes = (unsigned)(a.K * a.Kp * ES);
    if (a.n_major) {
      const int t0 = tile - xcd_idx, c0 = (int)fast_div((uint32_t)t0, g.fd_tiles_m) * BN;
      const int c1 = ((int)fast_div((uint32_t)min(t0 + per, nb - 1), g.fd_tiles_m) + 1) * BN;
      first = (unsigned)(c0 * a.Kp * ES);
      bytes = (unsigned)((min(c1, a.K) - c0) * a.Kp * ES);
    }
    touched = touch_filters<4>(rs_w, dump_base, first, bytes, xcd_idx * NW + wave, wgs * NW, lane);
  }

  auto issue_one = [&](int cc, int t, int i) {
    if (i < LW) {
      const int tw = (t + NSW) % 9, ccw = cc + (t + NSW) / 9;  // tap and chunk of the step being fetched
      lds_dma16(rs_w, wring_base + (unsigned)((tw % NSW) * WSTAGE + (i * NW + wave) * 64) * 16u,
                w_off[i] + (unsigned)((tw * a.C + ccw * CK) * ES));   // (kOob + a filter's length stays out of range)
    } else {
      const int xt = min(halo_first(t, XN) + (i - LW), XN - 1);   // which of this wave's halo loads
      issue_halo(xt, lds_base + (unsigned)(((cc + 1) & 1) * xbuf_slots) * 16u, (unsigned)((cc + 1) * CK * ES));
    }
  };

  acc_t acc[TN][TM];
#pragma unroll
  for (int tn = 0; tn < TN; ++tn)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tn][tm][v] = 0;

  LaneParams lp;
  finish_lane_params<IS_I8>(rawp, lp);

  const int lrow = lane & 31, lhalf = lane >> 5;
  // halo row of this lane's first pixel at tap (0, 0); its next one is XSTEP rows on (a block is two rows of a square tile)
  const int xrow0 = SQUARE ? (wm * TM * 2 + (lrow >> 4)) * SQP + (lrow & 15) : wm * WTM + lrow;
  constexpr int XSTEP = SQUARE ? 2 * SQP : 32;
  uint4 wf[2][KSW][TN], xf[2][KSW][TM];
  const int wlane = lds_slot(wn * WTN + lrow, lhalf);   // (k-vector 2 + lhalf of a row is two slots away: ^ 2)
  // where this lane's activations of step (cc, t) are; worked out anew for each step (those of all nine taps
  // would occupy the registers of the second operand set)
  int xslot[TM];
  auto locate_tap = [&](int cc, int t) {
    int xrow = xrow0;
    asm volatile("" : "+v"(xrow));
    xrow += (t / 3) * P + (t % 3);  // the tap is a shift of the halo rows
    const int xb = ((cc & 1) * (g.nxbuf - 1)) * xbuf_slots;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
      xslot[tm] = (XSTEP % 16 == 0 && tm) ? xslot[0] + tm * XSTEP * BKV : xb + lds_slot(xrow + tm * XSTEP, lhalf);  // (the swizzle repeats every 16 rows)
  };
  // the i-th operand read of a step, in the order the MFMAs use them
  auto read_one = [&](int t, int i, int buf) {
    const int k = i / (TN + TM), e = i % (TN + TM), ks = wk * KSW + k, kx = 2 * (ks & 1);
    if (e < TN) wf[buf][k][e] = wring[(t % NSW) * WSTAGE + (ks >> 1) * WPLANE + e * 32 * BKV + (wlane ^ kx)];
    else xf[buf][k][e - TN] = lds[(ks >> 1) * xplane + (xslot[e - TN] ^ kx)];
  };
  // ---- what the epilogue reads: the output pixels of this lane (the output pixel of a flat position o is the table's entry for o + P + 1) and
  //      its residual vectors, asked for behind step RES_AT of the last chunk, the last one that loads filters, so that they arrive under
  //      the steps behind it and no wait for filters is one for them.  (Layers with a residual 1 to 3 % faster than when asked for in the
  //      epilogue; two steps earlier less.  int8: asked for behind the last step, 1 to 3 % better than earlier.)
  constexpr int PPI = 64 / CG, ITS = 32 / PPI, NRES = TM_E * ITS, RES_AT = IS_I8 ? 8 : 5;
  const int epix = lane / CG, ecg = lane % CG;
  const bool vec_ok = (a.K & 7) == 0;
  const bool pre_res = (a.flags & F_RES) && vec_ok;
  unsigned mpix[TM_E][ITS];
  uint4 resv[TM_E][ITS];
  auto request_residual = [&]() {
#pragma unroll
    for (int tm = 0; tm < TM_E; ++tm)
#pragma unroll
      for (int it = 0; it < ITS; ++it) {
        const int pix = it * PPI + epix;
        mpix[tm][it] = ptab[(SQUARE ? ((wm * TM + tm_lo + tm) * 2 + (pix >> 4)) * SQP + (pix & 15) : wm * WTM + (tm_lo + tm) * 32 + pix) + P + 1];
      }
    if (pre_res) {
      const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.res), 0, (int)((unsigned)a.M * a.K * ES), 0x00020000);
#pragma unroll
      for (int tm = 0; tm < TM_E; ++tm)
#pragma unroll
        for (int it = 0; it < ITS; ++it) {
          const unsigned at = mpix[tm][it] != ~0u && ech < a.K ? (mpix[tm][it] * (unsigned)a.K + (unsigned)ech) * ES : kOob;
          if constexpr (IS_I8) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs_r, (int)at, 0, 0);
            resv[tm][it] = make_uint4(v[0], v[1], 0u, 0u);
          } else {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs_r, (int)at, 0, 0);
            resv[tm][it] = make_uint4(v[0], v[1], v[2], v[3]);
          }
        }
    }
  };
  // Step t multiplies the operands that step t - 1 read and reads those of step t + 1, so that LDS and matrix cores
  // work at the same time.  A step's loads were issued two steps before they are read.  LAST: the last chunk, behind
  // which nothing is left to load.
  auto step = [&](int cc, auto last_tag, auto tap_tag) {
    constexpr bool LAST = decltype(last_tag)::value;
    constexpr int t = decltype(tap_tag)::value, cur = t & 1;
    constexpr int FT = LAST ? 9 - NSW : 9;   // steps that have filters to load
    constexpr int nload = LAST ? (t < FT ? LW : 0) : loads_behind(t, LW, XN);
    constexpr int nread = LAST && t == 8 ? 0 : NR;
    if constexpr (nread > 0) {  // the operands this step reads have landed once only the loads behind step t - 1 are pending
      if (t == 0 && touched == 4) wait_loads<LW + 4>();
      else if (LAST && (t == RES_AT + 1 || t == RES_AT + 2) && pre_res) wait_loads<(t - 1 < FT ? LW : 0) + NRES>();   // (the residual's too)
      else wait_loads<t == 0 ? LW : (LAST ? (t - 1 < FT ? LW : 0) : loads_behind(t == 0 ? 8 : t - 1, LW, XN))>();
      __builtin_amdgcn_s_barrier();
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int k = m / (TN * TM), tn = m / TM % TN, tm = m % TM;
      acc[tn][tm] = Mma<IS_I8>::mma(wf[cur][k][tn], xf[cur][k][tm], acc[tn][tm]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = m; i < nload; i += NM) issue_one(cc, t, i);
#pragma unroll
      for (int i = 2 * m; i < nread && (i < 2 * m + 2 || m == NM - 1); ++i) read_one((t + 1) % 9, i, cur ^ 1);
      // where the next step reads, worked out while the last MFMAs run
      if (m == (2 * (NM - 2) >= NR ? NM - 2 : NM - 1)) locate_tap(cc + (t + 2) / 9, (t + 2) % 9);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (LAST && t == RES_AT) {
      request_residual();
      __builtin_amdgcn_sched_barrier(0);
    }
    // (the compiler may not sink a step's MFMAs to where the sums are used)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) asm volatile("" : "+v"(acc[tn][tm]));
  };
  auto chunk = [&](int cc, auto last_tag) {
    using std::integral_constant;
    step(cc, last_tag, integral_constant<int, 0>{});
    step(cc, last_tag, integral_constant<int, 1>{});
    step(cc, last_tag, integral_constant<int, 2>{});
    step(cc, last_tag, integral_constant<int, 3>{});
    step(cc, last_tag, integral_constant<int, 4>{});
    step(cc, last_tag, integral_constant<int, 5>{});
    step(cc, last_tag, integral_constant<int, 6>{});
    step(cc, last_tag, integral_constant<int, 7>{});
    step(cc, last_tag, integral_constant<int, 8>{});
    constexpr bool LAST = decltype(last_tag)::value;
    // (nine steps: the operands of the next chunk's first one are in the odd set)
    if constexpr (!LAST) {
#pragma unroll
      for (int k = 0; k < KSW; ++k) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) wf[0][k][tn] = wf[1][k][tn];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) xf[0][k][tm] = xf[1][k][tm];
      }
    }
    touched = 0;
  };
  locate_tap(0, 0);
  // the operands of the first step: everything but the filters of the steps behind it (and the touches) has landed
  if (touched == 4) wait_loads<(NSW - 1) * LW + 4>();
  else wait_loads<(NSW - 1) * LW>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < NR; ++i) read_one(0, i, 0);
  locate_tap(0, 1);
  for (int cc = 0; cc < g.ncc - 1; ++cc) chunk(cc, std::false_type{});
  chunk(g.ncc - 1, std::true_type{});

  // ---- epilogue: as in the implicit-GEMM kernel, with the flat position decoded back to a pixel
  wait_loads<NRES>();   // (nothing but the residual is in flight any more)
  __builtin_amdgcn_s_barrier();  // every wave is done reading
  constexpr int XCH = SK > 1 ? (TM * TN - TM_E * TN_E) * 4 * 64 : 0;  // slots a wave hands to the others of its tile
  acc_t fin[TN_E][TM_E];
  if constexpr (SK == 1) {
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) fin[tn][tm] = acc[tn][tm];
  } else {
    // every wave leaves the blocks that others finish, block by block in the order of their owners, and adds up its own
    uint4* give = lds + wave * XCH;
    constexpr int OWN = TM * TN / SK;   // blocks of an owner; block tm * TN + tn belongs to the wave with wk = block / OWN
#pragma unroll
    for (int b = 0; b < TM * TN; ++b) {
      const int owner = b / OWN;
      if (owner != wk) {   // (uniform)
        const int at = b - (owner > wk ? OWN : 0);
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          uint4 v;
          v.x = as_u32(acc[b % TN][b / TN][4 * q4]);
          v.y = as_u32(acc[b % TN][b / TN][4 * q4 + 1]);
          v.z = as_u32(acc[b % TN][b / TN][4 * q4 + 2]);
          v.w = as_u32(acc[b % TN][b / TN][4 * q4 + 3]);
          give[(at * 4 + q4) * 64 + lane] = v;
        }
      } else {
        fin[TN_E == 1 ? 0 : b % TN][0] = acc[b % TN][b / TN];
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int o = 1; o < SK; ++o) {
      const int from = (wk + o) % SK;   // (uniform)
      const uint4* take = lds + (from * (WAVES_M * WAVES_N) + wsub) * XCH + (wk - (wk > from ? 1 : 0)) * OWN * 4 * 64;
#pragma unroll
      for (int b = 0; b < OWN; ++b)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const uint4 v = take[(b * 4 + q4) * 64 + lane];
          const unsigned r[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (IS_I8) fin[b][0][4 * q4 + e] += (int)r[e];
            else fin[b][0][4 * q4 + e] += __builtin_bit_cast(float, r[e]);
          }
        }
    }
  }
  uint4* stg = lds + NW * XCH + wave * (32 * EP);
  const OutLoc ol = EXT ? locate_output(a, ech) : OutLoc{nullptr, 0, 0, 0};
#pragma unroll
  for (int tm = 0; tm < TM_E; ++tm) {
#pragma unroll
    for (int tn = 0; tn < TN_E; ++tn)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        uint4 v;
        v.x = as_u32(fin[tn][tm][4 * q4]);
        v.y = as_u32(fin[tn][tm][4 * q4 + 1]);
        v.z = as_u32(fin[tn][tm][4 * q4 + 2]);
        v.w = as_u32(fin[tn][tm][4 * q4 + 3]);
        stg[lrow * EP + tn * 8 + 2 * q4 + lhalf] = v;
      }
    // same wave wrote what it now reads: LDS operations of a wave execute in order
    uint4 kept[POOL ? 4 : 1];
#pragma unroll
    for (int it = 0; it < 32 / PPI; ++it) {
      const int pix = it * PPI + epix;
      const uint4 lo = stg[pix * EP + ecg * 2], hi = stg[pix * EP + ecg * 2 + 1];
      const unsigned raw[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      const unsigned m = mpix[tm][it];
      if constexpr (POOL) {
        kept[it] = make_uint4(0u, 0u, 0u, 0u);
        if (m != ~0u && ech < a.K) finish_store8<IS_I8, false>(a, raw, (int)m, ech, lp, ol, true, false, uint4{0u, 0u, 0u, 0u}, &kept[it]);
        continue;
      }
      if (m == ~0u || ech >= a.K) continue;  // not a pixel, or past Cout
      finish_store8<IS_I8, false, EXT>(a, raw, (int)m, ech, lp, ol, vec_ok, pre_res, resv[tm][it]);
    }
    if constexpr (POOL) {
      // a block is two rows of 16 outputs: a lane has columns epix and epix + 8 of both, the lane CG further the column to the
      // right.  (Even heights and widths: the four outputs of a maximum are all pixels or all not.)
      static_assert(!POOL || (SQUARE && !IS_I8 && CG == 8 && SK == 1 && !EXT), "two rows of 16 fp16 outputs in four passes of 8 pixels");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint4 v = max_half8(kept[h], kept[h + 2]);
        v = max_half8(v, make_uint4(__shfl_xor(v.x, CG, 64), __shfl_xor(v.y, CG, 64), __shfl_xor(v.z, CG, 64), __shfl_xor(v.w, CG, 64)));
        const unsigned m = mpix[tm][h];
        if ((epix & 1) || m == ~0u || ech >= a.K) continue;
        const unsigned x = m - fast_div(m, g.fd_w) * (unsigned)a.W;   // (row * W + x) -> (row / 2) * (W / 2) + x / 2
        *reinterpret_cast<uint4*>(static_cast<_Float16*>(g.y_pooled) + (size_t)((m + x) >> 2) * a.K + ech) = v;
      }
    }
  }
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
  if (!is_i8 && a.C == 64 && a.K <= 64 && t128 > 512 && t128 <= 1700 && halo_fits(a, is_i8, 2, 80 * 1024)) return 2;
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
