// The tile of the 3x3 kernel (conv_halo.hip, which describes it), for the kernels that run it.
#pragma once

#include "dma_common.hpp"

namespace relay {
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

// Fills in the arguments of a 128 x 64 tile with 128-byte chunks (all but the tile divisions), where the layer has that form.
bool conv_halo_group_args(const ConvArgs& a, HaloArgs& block, size_t& lds_bytes);
namespace {

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
// tile: what xcd_remap makes of the workgroup's place among the `workgroups` of this conv.  LDS: the launch's dynamic share.
template <bool IS_I8, int WAVES_M, int WAVES_N, int TM, int TN, int KP, int HB = 1, bool SQUARE = false, int SK = 1, bool EXT = false,
          bool POOL = false>
__device__ __forceinline__ void conv3x3_halo_tile(const HaloArgs& block, int tile, int place, int workgroups) {
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
  const int nb = workgroups, xcd_idx = place >> 3;
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
}  // namespace
}  // namespace relay
