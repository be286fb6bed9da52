// Depthwise 3x3 conv2d and the 1x1 conv2d behind it as one kernel, for layers of few pixels (small batches, deep layers) and for blocks
// of at most 128 channels.
//
// The patch kernel (dwpw.hip) cuts the channels into chunks and walks them behind a barrier per chunk.  That hides
// memory latency where there are many pixels, but a layer of few pixels is one long serial chain: 512 -> 512 at
// 14 x 14, batch 32 took 15.2 us there for 3.3 GFLOP and 13 MB, and at batch 1 two launches (4.8 + 4.6 us) beat it.
// Here a workgroup has a single barrier:
//   1. every thread computes depthwise outputs of 8 channels of two or four pixels (one above the other) at a time straight
//      from memory -- channels lie along the lanes, so a wave's load is a run of whole lines, taps in the
//      padding read zeros -- with the loads of its next pixels under way, and writes them, narrowed to fp16, into an
//      LDS tile that holds ALL channels of the rectangle;
//   2. behind the barrier a wave multiplies the tile with 32 output channels' filters, which it has brought
//      into an LDS ring of its own with global->LDS loads, requested before the depthwise work (the
//      whole reduction where it fits): it waits for its own loads only.
// The depthwise work is repeated by every workgroup of a pixel tile, so the channel tile is as wide as the grid allows:
// 64 channels where there are too few tiles to fill the chip, 256 where there are enough.
// Bound (cycles of a 16 x 64 tile of 512 channels, 10.9 K in all): the loads through the texture addresser at 64 bytes a
// clock (2.9 K), the depthwise multiply-adds (2.2 K with one wave per SIMD, half with two: a SIMD issues
// from two waves what one alone cannot), the fragments of the 1x1 conv through LDS (2.2 K), then latencies.  2 x 2 pixels per item (16
// loads for four outputs, not 24) was no faster, and slower where it leaves threads idle.
// Arithmetic and its order are those of the two separate kernels: the result equals the two launches bit for bit.
#include <cstdio>

#include "dma_common.hpp"
#include "dw_math.hpp"

namespace relay {
namespace {

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // four consecutive floats at any address

// 16 bytes per lane from memory to LDS: lane i's land at dst + i.  (The builtin, not lds_dma16: the compiler's waits for
// the register loads around these requests then leave them in flight.)
__device__ __forceinline__ void load_to_lds16(__amdgpu_buffer_rsrc_t rsrc, uint4* dst, unsigned voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, (int)voff, 0, 0, 0);
}

__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t rsrc, unsigned voff) {
  const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voff, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// What the host works out for a launch.
struct DirectGeom {
  int th, tw;                      // rectangle of output pixels, th a multiple of MR, th * tw <= BM
  int tiles_x, tiles_y, tiles_n;   // rectangles of an image, channel tiles
  int n_major;                     // consecutive workgroups share a channel tile (else a rectangle)
  int log_cv;                      // log2(C / 8)
  int nit;                         // items per thread
  FastDiv fd_x, fd_y, fd_n, fd_p, fd_tw;   // division by tiles_x, tiles_y, tiles_n, the rectangles of all images, tw
};

struct DirectArgs {
  DirectGeom g;
  DwPwArgs a;
};

// BM: rows of the tile (16: the matrix instruction's other 16 rows repeat them); WN: waves with 32 output channels each,
// of NW that share the depthwise work; NS: ring stages of 32 channels; CP: most channels / 32.  OCC: 0, a thread has the
// inputs of two items in registers, or the waves per SIMD for which it has those of one.  MR: output rows of an item.
// Four rows take 18 loads at stride 1 where twice two take 24, and one memory latency instead of two: with 256 or 128 channels
// and 64 x 128 tiles, a thread's whole share (128 -> 128 at 56 x 56, batch 32 21.4 -> 20.0 us; 512 -> 512 at 14 x 14 as 64 x 256
// 13.9 -> 13.2, as 32 x 256 9.5 -> 8.9 at batch 16 of 13 x 12).  Where fewer items than threads are left the two rows win.
template <int STRIDE, int BM, int WN, int NW, int NS, int CP, int OCC, int MR>
__global__ __launch_bounds__(64 * NW, OCC ? OCC : 1) void dwpw_fused_direct_kernel(const int workgroups, const DirectArgs block) {
  const DirectGeom& g = block.g;
  const DwPwArgs& a = block.a;
  constexpr int NT = 64 * NW, BN = 32 * WN;
  constexpr int TM = BM >= 32 ? BM / 32 : 1;
  constexpr int APL = BM * BKV + BKV;       // slots of a 32-channel plane of the tile (padded: the planes start on other banks)
  constexpr int FPL = 32 * BKV;             // slots of a ring stage: 32 filters x 64 bytes
  constexpr int EP = 9;                     // epilogue staging pitch
  constexpr int IH = (MR - 1) * STRIDE + 3; // input rows under an item's MR pixels
  static_assert(NS * FPL >= 32 * EP, "the staging block reuses the ring");
  static_assert(NS % 2 == 0 && NS >= 4, "whole groups of planes");
  static_assert(NW % WN == 0, "the waves share the first fill of the rings evenly");
  static_assert((CP * APL + WN * NS * FPL) * 16 <= 160 * 1024, "LDS of one CU");
  typedef Mma<false>::acc_t acc_t;
  __shared__ uint4 act[CP * APL];
  __shared__ uint4 ring[WN * NS * FPL];

  const ConvArgs& pw = a.pw;
  int place = xcd_remap((int)blockIdx.x, workgroups);   // (passes through: arithmetic on it stays behind the loads of all arguments)
  asm volatile("" : "+s"(place) : "s"(a.x), "s"(a.dw_w), "s"(a.dw_bias), "s"(a.dw_scale), "s"(a.dw_shift), "s"(a.dw_flags), "s"(a.N), "s"(a.H),
               "s"(a.W), "s"(a.C), "s"(a.Ho), "s"(a.Wo), "s"(a.stride), "s"(g.th), "s"(g.tw), "s"(g.tiles_x), "s"(g.tiles_y), "s"(g.tiles_n), "s"(g.n_major),
               "s"(g.log_cv), "s"(g.nit), "s"(g.fd_x.mul), "s"(g.fd_x.shift), "s"(g.fd_y.mul), "s"(g.fd_y.shift), "s"(g.fd_n.mul),
               "s"(g.fd_n.shift), "s"(g.fd_p.mul), "s"(g.fd_p.shift), "s"(g.fd_tw.mul), "s"(g.fd_tw.shift), "s"(pw.w), "s"(pw.y), "s"(pw.bias),
               "s"(pw.scale), "s"(pw.shift), "s"(pw.K), "s"(pw.Kp), "s"(pw.flags), "s"(pw.param_vec));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned t0 = (unsigned)place;
  const unsigned tq = fast_div(t0, g.n_major ? g.fd_p : g.fd_n);
  const unsigned rects = (unsigned)(g.tiles_x * g.tiles_y * a.N);
  const int tile_n = (int)(g.n_major ? tq : t0 - tq * (unsigned)g.tiles_n);
  const unsigned t1 = g.n_major ? t0 - tq * rects : tq;
  const unsigned t2 = fast_div(t1, g.fd_x);
  const int tx = (int)(t1 - t2 * (unsigned)g.tiles_x);
  const int n = (int)fast_div(t2, g.fd_y);
  const int ty = (int)t2 - n * g.tiles_y;
  const int oy0 = ty * g.th, ox0 = tx * g.tw, n0 = tile_n * BN;

  // ---- depthwise work: item = (MR pixels, one above the other; channel vector); a thread keeps its channel vector
  const int cvecs = 1 << g.log_cv;
  const int cv = tid & (cvecs - 1);
  const int groups = NT >> g.log_cv;              // items of a channel vector that the workgroup takes at a time
  const int nit = g.nit;
  const int pix_bytes = a.C * 2;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.x), 0, (int)((unsigned)a.N * a.H * a.W * a.C * 2u), 0x00020000);
  auto load_item = [&](int it, uint4(&xv)[IH][3]) {
    const int item = it * groups + (tid >> g.log_cv);
    const int py = (int)fast_div((unsigned)item, g.fd_tw), px = item - py * g.tw;
    const int iy = (oy0 + MR * py) * STRIDE - 1, ix = (ox0 + px) * STRIDE - 1;
    const bool live = MR * py < g.th;
    const unsigned base = (unsigned)(((n * a.H + iy) * a.W + ix) * pix_bytes + cv * 16);
#pragma unroll
    for (int r = 0; r < IH; ++r) {
      const bool rok = live && (unsigned)(iy + r) < (unsigned)a.H;
#pragma unroll
      for (int s = 0; s < 3; ++s)
        xv[r][s] = buffer_load16(rs, rok && (unsigned)(ix + s) < (unsigned)a.W ? base + (unsigned)((r * a.W + s) * pix_bytes) : kOob);
    }
  };
  // requested in the order of need: the first two items, the depthwise filters and constants, the 1x1 filters
  uint4 xa[IH][3], xb[IH][3];
  load_item(0, xa);
  if (!OCC && nit > 1) load_item(1, xb);
  uint4 wv[9];
  {
    const uint4* w = static_cast<const uint4*>(a.dw_w) + cv;   // [tap][C/8]
#pragma unroll
    for (int t = 0; t < 9; ++t) wv[t] = w[t << g.log_cv];
  }
  floatx4u sc[2] = {{1.f, 1.f, 1.f, 1.f}, {1.f, 1.f, 1.f, 1.f}}, sf[2] = {}, bb[2] = {};
  if (a.dw_flags & F_BN) {
    const floatx4u* s4 = reinterpret_cast<const floatx4u*>(a.dw_scale + cv * 8);
    const floatx4u* f4 = reinterpret_cast<const floatx4u*>(a.dw_shift + cv * 8);
    sc[0] = s4[0], sc[1] = s4[1], sf[0] = f4[0], sf[1] = f4[1];
  }
  if (a.dw_flags & F_BIAS) {
    const floatx4u* b4 = reinterpret_cast<const floatx4u*>(a.dw_bias + cv * 8);
    bb[0] = b4[0], bb[1] = b4[1];
  }

  // ---- the filters: the ring of wave w < WN holds its 32 output channels; all waves take part in the first fill
  const int planes = a.C >> 5;
  const int wn = wave % WN;
  const int srow = lane >> 2, sphys = lane & 3;
  const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(pw.w), 0, (int)((unsigned)pw.K * pw.Kp * 2u), 0x00020000);
  unsigned w_off[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = j * 16 + srow, ch = n0 + wn * 32 + row;
    w_off[j] = ch < pw.K ? (unsigned)((ch * pw.Kp + (sphys ^ lds_swizzle(row)) * 8) * 2) : kOob;
  }
  uint4* const my = ring + wn * (NS * FPL);
  const int fill = min(NS, planes);
  if (n0 + wn * 32 < pw.K)
    for (int p = wave / WN; p < fill; p += NW / WN)
#pragma unroll
      for (int j = 0; j < 2; ++j) load_to_lds16(rs_w, my + p * FPL + j * 64, w_off[j] + (unsigned)(p * 64));
  const bool mma_wave = wave < WN && n0 + wave * 32 < pw.K;   // (uniform)
  const int ech = n0 + wave * 32 + (lane & 3) * 8;
  RawLaneParams rawp;

  float mul[8], add[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float s1 = sc[e >> 2][e & 3];
    asm volatile("" : "+v"(s1));   // (not ahead of the requests above: the first use waits for everything older)
    mul[e] = s1;
    add[e] = bb[e >> 2][e & 3] * s1 + sf[e >> 2][e & 3];  // (acc + b)*sc + sf
  }
  const float relu_lo = (a.dw_flags & F_RELU) ? 0.f : -__builtin_inff();
  auto compute_item = [&](int it, const uint4(&xv)[IH][3]) {
    const int item = it * groups + (tid >> g.log_cv);
    const int py = (int)fast_div((unsigned)item, g.fd_tw), px = item - py * g.tw;
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      float dacc[8];
#pragma unroll
      for (int fr = 0; fr < 3; ++fr)
#pragma unroll
        for (int fs = 0; fs < 3; ++fs) {
          const uint4 xx = xv[i * STRIDE + fr][fs], ww = wv[fr * 3 + fs];
          const unsigned xh[4] = {xx.x, xx.y, xx.z, xx.w}, wr[4] = {ww.x, ww.y, ww.z, ww.w};
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            if (fr + fs == 0) {
              mul_mix_lo(dacc[2 * h], xh[h], wr[h]);
              mul_mix_hi(dacc[2 * h + 1], xh[h], wr[h]);
            } else {
              fma_mix_lo(dacc[2 * h], xh[h], wr[h]);
              fma_mix_hi(dacc[2 * h + 1], xh[h], wr[h]);
            }
          }
        }
      const int row = (MR * py + i) * g.tw + px;
      if (MR * py < g.th) act[(cv >> 2) * APL + lds_slot(row, cv & 3)] = scale_shift_narrow8(dacc, mul, add, relu_lo);
    }
  };
  if constexpr (OCC) {
    for (int it = 0; it < nit; ++it) {
      compute_item(it, xa);
      if (it + 1 < nit) load_item(it + 1, xa);
    }
  } else for (int it = 0; it < nit; it += 2) {
    compute_item(it, xa);
    if (it + 2 < nit) load_item(it + 2, xa);
    if (it + 1 < nit) {
      compute_item(it + 1, xb);
      if (it + 3 < nit) load_item(it + 3, xb);
    }
  }
  if (mma_wave) fetch_lane_params<false>(pw, ech, rawp);
  wait_loads<0>();
  __syncthreads();
  if (!mma_wave) return;

  // ---- the 1x1 conv: 32 channels x BM pixels of this wave, in the order of the separate kernel
  acc_t acc[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[tm][v] = 0;
  const int lrow = lane & 31, lhalf = lane >> 5;
  // a group of UP planes is multiplied while the fragments of the next are on their way from LDS
  // (three waves per SIMD cover each other's reads, and the registers of a second plane would spill: 128 -> 128 at 56 x 56 36 us)
  constexpr int UP = OCC >= 3 ? 1 : TM == 1 && NS % 8 == 0 ? 4 : 2;
  struct Frags {
    uint4 w[UP][2], x[UP][2][TM];
  };
  auto fetch = [&](int p, int st, Frags& f) {
#pragma unroll
    for (int u = 0; u < UP; ++u)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        f.w[u][k] = my[(st + u) * FPL + lds_slot(lrow, 2 * k + lhalf)];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) f.x[u][k][tm] = act[(p + u) * APL + lds_slot((tm * 32 + lrow) & (BM - 1), 2 * k + lhalf)];
      }
  };
  auto multiply = [&](int p, const Frags& f) {
#pragma unroll
    for (int u = 0; u < UP; ++u)
      if (p + u < planes) {   // (uniform; only the last group can be short)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int tm = 0; tm < TM; ++tm) acc[tm] = Mma<false>::mma(f.w[u][k], f.x[u][k][tm], acc[tm]);
      }
  };
  Frags fa, fb;
  fetch(0, 0, fa);
  if (planes <= NS) {   // the whole reduction is in the ring
    for (int p = 0; p < planes; p += 2 * UP) {
      if (p + UP < planes) fetch(p + UP, p + UP, fb);
      multiply(p, fa);
      if (p + 2 * UP < planes) fetch(p + 2 * UP, p + 2 * UP, fa);
      if (p + UP < planes) multiply(p + UP, fb);
    }
  } else {
    // group p + UP has landed when at most NS - 2 UP younger planes are in flight, and the fragments of group p are in
    // registers: its stages take the group NS planes further on
    // (planes past the end are requested with out-of-range offsets: every turn issues the same number of loads)
    int st = 0;
    const intx4 rs_w4 = make_rsrc(pw.w, (unsigned)pw.K * pw.Kp * 2u);
    const unsigned my_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint4*)(&ring[0]) + (unsigned)(wave * NS * FPL) * 16u;
    auto request_filters = [&](int plane, int s) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        lds_dma16(rs_w4, my_base + (unsigned)(s * FPL + j * 64) * 16u, plane < planes ? w_off[j] + (unsigned)(plane * 64) : kOob);
    };
    auto turn = [&](int p, Frags& cur, Frags& next) {
      wait_loads<2 * (NS - 2 * UP)>();
#pragma unroll
      for (int u = 0; u < UP; ++u) request_filters(p + NS + u, st + u);
      st = st + UP == NS ? 0 : st + UP;
      if (p + UP < planes) fetch(p + UP, st, next);
      multiply(p, cur);
    };
    for (int p = 0; p < planes; p += 2 * UP) {
      turn(p, fa, fb);
      if (p + UP < planes) turn(p + UP, fb, fa);
    }
  }

  // ---- epilogue of the 1x1 conv: transposition through the wave's ring, then 8 consecutive channels of a pixel per lane
  LaneParams lp;
  finish_lane_params<false>(rawp, lp);
  wait_loads<0>();   // (the requests past the end of the reduction still write zeros into the ring)
  uint4* stg = my;
  const OutLoc ol{nullptr, 0, 0, 0};
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      stg[lrow * EP + 2 * q + lhalf] =
          make_uint4(as_u32(acc[tm][4 * q]), as_u32(acc[tm][4 * q + 1]), as_u32(acc[tm][4 * q + 2]), as_u32(acc[tm][4 * q + 3]));
#pragma unroll
    for (int it = 0; it < (BM < 32 ? 1 : 2); ++it) {
      const int pix = it * 16 + (lane >> 2);
      const uint4 lo = stg[pix * EP + (lane & 3) * 2], hi = stg[pix * EP + (lane & 3) * 2 + 1];
      const unsigned raw[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      const int row = tm * 32 + pix;
      const int ry = (int)fast_div((unsigned)row, g.fd_tw), rx = row - ry * g.tw;
      const int oy = oy0 + ry, ox = ox0 + rx;
      if (ry >= g.th || oy >= a.Ho || ox >= a.Wo || ech >= pw.K) continue;
      finish_store8<false, false, false>(pw, raw, (n * a.Ho + oy) * a.Wo + ox, ech, lp, ol, true);
    }
  }
}

struct DirectTile {
  int bm, wn, nw, ns, cp, occ, mr;
};
// (at stride 2 four output rows would need nine input rows in registers)
constexpr int rows_of(int stride, int mr) { return stride == 1 ? mr : 2; }
// (index, rows, waves with filters, waves, ring stages, most channels / 32, OCC, MR at stride 1)
#define RELAY_DWPW_DIRECT(X) \
  X(0, 16, 2, 4, 8, 8, 0, 2) X(1, 32, 4, 4, 8, 8, 0, 2) X(2, 32, 8, 8, 8, 8, 0, 2) X(3, 16, 1, 8, 32, 32, 0, 2) X(4, 16, 2, 8, 16, 16, 0, 2) \
  X(5, 32, 2, 8, 16, 16, 0, 2) X(6, 32, 4, 8, 8, 16, 0, 2) X(7, 32, 8, 8, 6, 16, 0, 2) X(8, 64, 8, 8, 4, 16, 0, 2) X(9, 32, 8, 8, 6, 16, 2, 4) \
  X(10, 64, 8, 8, 4, 16, 2, 4) X(11, 64, 4, 4, 4, 4, 3, 4) X(12, 64, 4, 4, 4, 4, 3, 2)
#define RELAY_DWPW_DIRECT_ENTRY(i, bm, wn, nw, ns, cp, occ, mr) {bm, wn, nw, ns, cp, occ, mr},
constexpr DirectTile kDirect[] = {RELAY_DWPW_DIRECT(RELAY_DWPW_DIRECT_ENTRY)};
constexpr int kNumDirect = sizeof(kDirect) / sizeof(kDirect[0]);

// The rectangle of at most bm pixels, a multiple of mr rows high, that covers an image with the fewest tiles; of those
// the one with the smallest input patch.
void pick_rectangle(const DwPwArgs& a, int bm, int mr, int* th, int* tw) {
  long best_tiles = -1, best_patch = 0;
  for (int h = mr; h <= bm; h += mr) {
    const int w = bm / h < a.Wo ? bm / h : a.Wo;
    if (w < 1 || (h > mr && h > a.Ho + mr - 1)) break;
    const int nx = (a.Wo + w - 1) / w, wb = (a.Wo + nx - 1) / nx;   // (as narrow as the same number of tiles allows)
    const long tiles = (long)((a.Ho + h - 1) / h) * nx;
    const long patch = (long)((h - 1) * a.stride + 3) * ((wb - 1) * a.stride + 3);
    if (best_tiles < 0 || tiles < best_tiles || (tiles == best_tiles && patch < best_patch)) {
      best_tiles = tiles;
      best_patch = patch;
      *th = h;
      *tw = wb;
    }
  }
}

DirectGeom make_geom(const DwPwArgs& a, const DirectTile& t) {
  DirectGeom g;
  const int mr = rows_of(a.stride, t.mr);
  pick_rectangle(a, t.bm, mr, &g.th, &g.tw);
  g.tiles_x = (a.Wo + g.tw - 1) / g.tw;
  g.tiles_y = (a.Ho + g.th - 1) / g.th;
  g.tiles_n = (a.pw.K + t.wn * 32 - 1) / (t.wn * 32);
  // consecutive workgroups run on one XCD: they share what is larger, the filters or the activations
  g.n_major = (size_t)a.pw.K > (size_t)a.N * a.H * a.W;
  g.log_cv = 0;
  while ((8 << g.log_cv) < a.C) ++g.log_cv;
  g.fd_x = make_fastdiv((uint32_t)g.tiles_x);
  g.fd_y = make_fastdiv((uint32_t)g.tiles_y);
  g.fd_n = make_fastdiv((uint32_t)g.tiles_n);
  g.fd_p = make_fastdiv((uint32_t)(a.N * g.tiles_y * g.tiles_x));
  g.fd_tw = make_fastdiv((uint32_t)g.tw);
  const int groups = (t.nw * 64) >> g.log_cv;
  g.nit = (g.th / mr * g.tw + groups - 1) / groups;
  return g;
}

template <int STRIDE, int BM, int WN, int NW, int NS, int CP, int OCC, int MR>
hipError_t launch_direct_one(const DwPwArgs& a, hipStream_t st) {
  const DirectArgs block{make_geom(a, DirectTile{BM, WN, NW, NS, CP, OCC, MR}), a};
  const long wgs = (long)a.N * block.g.tiles_y * block.g.tiles_x * block.g.tiles_n;
  hipLaunchKernelGGL((dwpw_fused_direct_kernel<STRIDE, BM, WN, NW, NS, CP, OCC, MR>), dim3((unsigned)wgs), dim3(64 * NW), 0, st, (int)wgs, block);
  return hipGetLastError();
}

}  // namespace

int dwpw_direct_variant_count() { return kNumDirect; }

bool dwpw_direct_supported(const DwPwArgs& a, int v) {
  if (v < 0 || v >= kNumDirect) return false;
  const DirectTile& t = kDirect[v];
  const size_t lim = 0x7fffffffu;   // 32-bit buffer offsets, 2^31 marks "out of range"
  // (a power of two of channel vectors that the threads divide into)
  return (a.stride == 1 || a.stride == 2) && a.C >= 32 && (a.C & (a.C - 1)) == 0 && a.C <= t.cp * 32 && a.C <= t.nw * 512 && (a.pw.K & 7) == 0 &&
         (size_t)a.N * a.H * a.W * a.C * 2 <= lim && (size_t)a.pw.K * a.pw.Kp * 2 <= lim;
}

// From 64 channels on, the smallest tile whose workgroups fit the chip at once: a second round of such
// workgroups repeats the whole chain, and the chunked kernel or two launches are then as fast.  (Graph-timed; two
// launches or, with a star, the chunked kernel -> this one.)  One image: 64 -> 128 at 112 x 112 / 2 6.2 -> 4.4 us, 128 at 56 x 56
// 7.4 -> 4.5, 256 at 28 x 28 7.7 -> 4.4, 512 at 14 x 14 8.7 -> 5.5, 1024 at 7 x 7 9.8 -> 7.6.  4 images: 6.8* -> 5.7, 8.4* -> 5.9,
// 8.1 -> 5.8, 8.7 -> 7.3.  32 images: 256 -> 512 at 28 x 28 / 2 12.7* -> 9.8, 512 at 14 x 14 13.7* -> 13.0, 512 -> 1024 / 2 12.1 -> 9.7.
// Two rounds: 1024 at 7 x 7, 4 images 10.5 against 14.3.
// (A tile of up to 256 channels takes 3 us behind the launch with 16 pixels x 64 channels, 5 with 32 x 256, 7 with 64 x 256;
// with 512 channels 4.1 with 16 x 32, 5.5 with 32 x 64, 7.1 with 32 x 256, 10 with 64 x 256.)
// The tiles of four-row items come before those of two where every thread has one (512 channels in 32 rows, 256 in 64), and are passed by
// where their rectangles are too many (9 rows as 4 + 4 + 1).  At stride 2, where both have items of two rows, one item's inputs in registers
// instead of two is no slower: 19 blocks 0.99 to 1.01 of the time in 32 rows (512 at 28 x 28 / 2, 16 images 10.7 and 10.6 us), 0.96 to 0.99 in 64
// (32 images 15.4 and 14.8, 256 -> 512 11.1 and 10.8).
// Up to 128 channels on both sides, beyond one round: 64 x 128 tiles, three workgroups to a CU (49 KB of LDS, 150 registers), which
// cover each other's latencies where the chunked kernel waits at its barriers.  Operands from beyond the L2, chunked* or two launches -> this:
// 64 -> 128 / 2 at 82 x 103, 11 images 11.5 -> 8.2, at 100 x 90, 16 images 15.8 -> 10.2, at 112 x 112, 32 images 24.2* -> 23.0; 128 -> 128 at
// 50 x 45, 16 images 13.7* -> 11.1, at 56 x 56, 32 images 24.0* -> 20.0, at 112 x 112 79* -> 69; 128 -> 128 / 2 at 112 x 112 47.9 -> 34.0; 64 -> 64 at
// 56 x 56 17.7* -> 14.4, at 112 x 112, 32 images 51.8* -> 48.2 (the one size of these where two launches, 47.4, are faster).  64 channels take them also within one round of 64 x 256 (3 images at 56 x 56
// 5.15 -> 4.82), 128 do not (128 -> 128 / 2 at 90 x 70, 7 images 7.3 against 7.8).
int dwpw_direct_pick(const DwPwArgs& a) {
  if (a.C < 64) return -1;
  auto one_round = [&](int v) {
    if (!dwpw_direct_supported(a, v)) return false;
    const DirectGeom g = make_geom(a, kDirect[v]);
    return (long)a.N * g.tiles_y * g.tiles_x * g.tiles_n <= 256;
  };
  const bool thin = a.C <= 128 && a.pw.K <= 128;
  const int streams = a.C > 64 ? 11 : 12;   // (four-row items where every thread has one)
  if (a.C > 256) {
    for (int v : {3, 4, 5, 6, 9, 7, 10})
      if (one_round(v)) return v;
  } else {
    for (int v : {0, 1, 2})
      if (one_round(v)) return v;
    if (thin && a.C <= 64 && dwpw_direct_supported(a, streams)) return streams;
    if (a.C == 256 && one_round(10)) return 10;
  }
  if (one_round(8)) return 8;
  return thin && dwpw_direct_supported(a, streams) ? streams : -1;
}

// Is the block faster as this launch than as two?  Not where most of the 64 rows of many workgroups are empty (images far smaller than a
// tile; the work of a workgroup is that of a full one).  917 random blocks of up to 128 channels, images of 1 to 40 a side, that two launches
// were chosen for before: up to 512 workgroups, two to a CU, one launch took 0.54 to 0.98 of the time whatever the filling; beyond, with 1 row
// filled up to 3.9 times (4096 images of 1 x 1 7.5 -> 28.2 us), 4 rows 2.2 (2048 of 2 x 2 6.6 -> 12.1), 9 rows 2.0 (1024 of 3 x 3 6.9 -> 8.4).  From 13 rows
// on at 128 channels, from 16 or, beyond one round of three to a CU, 24 at 64, whose two launches are the cheaper ones, one of 535
// was slower by more than 2 % (6 %).
bool dwpw_direct_pays(const DwPwArgs& a) {
  const int v = dwpw_direct_pick(a);
  if (v < 0 || kDirect[v].occ != 3) return v >= 0;
  const DirectGeom g = make_geom(a, kDirect[v]);
  const long tiles = (long)a.N * g.tiles_y * g.tiles_x;
  const int rows = a.C > 64 ? 13 : tiles <= 768 ? 16 : 24;
  return tiles <= 512 || (long)a.N * a.Ho * a.Wo >= rows * tiles;
}

hipError_t launch_dwpw_direct(const DwPwArgs& a, int v, hipStream_t st) {
  switch (v) {
#define RELAY_DWPW_DIRECT_CASE(i, bm, wn, nw, ns, cp, occ, mr) \
  case i: return a.stride == 1 ? launch_direct_one<1, bm, wn, nw, ns, cp, occ, mr>(a, st) : launch_direct_one<2, bm, wn, nw, ns, cp, occ, 2>(a, st);
    RELAY_DWPW_DIRECT(RELAY_DWPW_DIRECT_CASE)
    default: return hipErrorInvalidValue;
  }
}

void dwpw_direct_kernel_name(const DwPwArgs& a, int v, char* buf, size_t len) {
  const DirectTile& t = kDirect[v];
  snprintf(buf, len, "dwpw_fused_direct_kernel<%d, %d, %d, %d, %d, %d, %d, %d>", a.stride, t.bm, t.wn, t.nw, t.ns, t.cp, t.occ,
           rows_of(a.stride, t.mr));
}

}  // namespace relay
