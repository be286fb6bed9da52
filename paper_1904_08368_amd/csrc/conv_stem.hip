// First-layer conv2d of at most four channels read from the NCHW image, with the 3x3 / stride 2 / pad 1 max pool behind it if
// there is one: one launch instead of a padded four-channel copy of the image, the conv over that copy and the pool
// (paper Section 4.1: same fused primitive functions, the layout change of Section 5.3 folded into their first loads).
//
// A workgroup owns a rectangle of TYC x TXC conv outputs (with a pool: the outputs under TYC/2 x TXC/2 pooled ones) and BN
// output channels.  The filters go straight to LDS; the image patch goes through registers, where the channel planes are
// interleaved to four channels per pixel, so that a filter row is a run of 16-byte operands along a patch row, as in the pooled
// tile of the staged kernel.  The finished tile takes the place of both, and leaves it in whole 8-channel vectors.  Sums per
// output: filter row by filter row, in one accumulator, or (MANY, the tiles for few outputs) in runs of per_run rows whose sums are
// added up in order: two, or as many as the waves of the small-tile kernel where the conv over the padded copy runs there, since
// a run's rounding error grows with its length (rms of the fp32 errors against 64 bits, 8 x 8 windows of 4 channels: one run 1.48e-7, two
// 1.14e-7, four 9.9e-8, which is also that of the small-tile kernel's four waves).
//
// Of the small tiles for few outputs one or two waves' worth of matrix work stand beside a patch of several hundred pixels, whose loads and
// deposits were half of the launch: HW more waves of the workgroup take their share of those and of the stores, and idle in between.
//
// What bounds it: latency -- the patch, then the stores -- hidden by three or four workgroups per CU.  (Workgroups that walk over
// several tiles, filters kept and the next patch in registers meanwhile, have room for two: 31.6 us against 25.4 for ResNet-18's
// first layer at batch 32; the padded copy, conv and pool apart take 6.2 + 22.3.)
#include <cstdio>

#include <atomic>

#include "dma_common.hpp"

namespace relay {
namespace {

template <bool IS_I8, int WM, int WN, int TM, int TN, int HW, int TYC, int TXC, int KS, bool MANY, bool POOL, bool PAIRS, int NI>
__global__ __launch_bounds__(64 * (WM * WN + HW), TM * TN > 1 || NI > 10 ? 3 : 4) void conv_stem_kernel(const int tiles, const StemArgs g) {
  constexpr int MW = WM * WN, NW = MW + HW, NT = 64 * NW, ES = IS_I8 ? 1 : 2, VE = 16 / ES, PXB = 4 * ES;
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32, WTM = TM * 32, WTN = TN * 32;
  constexpr int OPITCH = BN * ES + 8;   // (8 bytes spread the accumulator layout's writes over the banks)
  constexpr int FB = BN / 16;           // 1 KiB filter blocks of a filter row
  static_assert(TYC * TXC <= BM && (!POOL || (TYC % 2 == 1 && TXC % 2 == 1)), "");
  typedef typename Mma<IS_I8>::acc_t acc_t;
  typedef typename std::conditional<IS_I8, unsigned short, unsigned>::type pair_t;
  typedef typename std::conditional<IS_I8, unsigned char, unsigned short>::type one_t;
  const ConvArgs& a = g.a;
  extern __shared__ uint4 lds[];
  char* patch = reinterpret_cast<char*>(lds + a.R * BN * BKV);
  char* out = reinterpret_cast<char*>(lds);   // (over filters and patch, when nobody reads them any more)
  float* cst = reinterpret_cast<float*>(out + g.cst_at);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave % WM, wn = wave / WM;
  // (one batch of scalar loads; the workgroup's number passes through, so that arithmetic on it stays behind all of them)
  int tile = TM * TN > 1 ? xcd_remap((int)blockIdx.x, tiles) : (int)blockIdx.x;
  const void* ptr_w = a.w;
  asm volatile("" : "+s"(tile), "+s"(ptr_w) : "s"(a.x), "s"(a.y), "s"(a.bias), "s"(a.scale), "s"(a.shift), "s"(a.qbias), "s"(a.N), "s"(a.H), "s"(a.W),
               "s"(a.C), "s"(a.K), "s"(a.R), "s"(a.sh), "s"(a.sw), "s"(a.ph), "s"(a.pw), "s"(a.Ho), "s"(a.Wo), "s"(a.Kp), "s"(a.flags),
               "s"(g.y_pooled), "s"(g.Hp), "s"(g.Wp), "s"(g.per_run), "s"(g.tiles_img), "s"(g.tiles_row), "s"(g.pitch), "s"(g.cst_at),
               "s"(g.per_row), "s"(g.items), "s"(g.fd_img.mul), "s"(g.fd_img.shift), "s"(g.fd_row.mul), "s"(g.fd_row.shift), "s"(g.fd_items.mul),
               "s"(g.fd_items.shift));
  const int n0 = blockIdx.y * BN;

  // ---- filters and constants, once
  {
    const intx4 rs_w = make_rsrc(ptr_w, (unsigned)((size_t)a.K * a.Kp * ES));
    const unsigned base = (unsigned)(size_t)(__attribute__((address_space(3))) uint4*)(&lds[0]);
    const int srow = lane >> 2, sphys = lane & 3;
    for (int b = wave; b < a.R * FB; b += NW) {
      const int r = b / FB, row = (b % FB) * 16 + srow, ch = n0 + row;
      lds_dma16(rs_w, base + (unsigned)b * 1024u, ch < a.K ? (unsigned)((ch * a.Kp + r * (64 / ES) + (sphys ^ lds_swizzle(row)) * VE) * ES) : kOob);
    }
    if (tid < BN) {
      const int c = min(n0 + tid, a.K - 1);
      if constexpr (IS_I8) {
        cst[tid] = __builtin_bit_cast(float, (a.flags & F_BIAS) ? a.qbias[c] : 0);
      } else {
        const float sc = (a.flags & F_BN) ? a.scale[c] : 1.f, sf = (a.flags & F_BN) ? a.shift[c] : 0.f;
        cst[tid] = sc;
        cst[BN + tid] = ((a.flags & F_BIAS) ? a.bias[c] : 0.f) * sc + sf;
      }
    }
  }

  // ---- the tile: image, first conv row and column
  // (large tiles in the order of the other kernels, a run of them to an XCD: neighbouring patches share their lines of the image in its L2,
  //  and the layer behind finds these outputs in the L2 of the XCD that reads them.  First layer and the one behind it, ResNet-18 at
  //  batch 32 41.6 -> 38.7 us, int8 at batch 16 19.1 -> 17.9, MobileNet-v1 at batch 11 15.8 -> 14.1.  In a few small tiles the arithmetic
  //  costs what it gives: deep Q-network at batch 1 17.5 against 17.6.)
  const int t_n = (int)fast_div((uint32_t)tile, g.fd_img), t_rem = tile - t_n * g.tiles_img;
  const int t_ty = (int)fast_div((uint32_t)t_rem, g.fd_row), t_tx = t_rem - t_ty * g.tiles_row;
  const int c_y = POOL ? t_ty * (TYC - 1) - 1 : t_ty * TYC, c_x = POOL ? t_tx * (TXC - 1) - 1 : t_tx * TXC;
  const int iy0 = c_y * a.sh - a.ph, ix0 = c_x * a.sw - a.pw;

  // ---- its patch of the image: item i is pixel (or, where the width is even, the aligned pixel pair) i % per_row of row i / per_row.
  //      All loads first, from clamped places and without a use between them: one latency for all.
  unsigned v[NI][4];
  unsigned inside = 0;   // bit j: item j lies in the image
  const int col0 = PAIRS ? (ix0 & ~1) - ix0 : 0;   // patch column of a row's first item
  auto fetch = [&](auto nc_tag) {
    constexpr int NC = decltype(nc_tag)::value;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int i = min(j * NT + tid, g.items - 1);
      const int row = (int)fast_div((uint32_t)i, g.fd_items), p = i - row * g.per_row;
      const int iy = iy0 + row, gx = ix0 + col0 + (PAIRS ? 2 * p : p);
      if ((unsigned)iy < (unsigned)a.H && (unsigned)gx < (unsigned)a.W) inside |= 1u << j;   // (a pair is inside or outside as a whole)
      const unsigned at = ((unsigned)(t_n * a.C * a.H) + (unsigned)min(max(iy, 0), a.H - 1)) * (unsigned)a.W + (unsigned)min(max(gx, 0), PAIRS ? a.W - 2 : a.W - 1);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        v[j][c] = 0;
        if (c < NC) {
          const one_t* px = static_cast<const one_t*>(a.x) + (size_t)(at + (unsigned)(min(c, a.C - 1) * a.H) * (unsigned)a.W);
          v[j][c] = PAIRS ? (unsigned)*reinterpret_cast<const pair_t*>(px) : (unsigned)*px;
        }
      }
    }
  };
  auto pixel = [&](const unsigned (&w)[4], int shift) {   // the pixel at bit `shift` of the channel words
    if constexpr (IS_I8) {
      return ((w[0] >> shift) & 0xffu) | (((w[1] >> shift) & 0xffu) << 8) | (((w[2] >> shift) & 0xffu) << 16) | (((w[3] >> shift) & 0xffu) << 24);
    } else {
      return make_uint2(((w[0] >> shift) & 0xffffu) | ((w[1] >> shift) << 16), ((w[2] >> shift) & 0xffffu) | ((w[3] >> shift) << 16));
    }
  };
  auto deposit = [&](auto nc_tag) {
    constexpr int NC = decltype(nc_tag)::value;
    typedef typename std::conditional<IS_I8, unsigned, uint2>::type px_t;
    px_t* dst = reinterpret_cast<px_t*>(patch);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int i = j * NT + tid;
#pragma unroll
      for (int c = 0; c < NC; ++c) v[j][c] = ((inside >> j) & 1u) && c < a.C ? v[j][c] : 0u;
      if (i < g.items) {
        const int row = (int)fast_div((uint32_t)i, g.fd_items), p = i - row * g.per_row;
        const int col = col0 + (PAIRS ? 2 * p : p);
        if (col >= 0 && col < g.pitch) dst[row * g.pitch + col] = pixel(v[j], 0);
        if (PAIRS && col + 1 < g.pitch) dst[row * g.pitch + col + 1] = pixel(v[j], 8 * ES);
      }
    }
  };
  if (a.C == 4) {   // (uniform)
    fetch(std::integral_constant<int, 4>{});
    deposit(std::integral_constant<int, 4>{});
  } else {
    fetch(std::integral_constant<int, 3>{});
    deposit(std::integral_constant<int, 3>{});
  }

  const int lrow = lane & 31, lhalf = lane >> 5;
  const char* xs[TM];   // this lane's pixel of each block, at filter row 0
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int row = wm * WTM + tm * 32 + lrow, dy = min(row / TXC, TYC - 1), dx = row - (row / TXC) * TXC;   // (rows past the rectangle are no outputs)
    xs[tm] = patch + (dy * a.sh * g.pitch + dx * a.sw) * PXB + lhalf * 16;
  }
  uint4 wf[2][KS][TN], xf[2][KS][TM];
  // (an even fp16 stride: a pixel pair is a 16-byte vector; halves 16 bytes apart from lane to lane cost twice the LDS clocks)
  const bool wide = !IS_I8 && a.sw % 2 == 0;
  auto operands = [&](int r, int b, auto wide_tag) {
#pragma unroll
    for (int k = 0; k < KS; ++k) {
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) wf[b][k][tn] = lds[r * (BN * BKV) + lds_slot(wn * WTN + tn * 32 + lrow, 2 * k + lhalf)];
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) {
        if constexpr (decltype(wide_tag)::value) {
          xf[b][k][tm] = *reinterpret_cast<const uint4*>(xs[tm] + r * g.pitch * PXB + k * 32);
          continue;
        }
        const uint2* at = reinterpret_cast<const uint2*>(xs[tm] + r * g.pitch * PXB + k * 32);
        const uint2 lo = at[0], hi = at[1];
        xf[b][k][tm] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
    }
  };
  const ClipBounds qb = clip_bounds(a, a.flags & F_RELU);

  auto meet = [&]() {   // every wave's LDS reads and writes are done
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  wait_loads<0>();   // the filters
  meet();
  const bool multiplies = HW == 0 || wave < MW;   // (uniform; the others have brought their share and store theirs)
  acc_t acc[TN][TM];
  auto clear = [&]() {
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[tn][tm][e] = 0;
  };
  clear();
  auto multiply = [&](int b) {
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = Mma<IS_I8>::mma(wf[b][k][tn], xf[b][k][tm], acc[tn][tm]);
  };
  acc_t sum[MANY ? TN : 1][MANY ? TM : 1];   // ... of the runs behind
  auto end_run = [&]() {
#pragma unroll
    for (int tn = 0; tn < (MANY ? TN : 0); ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[tn][tm][e] += acc[tn][tm][e];
    clear();
  };
  if constexpr (MANY) {
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) sum[tn][tm] = acc[tn][tm];
  }
  auto reduce_rows = [&](auto wide_tag) {
    operands(0, 0, wide_tag);
    int left = g.per_run;   // rows until the run ends
    for (int r = 0; r < a.R; r += 2) {
      if (r + 1 < a.R) operands(r + 1, 1, wide_tag);
      multiply(0);
      if (MANY && --left == 0) {
        end_run();
        left = g.per_run;
      }
      if (r + 2 < a.R) operands(r + 2, 0, wide_tag);
      if (r + 1 < a.R) multiply(1);
      if (MANY && --left == 0) {   // (behind an odd number of rows it ends a run of nothing)
        end_run();
        left = g.per_run;
      }
    }
  };
  if (multiplies) {
    if (wide) reduce_rows(std::integral_constant<bool, !IS_I8>{});
    else reduce_rows(std::false_type{});
  }
  if constexpr (MANY) {
    end_run();
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = sum[tn][tm];
  }

  meet();   // (the tile takes the place of filters and patch)
  // ---- finish the accumulators where they are (element e of a block: pixel lane % 32, channel 8 (e / 4) + 4 (lane / 32) +
  //      e % 4), narrow, and collect the tile in LDS as [output][channel]
  auto narrow = [&](auto sat) {
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cb = wn * WTN + tn * 32 + 8 * q + 4 * lhalf;
        const float4 c0 = *reinterpret_cast<const float4*>(cst + cb);
        const float4 c1 = IS_I8 ? c0 : *reinterpret_cast<const float4*>(cst + BN + cb);
        const float m4[4] = {c0.x, c0.y, c0.z, c0.w}, a4[4] = {c1.x, c1.y, c1.z, c1.w};
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
          char* dst = out + (wm * WTM + tm * 32 + lrow) * OPITCH + cb * ES;
          if constexpr (IS_I8) {
            int c[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              c[e] = shift_round_clip<decltype(sat)::value>(acc[tn][tm][4 * q + e] + __builtin_bit_cast(int, m4[e]), a, qb);
            *reinterpret_cast<unsigned*>(dst) = pack_low_bytes(c[0], c[1], c[2], c[3]);
          } else {
            typedef float float2v __attribute__((ext_vector_type(2)));
            typedef _Float16 half2v __attribute__((ext_vector_type(2)));
            unsigned hw[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              // rounded to fp32 before it is narrowed, and relu as a packed maximum on the narrowed pair: as in the other kernels
              float f0 = acc[tn][tm][4 * q + 2 * e] * m4[2 * e] + a4[2 * e];
              float f1 = acc[tn][tm][4 * q + 2 * e + 1] * m4[2 * e + 1] + a4[2 * e + 1];
              asm("" : "+v"(f0), "+v"(f1));
              const float2v f = {f0, f1};
              half2v h = __builtin_convertvector(f, half2v);
              if (a.flags & F_RELU) h = __builtin_elementwise_max(h, half2v{(_Float16)0, (_Float16)0});
              hw[e] = __builtin_bit_cast(unsigned, h);
            }
            *reinterpret_cast<uint2*>(dst) = make_uint2(hw[0], hw[1]);
          }
        }
      }
  };
  if (multiplies) {
    if (!IS_I8 || qb.sat_ok) narrow(std::true_type{});
    else narrow(std::false_type{});
  }
  meet();

  // ---- whole 8-channel vectors to memory
  constexpr int GROUPS = BN / 8;
  auto vec = [&](int row, int gch) {
    const char* src = out + row * OPITCH + gch * 8 * ES;   // (8-byte aligned)
    uint4 o = make_uint4(0u, 0u, 0u, 0u);
    const uint2 lo = *reinterpret_cast<const uint2*>(src);
    o.x = lo.x;
    o.y = lo.y;
    if constexpr (!IS_I8) {
      const uint2 hi = *reinterpret_cast<const uint2*>(src + 8);
      o.z = hi.x;
      o.w = hi.y;
    }
    return o;
  };
  auto store = [&](void* y, size_t o, const uint4& u) {
    if constexpr (IS_I8) *reinterpret_cast<uint2*>(static_cast<int8_t*>(y) + o) = make_uint2(u.x, u.y);
    else *reinterpret_cast<uint4*>(static_cast<_Float16*>(y) + o) = u;
  };
  if (a.y) {   // (uniform) the conv outputs; with a pool those no other tile has as its own
    constexpr int D = POOL ? 1 : 0, OY = TYC - D, OX = TXC - D;
    for (int i = tid; i < OY * OX * GROUPS; i += NT) {
      const int px = i / GROUPS, gch = i - px * GROUPS, dy = px / OX + D, dx = px - (px / OX) * OX + D;
      const int oy = c_y + dy, ox = c_x + dx, ch = n0 + gch * 8;
      if (oy < a.Ho && ox < a.Wo && ch < a.K) store(a.y, ((size_t)(unsigned)(t_n * a.Ho + oy) * a.Wo + ox) * a.K + ch, vec(dy * TXC + dx, gch));
    }
  }
  if constexpr (POOL) {
    constexpr int PY = TYC / 2, PX = TXC / 2;
    for (int i = tid; i < PY * PX * GROUPS; i += NT) {
      const int pp = i / GROUPS, gch = i - pp * GROUPS, py = pp / PX, px = pp - py * PX;
      const int oy = (c_y + 1) / 2 + py, ox = (c_x + 1) / 2 + px, ch = n0 + gch * 8;
      if (oy >= g.Hp || ox >= g.Wp || ch >= a.K) continue;
      // (a window row or column outside the image: its centre again, which leaves the maximum as it is)
      const int rr[3] = {oy == 0 ? 1 : 0, 1, 2 * oy + 1 < a.Ho ? 2 : 1}, ss[3] = {ox == 0 ? 1 : 0, 1, 2 * ox + 1 < a.Wo ? 2 : 1};
      typedef _Float16 half2v __attribute__((ext_vector_type(2)));
      typedef short short2v __attribute__((ext_vector_type(2)));
      uint4 best;
      unsigned ev[2], od[2];  // int8: the even and the odd bytes of a word as the high bytes of 16-bit lanes
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const uint4 u = vec((2 * py + rr[r]) * TXC + 2 * px + ss[s], gch);
          if constexpr (IS_I8) {
            const unsigned uw[2] = {u.x, u.y};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const unsigned e = (uw[h] << 8) & 0xff00ff00u, o = uw[h] & 0xff00ff00u;
              if (r == 0 && s == 0) {
                ev[h] = e;
                od[h] = o;
              } else {
                ev[h] = __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(short2v, ev[h]), __builtin_bit_cast(short2v, e)));
                od[h] = __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(short2v, od[h]), __builtin_bit_cast(short2v, o)));
              }
            }
          } else if (r == 0 && s == 0) {
            best = u;
          } else {
            unsigned bw[4] = {best.x, best.y, best.z, best.w};
            const unsigned uw[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int h = 0; h < 4; ++h)
              bw[h] = __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(half2v, bw[h]), __builtin_bit_cast(half2v, uw[h])));
            best = make_uint4(bw[0], bw[1], bw[2], bw[3]);
          }
        }
      if constexpr (IS_I8) best = make_uint4((ev[0] >> 8) | od[0], (ev[1] >> 8) | od[1], 0u, 0u);
      store(g.y_pooled, ((size_t)(unsigned)(t_n * g.Hp + oy) * g.Wp + ox) * a.K + ch, best);
    }
  }
}

struct StemTile {
  int wm, wn, tm, tn, hw, tyc, txc;
  constexpr int threads() const { return 64 * (wm * wn + hw); }
  constexpr int multiplying() const { return 64 * wm * wn; }
  constexpr int bm() const { return wm * tm * 32; }
  constexpr int bn() const { return wn * tn * 32; }
};
// large and small, 64 and 32 channels, without and with a pool; the small ones without a pool once more with helpers (must match launch_stem)
constexpr StemTile kStem[] = {
    {4, 1, 2, 2, 0, 16, 16}, {4, 1, 2, 1, 0, 16, 16}, {2, 2, 1, 1, 0, 8, 8}, {2, 1, 1, 1, 0, 8, 8}, {4, 1, 2, 2, 0, 15, 17}, {2, 2, 1, 1, 0, 7, 9},
    {2, 2, 1, 1, 4, 8, 8}, {2, 1, 1, 1, 6, 8, 8},
};

int ksteps(const ConvArgs& a, bool is_i8) { return is_i8 ? (a.S <= 8 ? 1 : 0) : (a.S <= 4 ? 1 : a.S <= 8 ? 2 : 0); }

// fills what the tile needs; false: it does not take the layer
bool stem_geom(StemArgs& g, bool is_i8, int t, size_t& lds_bytes, int& items_per_thread) {
  const StemTile& s = kStem[t];
  const ConvArgs& a = g.a;
  const int es = is_i8 ? 1 : 2, ks = ksteps(a, is_i8);
  const bool pool = t == 4 || t == 5;
  if (ks == 0 || (pool && !is_i8 && ks != 2) || (is_i8 && (t == 1 || t == 3 || t == 7))) return false;
  g.pitch = ((s.txc - 1) * a.sw + (is_i8 ? 8 : 4) * ks + 1) / 2 * 2;
  const int rows = (s.tyc - 1) * a.sh + a.R;
  g.patch_bytes = (rows * g.pitch * 4 * es + 15) / 16 * 16;
  g.pairs = a.W % 2 == 0;
  g.per_row = g.pairs ? g.pitch / 2 + 1 : g.pitch;
  g.items = rows * g.per_row;
  items_per_thread = (g.items + s.threads() - 1) / s.threads();
  const int cy = pool ? s.tyc - 1 : s.tyc, cx = pool ? s.txc - 1 : s.txc;
  g.tiles_row = (a.Wo + cx - 1) / cx;
  g.tiles_img = ((a.Ho + cy - 1) / cy) * g.tiles_row;
  // (a launch holds fewer than 2^32 threads, and 65535 tiles of channels)
  if ((long)a.N * g.tiles_img * s.threads() >= (1L << 32) || (a.K + s.bn() - 1) / s.bn() > 65535) return false;
  g.tiles = a.N * g.tiles_img;
  g.fd_img = make_fastdiv((uint32_t)g.tiles_img);
  g.fd_row = make_fastdiv((uint32_t)g.tiles_row);
  g.fd_items = make_fastdiv((uint32_t)g.per_row);
  const int in = a.R * s.bn() * 64 + g.patch_bytes, out = s.bm() * (s.bn() * es + 8);
  g.cst_at = ((in > out ? in : out) + 15) / 16 * 16;
  lds_bytes = (size_t)g.cst_at + 2 * (size_t)s.bn() * 4;
  return items_per_thread <= (g.pairs ? 10 : 20) && lds_bytes <= 160 * 1024;
}

template <bool IS_I8, int WM, int WN, int TM, int TN, int HW, int TYC, int TXC, int KS, bool MANY, bool POOL, bool PAIRS, int NI>
hipError_t launch_stem_items(const StemArgs& g, size_t lds_bytes, hipStream_t st) {
  auto kern = conv_stem_kernel<IS_I8, WM, WN, TM, TN, HW, TYC, TXC, KS, MANY, POOL, PAIRS, NI>;
  static std::atomic<bool> raised{false};  // dynamic LDS above the default limit has to be asked for once per kernel
  if (!raised.load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    raised.store(true, std::memory_order_release);
  }
  constexpr int BN = WN * TN * 32;
  hipLaunchKernelGGL(kern, dim3(g.tiles, (g.a.K + BN - 1) / BN), dim3(64 * (WM * WN + HW)), lds_bytes, st, g.tiles, g);
  return hipGetLastError();
}

template <bool IS_I8, int WM, int WN, int TM, int TN, int HW, int TYC, int TXC, int KS, bool MANY, bool POOL>
hipError_t launch_stem_one(const StemArgs& g, size_t lds, int items, hipStream_t st) {
  if (g.pairs)
    return items <= 3 ? launch_stem_items<IS_I8, WM, WN, TM, TN, HW, TYC, TXC, KS, MANY, POOL, true, 3>(g, lds, st)
                      : launch_stem_items<IS_I8, WM, WN, TM, TN, HW, TYC, TXC, KS, MANY, POOL, true, 10>(g, lds, st);
  return items <= 6 ? launch_stem_items<IS_I8, WM, WN, TM, TN, HW, TYC, TXC, KS, MANY, POOL, false, 6>(g, lds, st)
                    : launch_stem_items<IS_I8, WM, WN, TM, TN, HW, TYC, TXC, KS, MANY, POOL, false, 20>(g, lds, st);
}

template <bool IS_I8, int KS>
hipError_t launch_stem_plain(const StemArgs& g, int t, size_t lds, int items, hipStream_t st) {
  if (t == 0) return launch_stem_one<IS_I8, 4, 1, 2, 2, 0, 16, 16, KS, false, false>(g, lds, items, st);
  if (t == 2) return launch_stem_one<IS_I8, 2, 2, 1, 1, 0, 8, 8, KS, true, false>(g, lds, items, st);
  if (t == 6) return launch_stem_one<IS_I8, 2, 2, 1, 1, 4, 8, 8, KS, true, false>(g, lds, items, st);
  if constexpr (!IS_I8) {
    if (t == 1) return launch_stem_one<false, 4, 1, 2, 1, 0, 16, 16, KS, false, false>(g, lds, items, st);
    if (t == 3) return launch_stem_one<false, 2, 1, 1, 1, 0, 8, 8, KS, true, false>(g, lds, items, st);
    if (t == 7) return launch_stem_one<false, 2, 1, 1, 1, 6, 8, 8, KS, true, false>(g, lds, items, st);
  }
  return hipErrorInvalidValue;
}

int stem_pick(StemArgs& g, bool is_i8, bool pool, size_t& lds, int& items) {
  const bool thin = !is_i8 && g.a.K <= 32 && !pool;
  const int large = pool ? 4 : thin ? 1 : 0, small = pool ? 5 : thin ? 3 : 2;
  const long tn = (g.a.K + kStem[large].bn() - 1) / kStem[large].bn();
  // Small tiles until the large ones occupy half the chip.  In networks, the copy, the conv (and the pool) apart / this launch: 7x7 / 2 with
  // pool, batch 1 fp16 9.6 / 7.6 us, int8 8.5 / 5.2, int8 batch 16 18.7 / 13.8, fp16 batch 7 of 197 x 251 18.9 / 12.6, batch 32 28.5 /
  // 25.4; 3x3 / 2 of 163 x 206, batch 11 11.2 / 7.1; 3x3 of 224 x 224, batch 32 71.1 / 57.0; 8x8 / 4 of one frame 5.7 / 5.7 and a launch less.
  // Also where the conv over the padded copy sums in several runs, whatever their number.
  const bool fits = stem_geom(g, is_i8, large, lds, items);
  if (fits && g.runs <= 1 && g.tiles * tn >= 128) return large;
  if (!stem_geom(g, is_i8, small, lds, items)) return -1;
  const int runs = g.runs > 2 ? g.runs : 2;
  g.per_run = (g.a.R + runs - 1) / runs;
  // With helpers where the chip holds all workgroups at once anyway, two to a CU: 8x8 / 4 of one frame 6.2 -> 4.7 us, of 32 7.2 -> 5.6; 7x7 / 2 of
  // 120 x 84 to 64 channels 5.4 -> 5.0, 3x3 of 4 60 x 84 5.1 either way.  The pooled tile gains 7 % up to one workgroup per CU and loses
  // 3 to 13 % beyond (its patch is two loads a thread as it is).
  const int helped = small == 2 ? 6 : 7;
  const long tiles = (long)g.tiles * ((g.a.K + kStem[small].bn() - 1) / kStem[small].bn());
  return !pool && tiles <= 512 && stem_geom(g, is_i8, helped, lds, items) ? helped : small;
}

}  // namespace

bool conv_stem_supported(const StemArgs& s, bool is_i8, bool pool) {
  StemArgs g = s;
  size_t lds;
  int items;
  const ConvArgs& a = g.a;
  if (a.C > 4 || a.K % 8 || (a.flags & F_RES) || (is_i8 && a.sw % 2) || a.W < 2) return false;
  if ((size_t)a.N * a.C * a.H * a.W >= (1u << 31) || (size_t)a.N * a.Ho * a.Wo >= (1u << 31) || (size_t)a.K * a.Kp >= (1u << 30)) return false;
  return stem_pick(g, is_i8, pool, lds, items) >= 0;
}

// One launch, or the padded copy, the conv (and the pool) apart?  Apart where every channel tile reads a large patch anew (a stride of
// four, more than 16 loads of four channels for each thread between them: 3 x 3 / 4 of 20 images 198 x 31 to 128 channels 11.4 us, apart
// 8.9; 8 x 8 / 4 of 40 71 x 202 with pool 20.7, 17.4), and where the two waves of the smallest tile read a large patch pixel by
// pixel (an odd width: 8 x 8 / 4 of 7 115 x 35 to 32 channels 7.3, 6.0).  Of 419 random first layers one launch was slower by 3 % or
// more on 18; with this rule 7 were, by 3 to 8 % and one by 12 %, and all together take 0.80 of the time.  With helpers none of 215 others
// that the rule takes is slower, and one of the 5 that it refuses would be faster (by 3 %).
bool conv_stem_pays(const StemArgs& s, bool is_i8, bool pool) {
  StemArgs g = s;
  size_t lds;
  int items;
  const int t = conv_stem_supported(s, is_i8, pool) ? stem_pick(g, is_i8, pool, lds, items) : -1;
  if (t < 0) return false;
  const int tn = (g.a.K + kStem[t].bn() - 1) / kStem[t].bn();
  items = (g.items + kStem[t].multiplying() - 1) / kStem[t].multiplying();   // (as without helpers)
  return !(tn > 1 && items * tn > 16) && !((t == 3 || t == 7) && !g.pairs && items >= 8);
}

hipError_t launch_conv_stem(const StemArgs& s, bool is_i8, bool pool, hipStream_t st) {
  StemArgs g = s;
  size_t lds;
  int items;
  const int t = stem_pick(g, is_i8, pool, lds, items);
  if (t == 4) return is_i8 ? launch_stem_one<true, 4, 1, 2, 2, 0, 15, 17, 1, false, true>(g, lds, items, st) : launch_stem_one<false, 4, 1, 2, 2, 0, 15, 17, 2, false, true>(g, lds, items, st);
  if (t == 5) return is_i8 ? launch_stem_one<true, 2, 2, 1, 1, 0, 7, 9, 1, true, true>(g, lds, items, st) : launch_stem_one<false, 2, 2, 1, 1, 0, 7, 9, 2, true, true>(g, lds, items, st);
  if (t < 0) return hipErrorInvalidValue;
  if (is_i8) return launch_stem_plain<true, 1>(g, t, lds, items, st);
  return ksteps(g.a, false) == 1 ? launch_stem_plain<false, 1>(g, t, lds, items, st) : launch_stem_plain<false, 2>(g, t, lds, items, st);
}

}  // namespace relay
