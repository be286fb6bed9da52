// The two 3x3 convs of a residual block as one launch, for blocks of 64 channels on few pixels (small batches).
//
// At batch 1 such a conv is 3.9 us of kernel and another 0.6 until the next one starts, of which its matrix instructions are 0.3: a chain of
// launch, argument fetch, first loads, reduction, store.  Here a workgroup computes a 4 x 8 rectangle of the block's outputs from the block's
// input: the 6 x 10 outputs of the first conv under it (60 of 64 rows; twice the work of that conv, which is the lesser part), narrowed to
// LDS as the second conv's input, and stored too, the rectangle's own ones, because the first conv's tensor belongs to the caller.  The input patch and the
// first conv's filters (72 KB in fp16) are requested at once, in the order of use, and the reduction follows them tap by tap; the
// second conv's are requested between its groups of taps.
// Bound: one wave a SIMD that issues, waits for LDS and multiplies.  Cycles of an fp16 workgroup (int8), 11.5 K (8.5 K) in all: 2.0 K (1.1 K) for the first
// requests, 4.5 K (2.3 K) for the first reduction, 1.0 K (1.7 K) for its tail, 2.8 K (1.6 K) for the second, 1.0 K (1.3 K) for that tail.  With all
// filters requested ahead of the first tap and operands read where they are multiplied it was 14.1 K (10.8 K).
// Measured: a block of one image of 56 x 56 called eagerly 14.6 -> 10.3 us (two calls instead of three), ResNet-18 at batch 1 77.2 -> 75.1, int8 65.5 ->
// 61.2; the block alone at the rule that chooses (api.cpp).
// The sums are grouped as igemm_small_kernel groups them (four waves over nine taps there: runs of three taps, added in order) and the
// tails are its tails, so both tensors are those of the two launches bit for bit.
#include <type_traits>

#include "dma_common.hpp"

namespace relay {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kChannels = 64, kTh = 4, kTw = 8;                       // outputs of a workgroup
constexpr int kMw = kTw + 2, kMid = (kTh + 2) * kMw;                  // first conv's outputs under them
constexpr int kIw = kTw + 4, kIn = (kTh + 4) * kIw;                   // input pixels under those

struct BlockArgs {
  int N, H, W, Kp;
  int tiles_row, tiles_img;
  FastDiv fd_img, fd_row;
  const void* x;
  const void* w[2];
  void* y[2];              // the first conv's outputs, the block's
  const void* scale[2];
  const void* shift[2];
  const void* bias[2];     // fp16: float, int8: int32
  unsigned flags[2];
  int lshift, rshift[2], round_add[2], clip_lo, clip_hi;   // int8: the quantized tails
};

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

template <bool IS_I8>
__global__ __launch_bounds__(256, IS_I8 ? 2 : 1) void conv_block_kernel(const int tiles, const BlockArgs g) {
  constexpr int ES = IS_I8 ? 1 : 2, PL = ES;             // planes of 64 bytes that a pixel or a filter tap has
  constexpr int WT = PL * kChannels * BKV;               // slots of a tap's filters
  constexpr int IROWS = 96, NB = PL * IROWS / 16, NI = (NB + 3) / 4;   // rows of an input plane, its blocks of 16 rows, loads of a wave
  constexpr int NA = IS_I8 ? 1 : 3;                      // runs of taps with a sum of their own
  typedef typename Mma16<IS_I8>::acc_t acc_t;
  static_assert(kIn <= IROWS && kMid <= 64, "the patches fit their rows");
  static_assert(2 + NI + 9 * PL <= 63 && 12 * PL <= 63, "vmcnt is a 6-bit counter");
  // filters of the first conv, of the second, input patch; behind the first reduction the first conv's outputs, and the block's on
  // their way out, take the place of the first filters
  __shared__ uint4 lds[18 * WT + PL * IROWS * BKV];
  __shared__ __align__(16) float cst[6 * kChannels];                   // scale, shift, bias of the first conv, then of the second (int8: bias alone)

  int tile = xcd_remap((int)blockIdx.x, tiles);
  const void* ptr_x = g.x;
  const void* ptr_w0 = g.w[0];
  const void* ptr_w1 = g.w[1];
#define RELAY_ASKED                                                                                                                        \
  "s"(g.N), "s"(g.H), "s"(g.W), "s"(g.Kp), "s"(g.tiles_row), "s"(g.tiles_img), "s"(g.fd_img.mul), "s"(g.fd_img.shift), "s"(g.fd_row.mul),  \
      "s"(g.fd_row.shift), "s"(g.y[0]), "s"(g.y[1]), "s"(g.bias[0]), "s"(g.bias[1]), "s"(g.flags[0]), "s"(g.flags[1])
  if constexpr (IS_I8)
    asm volatile("" : "+s"(tile), "+s"(ptr_x), "+s"(ptr_w0), "+s"(ptr_w1) : RELAY_ASKED, "s"(g.lshift), "s"(g.rshift[0]), "s"(g.rshift[1]),
                 "s"(g.round_add[0]), "s"(g.round_add[1]), "s"(g.clip_lo), "s"(g.clip_hi));
  else
    asm volatile("" : "+s"(tile), "+s"(ptr_x), "+s"(ptr_w0), "+s"(ptr_w1) : RELAY_ASKED, "s"(g.scale[0]), "s"(g.scale[1]), "s"(g.shift[0]), "s"(g.shift[1]));
#undef RELAY_ASKED
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = (int)fast_div((uint32_t)tile, g.fd_img), rem = tile - n * g.tiles_img;
  const int ty = (int)fast_div((uint32_t)rem, g.fd_row), tx = rem - ty * g.tiles_row;
  const int oy0 = ty * kTh, ox0 = tx * kTw;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint4*)(&lds[0]);
  const unsigned cst_base = (unsigned)(size_t)(__attribute__((address_space(3))) float*)(&cst[0]);
  uint4* const in = lds + 18 * WT;

  // ---- the loads, in the order of use; what the waits count on: two of constants, NI of the patch, 9 PL of the first conv's filters, then
  //      3 PL of the second's behind each of its first three groups of taps
  {
    // (64 words by 16 lanes; arrays that are not there read zeros; int8 has the biases alone, twice)
    auto constants = [&](const void* src, unsigned flag, int k) {
      if (lane < 16) lds_dma16(make_rsrc(src, flag ? kChannels * 4u : 0u), cst_base + (unsigned)(k * kChannels) * 4u, (unsigned)lane * 16u);
    };
    const unsigned bias0 = g.flags[0] & F_BIAS, bias1 = g.flags[1] & F_BIAS, bn0 = g.flags[0] & F_BN, bn1 = g.flags[1] & F_BN;
    const int odd = wave & 1;
    if constexpr (IS_I8) {
      constants(odd ? g.bias[1] : g.bias[0], odd ? bias1 : bias0, odd ? 5 : 2);
      constants(odd ? g.bias[1] : g.bias[0], odd ? bias1 : bias0, odd ? 5 : 2);
    } else {
      constants(wave == 0 ? g.scale[0] : wave == 1 ? g.shift[0] : wave == 2 ? g.bias[0] : g.scale[1], wave < 2 ? bn0 : wave == 2 ? bias0 : bn1, wave);
      constants(odd ? g.bias[1] : g.shift[1], odd ? bias1 : bn1, 4 + odd);
    }
  }
  const int lr4 = lane >> 2;      // staging: row of a block of 16, and (below) the piece that belongs in this lane's slot
  {
    const intx4 rs_x = make_rsrc(ptr_x, (unsigned)g.N * g.H * g.W * (kChannels * ES));
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int blk = __builtin_amdgcn_readfirstlane(min(j * 4 + wave, NB - 1)), plane = blk / (IROWS / 16), p = (blk - plane * (IROWS / 16)) * 16 + lr4;
      const int py = p / kIw, iy = oy0 - 2 + py, ix = ox0 - 2 + p - py * kIw;
      const bool ok = p < kIn && (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
      const unsigned at = (unsigned)(((n * g.H + iy) * g.W + ix) * (kChannels * ES) + plane * 64 + ((lane & 3) ^ lds_swizzle(p)) * 16);
      lds_dma16(rs_x, lds_base + (unsigned)(18 * WT + blk * 64) * 16u, ok ? at : kOob);
    }
  }
  const int w_ch = wave * 16 + lr4;
  const unsigned w_off = (unsigned)(w_ch * g.Kp * ES + ((lane & 3) ^ lds_swizzle(w_ch)) * 16);
  auto request_filters = [&](auto conv_tag, int from, int to) {   // of taps from .. to - 1
    constexpr int conv = decltype(conv_tag)::value;
    const intx4 rs_w = make_rsrc(conv ? ptr_w1 : ptr_w0, (unsigned)(kChannels * g.Kp * ES));
#pragma unroll
    for (int i = from * PL; i < to * PL; ++i)
      lds_dma16(rs_w, lds_base + (unsigned)(conv * 9 * WT + i * (kChannels * BKV) + wave * 64) * 16u, w_off + (unsigned)(i * 64));
  };
  const std::integral_constant<int, 0> first{};
  const std::integral_constant<int, 1> second{};
  request_filters(first, 0, 9);

  const int lr = lane & 15, lk = lane >> 4;   // matrix operand of this lane: row lr of a block of 16, k-vector lk
  auto meet = [&]() {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // k-steps (tap, plane) of either conv, taps from .. to - 1: TN x TM blocks of 16 channels x 16 pixels.  The operands of a step are on
  // their way from LDS while the step before it is multiplied (a wave is alone on its SIMD: nothing else covers that latency).
  auto steps = [&](auto& acc, auto from_tag, auto to_tag, const uint4* filters, const uint4* pixels, int plane_slots, int ch0, const int (&rows)[2], int pitch) {
    constexpr int TN = sizeof(acc[0]) / sizeof(acc[0][0]), FROM = decltype(from_tag)::value * PL, TO = decltype(to_tag)::value * PL;
    uint4 f[2][TN], x[2][2];
    auto read = [&](int s) {
      const int tap = s / PL, pl = s - tap * PL, shift = tap / 3 * pitch + tap % 3;
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) f[s & 1][tn] = filters[s * (kChannels * BKV) + lds_slot(ch0 + tn * 16 + lr, lk)];
#pragma unroll
      for (int tm = 0; tm < 2; ++tm) x[s & 1][tm] = pixels[pl * plane_slots + lds_slot(rows[tm] + shift, lk)];
    };
    read(FROM);
#pragma unroll
    for (int s = FROM; s < TO; ++s) {
      if (s + 1 < TO) read(s + 1);
      __builtin_amdgcn_sched_barrier(0);
      auto& sum = acc[IS_I8 ? 0 : s / PL / 3];
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) sum[tn][tm] = Mma16<IS_I8>::mma(f[s & 1][tn], x[s & 1][tm], sum[tn][tm]);
    }
  };
  auto clear = [&](acc_t& a) {
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = 0;
  };

  // ---- the first conv: 64 rows x 64 channels, a wave 32 x 32 of them
  const int wm = wave >> 1, wn = wave & 1;
  int rows[2];   // input pixel of tap (0, 0)
#pragma unroll
  for (int tm = 0; tm < 2; ++tm) {
    const int m = min(wm * 32 + tm * 16 + lr, kMid - 1), my = m / kMw;   // (rows past the patch repeat its last)
    rows[tm] = my * kIw + m - my * kMw;
  }
  acc_t acc[NA][2][2];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int b = 0; b < 4; ++b) clear(acc[i][b >> 1][b & 1]);
  auto taps = [&](auto from, auto to) { steps(acc, from, to, lds, in, IROWS * BKV, wn * 32, rows, kIw); };
  using std::integral_constant;
  // (the filters of a group of taps are there once every wave has waited for its share of them)
  wait_loads<PL * 8>();
  meet();
  request_filters(second, 0, 3);
  // the tails' factors and addends of this lane's channels: 16 wn + 4 lk (and 16 on) of the first conv, 16 wave + 4 lk of the second
  struct Tail {
    float4 mul, add;   // int8: add holds the bias
  };
  auto tail_of = [&](auto conv_tag, int ch) {
    constexpr int conv = decltype(conv_tag)::value;
    const float4* k = reinterpret_cast<const float4*>(cst + conv * 3 * kChannels + ch);
    const float4 b = k[2 * kChannels / 4];
    if constexpr (IS_I8) {
      return Tail{b, b};
    } else {
      const bool bn = (g.flags[conv] & F_BN) != 0;
      const float4 s = k[0], f = k[kChannels / 4];
      Tail v;
      v.mul = bn ? s : make_float4(1.f, 1.f, 1.f, 1.f);
      v.add = make_float4(b.x * v.mul.x + f.x, b.y * v.mul.y + f.y, b.z * v.mul.z + f.z, b.w * v.mul.w + f.w);  // (acc + b)*sc + sf
      return v;
    }
  };
  const Tail tail0[2] = {tail_of(first, wn * 32 + lk * 4), tail_of(first, wn * 32 + 16 + lk * 4)};
  const Tail tail1 = tail_of(second, wave * 16 + lk * 4);
  taps(integral_constant<int, 0>{}, integral_constant<int, 1>{});
  wait_loads<PL * 9>();
  meet();
  request_filters(second, 3, 6);
  taps(integral_constant<int, 1>{}, integral_constant<int, 3>{});
  wait_loads<PL * 9>();
  meet();
  request_filters(second, 6, 9);
  taps(integral_constant<int, 3>{}, integral_constant<int, 6>{});
  wait_loads<PL * 9>();
  meet();
  taps(integral_constant<int, 6>{}, integral_constant<int, 9>{});

  // ---- its tail: lane l of a block holds channels 4 (l / 16) .. + 3 of pixel l % 16
  typedef float float2v __attribute__((ext_vector_type(2)));
  typedef _Float16 half2v __attribute__((ext_vector_type(2)));
  // the sum of an element's runs, as raw bits
  auto total = [&](const auto& runs, int tn, int tm, int e) {
    if constexpr (IS_I8) {
      return as_u32(runs[0][tn][tm][e]);
    } else {
      float t = runs[0][tn][tm][e];
#pragma unroll
      for (int i = 1; i < NA; ++i) t += runs[i][tn][tm][e];
      return as_u32(t + 0.f);   // (the fourth wave's run is empty)
    }
  };
  // four channels from ch on of one pixel, finished as finish_store8 finishes eight; res: the residual's four values
  auto finish4 = [&](const unsigned (&raw)[4], auto conv_tag, const Tail& k, bool has_res, uint2 res) {
    constexpr int conv = decltype(conv_tag)::value;
    const float mul[4] = {k.mul.x, k.mul.y, k.mul.z, k.mul.w}, add[4] = {k.add.x, k.add.y, k.add.z, k.add.w};
    const bool relu = (g.flags[conv] & F_RELU) != 0;
    if constexpr (IS_I8) {
      ConvArgs a;
      a.rshift = g.rshift[conv], a.round_add = g.round_add[conv], a.clip_lo = g.clip_lo, a.clip_hi = g.clip_hi;
      const ClipBounds cb = clip_bounds(a, relu);
      int t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        t[e] = (int)raw[e] + __builtin_bit_cast(int, add[e]);
        if (has_res) t[e] += (int)(int8_t)(res.x >> (8 * e)) * (1 << g.lshift);
        t[e] = cb.sat_ok ? shift_round_clip<true>(t[e], a, cb) : shift_round_clip<false>(t[e], a, cb);
      }
      return make_uint2(pack_low_bytes(t[0], t[1], t[2], t[3]), 0u);
    } else {
      unsigned hw[2];
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = __builtin_bit_cast(float, raw[e]) * mul[e] + add[e];
      if (has_res) {
        const unsigned rw[2] = {res.x, res.y};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "+v"(t[2 * e]) : "v"(rw[e]));
          asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(t[2 * e + 1]) : "v"(rw[e]));
        }
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        asm("" : "+v"(t[2 * e]), "+v"(t[2 * e + 1]));   // (rounded to fp32 first, as everywhere)
        const float2v f = {t[2 * e], t[2 * e + 1]};
        half2v h = __builtin_convertvector(f, half2v);
        if (relu) h = __builtin_elementwise_max(h, half2v{(_Float16)0, (_Float16)0});
        hw[e] = __builtin_bit_cast(unsigned, h);
      }
      return make_uint2(hw[0], hw[1]);
    }
  };
  // where channels ch .. ch + 3 of a pixel lie in planes of `rows64` rows: slot, and the 8 (int8: 4) bytes in it
  auto place = [&](const uint4* at, int plane_slots, int row, int ch) {
    const int byte = ch * ES;
    return reinterpret_cast<const char*>(at) + ((byte >> 6) * plane_slots + lds_slot(row, (byte >> 4) & 3)) * 16 + (byte & 15);
  };
  auto put4 = [&](uint4* at, int row, int ch, uint2 v) {
    char* dst = const_cast<char*>(place(at, 64 * BKV, row, ch));
    if constexpr (IS_I8) *reinterpret_cast<unsigned*>(dst) = v.x;
    else *reinterpret_cast<uint2*>(dst) = v;
  };
  uint4* const mid = lds;                   // [64 rows] first conv's outputs,
  uint4* const out = lds + PL * 64 * BKV;   // [32] the block's
  wait_loads<0>();                          // (the second conv's filters)
  meet();                                   // nobody reads the first conv's filters any more
#pragma unroll
  for (int tm = 0; tm < 2; ++tm) {
    const int m = wm * 32 + tm * 16 + lr, my = m / kMw, mx = m - my * kMw;
    const int y = oy0 - 1 + my, x = ox0 - 1 + mx;
    const bool inside = m < kMid && (unsigned)y < (unsigned)g.H && (unsigned)x < (unsigned)g.W;   // (outside: the second conv's padding)
#pragma unroll
    for (int tn = 0; tn < 2; ++tn) {
      unsigned raw[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) raw[e] = total(acc, tn, tm, e);
      const int ch = wn * 32 + tn * 16 + lk * 4;
      const uint2 v = finish4(raw, first, tail0[tn], false, make_uint2(0u, 0u));
      put4(mid, m, ch, inside ? v : make_uint2(0u, 0u));
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  meet();

  // ---- 32 pixels x 8 vectors of 8 channels to memory, a piece per thread
  const int o = tid >> 3, oy = o >> 3, ox = o & 7, gch = (tid & 7) * 8;
  const bool live = oy0 + oy < g.H && ox0 + ox < g.W;
  auto store8 = [&](void* y, const char* src) {
    if (!live) return;
    const size_t at = ((size_t)(unsigned)(n * g.H + oy0 + oy) * g.W + ox0 + ox) * kChannels + gch;
    if constexpr (IS_I8) *reinterpret_cast<uint2*>(static_cast<int8_t*>(y) + at) = *reinterpret_cast<const uint2*>(src);
    else *reinterpret_cast<uint4*>(static_cast<_Float16*>(y) + at) = *reinterpret_cast<const uint4*>(src);
  };
  store8(g.y[0], place(mid, 64 * BKV, (oy + 1) * kMw + ox + 1, gch));

  // ---- the second conv: 32 rows x 64 channels, a wave 32 x 16 of them
  int rows2[2];
#pragma unroll
  for (int tm = 0; tm < 2; ++tm) rows2[tm] = (tm * 2 + (lr >> 3)) * kMw + (lr & 7);
  acc_t acc2[NA][1][2];
#pragma unroll
  for (int i = 0; i < NA; ++i) clear(acc2[i][0][0]), clear(acc2[i][0][1]);
  steps(acc2, integral_constant<int, 0>{}, integral_constant<int, 9>{}, lds + 9 * WT, mid, 64 * BKV, wave * 16, rows2, kMw);
  const bool has_res = (g.flags[1] & F_RES) != 0;
#pragma unroll
  for (int tm = 0; tm < 2; ++tm) {
    unsigned raw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) raw[e] = total(acc2, 0, tm, e);
    const int p = tm * 16 + lr, ch = wave * 16 + lk * 4;
    const char* res_at = place(in, IROWS * BKV, ((p >> 3) + 2) * kIw + (p & 7) + 2, ch);
    uint2 res = make_uint2(0u, 0u);
    if (has_res) {
      if constexpr (IS_I8) res.x = *reinterpret_cast<const unsigned*>(res_at);
      else res = *reinterpret_cast<const uint2*>(res_at);
    }
    put4(out, p, ch, finish4(raw, second, tail1, has_res, res));
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  meet();
  store8(g.y[1], place(out, 64 * BKV, o, gch));
}

}  // namespace

// Two 3x3 convs of 64 channels with the plain tails, the second on the first's outputs, in a buffer's range (for how many workgroups: api.cpp's block_plan).
bool conv_block_supported(const ConvArgs& a, const ConvArgs& b, bool is_i8) {
  for (const ConvArgs* c : {&a, &b})
    if (c->C != kChannels || c->K != kChannels || c->R != 3 || c->S != 3 || c->sh != 1 || c->sw != 1 || c->ph != 1 || c->pw != 1 ||
        c->xs_w != c->C || c->nseg || c->pool || c->qmode != QMODE_SHIFT || c->round_mode == ROUND_STOCHASTIC || c->clip_lo != a.clip_lo ||
        c->clip_hi != a.clip_hi)
      return false;
  if (a.N != b.N || a.H != b.H || a.W != b.W || (a.flags & F_RES)) return false;
  if ((size_t)a.M * kChannels * (is_i8 ? 1 : 2) > 0x7fffffffu) return false;
  return true;
}

long conv_block_workgroups(const ConvArgs& a) { return (long)a.N * ((a.H + kTh - 1) / kTh) * ((a.W + kTw - 1) / kTw); }

hipError_t launch_conv_block(const ConvArgs& a, const ConvArgs& b, bool is_i8, hipStream_t st) {
  BlockArgs g;
  g.N = a.N; g.H = a.H; g.W = a.W; g.Kp = a.Kp;
  g.tiles_row = (a.W + kTw - 1) / kTw;
  g.tiles_img = (a.H + kTh - 1) / kTh * g.tiles_row;
  g.fd_img = make_fastdiv((uint32_t)g.tiles_img);
  g.fd_row = make_fastdiv((uint32_t)g.tiles_row);
  g.x = a.x;
  for (int i = 0; i < 2; ++i) {
    const ConvArgs& c = i ? b : a;
    g.w[i] = c.w; g.y[i] = c.y; g.scale[i] = c.scale; g.shift[i] = c.shift; g.flags[i] = c.flags;
    g.bias[i] = is_i8 ? static_cast<const void*>(c.qbias) : c.bias;
    g.rshift[i] = c.rshift; g.round_add[i] = c.round_add;
  }
  g.lshift = b.lshift; g.clip_lo = b.clip_lo; g.clip_hi = b.clip_hi;
  const int tiles = a.N * g.tiles_img;
  if (is_i8) hipLaunchKernelGGL(conv_block_kernel<true>, dim3(tiles), dim3(256), 0, st, tiles, g);
  else hipLaunchKernelGGL(conv_block_kernel<false>, dim3(tiles), dim3(256), 0, st, tiles, g);
  return hipGetLastError();
}

}  // namespace relay
