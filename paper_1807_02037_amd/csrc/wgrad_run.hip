// Weight gradient of 2-D 3x3 stride-1 convolutions that keep the extents (padding 1), at least 48 channels on both sides.
//
// dw[kh][kw][c][k] = sum over positions of x[position + (kh - 1, kw - 1)][c] * dy[position][k].  Positions are numbered with one
// zero column behind every row and one zero row behind every image: index q = (n (H + 1) + h) (W + 1) + w.  A tap is then the
// same shift kh (W + 1) + kw of the index for every position, whatever row or image it is in, and the reduction is one run
// over q; products of a zero column or row add nothing.  14 x 14 maps fill 87 % of their numbers and 56 x 56 maps 96 %, where
// patches of 8 x 16 positions are 77 % and 87 % full.
//
// At a position that is none of dy's (zero column or row, behind the work-group's part) dy = 0 meets real pixels of x, which makes NaN of
// infinite ones in taps that never read them.  Such a sum is not finite, and a sum that is finite met no such pixel: a work-group
// that ends with one that is not goes over its part again with x masked at those positions, so that infinities and NaN
// reach the entries that read them and no others (256 -> 256, 14 x 14, batch 256 81 -> 195 us with one infinity).  Finite tensors pay for
// the look at the sums alone, 0.3 us (16.3 -> 16.6 at 256 -> 256, 14 x 14, batch 8).
//
// A work-group of eight waves, one per compute unit, owns 64 input channels x KT output channels of all nine taps and a part of
// the run.  A wave has one 32 x 32 block of them (nine accumulators); the groups of waves that cover the tile take turns at
// 16 positions each, and their sums meet in LDS.  x goes from memory straight into a ring of pixels in LDS, each pixel once, dy
// into three buffers, both two steps of 128 positions ahead; the operands are read with the LDS transpose read, one round
// ahead of their products.  Of a filter row the first and the last tap are read, from 16-byte aligned registers each, and the middle one is
// cut out of the two: nine products take fourteen reads of 8 bytes a lane and twelve shifts (cutting the last tap out as well took
// three reads less and twelve register moves more; with the bank conflicts below, 256 -> 256 at 14 x 14, batch 256 81.0 / 79.8, 128 -> 128 at 28 x 28,
// batch 64 30.6 / 29.8, 512 -> 512 at 7 x 7, batch 256 81.3 / 79.6).
//
// What bounds it, on the layers with many positions, is no single pipe: at 14 x 14 and larger the matrix pipes are busy 37 % of the cycles
// (936 TFLOP/s with the zero column and row, 0.59 of what a loop on registers reaches on random operands), LDS is active in 20 %, without
// bank conflicts in the reads (with pairs of 16-byte slots permuted, which fits reads of 16 lanes at a time and not of 32, two fifths of 27 %); without its LDS reads the kernel is 1 us faster, without the loads of x and dy 8 us, of 66
// at 256 -> 256.  Two waves a SIMD meet at a barrier every 128 positions.  On the layers with one tile it is the partial filters, written
// and added.  Both parameter gradients, us, patches of 8 x 16 positions / this kernel: 256 -> 256 at 14 x 14, batch 256 93 -> 74 (804
// TFLOP/s); 128 -> 128 at 28 x 28, batch 128 57 -> 46; 512 -> 512 at 7 x 7, batch 256 92 -> 81; 64 -> 64 at 56 x 56, batch 64 36 -> 32;
// 384 -> 320 at 9 x 9, batch 210 218 -> 58; 88 -> 88 layers of 4 Ki positions 13 -> 13.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"

namespace lms {

namespace {


constexpr int RUN_NT = 512, STEP = 128, PIX_B = 128;
constexpr int RING = 5 * STEP, RING_PAD = 32;                     // pixels of x in LDS; first ones once more behind the end
constexpr int RUN_SUMS = 4 * 9 * 4 * 64 * 16;                     // the sums of four waves
// KT output channels of a work-group: 64, two groups of four waves, or 32, four groups of two
template <int KT>
struct RunTile {
  static constexpr int Y_PIX = KT * 2, Y_BUF = STEP * Y_PIX, YV = KT / 32;      // bytes of a pixel of dy; loads per thread and step
  static constexpr int G = KT == 64 ? 2 : 4, ROUNDS = 8 / G;      // groups; 16-position rounds of a group per step
  static constexpr int LDS_X = (RING + RING_PAD) * PIX_B, FLAGS = LDS_X + 3 * Y_BUF > RUN_SUMS ? LDS_X + 3 * Y_BUF : RUN_SUMS, LDS = FLAGS + 64;
};

struct WRunP {
  const uint16_t* X;
  const uint16_t* DY;
  float* part;
  float* cs_part;              // partial column sums of dy [split][ky], or null
  int batch, H, W, cx, ky;
  int ctiles, ktiles, splits;
  int q_total, q_per_split;    // q_per_split: multiple of 32
  int inc_h, inc_w, inc_m;     // a step of 128 positions: rows, columns, pixels in memory
  int above;                   // images that hold the step before the first image
};

template <int KT, bool CS>
__global__ __launch_bounds__(RUN_NT, 2) void wgrad_run_kernel(WRunP p) {
  typedef RunTile<KT> T;
  constexpr int G = T::G, YV = T::YV;
  extern __shared__ __attribute__((aligned(256))) unsigned char lds_run[];
  // the tiles of one split read the same pixels: on one XCD they share them in its L2
  int b = p.ctiles * p.ktiles > 1 ? xcd_order(p.ctiles * p.ktiles * p.splits) : (int)blockIdx.x;
  if (b < 0) return;
  const int cc = b % p.ctiles; b /= p.ctiles;
  const int kt = b % p.ktiles; b /= p.ktiles;
  const int split = b;
  const int c0 = cc * 64, k0 = kt * KT;
  const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = wave8 / (8 / G), wave = wave8 % (8 / G);
  const int cq = wave & 1, kq = wave >> 1;                        // which 32 channels of x, of dy
  const int Wp = p.W + 1, Hp = p.H + 1, img = Hp * Wp;

  const int q0 = split * p.q_per_split;
  const int qlen = p.q_total - q0 < p.q_per_split ? p.q_total - q0 : p.q_per_split;
  const int steps = (qlen + STEP - 1) / STEP;

  // ---- this thread's vectors of a step: pixel tid / 8 (and 64 on), 16-byte slot tid % 8; every two pixels the halves of one are
  // swapped, so that the four pixels x 64 bytes that LDS serves at a time fall into different banks (32 channels of dy: they do anyway) ----
  const int px = tid >> 3, ch = ((tid & 7) ^ ((px & 2) << 1)) * 8;
  const int y_px = KT == 64 ? px : tid >> 2, y_c = KT == 64 ? ch : (tid & 3) * 8;
  const bool xc_ok = c0 + ch < p.cx, yc_ok = k0 + y_c < p.ky;
  const int xs = q0 - STEP;                                       // x is there from the step before the first on
  int n0 = (xs + img * p.above) / img - p.above;                  // image of its first pixel
  n0 = n0 < 0 ? 0 : n0;
  const long long plane = (long long)p.H * p.W;
  const v4u rs_x = buffer_rsrc(p.X + n0 * plane * p.cx, (p.batch - n0) * plane * p.cx * 2);
  const v4u rs_y = buffer_rsrc(p.DY + n0 * plane * p.ky, (p.batch - n0) * plane * p.ky * 2);
  // positions move by a step without divisions: row and column (the zero ones too) and pixel of the tensor, counted from n0
  struct Pos { int h, w, m; };
  auto start = [&](int q) {
    const unsigned t = (unsigned)(q + img * p.above);
    const int n = (int)(t / (unsigned)img) - p.above, r = (int)(t % (unsigned)img);
    const int h = r / Wp, w = r % Wp;
    return Pos{h, w, ((n - n0) * p.H + h) * p.W + w};             // above the first image: m negative, beyond the buffer
  };
  auto advance = [&](Pos& s) {
    s.w += p.inc_w; s.h += p.inc_h; s.m += p.inc_m;
    if (s.w >= Wp) { s.w -= Wp; ++s.h; --s.m; }
    if (s.h >= Hp) { s.h -= Hp; s.m -= p.W; }
  };
  Pos xp[2], yp;
  const unsigned lds0 = (unsigned)(uintptr_t)lds_run;
  const unsigned lds_x = __builtin_amdgcn_readfirstlane(lds0 + wave8 * 1024);
  const unsigned lds_y = __builtin_amdgcn_readfirstlane(lds0 + T::LDS_X + wave8 * 1024);
  int fill;                                                       // ring pixel of the next step of x
  int ym[2][2];                                                   // KT 64: pixels of the two steps that x is ahead of dy; -1: zeros
  const int x_pitch = p.cx * 2, y_pitch = p.ky * 2, x_ch = (c0 + ch) * 2, y_ch = (k0 + y_c) * 2;
  auto fetch_x = [&]() {
    unsigned o[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bool in = xp[j].h < p.H && xp[j].w < p.W;
      o[j] = xc_ok && in ? (unsigned)(xp[j].m * x_pitch + x_ch) : DMA_OOB;
      if constexpr (KT == 64) {
        ym[0][j] = ym[1][j];
        ym[1][j] = yc_ok && in ? xp[j].m : -1;
      }
      load_lds16(rs_x, lds_x + (fill + 64 * j) * PIX_B, o[j], 0);
      advance(xp[j]);
    }
    // the first pixels of the ring once more behind its end, for reads that begin before it
    if (fill == 0 && wave8 < RING_PAD / 8) load_lds16(rs_x, lds_x + RING * PIX_B, o[0], 0);
    fill += STEP;
    if (fill == RING) fill = 0;
  };
  auto fetch_y = [&](int step, int buf) {                         // KT 64: the step before the one that fetch_x has just asked for
#pragma unroll
    for (int j = 0; j < YV; ++j) {
      int m;
      if constexpr (KT == 64) m = ym[0][j];
      else {
        m = yc_ok && yp.h < p.H && yp.w < p.W ? yp.m : -1;
        advance(yp);
      }
      const bool ok = m >= 0 && step * STEP + y_px + 64 * j < qlen;
      load_lds16(rs_y, lds_y + buf * T::Y_BUF + j * 64 * PIX_B, ok ? (unsigned)(m * y_pitch + y_ch) : DMA_OOB, 0);
    }
  };

  // ---- LDS read addresses: a 16-lane group reads four pixels (lane / 4) x 16 channels; tap (kh, 0) of a position is
  // 8 a + b pixels into the step before its own: b here, 8 a with the step and the 16 positions in a scalar ----
  const int li = lane & 15, lg = lane >> 4, row = (lg >> 1) * 8 + (li >> 2);
  auto at = [&](int r, int pair) { return r * PIX_B + ((pair ^ (r & 2)) << 5) + (li & 3) * 8; };
  const int xpair = cq * 2 + (lg & 1), ypair = kq * 2 + (lg & 1);
  int xa[3][2], ya, xb[3];
#pragma unroll
  for (int kh = 0; kh < 3; ++kh) {
    const int s = STEP - 1 + (kh - 1) * Wp;
    xb[kh] = s & ~7;
    xa[kh][0] = at((s & 7) + row, xpair);
    xa[kh][1] = at((s & 7) + row + 2, xpair);
  }
  ya = KT == 64 ? at(row, ypair) : row * T::Y_PIX + (lg & 1) * 32 + (li & 3) * 8;

  f32x16 acc[9], cs;
#pragma unroll
  for (int v = 0; v < 16; ++v) cs[v] = 0.f;
  const bool cs_on = CS && cc == 0;

  int base, ybuf;                                                 // ring pixel of the step, buffer of its dy
  // 16 positions: operands as they come from LDS, and their products.  They are read one round ahead: with reads and products
  // in turn each of the four waits of a round cost an LDS round trip.
  struct Frag { v2u y[2], x[3][2][2]; };
  auto load = [&](Frag& f, int j) {
    const int ks = G * j + g;
    const unsigned char* sy = lds_run + T::LDS_X + ybuf * T::Y_BUF + ks * 16 * T::Y_PIX;
#pragma unroll
    for (int i = 0; i < 2; ++i) f.y[i] = tr_read(sy + ya + 4 * i * T::Y_PIX);
#pragma unroll
    for (int kh = 0; kh < 3; ++kh) {
      int s = base + ks * 16 + xb[kh];
      if (s >= RING) s -= RING;
      const unsigned char* sx = lds_run + s * PIX_B;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f.x[kh][0][i] = tr_read(sx + xa[kh][0] + 4 * i * PIX_B);
        f.x[kh][1][i] = tr_read(sx + xa[kh][1] + 4 * i * PIX_B);
      }
    }
  };
  // masked: the positions of step st, round j that are dy's keep their x
  auto mul = [&](const Frag& f, auto masked_c, int st, int j) {
    v4u m = {~0u, ~0u, ~0u, ~0u};
    if constexpr (decltype(masked_c)::value) {
      int r = st * STEP + (G * j + g) * 16 + 8 * (lane >> 5);
      int h = (int)((unsigned)(q0 + r) % (unsigned)img), w = h % Wp;
      h /= Wp;
#pragma unroll
      for (int e = 0; e < 8; ++e, ++r) {
        if (!(r < qlen && h < p.H && w < p.W)) m[e >> 1] &= (e & 1) ? 0xffffu : 0xffff0000u;
        if (++w == Wp) { w = 0; if (++h == Hp) h = 0; }
      }
    }
    const bf16x8 yf = __builtin_bit_cast(bf16x8, v4u{f.y[0][0], f.y[0][1], f.y[1][0], f.y[1][1]});
#pragma unroll
    for (int kh = 0; kh < 3; ++kh) {
      const v4u f0 = {f.x[kh][0][0][0], f.x[kh][0][0][1], f.x[kh][0][1][0], f.x[kh][0][1][1]};      // two positions a word
      const v4u f2 = {f.x[kh][1][0][0], f.x[kh][1][0][1], f.x[kh][1][1][0], f.x[kh][1][1][1]};
      const v4u f1 = {__builtin_amdgcn_alignbit(f2[0], f0[0], 16), __builtin_amdgcn_alignbit(f2[1], f0[1], 16),
                      __builtin_amdgcn_alignbit(f2[2], f0[2], 16), __builtin_amdgcn_alignbit(f2[3], f0[3], 16)};
      acc[kh * 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f0 & m), yf, acc[kh * 3], 0, 0, 0);
      acc[kh * 3 + 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f2 & m), yf, acc[kh * 3 + 2], 0, 0, 0);
      acc[kh * 3 + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f1 & m), yf, acc[kh * 3 + 1], 0, 0, 0);
    }
  };

  // x step i (i = 0: the step before the first) is needed by steps i - 2 to i of dy.  Step st asks for x step st + 4 and dy step
  // st + 2, into the pixels of x step st - 1 and the buffer of dy step st - 1.  Per step a wave has 2 + YV loads, one more with the
  // pixels behind the ring's end.
  auto loop = [&](auto sums_c, auto masked_c) {
    constexpr bool SUMS = decltype(sums_c)::value;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) xp[j] = start(xs + px + 64 * j);
    if constexpr (KT == 32) yp = start(q0 + y_px);
    fill = base = ybuf = 0;
    fetch_x();
    fetch_x();
    fetch_x();
    fetch_y(0, 0);
    fetch_x();
    fetch_y(1, 1);
#pragma unroll 1
    for (int st = 0; st < steps; ++st) {
      if (st + 1 < steps) wait_barrier<2 + YV>();
      else wait_barrier<0>();
      // rounds of this half, two at a time; those beyond the last position multiply zeros
      const int rest = qlen - st * STEP, n = rest >= STEP ? T::ROUNDS : (rest - g * 16 + 16 * G - 1) / (16 * G);
      Frag fa, fb;
      load(fa, 0);
      if (st + 2 < steps) {
        fetch_x();
        fetch_y(st + 2, ybuf == 0 ? 2 : ybuf - 1);
      }
#pragma unroll 1
      for (int j = 0; j < n; j += 2) {
        load(fb, j + 1);
        mul(fa, masked_c, st, j);
        if constexpr (SUMS) {                                     // the quadrants of a column share the sums
          const __bf16 o = (__bf16)1.f;
          const bf16x8 ones = {o, o, o, o, o, o, o, o};
          v4u yf;
#pragma unroll
          for (int i = 0; i < 4; ++i) yf[i] = cq == 0 ? fa.y[i >> 1][i & 1] : fb.y[i >> 1][i & 1];
          cs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, __builtin_bit_cast(bf16x8, yf), cs, 0, 0, 0);
        }
        load(fa, j + 2 < n ? j + 2 : j);
        mul(fb, masked_c, st, j + 1);
      }
      base += STEP;
      if (base == RING) base = 0;
      ybuf = ybuf == 2 ? 0 : ybuf + 1;
    }
  };
  if (cs_on) loop(std::true_type{}, std::false_type{});
  else loop(std::false_type{}, std::false_type{});
  float most = 0.f;
#pragma unroll
  for (int t = 0; t < 9; ++t) most = magnitude(acc[t], most);
  int* flags = reinterpret_cast<int*>(lds_run + T::FLAGS);        // per wave
  flags[wave8] = __builtin_amdgcn_ballot_w64(!(most < __builtin_inff())) != 0;
  __syncthreads();
  int again = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) again |= flags[i];
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(again), 0)) {                    // the sums of dy stand
    loop(std::false_type{}, std::true_type{});
    __syncthreads();
  }

  // ---- of four groups the last two leave their sums to the first two; two then exchange theirs: one finishes taps 0 to 4,
  // the other the rest ----
  float4* sums = reinterpret_cast<float4*>(lds_run);
  auto slot = [&](int t, int q) -> float4& { return sums[((wave8 % 4 * 9 + t) * 4 + q) * 64 + lane]; };
  if constexpr (G == 4) {
    if (g >= 2) {
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) slot(t, q) = make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
    }
    __syncthreads();
    if (g < 2) {
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 o = slot(t, q);
          acc[t][4 * q] += o.x; acc[t][4 * q + 1] += o.y; acc[t][4 * q + 2] += o.z; acc[t][4 * q + 3] += o.w;
        }
    }
    __syncthreads();
  }
  const int c = c0 + cq * 32 + 4 * (lane >> 5), k = k0 + kq * 32 + (lane & 31);
  const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(p.part + (long long)split * 9 * p.cx * p.ky, 0, 9 * p.cx * p.ky * 4, 0x00020000);
  const unsigned out_off = k < p.ky ? (unsigned)((c * p.ky + k) * 4) : DMA_OOB;
  auto half = [&](auto g_c) {
    constexpr int MINE = decltype(g_c)::value == 0 ? 0 : 5, MINE_END = decltype(g_c)::value == 0 ? 5 : 9;
#pragma unroll
    for (int t = 0; t < 9; ++t)
      if (t < MINE || t >= MINE_END)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          sums[((wave * 9 + t) * 4 + q) * 64 + lane] = make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int t = MINE; t < MINE_END; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 o = sums[((wave * 9 + t) * 4 + q) * 64 + lane];
        const float v[4] = {acc[t][4 * q] + o.x, acc[t][4 * q + 1] + o.y, acc[t][4 * q + 2] + o.z, acc[t][4 * q + 3] + o.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned o = c + 8 * q + e < p.cx ? out_off + (unsigned)(((t * p.cx + 8 * q + e) * p.ky) * 4) : DMA_OOB;
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v[e]), out, (int)o, 0, 0);
        }
      }
  };
  if (g == 0) half(std::integral_constant<int, 0>{});
  else if (g == 1) half(std::integral_constant<int, 1>{});
  else __syncthreads();                                           // the one in half
  if (cs_on) {
    float* sh = reinterpret_cast<float*>(lds_run);
    __syncthreads();                                              // the sums above have been read
    if (lane < 32) sh[(g * 2 + cq) * KT + kq * 32 + lane] = cs[0];      // every row of the product with ones is the sum
    __syncthreads();
    if (tid < KT && k0 + tid < p.ky) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < 2 * G; ++i) t += sh[i * KT + tid];
      p.cs_part[(long long)split * p.ky + k0 + tid] = t;
    }
  }
}

RunPlan run_plan_kt(long long batch, int h, int w, int cx, int ky, int kt, long long room) {
  RunPlan r;
  r.kt = kt;
  r.ctiles = (cx + 63) / 64; r.ktiles = (ky + kt - 1) / kt;
  r.q = batch * (h + 1) * (w + 1);
  // One work-group per compute unit, of at least 96 positions: shorter ones cost more in partial filters than they save
  // (us, at least 32 / 64 / 128 / 192 positions: 376 -> 56, 25 x 24, batch 2 17.9 / 13.7 / 14.3 / 13.8; 240 -> 216, 16 x 16
  // 15.4 / 13.7 / 13.3 / 14.2; 512 -> 184, 16 x 16, batch 5 21.2 / 19.0 / 19.1 / 19.0).
  const int tiles = r.ctiles * r.ktiles;
  long long splits = tiles < 256 ? 256 / tiles : 1;
  const long long units = (r.q + 31) / 32, most = r.q < 96 ? 1 : r.q / 96;
  if (splits > most) splits = most;
  // ... and no more of them than the workspace has room for
  if (splits > room) splits = room;
  const long long per = (units + splits - 1) / splits;
  r.q_per_split = (int)(per * 32 < 0x7fffffff ? per * 32 : 0x7fffffff);
  r.splits = (int)((units + per - 1) / per);
  return r;
}

// 64 output channels of a work-group, or 32: twice the steps of a work-group, 1.28 us each and not 2.05, for half the partial
// filters (0.27 us a MB, written and added), and 1.3 us to add two more groups' sums.  Both parameter gradients, us, 64 / 32: 64 -> 64 at
// 56 x 56, batch 64 33.9 / 32.2; 256 -> 256 at 14 x 14, batch 8 22.0 / 19.1, batch 256 73.6 / 82.3; 64 -> 184, 12 x 12, batch 89 20.5 / 17.4;
// 128 -> 128, 28 x 28, batch 128 45.9 / 48.0; 208 -> 136, 9 x 7, batch 7 (as many partial filters) 12.4 / 13.0.
RunPlan run_plan(long long batch, int h, int w, int cx, int ky, long long room) {
  const RunPlan a = run_plan_kt(batch, h, w, cx, ky, 64, room), b = run_plan_kt(batch, h, w, cx, ky, 32, room);
  auto cost = [&](const RunPlan& r, double step) { return r.q_per_split * step / STEP + 0.27e-6 * 36 * cx * ky * r.splits; };
  return cost(b, 1.28) + 1.3 < cost(a, 2.05) ? b : a;
}

template <int KT, bool CS>
hipError_t launch_run_t(const WRunP& p, unsigned grid, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(wgrad_run_kernel<KT, CS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, RunTile<KT>::LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((wgrad_run_kernel<KT, CS>), dim3(grid), dim3(RUN_NT), RunTile<KT>::LDS, s, p);
  return hipGetLastError();
}

}  // namespace

// Offsets within a work-group's part of the run have 31 bits.
RunPlan wgrad_run_plan(long long batch, const int* asp, const int* osp, const int* filt, const int* pad, int cx, int ky) {
  static const bool off = getenv("LMS_NO_WGRAD_RUN") != nullptr;   // tuning aid
  const RunPlan none{};
  if (off || filt[0] != 1 || filt[1] != 3 || filt[2] != 3 || pad[0] != 0 || pad[1] != 1 || pad[2] != 1 || asp[0] != 1) return none;
  if (asp[1] != osp[1] || asp[2] != osp[2] || cx < 48 || ky < 48 || (cx & 7) != 0 || (ky & 7) != 0) return none;
  const int h = asp[1], w = asp[2];
  if (w > 126 || batch < 1 || batch * (h + 1LL) * (w + 1) >= 0x40000000LL) return none;
  const RunPlan r = run_plan(batch, h, w, cx, ky, wgrad_patch_splits(batch, asp, osp, filt, pad, cx, ky));
  return (r.q_per_split + 1024LL + 2LL * (h + 1) * (w + 1)) * (cx > ky ? cx : ky) * 2 < 0x7fffffffLL && (long long)r.ctiles * r.ktiles * r.splits < 0x7fffff00LL &&
         36LL * cx * ky < 0x40000000LL ? r : none;
}

hipError_t launch_wgrad_run(const RunPlan& r, const uint16_t* X, const uint16_t* DY, float* part, long long batch, const int* osp, int cx, int ky,
                            float* cs_part, hipStream_t s) {
  WRunP p{};
  p.X = X; p.DY = DY; p.part = part; p.cs_part = cs_part;
  p.batch = (int)batch; p.H = osp[1]; p.W = osp[2]; p.cx = cx; p.ky = ky;
  p.ctiles = r.ctiles; p.ktiles = r.ktiles; p.splits = r.splits;
  p.q_total = (int)r.q; p.q_per_split = r.q_per_split;
  const int wp = p.W + 1, img = (p.H + 1) * wp, left = STEP % img, images = STEP / img;
  p.inc_h = left / wp; p.inc_w = left % wp;
  p.inc_m = images * p.H * p.W + p.inc_h * p.W + p.inc_w;
  p.above = (STEP + img - 1) / img;
  const int tiles = r.ctiles * r.ktiles;
  const unsigned grid = (unsigned)(tiles > 1 ? xcd_grid((long long)tiles * r.splits) : r.splits);
  if (r.kt == 64) return cs_part ? launch_run_t<64, true>(p, grid, s) : launch_run_t<64, false>(p, grid, s);
  return cs_part ? launch_run_t<32, true>(p, grid, s) : launch_run_t<32, false>(p, grid, s);
}

}  // namespace lms
