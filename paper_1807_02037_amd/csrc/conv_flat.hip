// 3x3 and 3x3x3 stride-1 convolutions that keep the extents (padding 1), forward and data gradient.
//
// A tile is BM consecutive positions of the batch in memory order, whatever rows and images they belong to, so no
// tile is padded: patches of 8 x 16 positions are 77 % full on the 14 x 14, 28 x 28 and 7 x 7 maps of ResNet-50 and fill worse
// still on odd extents.  The input pixels that the nine taps of a tile touch are one contiguous run of BM + 2 W + 2 rows;
// for every block of 32 channels the run goes straight to LDS (buffer loads that write LDS) while the block before it is
// multiplied, and a tap is a shift by kh * W + kw pixels.  Where a tap leaves the image, the lane reads zeros instead, with the longer filter
// rings from the LDS banks its pixel would have come from: its nine addresses are worked out once per tile.  The filter streams through a ring of LDS buffers one
// filter row (three taps x BN x 32 channels) a stage, one barrier each.  Products are taken transposed and leave through
// wave_epilogue.  The forward pass reads the filter as it is stored, through the LDS transpose read: packing it first was a launch of
// 3 to 5 us (us, packed / as stored: 72 -> 40 at 45 x 37, batch 3 12.5 / 8.8; 256 -> 256 at 14 x 14, batch 256 64.8 / 61.7, 16^3 30.6 /
// 25.8; 64 -> 64 at 64^3 60.3 / 55.9; 100 random layers 0.82 of the time, none slower by more than 2 %).
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"

namespace lms {

namespace {

template <int BM_, int BN_, int WM_, int WN_, int AV_, int NB_, int G_ = 1>
struct FlatTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, G = G_;
  static constexpr int NT = NTHREADS * G;                         // threads of the work-group
  static constexpr int AV = AV_;                                  // input loads per thread and block
  static constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  static_assert(WM * WN == 4, "four waves a group");
  static constexpr int BV = (3 * BN * 4 + NTHREADS - 1) / NTHREADS;       // filter loads per thread and stage
  static constexpr int B_STAGE = BV * NTHREADS * 16;
  static constexpr int NB = NB_;                                  // filter ring, 2 to 4 stages
  // Loads between the products (stage).  Only tiles that do so pay for an address of zeros per tap and an offset for blocks that are not there: the
  // others got nothing from them and lost, in volumes with at most 32 outputs, 2 % (us, forward, without / with: 32 -> 32 at 18 x 18 x 19
  // 6.3 / 6.4, 224 -> 24 at 17^3 24.2 / 24.8).
  static constexpr bool SPREAD = NB > 2 && TM * TN > 1;
  static constexpr int MAXPIX = AV * NTHREADS / 4;                // input pixels at most
  static constexpr int LPR = WTN / 8, RPI = 64 / LPR, QV = 32 / RPI;
};

// Input pixels of a tile, rounded to the 16 pixels a wave loads at once, and 256 bytes of zeros (all banks) behind them.
__host__ __device__ inline int flat_pixels(int bm, int w) { return (bm + 2 * w + 2 + 15) / 16 * 16; }
__host__ __device__ inline int flat_abuf(int bm, int w) { return flat_pixels(bm, w) * 64 + 256; }

// LDS of a group: filter ring, two input buffers, a place for loads that nobody needs.
template <typename T>
__host__ __device__ inline int flat_group_lds(int w) { return T::NB * T::B_STAGE + 2 * flat_abuf(T::BM, w) + 1024; }

template <typename T, bool P3D, bool FLIP>
__global__ __launch_bounds__(T::NT, 2) void conv_flat_kernel(IgemmP p) {
  constexpr int TM = T::TM, TN = T::TN, BV = T::BV, AV = T::AV, NB = T::NB, G = T::G, KD = P3D ? 3 : 1;
  extern __shared__ __attribute__((aligned(256))) unsigned char flat_smem[];
  const int per_xcd = (p.ntiles + 7) / 8;
  const int tile = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (tile >= p.ntiles) return;
  const int n0 = (tile % p.ntiles_n) * T::BN;
  const long long m0 = (long long)(tile / p.ntiles_n) * T::BM;
  const int W = p.osp[2], H = p.osp[1];

  const int tid = threadIdx.x & (NTHREADS - 1), lane = tid & 63, wave = tid >> 6;      // within the group
  const int grp = G > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / NTHREADS) : 0;
  const int wm = wave / T::WN, wn = wave % T::WN, half = lane >> 5;

  // ---- LDS of the group ----
  const int npix = flat_pixels(T::BM, W), abuf = flat_abuf(T::BM, W);
  unsigned char* sB = flat_smem + grp * flat_group_lds<T>(W);
  unsigned char* sA = sB + NB * T::B_STAGE;
  const unsigned lds0 = (unsigned)(uintptr_t)sB;                  // LDS address: the low half of the generic one
  const unsigned ldsA = lds0 + NB * T::B_STAGE, ldsX = ldsA + 2 * abuf;
  if (tid < 32) *reinterpret_cast<uint4*>(sA + (tid >> 4) * abuf + npix * 64 + (tid & 15) * 16) = make_uint4(0, 0, 0, 0);

  // ---- operands of the epilogue, fetched ahead ----
  const int cg = (lane % T::LPR) * 8, n = n0 + wn * T::WTN + cg;
  const int er = wm * T::WTM + lane / T::LPR;
  const EpiBuffers eb(p, m0, grp == 0 ? (p.M - m0) * p.nout * 2 : 0);                 // group 0 writes
  const unsigned col = n < p.nout ? (unsigned)(n * 2) : DMA_OOB;
  auto out_off = [&](int r) -> unsigned { return col + (unsigned)(r * p.nout * 2); };   // rows beyond the last lie beyond the buffer
  constexpr int EV = TM * T::QV;
  uint4 pre_add[EV], pre_mask[EV];
#pragma unroll
  for (int q = 0; q < EV; ++q) {
    const unsigned o = out_off(er + (q / T::QV) * 32 + (q % T::QV) * T::RPI);
    pre_add[q] = EpiBuffers::get(eb.add, o);
    pre_mask[q] = EpiBuffers::get(eb.mask, o);
  }

  // ---- input loads: pixel j of the buffer is row m0 - W - 1 + j of the tensor, channel slot g sits at g ^ ((j >> 2) & 3) ----
  const int apix = tid >> 2, ag = (tid & 3) ^ ((apix >> 2) & 3);
  const long long plane = (long long)H * W, arow0 = m0 - W - 1 - (P3D ? plane : 0);
  const v4u rs_a = buffer_rsrc(p.A + arow0 * p.red, 0x7fffffff);  // rows outside the tensor are never asked for
  const unsigned a_off = (unsigned)((apix * p.red + ag * 8) * 2), a_plane = (unsigned)(plane * p.red * 2);
  unsigned a_in[KD];                                              // bit j: pixel apix + 64 j of this plane's run is a row of the tensor
#pragma unroll
  for (int kd = 0; kd < KD; ++kd) {
    a_in[kd] = 0;
#pragma unroll
    for (int j = 0; j < AV; ++j) {
      const int pix = apix + j * (NTHREADS / 4);
      const long long row = arow0 + kd * plane + pix;
      if (pix < npix && row >= 0 && row < p.M) a_in[kd] |= 1u << j;
    }
  }
  const unsigned ldsA_w = __builtin_amdgcn_readfirstlane(ldsA + wave * 1024), ldsX_u = __builtin_amdgcn_readfirstlane(ldsX);
  const int wpix = __builtin_amdgcn_readfirstlane(wave * 16);
  // block vb of the layer: channel block vb / KD, input plane vb % KD; the group takes vb = grp, grp + G, ...
  const int nblocks = ((p.red + BK - 1) / BK) * KD, nlocal = (nblocks + G - 1) / G;
  struct Run { bool ok; unsigned in, so; };                       // what the loads of a block share: channels there, pixels there, offset
  auto run_a = [&](int lb) {
    const int vb = lb * G + grp, chunk = vb / KD, kd = vb % KD;
    unsigned in = a_in[0];
    if constexpr (P3D) in = kd == 0 ? a_in[0] : (kd == 1 ? a_in[1] : a_in[2]);
    return Run{vb < nblocks && chunk * BK + ag * 8 < p.red, in, (P3D ? kd * a_plane : 0) + chunk * (BK * 2)};
  };
  auto load_a = [&](const Run& r, int lb, int j) {
    const unsigned dst = j * (NTHREADS / 4) + wpix < npix ? ldsA_w + (lb & 1) * abuf + j * NTHREADS * 16 : ldsX_u;   // uniform
    load_lds16(rs_a, dst, r.ok && ((r.in >> j) & 1) ? a_off : DMA_OOB, (unsigned)(j * (NTHREADS / 4) * p.red * 2) + r.so);
  };
  auto fetch_a = [&](int lb) {
    const Run r = run_a(lb);
#pragma unroll
    for (int j = 0; j < AV; ++j) load_a(r, lb, j);
  };
  // ---- filter loads.  Data gradient: row (tap of the filter row, output channel), channel slot g at g ^ ((n >> 2) & 3).  Forward: the
  // filter as stored, row (tap, input channel) of BN output channels for the transpose read.  LDS serves 32 lanes of that read at a
  // time, four rows x 64 bytes; rows of 64 channels swap their halves every two rows, so that the four fall into different banks
  // (a swap of neighbouring slots, made for four rows x 32 bytes, cost a conflict in every read, and with the zeros at one place 43 % of
  // the LDS cycles were conflicts; us: 512 -> 512 at 7 x 7, batch 32 17.2 / 15.3, 256 -> 256 at 16^3 24.6 / 23.9, 96 -> 160 at 23 x 21,
  // batch 16 8.2 / 7.6; nothing where a launch has two rounds of tiles) ----
  const v4u rs_b = buffer_rsrc(p.B, (long long)(9 * KD) * p.nout * p.red * 2);
  unsigned b_off[BV];
  int b_k[BV];
#pragma unroll
  for (int j = 0; j < BV; ++j) {
    const int v = tid + j * NTHREADS;
    if constexpr (FLIP) {
      const int row = v >> 2, nr = row % T::BN, tl = row / T::BN;
      b_k[j] = ((v & 3) ^ ((nr >> 2) & 3)) * 8;
      b_off[j] = tl < 3 && n0 + nr < p.nout ? (unsigned)(((tl * p.nout + n0 + nr) * p.red + b_k[j]) * 2) : DMA_OOB;
    } else {
      constexpr int SPR = T::BN / 8;
      const int row = v / SPR, g = v % SPR, tl = row / BK, ch = (T::BN == 64 ? g ^ ((row & 2) << 1) : g) * 8;
      b_k[j] = row % BK;
      b_off[j] = tl < 3 && n0 + ch < p.nout ? (unsigned)(((tl * p.red + b_k[j]) * p.nout + n0 + ch) * 2) : DMA_OOB;
    }
  }
  const unsigned b_chunk = (unsigned)(FLIP ? BK * 2 : BK * 2 * p.nout);
  const unsigned ldsB_w = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
  struct Row { bool ok; int c0; unsigned so; };                   // of a filter row
  auto row_b = [&](int lb, int u) {
    const int vb = lb * G + grp, chunk = vb / KD, kd = FLIP ? KD - 1 - vb % KD : vb % KD;
    const bool ok = vb < nblocks;                                 // beyond the last block no offset beyond the buffer either (without SPREAD only the
                                                                  // block that a second group lacks is asked for, whose offset lies inside)
    return Row{ok, chunk * BK, !T::SPREAD || ok ? (unsigned)(kd * 3 + u) * 3 * p.nout * p.red * 2 + chunk * b_chunk : 0};
  };
  auto load_b = [&](const Row& r, int buf, int j) {
    load_lds16(rs_b, ldsB_w + buf * T::B_STAGE + j * NTHREADS * 16, r.ok && r.c0 + b_k[j] < p.red ? b_off[j] : DMA_OOB, r.so);
  };
  auto fetch_b = [&](int lb, int u, int buf) {
    const Row r = row_b(lb, u);
#pragma unroll
    for (int j = 0; j < BV; ++j) load_b(r, buf, j);
  };

  // ---- LDS read addresses: per 32-position group and tap the pixel, or the zeros ----
  int a_rd[TM][9], a_d[TM];                                       // a_d: depth of the lane's position
  const int a_zero = npix * 64 + (lane & 3) * 64;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = wm * T::WTM + i * 32 + (lane & 31);
    const unsigned t = (unsigned)(m0 + r < p.M ? m0 + r : 0);     // M < 2^31: flat_eligible
    const int w = (int)(t % (unsigned)W), h = (int)((t / (unsigned)W) % (unsigned)H);
    a_d[i] = P3D ? (int)((t / (unsigned)W / (unsigned)H) % (unsigned)p.osp[0]) : 0;
#pragma unroll
    for (int kh = 0; kh < 3; ++kh)
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const int pix = r + kh * W + kw;
        const bool in = (unsigned)(h + kh - 1) < (unsigned)H && (unsigned)(w + kw - 1) < (unsigned)W;
        const int at = pix * 64 + ((half ^ ((pix >> 2) & 3)) << 4);
        a_rd[i][kh * 3 + kw] = in ? at : T::SPREAD ? npix * 64 + (at & 255) : a_zero;
      }
  }
  // data gradient: per 16 channels of the reduction; forward: their first four rows of the lane's half, and the next four
  int b_rd[TN][2];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int nr = wn * T::WTN + j * 32 + (lane & 31);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (FLIP) {
        b_rd[j][i] = nr * 64 + (((i * 2 + half) ^ ((nr >> 2) & 3)) << 4);
      } else {
        const int li = lane & 15, lg = lane >> 4, row = (lg >> 1) * 8 + (li >> 2) + 4 * i, pair = wn * (T::WTN / 16) + j * 2 + (lg & 1);
        b_rd[j][i] = row * T::BN * 2 + ((T::BN == 64 ? pair ^ (row & 2) : pair) << 5) + (li & 3) * 8;
      }
    }
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // Stage st = 3 lb + u multiplies filter row u of the group's block lb.  It asks for the input of block lb + 1 (at u = 0,
  // into the buffer of block lb - 1), then for the filter row NB - 1 stages on; so when stage st begins, what it needs is
  // older than the filter rows asked for in the NB - 2 stages before it, and than the next input among them.
  // SPREAD: with three buffers or more the loads go out a few at a time between the products, since with all at the head of a stage every wave of the
  // compute unit stands behind them before its first product; beyond the last block they write zeros, for a branch around them
  // costs what they gain.  With two buffers a load has one stage to arrive in and goes first, and so it does where a step is one product.
  const int nstages = 3 * nlocal;
  fetch_a(0);
#pragma unroll
  for (int st = 0; st < NB - 1; ++st)
    if (st < nstages) fetch_b(st / 3, st % 3, st);
  int a_cur[TM][9];                                               // addresses of the block: zeros where its plane is outside
  auto stage = [&](int lb, auto u_c, auto bbuf_c) {
    constexpr int u = decltype(u_c)::value, bbuf = decltype(bbuf_c)::value;
    const int left = nstages - 1 - (3 * lb + u);                  // stages after this one
    const bool more = lb + 1 < nlocal;
    constexpr bool a_newer = u > 0 && u <= NB - 2;                // the next input was asked for in the last NB - 2 stages
    constexpr int NEXT_A = u == 0 ? AV : 0, LOADS = NEXT_A + BV, PER = (LOADS + 5) / 6;
    if constexpr (T::SPREAD) wait_barrier<(NB - 2) * BV + (a_newer ? AV : 0)>();
    else if (left == 0) wait_barrier<0>();
    else if (a_newer && more) wait_barrier<(NB - 2) * BV + AV>();
    else wait_barrier<(NB - 2) * BV>();
    if (!T::SPREAD && u == 0 && more) fetch_a(lb + 1);
    if (!T::SPREAD && left >= NB - 1) {
      constexpr int fu = (u + NB - 1) % 3;
      fetch_b(lb + (u + NB - 1) / 3, fu, (bbuf + NB - 1) % NB);
    }
    if constexpr (P3D && u == 0) {
      const int kd = (lb * G + grp) % KD;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const bool in = (unsigned)(a_d[i] + kd - 1) < (unsigned)p.osp[0];
#pragma unroll
        for (int q = 0; q < 9; ++q) a_cur[i][q] = in ? a_rd[i][q] : a_zero;      // a whole plane: most lanes of a read
      }
    }
    const int (&ar)[TM][9] = P3D ? a_cur : a_rd;
    const Run ra = run_a(lb + 1);
    const Row rb = row_b(lb + (u + NB - 1) / 3, (u + NB - 1) % 3);
    const unsigned char* b = sB + bbuf * T::B_STAGE;
    const unsigned char* a = sA + (lb & 1) * abuf;
    // operands are read this many steps ahead of their products: with one product a step the LDS latency shows
    constexpr int NSTEP = 6, DEPTH = TM * TN == 1 ? 3 : 1;
    bf16x8 af[DEPTH + 1][TM], bfr[DEPTH + 1][TN];
    auto load = [&](int st) {
      const int tl = st / 2, ks = st % 2;
      const int tap = (FLIP ? 2 - u : u) * 3 + (FLIP ? 2 - tl : tl);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (FLIP) bfr[st % (DEPTH + 1)][j] = *reinterpret_cast<const bf16x8*>(b + b_rd[j][ks] + tl * T::BN * 64);
        else bfr[st % (DEPTH + 1)][j] = tr_frag(b + b_rd[j][0] + (tl * BK + ks * 16) * T::BN * 2, b + b_rd[j][1] + (tl * BK + ks * 16) * T::BN * 2);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) af[st % (DEPTH + 1)][i] = *reinterpret_cast<const bf16x8*>(a + (ar[i][tap] ^ (ks * 32)));
    };
#pragma unroll
    for (int st = 0; st < DEPTH; ++st) load(st);
#pragma unroll
    for (int st = 0; st < NSTEP; ++st) {
      if (st + DEPTH < NSTEP) load(st + DEPTH);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[st % (DEPTH + 1)][j], af[st % (DEPTH + 1)][i], acc[i][j], 0, 0, 0);
      if constexpr (T::SPREAD) {
#pragma unroll
        for (int q = st * PER; q < (st + 1) * PER && q < LOADS; ++q) {
          if (q < NEXT_A) load_a(ra, lb + 1, q);
          else load_b(rb, (bbuf + NB - 1) % NB, q - NEXT_A);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (T::SPREAD) return;
    constexpr int READS = TM + (FLIP ? TN : 2 * TN);
    __builtin_amdgcn_sched_group_barrier(0x100, READS * DEPTH, 0);
#pragma unroll
    for (int st = 0; st < NSTEP; ++st) {
      if (st + DEPTH < NSTEP) __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
    }
  };
  // three stages a block: the ring is where it was after NB blocks (three buffers: after each)
  constexpr int PERIOD = NB == 3 ? 1 : NB;
  for (int lb0 = 0; lb0 < nlocal; lb0 += PERIOD)
    unrolled<PERIOD>([&](auto b_c) {
      constexpr int bi = decltype(b_c)::value;
      if (lb0 + bi < nlocal) unrolled<3>([&](auto u) { stage(lb0 + bi, u, std::integral_constant<int, (3 * bi + decltype(u)::value) % NB>{}); });
    });
  if constexpr (T::SPREAD) wait_loads();                          // the zeros beyond the last block
  __syncthreads();                                                // LDS is free
  if constexpr (G > 1) {
    float4* sums = reinterpret_cast<float4*>(flat_smem);
    auto slot = [&](int g, int i, int j, int q) -> float4& { return sums[((((g - 1) * 4 + wave) * TM + i) * TN + j) * 256 + q * 64 + lane]; };
    if (grp > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            slot(grp, i, j, q) = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int g = 1; g < G; ++g)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float4 t = slot(g, i, j, q);
              acc[i][j][4 * q] += t.x; acc[i][j][4 * q + 1] += t.y; acc[i][j][4 * q + 2] += t.z; acc[i][j][4 * q + 3] += t.w;
            }
    }
    __syncthreads();
    if (grp > 0) return;
  }
  wave_epilogue<T::WTN, TM, TN>(p, eb, acc, flat_smem + wave * epi_wave_bytes(T::WTN), pre_add, pre_mask, n, n < p.nout, er, out_off);
}

template <typename T, bool P3D, bool FLIP>
hipError_t launch_flat_t(IgemmP& p, hipStream_t s) {
  const int ring = T::G * flat_group_lds<T>(p.osp[2]), epi = 4 * epi_wave_bytes(T::WTN), sums = (T::G - 1) * T::BM * T::BN * 4;
  int lds = ring > epi ? ring : epi;
  if (sums > lds) lds = sums;
  if (lds > 163840) return hipErrorInvalidValue;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_flat_kernel<T, P3D, FLIP>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
  if (attr != hipSuccess) return attr;
  p.ntiles_n = (p.nout + T::BN - 1) / T::BN;
  const long long mt = (p.M + T::BM - 1) / T::BM;
  if (mt * p.ntiles_n > 0x7fffff00LL) return hipErrorInvalidValue;
  p.ntiles = (int)(mt * p.ntiles_n);
  hipLaunchKernelGGL((conv_flat_kernel<T, P3D, FLIP>), dim3(8 * ((p.ntiles + 7) / 8)), dim3(T::NT), lds, s, p);
  return hipGetLastError();
}

typedef FlatTile<256, 64, 4, 1, 8, 2> Flat256x64;
typedef FlatTile<256, 64, 4, 1, 6, 3> Flat256x64n3;
typedef FlatTile<128, 64, 2, 2, 6, 2> Flat128x64;
typedef FlatTile<128, 64, 2, 2, 6, 3> Flat128x64n3;
typedef FlatTile<128, 64, 2, 2, 4, 4> Flat128x64n4;
typedef FlatTile<64, 64, 2, 2, 6, 3> Flat64;
typedef FlatTile<64, 64, 2, 2, 5, 3, 2> Flat64g2;
typedef FlatTile<256, 32, 4, 1, 8, 2> Flat256x32;
typedef FlatTile<128, 32, 4, 1, 6, 3> Flat128x32;

// The widest tile leaves room for a second work-group on a compute unit up to 87 positions a row.
bool wide_fits(int w) { return flat_group_lds<Flat256x64>(w) <= 81920; }

bool long_fits(int w) { return flat_group_lds<Flat256x32>(w) <= 81920; }    // 256 x 32: up to 119

long long flat_tiles(const IgemmP& p, int bm, int bn) { return ((p.M + bm - 1) / bm) * ((p.nout + bn - 1) / bn); }

// At most 32 output channels: tiles of 256 positions where two of their work-groups share a compute unit, unless tiles of 128
// all run at once (us, 256 / 128 positions: 2-D 16 -> 16, 62 x 31, batch 46 8.2 / 7.4; 32 <- 64, 96 x 96, batch 8 8.1 / 8.9;
// 64 -> 32, 120 x 120, batch 12 18.4 / 17.3).
bool narrow_256(const IgemmP& p) {
  const int w = p.osp[2];
  return long_fits(w) && flat_tiles(p, 256, 32) >= 256 && flat_tiles(p, 128, 32) > 256LL * (163840 / flat_group_lds<Flat128x32>(w));
}

// Layers that patches (conv_halo.hip) are faster on, us, this kernel (forward: with the filter packed first) / patches:
//   3-D, at most 32 outputs, up to 64 Ki positions: data gradients (24 <- 40, 16^3 9.4 / 8.3; 16 <- 208, 16^3 24 / 18) and, but for
//   short reductions on less than one tile per compute unit, forward passes (128 -> 16, 24 x 40 x 36 21 / 18; but
//   32 -> 32, 16^3 8.3 / 9.2); beyond one round of tiles where patches are full (64 -> 16, 80^3 64 / 59; but 48^3, 432 tiles, 18.7 / 22.3)
//   3-D, more outputs: long reductions on full patches of large volumes (192 -> 192, 80^3 855 / 811; but 64 -> 64 108 / 109)
//   2-D data gradients of one short block (16 <- 16, 112 x 112, batch 8 6.7 / 6.4); long reductions on full patches where rows
//   are too long for 256 x 64 (256 -> 256, 112 x 112, batch 16 248 / 240; but 104 x 104, 93 % full, 114 / 118); rows of 120
//   positions, where 256 x 32 does not fit either (256 -> 256, batch 12 227 / 215; 32 <- 64 19 / 18)
bool patches_win(const IgemmP& p) {
  if (!halo_eligible(p)) return false;
  const bool p3d = p.filt[0] == 3, dgrad = p.mode == 1;
  const double full = p3d ? patch_use(p, 4, 4, 8) : patch_use(p, 1, 8, 16);
  if (!p3d) {
    const int w = p.osp[2];
    if (!long_fits(w) && (p.red >= 192 || p.nout <= 32) && full >= 0.9) return true;
    return full >= 0.95 && ((dgrad && p.nout <= 32 && p.red <= 16 && p.M >= 65536) || (!wide_fits(w) && p.nout > 32 && p.red >= 192));
  }
  if (p.nout > 32) return p.red >= 128 && p.M >= 262144 && full >= 0.95;
  if (p.M <= 65536) return dgrad || p.red > 64 || p.M > 32768;
  return flat_tiles(p, 256, 32) > 512 && full >= 0.95;
}

// The longest ring that leaves room for a second work-group on a compute unit (us, forward / data gradient, ring of two, loads at the
// head of a stage / three, loads spread / four: 256 x 64: 256 -> 256, 14 x 14, batch 256 59.8 / 65.8, 56.6 / 63.6; 512 -> 512, 14 x 14, batch 96 87 / 96,
// 80 / 89; 128 -> 128, 28 x 28, batch 128 33.9 / 39.3, 31.7 / 37.9; 128 -> 128, 32^3 30.9 / 29.8, 28.1 / 28.7; 64 -> 64, 56 x 56, where
// three leave no room, 24 / 30 for one work-group.  128 x 64: 256 -> 256, 14 x 14, batch 32 15.6 / 19.1, 13.0 / 16.7, 11.4 / 15.5; 512 -> 512, 7 x 7, batch
// 64 27.3 / 32.4, 20.1 / 26.1, 18.3 / 24.2; 128 -> 128, 24^3 21.5 / 21.8, 20.0 / 19.0, 19.8 / 19.1).  With 128 x 64 one or two blocks of the
// reduction are over before a long ring pays (us, ring of two / three or four: forward 32 -> 104, 62 x 62, batch 5 6.35 / 6.65, 24 -> 72, 43 x 55, batch 9 6.3 / 6.5; data gradient
// 64 <- 56, 26 x 72, batch 25 8.6 / 8.9; 64 -> 64, 40 x 40, batch 32 8.1 / 7.8 by itself, but in a network 9.1 / 9.5).
template <typename T>
bool pair_fits(int w) { return flat_group_lds<T>(w) <= 81920 && flat_pixels(T::BM, w) <= T::MAXPIX; }
template <bool P3D, bool FLIP>
hipError_t launch_256x64(IgemmP& p, hipStream_t s) {
  if (pair_fits<Flat256x64n3>(p.osp[2])) return launch_flat_t<Flat256x64n3, P3D, FLIP>(p, s);
  return launch_flat_t<Flat256x64, P3D, FLIP>(p, s);
}
template <bool P3D, bool FLIP>
hipError_t launch_128x64(IgemmP& p, hipStream_t s) {
  const int blocks = (p.red + BK - 1) / BK * (P3D ? 3 : 1);
  if (blocks >= 3 && pair_fits<Flat128x64n4>(p.osp[2])) return launch_flat_t<Flat128x64n4, P3D, FLIP>(p, s);
  if (blocks >= 3 && pair_fits<Flat128x64n3>(p.osp[2])) return launch_flat_t<Flat128x64n3, P3D, FLIP>(p, s);
  if constexpr (P3D) return hipErrorInvalidValue;                 // rows of at most 87 (flat_eligible): three fit
  else return launch_flat_t<Flat128x64, P3D, FLIP>(p, s);
}

template <bool P3D, bool FLIP>
hipError_t launch_flat_f(IgemmP& p, hipStream_t s) {
  // us, forward / data gradient, rings of two and of three for 64 x 64 and the filter packed first; before: patches of 8 x 16 or 4 x 4 x 8 positions, or the general kernel where they fill badly.
  //                                                     before         256 x 64     128 x 64    64 x 64     64 x 64, two groups
  //   2-D 256 -> 256, 14 x 14, batch 256                81 / 85        65 / 68      69 / 73     89 / 93     107 / 118
  //   2-D 512 -> 512, 7 x 7, batch 256                  81 / 88        62 / 67      77 / 84     98 / 105    108 / 116
  //   2-D 96 -> 160, 23 x 21, batch 16                  15.4 / 17.6    17.0 / 20.6  15.0 / 17.5 14.4 / 14.6 18.6 / 15.3
  //   2-D 72 -> 40, 45 x 37, batch 3                    14.8 / 10.0    16.5 / 11.5  14.2 / 9.2  12.6 / 8.6  13.3 / 8.1
  //   3-D 128 -> 128, 32^3                              40 / 37        37 / 33      38 / 35     50 / 47     54 / 51
  //   3-D 256 -> 256, 16^3                              40 / 37        56 / 52      45 / 41     35 / 31     31 / 27
  //   3-D 96 -> 144, 13 x 13 x 12                       67 / 94        29 / 36      24 / 29     20 / 21     19 / 20
  //   2-D 512 -> 512, 7 x 7, batch 32                                                       25 / 30     23 / 27
  // So the widest tile of which there is one per compute unit; below that, the reduction is shared by two groups of
  // waves where it is long enough (8 blocks) to pay for adding their sums and one such work-group, all that a compute
  // unit holds, is enough for each (2-D 256 -> 256, 45 x 37, batch 3, 316 tiles: 21 / 17 us, with 128 x 64 18 / 13).
  // Where rows are too long for the widest tile, 256 x 32 has the shorter runs of filter and twice the tiles (us, 128 x 64 /
  // 256 x 32 / patches: 2-D 256 -> 256, 96 x 96, batch 24 284 / 268 / 263; 128 -> 128, 112 x 112, batch 16 76 / 73 / 73;
  // 96 -> 96, 112 x 112, batch 16 59 / 48 / 57).
  const bool wide = wide_fits(p.osp[2]);
  if (p.nout <= 32) return narrow_256(p) ? launch_flat_t<Flat256x32, P3D, FLIP>(p, s) : launch_flat_t<Flat128x32, P3D, FLIP>(p, s);
  if (!wide && long_fits(p.osp[2]) && flat_tiles(p, 256, 32) >= 512) return launch_flat_t<Flat256x32, P3D, FLIP>(p, s);
  if (wide && flat_tiles(p, 256, 64) >= 256) return launch_256x64<P3D, FLIP>(p, s);
  if (flat_tiles(p, 128, 64) >= 256) return launch_128x64<P3D, FLIP>(p, s);
  const int blocks = (p.red + BK - 1) / BK * (P3D ? 3 : 1);
  if (blocks >= 8) {
    if (flat_tiles(p, 64, 64) <= 256) return launch_flat_t<Flat64g2, P3D, FLIP>(p, s);
    if (flat_tiles(p, 64, 64) <= 512) return launch_128x64<P3D, FLIP>(p, s);
  }
  return launch_flat_t<Flat64, P3D, FLIP>(p, s);
}

}  // namespace

bool flat_eligible(const IgemmP& p) {
  static const bool off = getenv("LMS_NO_FLAT") != nullptr;   // tuning aid
  const bool p3d = p.filt[0] == 3;
  if (off || p.small || !aligned16(p) || (p.filt[0] != 1 && !p3d) || p.filt[1] != 3 || p.filt[2] != 3 || p.pad[0] != (p3d ? 1 : 0) || p.pad[1] != 1 || p.pad[2] != 1) return false;
  for (int i = 0; i < 3; ++i)
    if (p.stride[i] != 1 || p.asp[i] != p.osp[i]) return false;
  if ((p.red & 7) != 0 || (p.nout & 7) != 0 || p.osp[2] > 120 || p.M >= 0x7fffffffLL) return false;
  // Volumes of wider rows stay with patches: 64 -> 64 at 48 x 96 x 96 took 130 us with the 128 x 64 tile and 107 there, while
  // 64^3 took 61 with the 256 x 64 tile and 66 there.
  if (p3d && (!wide_fits(p.osp[2]) || 4LL * p.osp[1] * p.osp[2] * p.red >= 0x3fffffffLL)) return false;
  if (patches_win(p)) return false;
  return (long long)27 * p.nout * p.red < 0x3fffffffLL && 600LL * (p.red > p.nout ? p.red : p.nout) < 0x3fffffffLL;
}

hipError_t launch_flat(IgemmP& p, hipStream_t s) {
  if (split_eligible(p)) return launch_split(p, s);               // few tiles, or one for a compute unit
  if (p.filt[0] == 3) return p.mode == 1 ? launch_flat_f<true, true>(p, s) : launch_flat_f<true, false>(p, s);
  return p.mode == 1 ? launch_flat_f<false, true>(p, s) : launch_flat_f<false, false>(p, s);
}

}  // namespace lms
