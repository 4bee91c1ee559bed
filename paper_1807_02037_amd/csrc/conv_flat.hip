// 3x3 stride-1 convolutions that keep the extents (padding 1), 2-D, forward and data gradient.
//
// A tile is BM consecutive positions of the batch in memory order, whatever rows and images they belong to, so no
// tile is padded: patches of 8 x 16 positions are 77 % full on the 14 x 14, 28 x 28 and 7 x 7 maps of ResNet-50 and fill worse
// still on odd extents.  The input pixels that the nine taps of a tile touch are one contiguous run of BM + 2 W + 2 rows;
// for every block of 32 channels the run goes straight to LDS (buffer loads that write LDS) while the block before it is
// multiplied, and a tap is a shift by kh * W + kw pixels.  Where a tap leaves the image, the lane reads a pixel of zeros
// instead: its nine addresses are worked out once per tile.  The filter streams through a ring of LDS buffers one
// filter row (three taps x BN x 32 channels) a stage, one barrier each.  Products are taken transposed and leave through
// wave_epilogue.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"

namespace lms {

namespace {

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<N, I + 1>(f);
  }
}

template <int BM_, int BN_, int WM_, int WN_, int AVS_>
struct FlatTile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int AVS = AVS_;                                // input loads per thread in each of two stages of a channel block
  static constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  static_assert(WM * WN == 4, "four waves");
  static constexpr int BV = (3 * BN * 4 + NTHREADS - 1) / NTHREADS;       // filter loads per thread and stage
  static constexpr int B_STAGE = BV * NTHREADS * 16;
  static constexpr int NB = 2;                                    // filter ring
  static constexpr int MAXPIX = 2 * AVS * NTHREADS / 4;           // input pixels at most
  static constexpr int LPR = WTN / 8, RPI = 64 / LPR, QV = 32 / RPI;
};

// Input pixels of a tile, the pixel of zeros behind them (64 bytes, any slot), rounded to the 16 pixels a wave loads at once.
__host__ __device__ inline int flat_pixels(int bm, int w) { return (bm + 2 * w + 2 + 15) / 16 * 16; }
__host__ __device__ inline int flat_abuf(int bm, int w) { return flat_pixels(bm, w) * 64 + 256; }

template <typename T, bool FLIP>
__global__ __launch_bounds__(NTHREADS, 2) void conv_flat_kernel(IgemmP p) {
  constexpr int TM = T::TM, TN = T::TN, BV = T::BV, AVS = T::AVS, NB = T::NB;
  extern __shared__ __attribute__((aligned(256))) unsigned char flat_smem[];
  const int per_xcd = (p.ntiles + 7) / 8;
  const int tile = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (tile >= p.ntiles) return;
  const int n0 = (tile % p.ntiles_n) * T::BN;
  const long long m0 = (long long)(tile / p.ntiles_n) * T::BM;
  const int W = p.osp[2], H = p.osp[1];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / T::WN, wn = wave % T::WN, half = lane >> 5;

  // ---- LDS: filter ring, two input buffers (pixels, then zeros), a place for loads that nobody needs ----
  const int npix = flat_pixels(T::BM, W), abuf = flat_abuf(T::BM, W);
  unsigned char* sB = flat_smem;
  unsigned char* sA = flat_smem + NB * T::B_STAGE;
  const unsigned lds0 = (unsigned)(uintptr_t)flat_smem;           // LDS address: the low half of the generic one
  const unsigned ldsA = lds0 + NB * T::B_STAGE, ldsX = ldsA + 2 * abuf;
  if (tid < 32) *reinterpret_cast<uint4*>(sA + (tid >> 4) * abuf + npix * 64 + (tid & 15) * 16) = make_uint4(0, 0, 0, 0);

  // ---- operands of the epilogue, fetched ahead ----
  const int cg = (lane % T::LPR) * 8, n = n0 + wn * T::WTN + cg;
  const int er = wm * T::WTM + lane / T::LPR;
  const EpiBuffers eb(p, m0, (p.M - m0) * p.nout * 2);
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
  const long long arow0 = m0 - W - 1;
  const v4u rs_a = buffer_rsrc(p.A + arow0 * p.red, 0x7fffffff);  // rows outside the tensor are never asked for
  const unsigned a_off = (unsigned)((apix * p.red + ag * 8) * 2);
  unsigned a_in = 0;                                              // bit j: pixel apix + 64 j is a row of the tensor
#pragma unroll
  for (int j = 0; j < 2 * AVS; ++j) {
    const int pix = apix + j * (NTHREADS / 4);
    const long long row = arow0 + pix;
    if (pix < npix && row >= 0 && row < p.M) a_in |= 1u << j;
  }
  const unsigned ldsA_w = __builtin_amdgcn_readfirstlane(ldsA + wave * 1024), ldsX_u = __builtin_amdgcn_readfirstlane(ldsX);
  const int wpix = __builtin_amdgcn_readfirstlane(wave * 16);
  auto fetch_a = [&](int chunk, int part) {                       // part 0 or 1: AVS loads per thread each
    const bool ok = chunk * BK + ag * 8 < p.red;
#pragma unroll
    for (int jj = 0; jj < AVS; ++jj) {
      const int j = part * AVS + jj;
      const unsigned dst = j * (NTHREADS / 4) + wpix < npix ? ldsA_w + (chunk & 1) * abuf + j * NTHREADS * 16 : ldsX_u;   // uniform
      load_lds16(rs_a, dst, ok && ((a_in >> j) & 1) ? a_off : DMA_OOB, (unsigned)(j * (NTHREADS / 4) * p.red * 2 + chunk * (BK * 2)));
    }
  };
  // ---- filter loads: row (tap of the filter row, output channel), channel slot g at g ^ ((n >> 2) & 3) ----
  const v4u rs_b = buffer_rsrc(p.B, (long long)9 * p.nout * p.red * 2);
  unsigned b_off[BV];
  int b_k[BV];
#pragma unroll
  for (int j = 0; j < BV; ++j) {
    const int v = tid + j * NTHREADS, row = v >> 2, nr = row % T::BN, tl = row / T::BN;
    b_k[j] = ((v & 3) ^ ((nr >> 2) & 3)) * 8;
    b_off[j] = tl < 3 && n0 + nr < p.nout ? (unsigned)(((tl * p.nout + n0 + nr) * p.red + b_k[j]) * 2) : DMA_OOB;
  }
  const unsigned ldsB_w = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
  auto fetch_b = [&](int chunk, int u, int buf) {
    const unsigned so = (unsigned)u * 3 * p.nout * p.red * 2 + chunk * (BK * 2);
#pragma unroll
    for (int j = 0; j < BV; ++j)
      load_lds16(rs_b, ldsB_w + buf * T::B_STAGE + j * NTHREADS * 16, chunk * BK + b_k[j] < p.red ? b_off[j] : DMA_OOB, so);
  };

  // ---- LDS read addresses: per 32-position group and tap the pixel, or the zeros ----
  int a_rd[TM][9];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = wm * T::WTM + i * 32 + (lane & 31);
    const unsigned t = (unsigned)(m0 + r < p.M ? m0 + r : 0);     // host guarantees M < 2^31
    const int w = (int)(t % (unsigned)W), h = (int)((t / (unsigned)W) % (unsigned)H);
#pragma unroll
    for (int kh = 0; kh < 3; ++kh)
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const int pix = r + kh * W + kw;
        const bool in = (unsigned)(h + kh - 1) < (unsigned)H && (unsigned)(w + kw - 1) < (unsigned)W;
        a_rd[i][kh * 3 + kw] = in ? pix * 64 + ((half ^ ((pix >> 2) & 3)) << 4) : npix * 64 + (lane & 3) * 64;
      }
  }
  int b_rd[TN][2];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int nr = wn * T::WTN + j * 32 + (lane & 31);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) b_rd[j][ks] = nr * 64 + (((ks * 2 + half) ^ ((nr >> 2) & 3)) << 4);
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int nchunks = (p.red + BK - 1) / BK;
  fetch_b(0, 0, 0);
  fetch_a(0, 0);
  fetch_a(0, 1);
  // Filter row u of channel block `chunk`, the buffers of both as compile-time parities of the stage.  Order of the loads:
  // every stage asks for the next stage's filter row, then the first two stages of a block for half of the next
  // block's input each; so what the next stage needs is older than those AVS input loads.
  auto stage = [&](int chunk, auto u_c, auto bbuf_c, bool last) {
    constexpr int u = decltype(u_c)::value, bbuf = decltype(bbuf_c)::value;
    if (u == 0 || chunk + 1 >= nchunks) wait_barrier<0>();
    else wait_barrier<AVS>();
    if (!last) fetch_b(u == 2 ? chunk + 1 : chunk, (u + 1) % 3, bbuf ^ 1);
    if (u < 2 && chunk + 1 < nchunks) fetch_a(chunk + 1, u);
    const unsigned char* b = sB + bbuf * T::B_STAGE;
    const unsigned char* a = sA + (chunk & 1) * abuf;
    constexpr int NSTEP = 6, DEPTH = 1;
    bf16x8 af[DEPTH + 1][TM], bfr[DEPTH + 1][TN];
    auto load = [&](int st) {
      const int tl = st / 2, ks = st % 2;
      const int tap = (FLIP ? 2 - u : u) * 3 + (FLIP ? 2 - tl : tl);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[st % (DEPTH + 1)][j] = *reinterpret_cast<const bf16x8*>(b + b_rd[j][ks] + tl * T::BN * 64);
#pragma unroll
      for (int i = 0; i < TM; ++i) af[st % (DEPTH + 1)][i] = *reinterpret_cast<const bf16x8*>(a + (a_rd[i][tap] ^ (ks * 32)));
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
    }
    __builtin_amdgcn_sched_group_barrier(0x100, (TM + TN) * DEPTH, 0);
#pragma unroll
    for (int st = 0; st < NSTEP; ++st) {
      if (st + DEPTH < NSTEP) __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
    }
  };
  // three stages a block: the filter buffer's parity alternates from block to block
  for (int chunk = 0; chunk < nchunks; chunk += 2) {
    unrolled<3>([&](auto u) { stage(chunk, u, std::integral_constant<int, decltype(u)::value & 1>{}, chunk + 1 >= nchunks && decltype(u)::value == 2); });
    if (chunk + 1 < nchunks)
      unrolled<3>([&](auto u) { stage(chunk + 1, u, std::integral_constant<int, (decltype(u)::value + 1) & 1>{}, chunk + 2 >= nchunks && decltype(u)::value == 2); });
  }
  __syncthreads();                                                // LDS is free for the epilogue
  wave_epilogue<T::WTN, TM, TN>(p, eb, acc, flat_smem + wave * epi_wave_bytes(T::WTN), pre_add, pre_mask, n, n < p.nout, er, out_off);
}

template <typename T, bool FLIP>
hipError_t launch_flat_t(IgemmP& p, hipStream_t s) {
  const int ring = T::NB * T::B_STAGE + 2 * flat_abuf(T::BM, p.osp[2]) + 1024, epi = 4 * epi_wave_bytes(T::WTN);
  const int lds = ring > epi ? ring : epi;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_flat_kernel<T, FLIP>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
  if (attr != hipSuccess) return attr;
  p.ntiles_n = (p.nout + T::BN - 1) / T::BN;
  const long long mt = (p.M + T::BM - 1) / T::BM;
  if (mt * p.ntiles_n > 0x7fffff00LL || p.M >= 0x7fffffffLL) return hipErrorInvalidValue;
  p.ntiles = (int)(mt * p.ntiles_n);
  hipLaunchKernelGGL((conv_flat_kernel<T, FLIP>), dim3(8 * ((p.ntiles + 7) / 8)), dim3(NTHREADS), lds, s, p);
  return hipGetLastError();
}

template <bool FLIP>
hipError_t launch_flat_f(IgemmP& p, hipStream_t s) {
  auto tiles = [&](int bm, int bn) { return ((p.M + bm - 1) / bm) * ((p.nout + bn - 1) / bn); };
  // the widest tile leaves room for a second work-group on a compute unit up to 87 positions a row
  const bool wide = 2 * FlatTile<256, 64, 4, 1, 4>::B_STAGE + 2 * flat_abuf(256, p.osp[2]) + 1024 <= 81920;
  if (p.nout <= 32) return tiles(256, 32) >= 256 ? launch_flat_t<FlatTile<256, 32, 4, 1, 4>, FLIP>(p, s) : launch_flat_t<FlatTile<128, 32, 4, 1, 3>, FLIP>(p, s);
  if (wide && tiles(256, 64) >= 256) return launch_flat_t<FlatTile<256, 64, 4, 1, 4>, FLIP>(p, s);
  if (tiles(128, 64) >= 256) return launch_flat_t<FlatTile<128, 64, 2, 2, 3>, FLIP>(p, s);
  return launch_flat_t<FlatTile<64, 64, 2, 2, 3>, FLIP>(p, s);
}

}  // namespace

bool flat_eligible(const IgemmP& p) {
  static const bool off = getenv("LMS_NO_FLAT") != nullptr;   // tuning aid
  if (off || p.small || p.filt[0] != 1 || p.filt[1] != 3 || p.filt[2] != 3 || p.pad[0] != 0 || p.pad[1] != 1 || p.pad[2] != 1) return false;
  for (int i = 0; i < 3; ++i)
    if (p.stride[i] != 1 || p.asp[i] != p.osp[i]) return false;
  if ((p.red & 7) != 0 || (p.nout & 7) != 0 || p.osp[2] > 120) return false;
  return (long long)9 * p.nout * p.red < 0x3fffffffLL && 600LL * p.red < 0x3fffffffLL;
}

hipError_t launch_flat(IgemmP& p, hipStream_t s) { return p.mode == 1 ? launch_flat_f<true>(p, s) : launch_flat_f<false>(p, s); }

}  // namespace lms
