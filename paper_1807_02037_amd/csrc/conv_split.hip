// 3x3 and 3x3x3 stride-1 convolutions that keep the extents (padding 1), forward and data gradient, where there is at most one tile
// of 64 positions x 64 channels for a compute unit: the reduction of a tile is split among its four waves.
//
// Such layers are a serial chain of stages on every compute unit, and waves that share tiles of LDS go through it in step: without products
// the two-group tile of conv_flat.hip takes 39 of 47 us (512 -> 256 at 16^3), without loads 33, without reads from LDS 35, without barriers
// 40.  Here a wave owns the whole tile and every fourth unit of the reduction: one filter row (three taps) x 64 input channels.  It loads
// the unit's input (rows of positions, whole 128-byte lines) and its filter, four kilobytes a stage and five stages ahead, into LDS of its own, waits for
// nothing but its own loads, and reads one operand of 1 KiB a product, half of what four waves of 32 x 32 read.  At the end the four
// sums meet in LDS in the order of the waves.  No pipe is full: at 256 -> 256, 16^3 36 units of 33 KB arrive in 21.5 us, 55 B/ns on average of the 124 that
// four waves with as much in flight take from an L2; what fills the rest of its one round was not taken apart.
// us, forward / data gradient, conv_flat.hip / here: 256 -> 256 at 16^3 26.8 / 25.1, 23.1 / 21.4; 256 -> 256 at 14^3 21.9 / 22.1, 18.1 / 18.3;
// tiles of 32 positions: 192 -> 192 at 12^3 17.8 / 17.5, 12.6 / 13.3; 128 -> 128 at 16^3 13.6 / 13.2, 10.6 / 11.0; 64 -> 128 at 16^3 10.0 / 12.8, 7.8 / 10.3;
// 256 -> 256 at 14 x 14, batch 8 9.5 / 14.1, 8.1 / 13.0; 512 -> 512 at 7 x 7, batch 4 14.8 / 20.5, 14.2 / 17.2.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"

namespace lms {

namespace {


// At most N of this wave's memory loads may still be in flight, and its LDS reads have come back.
template <int N>
__device__ __forceinline__ void wait_own() {
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

constexpr int CB = 64, SPLIT_BN = 64, LINE = 128;                 // channels of a unit; output channels; bytes of a row in LDS
constexpr int STAGES = 6, B_STAGE = 4096, BV = 4;                 // of a unit; filter bytes and loads of a stage

template <int TM_>
struct SplitTile {
  static constexpr int TM = TM_, TN = 2, BM = 32 * TM, NB = 5;    // NB: filter stages in LDS
  static constexpr int AV = (BM + 2 + 7) / 8, A_BUF = AV * 1024;  // input loads of a unit, eight rows each
  static constexpr int ZEROS = 2 * A_BUF + NB * B_STAGE, WAVE_LDS = ZEROS + 256;
  static constexpr int SUMS = TM * TN * 4 * 4096, LDS = 4 * WAVE_LDS > SUMS + 4 * epi_wave_bytes(32) ? 4 * WAVE_LDS : SUMS + 4 * epi_wave_bytes(32);
};

__device__ __forceinline__ int row_swizzle(int row) { return (row >> 1) & 7; }

template <typename T, bool P3D, bool FLIP>
__global__ __launch_bounds__(256, 1) void conv_split_kernel(IgemmP p) {
  constexpr int TM = T::TM, TN = T::TN, AV = T::AV, NB = T::NB, KD = P3D ? 3 : 1;
  extern __shared__ __attribute__((aligned(256))) unsigned char split_smem[];
  const int tile = xcd_order(p.ntiles);
  if (tile < 0) return;
  const int n0 = (tile % p.ntiles_n) * SPLIT_BN, m0 = (tile / p.ntiles_n) * T::BM;
  const int H = p.osp[1], W = p.osp[2];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), half = lane >> 5;

  unsigned char* sA = split_smem + wave * T::WAVE_LDS;
  const unsigned ldsA = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)sA), ldsB = ldsA + 2 * T::A_BUF;

  // ---- operands of the epilogue, fetched ahead: wave b finishes block b of 32 x 32 ----
  const int bi = wave / TN, bj = wave % TN, n = n0 + bj * 32 + (lane & 3) * 8, er = bi * 32 + (lane >> 2);
  const bool mine = wave < TM * TN;
  const EpiBuffers eb(p, m0, mine ? (p.M - m0) * p.nout * 2 : 0);
  const unsigned col = n < p.nout ? (unsigned)(n * 2) : DMA_OOB;
  auto out_off = [&](int r) -> unsigned { return col + (unsigned)(r * p.nout * 2); };
  uint4 pre_add[2], pre_mask[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    pre_add[q] = EpiBuffers::get(eb.add, out_off(er + 16 * q));
    pre_mask[q] = EpiBuffers::get(eb.mask, out_off(er + 16 * q));
  }

  // ---- loads.  Unit: 64 channels of one input row of the filter (kd, kh).  Its input: rows m0 - 1 ... of that shift, 128 bytes each,
  // slot g at g ^ row_swizzle: rows before the tensor have offsets beyond it, as have those behind ----
  const int lr = lane >> 3, nunits = ((p.red + CB - 1) / CB) * KD * 3;
  const v4u rs_a = buffer_rsrc(p.A, p.M * p.red * 2), rs_b = buffer_rsrc(p.B, 9LL * KD * p.nout * p.red * 2);
  const int ch_e = ((lane & 7) ^ (lane >> 4)) * 8, ch_o = ch_e ^ 32;         // of even and odd loads
  auto fetch_a = [&](int u, int buf) {
    const int chunk = u / (3 * KD), kd = P3D ? u / 3 % 3 : 0, kh = u % 3;
    const int row = m0 - 1 + (kh - 1) * W + (P3D ? (kd - 1) * H * W : 0) + lr;
    const unsigned base = (unsigned)((row * p.red + chunk * CB) * 2);
    const bool ok = u < nunits;
    const unsigned e = ok && chunk * CB + ch_e < p.red ? base + ch_e * 2 : DMA_OOB, o = ok && chunk * CB + ch_o < p.red ? base + ch_o * 2 : DMA_OOB;
#pragma unroll
    for (int j = 0; j < AV; ++j) {
      const unsigned v = j & 1 ? o : e;
      load_lds16(rs_a, ldsA + buf * T::A_BUF + j * 1024, v == DMA_OOB ? v : v + (unsigned)(j * 16 * p.red), 0);
    }
  };
  // Filter, a stage: forward 32 input channels of a tap, as stored (rows of 64 output channels for the transpose read); data gradient
  // 32 output channels (rows of 64 of the reduction)
  const int nch = ((lane & 7) ^ ((lr & 2) << 1)) * 8;
  const unsigned b_fwd = n0 + nch < p.nout ? (unsigned)((lr * p.nout + n0 + nch) * 2) : DMA_OOB;
  const unsigned b_bwd_e = (unsigned)((lr * p.red + ch_e) * 2), b_bwd_o = (unsigned)((lr * p.red + ch_o) * 2);
  auto fetch_b = [&](int u, int s, int slot) {
    const int chunk = u / (3 * KD), kd = P3D ? u / 3 % 3 : 0, kh = u % 3, kw = s >> 1;
    const int tap = FLIP ? ((KD - 1 - kd) * 3 + 2 - kh) * 3 + 2 - kw : (kd * 3 + kh) * 3 + kw;
    const bool ok = u < nunits;
    const int r0 = (s & 1) * 32, base = FLIP ? n0 + r0 : chunk * CB + r0, rows = ok ? (FLIP ? p.nout : p.red) - base : 0;     // rows from base on
    unsigned so = ok ? (unsigned)(FLIP ? ((tap * p.nout + base) * p.red + chunk * CB) * 2 : (tap * p.red + base) * p.nout * 2) : 0;
    const unsigned step = (unsigned)(16 * (FLIP ? p.red : p.nout));
#pragma unroll
    for (int j = 0; j < BV; ++j) {
      unsigned v = b_fwd;
      if constexpr (FLIP) v = chunk * CB + (j & 1 ? ch_o : ch_e) < p.red ? (j & 1 ? b_bwd_o : b_bwd_e) : DMA_OOB;
      load_lds16(rs_b, ldsB + slot + j * 1024, j * 8 < rows ? v : DMA_OOB, j * 8 < rows ? so : 0);      // no scalar offset beyond the buffer
      so += step;
    }
  };
  const int nu = wave < nunits ? (nunits - wave + 3) / 4 : 0;     // units wave, wave + 4, ...
  if (nu > 0) {
    fetch_a(wave, 0);
#pragma unroll
    for (int s = 0; s < NB; ++s) fetch_b(wave, s, s * B_STAGE);
  }

  // ---- LDS read addresses ----
  if (lane < 16) *reinterpret_cast<uint4*>(sA + T::ZEROS + lane * 16) = make_uint4(0, 0, 0, 0);
  int a_off[TM][3], a_h[TM], a_d[TM];                             // per tap of a filter row
  bool a_w[TM][3];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = i * 32 + (lane & 31);
    const unsigned t = (unsigned)(m0 + r < p.M ? m0 + r : 0);
    const int w = (int)(t % (unsigned)W);
    a_h[i] = (int)((t / (unsigned)W) % (unsigned)H);
    a_d[i] = P3D ? (int)((t / (unsigned)W / (unsigned)H) % (unsigned)p.osp[0]) : 0;
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) {
      a_off[i][kw] = (r + kw) * LINE + ((half ^ row_swizzle(r + kw)) << 4);
      a_w[i][kw] = (unsigned)(w + kw - 1) < (unsigned)W;
    }
  }
  int b_rd[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    if constexpr (FLIP) {
      b_rd[j] = (lane & 31) * LINE + ((half ^ row_swizzle(lane & 31)) << 4);
    } else {
      const int li = lane & 15, lg = lane >> 4, row = (lg >> 1) * 8 + (li >> 2), pair = j * 2 + (lg & 1);
      b_rd[j] = row * LINE + ((pair ^ (row & 2)) << 5) + (li & 3) * 8;
    }
  }
  int a_cur[TM][3];
  auto unit_addresses = [&](int u, int buf) {
    const int kd = P3D ? u / 3 % 3 : 0, kh = u % 3;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const bool in = (unsigned)(a_h[i] + kh - 1) < (unsigned)H && (!P3D || (unsigned)(a_d[i] + kd - 1) < (unsigned)p.osp[0]);
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) a_cur[i][kw] = in && a_w[i][kw] ? a_off[i][kw] + buf * T::A_BUF : T::ZEROS + (a_off[i][kw] & 255);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // Operands of a stage.  Forward: 16-channel steps of the half, input and filter.  Data gradient: the filter of 32 output channels, all
  // four steps; the input of the tap with the first half.
  constexpr int NA = FLIP ? 4 : 2, NBF = FLIP ? 4 : 2;
  bf16x8 af[FLIP ? 3 : 2][NA][TM], bfr[2][NBF][FLIP ? 1 : TN];
  auto load = [&](auto s_c, int slot) {
    constexpr int s = decltype(s_c)::value, kw = s >> 1, hf = s & 1, set = s & 1, aset = FLIP ? kw : set;
    const unsigned char* b = sA + 2 * T::A_BUF + slot;
    if constexpr (FLIP) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) bfr[set][ks][0] = *reinterpret_cast<const bf16x8*>(b + (b_rd[0] ^ (ks * 32)));
      if constexpr (hf == 0)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int i = 0; i < TM; ++i) af[aset][ks][i] = *reinterpret_cast<const bf16x8*>(sA + (a_cur[i][kw] ^ (ks * 32)));
    } else {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[set][ks][j] = tr_frag(b + b_rd[j] + ks * 16 * LINE, b + b_rd[j] + (ks * 16 + 4) * LINE);
#pragma unroll
        for (int i = 0; i < TM; ++i) af[set][ks][i] = *reinterpret_cast<const bf16x8*>(sA + (a_cur[i][kw] ^ ((hf * 2 + ks) * 32)));
      }
    }
  };
  auto mul = [&](auto s_c) {
    constexpr int s = decltype(s_c)::value, kw = s >> 1, hf = s & 1, set = s & 1, aset = FLIP ? kw : set;
    if constexpr (FLIP) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i][hf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][ks][0], af[aset][ks][i], acc[i][hf], 0, 0, 0);
    } else {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][ks][j], af[set][ks][i], acc[i][j], 0, 0, 0);
    }
  };

  // Stage t multiplies what was read from LDS in stage t - 1, reads for stage t + 1 and asks for the filter of stage t + NB, into the place of
  // its own, which has been read; the next unit's input is asked for in the first stage of a unit.  A wave waits for nothing but its own loads.
  if (nu > 0) {
    unit_addresses(wave, 0);
    wait_own<(NB - 1) * BV>();
    load(std::integral_constant<int, 0>{}, 0);
    int slot = 0;
    for (int k = 0; k < nu; ++k) {
      const int u = wave + 4 * k, buf = k & 1;
      unrolled<STAGES>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        constexpr bool a_newer = s >= 1 && s <= NB - 1;           // than the filter of the next stage
        wait_own<(NB - 2) * BV + (a_newer ? AV : 0)>();
        fetch_b(s + NB < STAGES ? u : u + 4, (s + NB) % STAGES, slot);
        if constexpr (s == 0) fetch_a(u + 4, buf ^ 1);
        slot = slot == (NB - 1) * B_STAGE ? 0 : slot + B_STAGE;
        if constexpr (s == STAGES - 1) unit_addresses(u + 4, buf ^ 1);
        load(std::integral_constant<int, (s + 1) % STAGES>{}, slot);
        mul(s_c);
      });
    }
  }

  // ---- the four waves' sums of a block meet in LDS, in the order of the waves ----
  wait_barrier<0>();
  float4* sums = reinterpret_cast<float4*>(split_smem);
#pragma unroll
  for (int b = 0; b < TM * TN; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x16& a = acc[b / TN][b % TN];
      sums[(b * 4 + wave) * 256 + q * 64 + lane] = make_float4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
    }
  __syncthreads();
  if (!mine) return;
  f32x16 total[1][1];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float4 t = sums[wave * 4 * 256 + q * 64 + lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 o = sums[(wave * 4 + w) * 256 + q * 64 + lane];
      t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
    }
    total[0][0][4 * q] = t.x; total[0][0][4 * q + 1] = t.y; total[0][0][4 * q + 2] = t.z; total[0][0][4 * q + 3] = t.w;
  }
  wave_epilogue<32, 1, 1>(p, eb, total, split_smem + T::SUMS + wave * epi_wave_bytes(32), pre_add, pre_mask, n, n < p.nout, er, out_off);
}

template <typename T, bool P3D, bool FLIP>
hipError_t launch_split_t(IgemmP& p, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_split_kernel<T, P3D, FLIP>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
  if (attr != hipSuccess) return attr;
  p.ntiles_n = (p.nout + SPLIT_BN - 1) / SPLIT_BN;
  p.ntiles = (int)((p.M + T::BM - 1) / T::BM * p.ntiles_n);
  hipLaunchKernelGGL((conv_split_kernel<T, P3D, FLIP>), dim3((unsigned)xcd_grid(p.ntiles)), dim3(256), T::LDS, s, p);
  return hipGetLastError();
}

// Positions of a tile, 0: not here.  A unit is padded to 64 channels, so they have to be mostly there (72 -> 136 at 14 x 14, batch 10 6.1 / 6.5,
// 96 -> 96 at 20 x 20, batch 3 5.8 / 6.0, but at 10^3 48 -> 48 9.6 / 7.3).  Tiles of 32 positions fill the chip where there are too few of 64.  In the
// plane one tile of 64 positions a compute unit pays in long data gradients only (forward / data gradient 512 -> 512 at 7 x 7, batch 32 15.6 / 21.1,
// 16.2 / 19.9; 256 -> 256 at 14 x 14, batch 16 10.0 / 14.4, 9.9 / 14.4), and in volumes with units that are full (128 <- 96 at 20^3 12.2 / 13.0).  In
// the plane three units leave a wave idle and six the sums to pay for: forward passes of one block of 64 channels and data gradients of
// up to 160 channels lose (forward 64 -> 120 at 8 x 8, batch 5 4.6 / 5.1, 56 -> 88 at 9 x 9, batch 11 4.9 / 5.2; data gradient 112 <- 64 at 9 x 9,
// batch 4 7.9 / 8.4, 56 <- 160 at 10 x 10, batch 8 10.6 / 11.0, 344 <- 120 at 12 x 12, batch 3 6.4 / 6.6).
int split_rows(const IgemmP& p) {
  const bool p3d = p.filt[0] == 3;
  const long long cols = (p.nout + SPLIT_BN - 1) / SPLIT_BN, t32 = (p.M + 31) / 32 * cols, t64 = (p.M + 63) / 64 * cols;
  const int padded = (p.red + CB - 1) / CB * CB;
  if (p.nout <= 32 || t64 > 256 || (!p3d && p.red <= (p.mode == 1 ? 160 : CB))) return 0;
  if (t32 <= 256) return (p3d ? 4 * p.red >= 3 * padded : 5 * p.red >= 4 * padded) ? 32 : 0;
  return (p3d ? 4 * p.red > 3 * padded : p.mode == 1 && p.red >= 512) ? 64 : 0;
}

template <bool P3D, bool FLIP>
hipError_t launch_split_f(IgemmP& p, hipStream_t s) {
  if (split_rows(p) == 32) return launch_split_t<SplitTile<1>, P3D, FLIP>(p, s);
  if constexpr (P3D || FLIP) return launch_split_t<SplitTile<2>, P3D, FLIP>(p, s);
  else return hipErrorInvalidValue;                               // in the plane 64 positions are for data gradients: split_rows
}

}  // namespace

// Of the layers that conv_flat.hip takes; offsets into both tensors have 31 bits, rows before the first ones included.
bool split_eligible(const IgemmP& p) {
  const long long plane = (long long)p.osp[1] * p.osp[2];
  return split_rows(p) != 0 && (p.M + 2 * (plane + p.osp[2] + 128)) * p.red < 0x3fffffffLL && 27LL * p.nout * p.red < 0x3fffffffLL;
}

hipError_t launch_split(IgemmP& p, hipStream_t s) {
  if (p.filt[0] == 3) return p.mode == 1 ? launch_split_f<true, true>(p, s) : launch_split_f<true, false>(p, s);
  return p.mode == 1 ? launch_split_f<false, true>(p, s) : launch_split_f<false, false>(p, s);
}

}  // namespace lms
