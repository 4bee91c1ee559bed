// Pointwise (1x1 / 1x1x1, no padding) convolutions as one matrix product over channels-last rows:
//   forward          out[m][k] = epi(sum_c x[row(m)][c] * w[c][k])        (row(m): the input row under a stride)
//   data gradient    dx[row(m)][c] = epi(sum_k dy[m][k] * w[c][k])
//   transposed convolution with window = stride: see UP below.
//
// With the channel counts of CNN bottlenecks these layers are bound by the passes over the activations, or, on the small
// maps of the late stages, by how fast tiles can be fed: both ask for loads in flight.  Tiles of both operands go from
// memory straight to LDS (16-byte buffer loads that write LDS: no registers, no LDS store instructions; offsets beyond
// the descriptor read zeros, so ragged tiles need no branches), 64 reduction channels a stage (a whole 128-byte line of
// a row: with 32 every line crossed from the L2 twice) in two buffers with one barrier per stage; the second work-group
// of the compute unit covers what one stage of lookahead does not (with 128 x 128 three buffers and one work-group were
// 40 % slower; 256 x 128 has them, see launch_pw_shape).  The
// filter stays as it lies in memory: the forward pass reads its [c][k] tile with the gfx950 LDS transpose read, the data
// gradient reads rows [c][k] as they are ([n][r] for it).  A wave of the widest tile owns 64 x 64 outputs, one LDS read
// per product.  Products are taken transposed (filter fragment first): a lane holds four consecutive channels of a
// position and writes them to LDS as one vector; each wave turns 32 positions at a time through its own piece of LDS,
// without a barrier, and stores full lines.  The stores go around the L2s: a result is as large as what the L2s hold,
// and on its way through evicts the operand tiles that neighbouring work-groups share (forward 2048 -> 512 on 7 x 7 at
// batch 256 45 -> 34 us, data gradient 64 <- 256 on 56 x 56 at batch 128 86 -> 73 us; nowhere slower).
//
// Measured: see launch_pw_shape.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"

namespace lms {

namespace {


constexpr int PK = 64;        // reduction channels per stage
constexpr int SL = PK / 8;    // 16-byte slots of a row of PK channels
__device__ __forceinline__ int pw_swz(int row) { return (row >> 1) & 7; }

enum { PW_FWD = 0, PW_DGRAD = 1, PW_UP = 2 };

template <int BM_, int BN_, int WM_, int WN_, int BUFS_ = 2>
struct PwTile {
  static constexpr int BUFS = BUFS_;                              // stages in LDS
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int NT = 64 * WM * WN;                         // threads
  static constexpr int WTM = BM / WM, WTN = BN / WN;              // outputs of a wave
  static constexpr int TM = WTM / 32, TN = WTN / 32;
  static constexpr int A_BYTES = BM * PK * 2, B_BYTES = BN * PK * 2;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int AV = A_BYTES / (16 * NT), BV = B_BYTES / (16 * NT);   // loads per thread and stage
  static constexpr int EPI_WAVE = epi_wave_bytes(WTN);
  static constexpr int LDS_BYTES = BUFS * STAGE > WM * WN * EPI_WAVE ? BUFS * STAGE : WM * WN * EPI_WAVE;
  static constexpr int LPR = WTN / 8;                             // lanes per output row in the epilogue
  static constexpr int RPI = 64 / LPR;                            // rows per instruction
  static constexpr int QV = 32 / RPI;                             // vectors per lane and 32 positions
  static constexpr int OCC = 163840 / LDS_BYTES * (NT / 256) < 4 ? 163840 / LDS_BYTES * (NT / 256) : 4;   // waves per SIMD
};

// Row of the strided grid (extents big) under row m of the small one (extents small).
__device__ __forceinline__ long long pw_strided_row(long long m, const int* small, const int* big, const int* stride) {
  unsigned t = (unsigned)m;                                       // host guarantees M < 2^31
  const unsigned w = t % (unsigned)small[2]; t /= (unsigned)small[2];
  const unsigned h = t % (unsigned)small[1]; t /= (unsigned)small[1];
  const unsigned d = t % (unsigned)small[0]; t /= (unsigned)small[0];
  return (((long long)t * big[0] + d * stride[0]) * big[1] + h * stride[1]) * (long long)big[2] + w * stride[2];
}

// UP: transposed convolution with window = stride.  Every output position takes one filter tap (the parity of its
// coordinates), so the layer is one product of the input with taps x k virtual output channels: column n is channel
// n % k of tap n / k, filter element w[tap][c][n % k], written to the output position stride * input position + tap.
// The input tile is read once for all taps of a column tile, and the taps that differ in the last coordinate only are
// neighbours in memory, so their channels leave as one contiguous run.
// STRIDED: rows are gathered (forward) or scattered (data gradient: the positions a stride leaves under a dy row; the others, up
// to the next one along each axis, get the epilogue of zero from the same work-group behind the product, or from
// strided_rest_kernel).
template <typename T, int MODE, bool STRIDED>
__global__ __launch_bounds__(T::NT, T::OCC) void pw_kernel(IgemmP p) {
  constexpr bool UP = MODE == PW_UP;
  constexpr int BN = T::BN, PM = T::BM, TM = T::TM, TN = T::TN, AV = T::AV, BV = T::BV;
  constexpr int ROWB = BN * 2;                                    // bytes of a filter row of the [r][n] tile
  extern __shared__ __attribute__((aligned(16))) unsigned char pw_smem[];

  const int per_xcd = (p.ntiles + 7) / 8;
  const int tile = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (tile >= p.ntiles) return;
  const int nv = (UP ? p.up[0] * p.up[1] * p.up[2] : 1) * p.nout;           // columns, virtual ones included
  const int n0 = (tile % p.ntiles_n) * BN;
  const long long m0 = (long long)(tile / p.ntiles_n) * PM;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / T::WN, wn = wave % T::WN;
  const int half = lane >> 5, li = lane & 15, lg = lane >> 4;

  // ---- operand of the epilogue: row and column of this lane's vectors; output rows relative to that of m0 ----
  const int cg = (lane % T::LPR) * 8, n = n0 + wn * T::WTN + cg;
  const int er = wm * T::WTM + lane / T::LPR;                     // tile row of vector (0, 0)
  __shared__ unsigned s_row[UP || (STRIDED && MODE == PW_DGRAD) ? PM : 1];
  __shared__ unsigned s_left[STRIDED && MODE == PW_DGRAD ? PM : 1];   // rest: positions along each axis, 8 bits each
  long long o_base = m0;                                          // output row that s_row counts from
  if constexpr (UP || (STRIDED && MODE == PW_DGRAD)) {
    const int* big = p.osp;
    const int* st = UP ? p.up : p.stride;
    o_base = pw_strided_row(m0, p.asp, big, st);
    if (tid < PM) s_row[tid] = (unsigned)(pw_strided_row(m0 + tid < p.M ? m0 + tid : m0, p.asp, big, st) - o_base);
    if (STRIDED && MODE == PW_DGRAD && tid < PM) {
      unsigned t = (unsigned)(m0 + tid), left = 0;
#pragma unroll
      for (int i = 2; i >= 0; --i) {
        const int at = (int)(t % (unsigned)p.asp[i]) * st[i];
        t /= (unsigned)p.asp[i];
        left = left << 8 | (unsigned)(big[i] - at < st[i] ? big[i] - at : st[i]);
      }
      s_left[tid] = m0 + tid < p.M ? left : 0;
    }
    __syncthreads();
  }
  long long up_tap = 0;                                           // UP: this lane's columns lie in one tap
  int up_n = n;
  if (UP && n < nv) {
    int t = n / p.nout;
    up_n = n - t * p.nout;
    const int tw = t % p.up[2]; t /= p.up[2];
    const int th = t % p.up[1];
    up_tap = ((long long)(t / p.up[1]) * p.osp[1] + th) * p.osp[2] + tw;
  }
  const long long o_rows = UP || (STRIDED && MODE == PW_DGRAD) ? p.M_out - o_base : p.M - m0;
  const EpiBuffers eb(p, o_base, o_rows * p.nout * 2);
  const unsigned col = n < nv ? (unsigned)((up_tap * p.nout + up_n) * 2) : DMA_OOB;
  auto out_off = [&](int r) -> unsigned {
    if constexpr (UP || (STRIDED && MODE == PW_DGRAD)) return m0 + r < p.M ? col + s_row[r] * (unsigned)(p.nout * 2) : DMA_OOB;
    else return col + (unsigned)(r * p.nout * 2);                 // rows beyond the last lie beyond the buffer
  };
  constexpr int EV = TM * T::QV;
  uint4 pre_add[EV], pre_mask[EV];
#pragma unroll
  for (int q = 0; q < EV; ++q) {
    const unsigned o = out_off(er + (q / T::QV) * 32 + (q % T::QV) * T::RPI);
    pre_add[q] = EpiBuffers::get(eb.add, o);
    pre_mask[q] = EpiBuffers::get(eb.mask, o);
  }

  // ---- loads: vector v of a stage's tile goes to LDS bytes [16 v, 16 v + 16); which channels it holds is permuted within
  // a row so that the reads below fall into different banks ----
  const long long a_row0 = STRIDED && MODE == PW_FWD ? pw_strided_row(m0, p.osp, p.asp, p.stride) : m0;
  const long long a_rows = STRIDED && MODE == PW_FWD ? p.M_in - a_row0 : p.M - m0;
  v4u rs_a = buffer_rsrc(p.A + a_row0 * p.red, a_rows * p.red * 2), rs_b = buffer_rsrc(p.B, (long long)nv * p.red * 2);
  if constexpr (STRIDED && MODE == PW_DGRAD)                      // the same for all lanes, which the compiler loses sight of here
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      rs_a[i] = __builtin_amdgcn_readfirstlane(rs_a[i]);
      rs_b[i] = __builtin_amdgcn_readfirstlane(rs_b[i]);
    }
  const unsigned lds0 = (unsigned)(uintptr_t)pw_smem;             // LDS address: the low half of the generic one
  unsigned a_off[AV], b_off[BV];
  int a_k[AV], b_k[BV];                                           // reduction channel of the vector within the stage
#pragma unroll
  for (int j = 0; j < AV; ++j) {
    const int v = tid + j * T::NT, row = v / SL;
    a_k[j] = ((v % SL) ^ pw_swz(row)) * 8;
    long long src = row;
    if constexpr (STRIDED && MODE == PW_FWD) src = pw_strided_row(m0 + row < p.M ? m0 + row : m0, p.osp, p.asp, p.stride) - a_row0;
    a_off[j] = m0 + row < p.M ? (unsigned)((src * p.red + a_k[j]) * 2) : DMA_OOB;
  }
#pragma unroll
  for (int j = 0; j < BV; ++j) {
    const int v = tid + j * T::NT;
    if constexpr (MODE == PW_DGRAD) {                             // rows n of PK reduction channels
      const int row = v / SL;
      b_k[j] = ((v % SL) ^ pw_swz(row)) * 8;
      b_off[j] = n0 + row < nv ? (unsigned)(((n0 + row) * p.red + b_k[j]) * 2) : DMA_OOB;
    } else {                                                      // rows r of BN columns
      const int r = v / (BN / 8), slot = v % (BN / 8);
      const int blk = (slot >> 2) ^ (BN == 128 ? r & 3 : (r >> 1) & 1);
      const int col = n0 + blk * 32 + (slot & 3) * 8;
      b_k[j] = r;
      const int t = UP ? col / p.nout : 0;
      b_off[j] = col < nv ? (unsigned)(((t * p.red + r) * p.nout + col - t * p.nout) * 2) : DMA_OOB;
    }
  }
  const unsigned a_step = PK * 2, b_step = MODE == PW_DGRAD ? PK * 2 : (unsigned)(PK * p.nout * 2);
  const int niter = (p.red + PK - 1) / PK;
  const unsigned lds_w = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
  // the last stage may be partial: zeros, whatever lies behind, and nothing but zeros in the stages after it (whose scalar offset is 0: one
  // beyond the buffer would have to be compared with what is left of it)
  auto load_a = [&](int it, int buf, int j) {
    const bool whole = (it + 1) * PK <= p.red;
    load_lds16(rs_a, lds_w + buf * T::STAGE + j * T::NT * 16, whole || it * PK + a_k[j] < p.red ? a_off[j] : DMA_OOB, it < niter ? it * a_step : 0);
  };
  auto load_b = [&](int it, int buf, int j) {
    const bool whole = (it + 1) * PK <= p.red;
    load_lds16(rs_b, lds_w + buf * T::STAGE + T::A_BYTES + j * T::NT * 16, whole || it * PK + b_k[j] < p.red ? b_off[j] : DMA_OOB, it < niter ? it * b_step : 0);
  };
  auto fetch = [&](int it, int buf) {
#pragma unroll
    for (int j = 0; j < AV; ++j) load_a(it, buf, j);
#pragma unroll
    for (int j = 0; j < BV; ++j) load_b(it, buf, j);
  };

  // ---- LDS read addresses ----
  int a_rd[PK / 16], b_rd[TN][PK / 16];
  {
    const int row = wm * T::WTM + (lane & 31);
#pragma unroll
    for (int ks = 0; ks < PK / 16; ++ks) a_rd[ks] = row * (PK * 2) + (((ks * 2 + half) ^ pw_swz(row)) << 4);
  }
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int ks = 0; ks < PK / 16; ++ks) {
      if constexpr (MODE == PW_DGRAD) {
        const int row = wn * T::WTN + j * 32 + (lane & 31);
        b_rd[j][ks] = row * (PK * 2) + (((ks * 2 + half) ^ pw_swz(row)) << 4);
      } else {
        const int r = ks * 16 + 8 * (lg >> 1) + (li >> 2);
        const int blk = (wn * TN + j) ^ (BN == 128 ? r & 3 : (r >> 1) & 1);
        b_rd[j][ks] = r * ROWB + blk * 64 + 32 * (lg & 1) + 8 * (li & 3);
      }
    }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  constexpr int AHEAD = T::BUFS - 1;                              // stages asked for ahead
#pragma unroll
  for (int it = 0; it < AHEAD; ++it) fetch(it, it);               // red >= 32: pw_channels
  auto stage = [&](int it, auto buf_c) {
    constexpr int buf = decltype(buf_c)::value, next = (buf + AHEAD) % T::BUFS;
    // stage `it` has landed; the barrier says so for every wave, and that every wave is done with the buffer that the
    // next request writes.  With three buffers the loads go out between the products, beyond the last stage too (no branch).
    constexpr bool SPREAD = T::BUFS > 2;
    wait_barrier<(AHEAD - 1) * (AV + BV)>();
    if (!SPREAD && it + 1 < niter) fetch(it + 1, next);
    const unsigned char* a = pw_smem + buf * T::STAGE;
    const unsigned char* b = a + T::A_BYTES;
    constexpr int NKS = PK / 16;
    bf16x8 af[2][TM], bfr[2][TN];                                 // operands are read one step ahead of their products
    auto load = [&](int ks) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (MODE == PW_DGRAD) bfr[ks & 1][j] = *reinterpret_cast<const bf16x8*>(b + b_rd[j][ks]);
        else bfr[ks & 1][j] = tr_frag(b + b_rd[j][ks], b + b_rd[j][ks] + 4 * ROWB);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) af[ks & 1][i] = *reinterpret_cast<const bf16x8*>(a + a_rd[ks] + i * 64 * PK);
    };
    load(0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      if (ks + 1 < NKS) load(ks + 1);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks & 1][j], af[ks & 1][i], acc[i][j], 0, 0, 0);
      if constexpr (SPREAD) {
        constexpr int PER = (AV + BV + NKS - 1) / NKS;
#pragma unroll
        for (int q = ks * PER; q < (ks + 1) * PER && q < AV + BV; ++q) {
          if (q < BV) load_b(it + AHEAD, next, q);
          else load_a(it + AHEAD, next, q - BV);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (SPREAD) return;
    constexpr int NRD = TM + (MODE == PW_DGRAD ? 1 : 2) * TN;     // LDS reads of a step
    __builtin_amdgcn_sched_group_barrier(0x100, NRD, 0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      if (ks + 1 < NKS) __builtin_amdgcn_sched_group_barrier(0x100, NRD, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
    }
  };
  for (int it = 0; it < niter; it += T::BUFS)
    unrolled<T::BUFS>([&](auto k) {
      if (it + decltype(k)::value < niter) stage(it + decltype(k)::value, k);
    });
  if constexpr (T::BUFS > 2) wait_loads();
  __syncthreads();                                                // the ring is free for the epilogue

  wave_epilogue<T::WTN, TM, TN>(p, eb, acc, pw_smem + wave * T::EPI_WAVE, pre_add, pre_mask, UP ? up_n : n, n < nv, er, out_off);

  if constexpr (STRIDED && MODE == PW_DGRAD) {
    if (!p.rest) return;
    constexpr int VPR = BN / 8, RL = T::NT / VPR, RV = PM / RL < 4 ? PM / RL : 4;   // vectors of a row, rows side by side, rows at a time
    const int rn = n0 + tid % VPR * 8;
    const EpiCoef none = {};
    const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int ad = 0; ad < p.stride[0]; ++ad)
      for (int ah = 0; ah < p.stride[1]; ++ah)
        for (int aw = 0; aw < p.stride[2]; ++aw) {
          if ((ad | ah | aw) == 0) continue;
          const unsigned delta = (unsigned)((ad * p.osp[1] + ah) * p.osp[2] + aw);
          for (int r0 = tid / VPR; r0 < PM; r0 += RV * RL) {
            unsigned o[RV];
            uint4 a[RV], m[RV];
#pragma unroll
            for (int v = 0; v < RV; ++v) {
              const unsigned left = s_left[r0 + v * RL];
              const bool ok = rn < p.nout && ad < (int)(left & 255) && ah < (int)(left >> 8 & 255) && aw < (int)(left >> 16 & 255);
              o[v] = ok ? ((s_row[r0 + v * RL] + delta) * (unsigned)p.nout + (unsigned)rn) * 2u : DMA_OOB;
              a[v] = EpiBuffers::get(eb.add, o[v]);
              m[v] = EpiBuffers::get(eb.mask, o[v]);
            }
#pragma unroll
            for (int v = 0; v < RV; ++v) eb.put(o[v], epilogue_pack8(p, none, zero, a[v], m[v]));
          }
        }
  }
}

// Data gradient of a strided pointwise layer, the positions no dy row lies under: the epilogue of zero.  A pure stream
// (addend and mask in, dx out), one 8-channel vector per thread and round, rows of the grid in memory order.
__global__ __launch_bounds__(NTHREADS) void strided_rest_kernel(IgemmP p, long long rows, int vpr) {
  const long long total = rows * vpr, step = (long long)gridDim.x * NTHREADS;
  for (long long i = (long long)blockIdx.x * NTHREADS + threadIdx.x; i < total; i += step) {
    const long long row = i / vpr;
    unsigned t = (unsigned)row;                                   // host guarantees rows < 2^31
    const unsigned w = t % (unsigned)p.osp[2]; t /= (unsigned)p.osp[2];
    const unsigned h = t % (unsigned)p.osp[1]; t /= (unsigned)p.osp[1];
    const unsigned d = t % (unsigned)p.osp[0];
    if (w % p.stride[2] == 0 && h % p.stride[1] == 0 && d % p.stride[0] == 0) continue;
    uint4 addq = make_uint4(0, 0, 0, 0), maskq = addq;
    if (p.add) addq = *reinterpret_cast<const uint4*>(p.add + i * 8);
    if (p.mask) maskq = *reinterpret_cast<const uint4*>(p.mask + i * 8);
    EpiCoef none;
    const float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    __builtin_nontemporal_store(__builtin_bit_cast(v4u, epilogue_pack8(p, none, v, addq, maskq)), reinterpret_cast<v4u*>(p.out + i * 8));
  }
}

template <typename T, int MODE, bool STRIDED>
hipError_t launch_pw_t(IgemmP& p, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(pw_kernel<T, MODE, STRIDED>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
  if (attr != hipSuccess) return attr;
  const int npar = MODE == PW_UP ? p.up[0] * p.up[1] * p.up[2] : 1;
  p.ntiles_n = (npar * p.nout + T::BN - 1) / T::BN;
  const long long mt = (p.M + T::BM - 1) / T::BM;
  if (mt * p.ntiles_n > 0x7fffff00LL || p.M >= 0x7fffffffLL) return hipErrorInvalidValue;
  p.ntiles = (int)(mt * p.ntiles_n);
  const int grid = 8 * ((p.ntiles + 7) / 8);
  const int ring = p.red > PK || T::BUFS > 2 ? T::BUFS * T::STAGE : T::STAGE, epi = T::WM * T::WN * T::EPI_WAVE;
  hipLaunchKernelGGL((pw_kernel<T, MODE, STRIDED>), dim3(grid), dim3(T::NT), ring > epi ? ring : epi, s, p);
  return hipGetLastError();
}

typedef PwTile<128, 128, 2, 2> Tile0;
typedef PwTile<64, 128, 2, 2> Tile1;
typedef PwTile<128, 64, 2, 2> Tile2;
typedef PwTile<64, 64, 2, 2> Tile3;
typedef PwTile<256, 128, 4, 2, 3> Tile4;

// Tile by shape (us on ResNet-50 layers, three sets of tensors in turn so that nothing stays cached; batch 128 at 56 x 56 and
// 28 x 28, 256 below; before: 128-position tiles staged through registers, data gradients of narrowing layers on the general
// kernel with 64 x 128 tiles):
//                                           before   128x128  64x128  128x64  64x64
//   forward 64 -> 256, 56 x 56, residual      95       88       97      99     101     long stores: wide tiles
//   forward 1024 -> 256, 14 x 14              61       53       63      64      68     long reductions: fewest re-reads
//   forward 2048 -> 512, 7 x 7                50       34       48      48      49     (392 tiles of 128 x 128)
//   data gradient 64 <- 256, 56 x 56          89       93       85      73      72     64 channels: no wider than they are
//   data gradient 256 <- 64, 56 x 56         134      147      130     135     138     mask and addend in, short reduction:
//   data gradient 1024 <- 256, 14 x 14       105       96       89      91      93     more work-groups in flight
//   forward 400 -> 176, 16 x 21 x 24          14.4     12.4     11.0    11.8     9.8   few tiles: smaller ones fill the chip
// Products with a ReLU mask and at most 512 reduction channels take 64 x 128, others 128 x 128, and both step down to tiles of which there are at
// least 256, one per compute unit.  From 384 channels on masked ones take 128 x 128 too, but under a stride, where the last round of two a compute unit is at least three
// quarters full.  900 layers, time against 64 x 128: those 592 0.92 (three 3 to 6 % slower); of the others, up to 1.17, 182 lose and 59 would gain (us, data
// gradient 640 <- 384, 28 x 28, batch 128 107.3 / 97.5; 256 <- 512, batch 100 48.5 / 44.5, with addend 57.1 / 52.6; but 400 <- 464, 23 x 23, batch 31, 516
// tiles 18.2 / 21.2; 136 <- 512, 64 x 64, batch 4, 256 tiles 9.2 / 10.5; under a stride 256 <- 512, 56 x 56, batch 128 147.8 / 159.8).
//   Long reductions: what arrives in LDS is the bound, the rows of x that two work-groups share and the filter, which the L2s deliver
// behind the misses of the activations (a loop of nothing but these loads: 512 tiles of 128 rows x 2 KB once 27 us, twice with the filter
// 42, whatever number of stages ahead).  256 x 128 takes the filter half as often; one work-group of eight waves, three stages in LDS, loads between
// the products: see long_lines.

// 256 x 128 tiles, of which a compute unit holds one: where the activation comes from memory (from 88 MB on three of them exceed the last-level
// cache) in whole lines and the columns fill their tiles by more than three quarters, or where there is one column of tiles and its last round is
// three quarters full.  1200 layers with at least 256 such tiles, time against 128 x 128 or 64 x 128: those 201 0.93 (two 3 to 4 % slower) and those 69 0.96
// (one 5 % slower); of the others, 0.83 to 1.52, 415 lose (us, forward 656 -> 752, 7 x 7, batch 221 17.2 / 26.2; 640 -> 256 at 256 x 140
// 22.5 / 24.9; data gradient 224 <- 784, 35 x 35, batch 28, addend 37.5 / 44.9) and 236 would gain.  Forward 1024 -> 256, 14 x 14, batch 256, residual
// 51.0 / 45.5 (all directions of the layer in turn 167 / 164); data gradient 256 <- 1024 56.9 / 51.5; beyond 512 columns the masks and addends of data gradients outweigh it (656 <- 1024 5 % slower).
bool long_lines(const IgemmP& p, long long cols, bool dgrad) {
  const long long ct = (cols + 127) / 128, tiles = (p.M + 255) / 256 * ct;
  if (tiles < 256 || 256LL * (p.red > p.nout ? p.red : p.nout) >= 0x3fffffffLL) return false;    // 32-bit offsets into the rows of a tile
  if (ct == 1) return p.red >= (dgrad ? 768 : 576) && 4 * tiles >= 3 * ((tiles + 255) / 256 * 256);
  return p.red >= 960 && (p.red & 63) == 0 && 2LL * p.M * p.red >= 88000000 && 4 * cols > 3 * 128 * ct && !(dgrad && cols > 512);
}

// 160 and 192 columns waste a quarter or more of two 128-wide tiles, and three of 64 store whole halves of lines, which those of 168 to 184
// columns do not (forward 48 -> 184, 108 x 108, batch 72 103 / 183 us).  It pays while the reduction is short and the epilogue has little to read and
// write.  1000 layers of 160 to 192 columns, reductions of 32 to 1024, time against 128 x 128 or 64 x 128: those 336 0.87 (four 2 to 5 % slower, all under a
// stride; us, forward 64 -> 160, 56 x 56, batch 11 8.6 / 5.9, 96 -> 192, batch 29 16.1 / 13.7; data gradient 160 <- 224, 14 x 14, batch 438 21.8 / 18.1);
// of the others 303 lose and 233 would gain.  Transposed convolutions store shorter pieces of rows and were not measured.
bool half_lines(const IgemmP& p, long long cols, long long rows) {
  const double bytes = 2.0 * (double)rows * p.nout * (1 + (p.add != nullptr) + (p.mask != nullptr));
  return cols > 152 && cols <= 192 && (cols & 31) == 0 && p.red <= 256 && (bytes <= 60e6 || (cols <= 160 && p.red <= 192)) && (p.M + 127) / 128 >= 256;
}

template <int MODE, bool STRIDED>
hipError_t launch_pw_shape(IgemmP& p, hipStream_t s) {
  const long long cols = (MODE == PW_UP ? (long long)p.up[0] * p.up[1] * p.up[2] : 1) * p.nout;
  auto tiles = [&](int bm, int bn) { return ((p.M + bm - 1) / bm) * ((cols + bn - 1) / bn); };
  if (cols <= 64) return tiles(128, 64) >= 256 ? launch_pw_t<Tile2, MODE, STRIDED>(p, s) : launch_pw_t<Tile3, MODE, STRIDED>(p, s);
  if (MODE != PW_UP && half_lines(p, cols, MODE == PW_DGRAD && STRIDED ? p.M_out : p.M)) return launch_pw_t<Tile2, MODE, STRIDED>(p, s);
  if constexpr (!STRIDED && MODE != PW_UP)
    if (long_lines(p, cols, MODE == PW_DGRAD)) return launch_pw_t<Tile4, MODE, STRIDED>(p, s);
  const bool narrow = p.mask && p.red <= 512 && (STRIDED || p.red < 384 || 4 * tiles(128, 128) < 3 * ((tiles(128, 128) + 511) / 512 * 512));
  if (!narrow && tiles(128, 128) >= 256) return launch_pw_t<Tile0, MODE, STRIDED>(p, s);
  return tiles(64, 128) >= 256 ? launch_pw_t<Tile1, MODE, STRIDED>(p, s) : launch_pw_t<Tile3, MODE, STRIDED>(p, s);
}

// Where the product's work-groups also write the positions between the strides, instead of a launch of its own: one launch
// less, and both halves of a row pair are in flight together.  us, apart / inside (stride 2, addend and mask): 256 <- 512, n 128,
// 56 x 56 169 / 149; 64 <- 128, n 32, 56 x 56 13.1 / 8.9; 256 <- 512, n 2, 14 x 14 10.8 / 7.8; 512 <- 128, n 64, 57 x 55 130 / 123.
// Beyond the caches the separate kernel's whole rows in memory order win where a tile's piece of a row is not whole
// lines (648 <- 400, n 32, 95 x 46 144 / 170; 440 <- 184, n 16, 68 x 100 73 / 86), and its streaming beside long reductions
// (512 <- 1024, n 128, 28 x 28 92.8 / 95.5).  Strides of more than 8 positions leave too few work-groups for the stream.
bool pw_rest_inside(const IgemmP& p) {
  if (p.stride[0] * (long long)p.stride[1] * p.stride[2] > 8) return false;
  const double bytes = 2.0 * (double)p.M * p.nout * (1 + (p.add != nullptr) + (p.mask != nullptr));
  return bytes <= 100e6 || ((p.nout & 63) == 0 && p.red <= 512);
}

// Data gradients under a stride: the general kernel or the product here.  Where the positions that no dy row lies under take a
// second launch, us, general / here (stride 2, batch n; 250 layers measured):
//   64 <- 128, n 16, 28 x 28   6.3 / 8.8       64 <- 128, n 32, 56 x 56   14 / 12       256 <- 512, n 2, 14 x 14   12.8 / 10.0
//   32 <- 64, n 16, 56 x 56    6.4 / 8.7       64 <- 128, n 128, 56 x 56  40 / 33       512 <- 256, n 2, 14 x 14   9.2 / 8.5
//   128 <- 192, n 6, 30 x 29   7.9 / 9.0       128 <- 192, n 16, 56 x 56  14 / 13       64 <- 512, n 6, 30 x 29    9.1 / 10.1
// So the second launch has to pay: 0.8 G products over all positions (2 G where few columns fill the tile badly: 48 <- 72,
// n 128, 56 x 56 32 / 35), or a filter so large that the general kernel waits for its long reductions.  Beyond the
// caches, tensors much wider than dy are bound by the writes, and it writes whole rows in order (1024 <- 64, n 64,
// 56 x 56 235 / 271; odd extents cost it more: 512 <- 128, n 64, 57 x 55 158 / 127).  With one launch in two dimensions the
// line is at 0.12 G: 176 <- 192, n 6, 40 x 41 9.1 / 6.7; 168 <- 296, n 4, 34 x 88 11.4 / 7.3; 128 <- 192, n 6, 30 x 29 8.2 / 7.6;
// 72 <- 64, n 1, 22 x 107 (0.01 G) 6.6 / 7.0.
bool strided_dgrad_general(const IgemmP& p) {
  const double macs = (double)p.M * p.nout * p.red;
  bool whole = true;
  for (int i = 0; i < 3; ++i) whole = whole && p.osp[i] % p.stride[i] == 0;
  if (p.nout >= 4 * p.red && p.M * p.nout >= (whole ? 100000000LL : 200000000LL)) return true;
  if ((long long)p.stride[0] * p.stride[1] * p.stride[2] <= 4 && pw_rest_inside(p)) return macs < 1.2e8 && (long long)p.nout * p.red < 100000;
  return macs < (p.nout < 64 && p.red < 128 ? 2e9 : 8e8) && (long long)p.nout * p.red < 100000;
}

bool pw_channels(const IgemmP& p, long long columns) {
  // 16-byte vectors of both operands, 32-bit offsets into the filter and into the 128 rows of a tile, tiles not mostly padding
  if (128LL * (p.red > p.nout ? p.red : p.nout) >= 0x3fffffffLL) return false;
  return !p.small && aligned16(p) && (p.red & 7) == 0 && (p.nout & 7) == 0 && p.nout >= 32 && p.red >= 32 && columns * p.red < 0x3fffffffLL;
}

}  // namespace

bool pw_eligible(const IgemmP& p) {
  static const bool off = getenv("LMS_NO_PW") != nullptr;   // tuning aid
  if (off || p.taps != 1) return false;
  bool strided = false;
  long long rows = 4LL * 256;                               // rows of the wider grid that a tile may span: 32-bit offsets from its first one
  for (int i = 0; i < 3; ++i) {
    if (p.filt[i] != 1 || p.stride[i] < 1 || p.pad[i] != 0) return false;
    rows *= p.stride[i];
    strided = strided || p.stride[i] != 1;
  }
  const int* big = p.mode == 0 ? p.asp : p.osp;
  if (strided && p.mode == 1 && strided_dgrad_general(p)) return false;
  rows += 2LL * p.stride[1] * big[2] + 2LL * p.stride[0] * big[1] * (long long)big[2];
  return pw_channels(p, p.nout) && (!strided || rows * (p.red > p.nout ? p.red : p.nout) < 0x3fffffffLL);
}

// Transposed convolution with window = stride (1 or 2 per axis), filter read as stored.
bool pw_up_eligible(const IgemmP& p) {
  static const bool off = getenv("LMS_NO_PW") != nullptr;   // tuning aid
  if (off) return false;
  for (int i = 0; i < 3; ++i)
    if (p.up[i] < 1 || p.up[i] > 2 || p.osp[i] != p.asp[i] * p.up[i]) return false;
  // output rows that a tile may span: 32-bit offsets from its first one
  const long long rows = 4LL * 256 * 8 + 4LL * p.osp[2] + 4LL * p.osp[1] * p.osp[2];
  return pw_channels(p, 8LL * p.nout) && rows * p.nout < 0x3fffffffLL;
}

hipError_t launch_pw(IgemmP& p, hipStream_t s) {
  if (p.up[0] > 0) {
    p.M_out = p.M * p.up[0] * p.up[1] * p.up[2];
    return launch_pw_shape<PW_UP, false>(p, s);
  }
  const bool strided = p.stride[0] != 1 || p.stride[1] != 1 || p.stride[2] != 1;
  if (p.mode == 0) {
    p.M_in = p.M / ((long long)p.osp[0] * p.osp[1] * p.osp[2]) * p.asp[0] * p.asp[1] * p.asp[2];
    if (strided) return launch_pw_shape<PW_FWD, true>(p, s);
    return launch_pw_shape<PW_FWD, false>(p, s);
  }
  if (!strided) return launch_pw_shape<PW_DGRAD, false>(p, s);
  const long long rows = p.M_out = p.M;                     // dx rows; the product runs over the dy rows
  p.rest = pw_rest_inside(p);
  if (rows >= 0x7fffffffLL) return hipErrorInvalidValue;
  p.M = rows / ((long long)p.osp[0] * p.osp[1] * p.osp[2]) * p.asp[0] * p.asp[1] * p.asp[2];
  if (p.rest) return launch_pw_shape<PW_DGRAD, true>(p, s);
  const int vpr = p.nout / 8;
  const long long blocks = (rows * vpr + NTHREADS * 4 - 1) / (NTHREADS * 4);
  hipLaunchKernelGGL(strided_rest_kernel, dim3((unsigned)(blocks < 1 ? 1 : (blocks > 65536 ? 65536 : blocks))), dim3(NTHREADS), 0, s, p, rows, vpr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_pw_shape<PW_DGRAD, true>(p, s);
}

}  // namespace lms
