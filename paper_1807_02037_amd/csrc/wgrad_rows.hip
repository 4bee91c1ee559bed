// Weight gradient of 1x1 (1x1x1) convolutions: dw[c][k] = sum over output positions of x[pos * stride][c] * dy[pos][k].
//
// Both operands lie position-major with channels contiguous (with a stride, the rows of x are gathered), and the reduction
// runs over positions: blocks of PB positions of both tensors go from memory straight to LDS as they lie (buffer loads that
// write LDS; rows and channels beyond the last read zeros), and the MFMA operands (8 consecutive positions per lane) are
// read with the gfx950 LDS transpose read.  A wave owns 64 x 64 filter entries, so a product needs one 16-byte LDS read.
// A work-group of eight waves, one per compute unit, covers TC x TK entries of the filter with G = 8 / (tiles of a wave)
// groups of waves: each group reduces its own blocks of positions (group g the blocks g, g + G, ...) through its own
// pair of LDS buffers, one barrier per round, and the groups' sums meet in LDS at the end.  So the partial filters that
// have to be written and read again number one per work-group and not one per group, and narrow filters (64 x 64: eight
// groups) keep all waves at work.  The partials of the work-groups are summed in a fixed order by the caller.
//
// Measured with the sums that follow, us (MI355X, ResNet-50 layers, three sets of tensors in turn; before: eight waves on one
// tile, blocks staged through two register sets, of which the compiler waited for both, tiles of a split on all XCDs):
//   1024 x 256 at 14 x 14, batch 256 53 -> 42; 256 x 512 stride 2 at 56 x 56, batch 128 69 -> 53; 512 x 2048 at 7 x 7, batch 256
//   51 -> 43; 64 x 256 at 56 x 56, batch 128 52 (257 MB: bound by memory); U-Net up-convolutions 64 -> 32 at 64^3 12 -> 8.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"

namespace lms {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));

constexpr int RT = 512;      // threads per work-group

// Position of a row in a grid, stepped by a constant number of rows without divisions.
struct RowPos {
  int n, d, h, w;
};
__host__ __device__ __forceinline__ RowPos row_pos(unsigned m, const int* sp) {
  RowPos q;
  q.w = m % (unsigned)sp[2]; m /= (unsigned)sp[2];
  q.h = m % (unsigned)sp[1]; m /= (unsigned)sp[1];
  q.d = m % (unsigned)sp[0];
  q.n = m / (unsigned)sp[0];
  return q;
}
__device__ __forceinline__ void row_step(RowPos& q, const RowPos& by, const int* sp) {
  q.w += by.w; q.h += by.h; q.d += by.d; q.n += by.n;
  if (q.w >= sp[2]) { q.w -= sp[2]; ++q.h; }
  if (q.h >= sp[1]) { q.h -= sp[1]; ++q.d; }
  if (q.d >= sp[0]) { q.d -= sp[0]; ++q.n; }
}

struct WRowsP {
  const uint16_t* X;
  const uint16_t* DY;
  float* part;
  long long rows;
  int cx, ky;
  int ctiles, ktiles, splits;
  int rows_per_split;        // multiple of the positions of a round
  int asp[3], osp[3], stride[3];   // strided variant: x is gathered at output position * stride
  // gathered-dy variant (weight gradient of a transposed convolution with window = stride): rows run over the
  // positions of x (extents asp), column j of the virtual dy is channel j % kk of tap j / kk, read at the output
  // position (extents osp) x-position * stride + tap
  int kk;
  RowPos step, vstep;        // both gathering variants: the rows of a round, and those between a thread's vectors, in extents
  // column sums of dy on the side (plain and strided variants): partial sums [split][ky], written by the
  // work-groups of the first channel tile of x; the caller adds them over the splits
  float* cs_part;
};

enum { ROWS_PLAIN = 0, ROWS_STRIDED_X = 1, ROWS_GATHERED_DY = 2 };

template <int TC_, int TK_, int PB_>
struct RowsTile {
  static constexpr int TC = TC_, TK = TK_, PB = PB_;         // PB: positions of a block
  static constexpr int WPG = (TC / 64) * (TK / 64);          // waves of a group
  static constexpr int G = 8 / WPG;
  static constexpr int GT = 64 * WPG;                        // threads of a group
  static constexpr int X_BYTES = PB * TC * 2, Y_BYTES = PB * TK * 2;
  static constexpr int XV = X_BYTES / (16 * GT), YV = Y_BYTES / (16 * GT);   // loads per thread and block
  static constexpr int BUF = X_BYTES + Y_BYTES;
  static constexpr int RING = G * 2 * BUF;
  static constexpr int SUMS = G * TC * TK * 4;               // the groups' sums
  static constexpr int LDS_BYTES = RING > SUMS ? RING : SUMS;
  static_assert(WPG * G == 8 && LDS_BYTES <= 163840, "eight waves, the LDS of a compute unit");
};

__device__ __forceinline__ bf16x8 tr_frag8(const unsigned char* p0, const unsigned char* p1) {
  const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p0);
  const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p1);
  const v8s r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// 64-byte blocks of row r of an LDS tile of T channels are permuted by this, so that the four rows of a transpose read
// fall into different quarters of the banks.
template <int T>
__device__ __forceinline__ int rows_swz(int r) { return T >= 128 ? r & 3 : (r >> 1) & 1; }

// CS: the work-groups of channel tile 0 of x also add up the rows of dy (every row of dy passes through exactly one of them
// per column tile): the bias / shift gradient as products of dy with a fragment of ones.
template <typename T, int MODE, bool CS>
__global__ __launch_bounds__(RT, 2) void wgrad_rows_kernel(WRowsP p) {
  static_assert(!CS || MODE != ROWS_GATHERED_DY, "column sums are kept for the plain and strided variants only");
  constexpr int TC = T::TC, TK = T::TK, PB = T::PB, G = T::G, XV = T::XV, YV = T::YV;
  constexpr int XVR = TC / 8, YVR = TK / 8;                  // vectors of a row
  constexpr int XRS = T::GT / XVR, YRS = T::GT / YVR;        // rows between a thread's vectors
  static_assert(XRS % 4 == 0 && YRS % 4 == 0, "a thread's rows have the same permutation");
  extern __shared__ __attribute__((aligned(256))) unsigned char lds_rows[];

  // the tiles of one split read the same rows: on one XCD they share them in its L2
  int b = p.ctiles * p.ktiles > 1 ? xcd_order(p.ctiles * p.ktiles * p.splits) : (int)blockIdx.x;
  if (b < 0 || b >= p.ctiles * p.ktiles * p.splits) return;
  const int ct = b % p.ctiles; b /= p.ctiles;
  const int kt = b % p.ktiles; b /= p.ktiles;
  const int split = b;
  const int c0 = ct * TC, k0 = kt * TK;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = wave / T::WPG, wq = wave % T::WPG, gt = tid - g * T::GT;
  const int wc = (wq % (TC / 64)) * 64, wk = (wq / (TC / 64)) * 64;
  const int li = lane & 15, lg = lane >> 4;

  const long long lo = (long long)split * p.rows_per_split;
  const long long hi = lo + p.rows_per_split < p.rows ? lo + p.rows_per_split : p.rows;
  const int rounds = hi > lo ? (int)((hi - lo + G * PB - 1) / (G * PB)) : 0;

  // ---- this thread's vectors of a block: LDS vector v of the tile (16 bytes) holds row v / XVR, permuted 64-byte block ----
  const int xr = gt / XVR, yr = gt % T::GT / YVR;
  auto column = [](int slot, int swz) { return ((slot >> 2) ^ swz) * 32 + (slot & 3) * 8; };
  const int xc = column(gt % XVR, rows_swz<TC>(xr)), yc = column(gt % YVR, rows_swz<TK>(yr));
  const bool x_ok = c0 + xc < p.cx, y_ok = k0 + yc < p.ky;
  unsigned x_off = x_ok ? (unsigned)((xr * p.cx + c0 + xc) * 2) : DMA_OOB;
  unsigned y_off = y_ok ? (unsigned)((yr * p.ky + k0 + yc) * 2) : DMA_OOB;
  // strided / gathered variants: where the thread's rows are, and the first of them in the wave (uniform; lane 0 has it), which
  // 32-bit offsets count from.  One division per extent finds a thread's first row, the others are stepped to: with
  // six positions found by division a small layer spent a third of its time on them ((2, 7, 9) 128 -> 64 10.1 us, now 9.6).
  constexpr int XP = MODE == ROWS_STRIDED_X ? XV : 1, YP = MODE == ROWS_GATHERED_DY ? YV : 1;
  RowPos xpos[XP], ypos[YP], first{};
  const int* small = MODE == ROWS_GATHERED_DY ? p.asp : p.osp;
  const int* big = MODE == ROWS_GATHERED_DY ? p.osp : p.asp;
  auto big_row = [&](const RowPos& q) {
    return (((long long)q.n * big[0] + q.d * p.stride[0]) * big[1] + q.h * p.stride[1]) * (long long)big[2] + q.w * p.stride[2];
  };
  unsigned y_tap = 0;
  auto positions = [&](RowPos* pos, int count, int row) {
    pos[0] = row_pos((unsigned)(lo + g * PB + row), small);
#pragma unroll
    for (int j = 1; j < count; ++j) {
      pos[j] = pos[j - 1];
      row_step(pos[j], p.vstep, small);
    }
    auto lane0 = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    first = RowPos{lane0(pos[0].n), lane0(pos[0].d), lane0(pos[0].h), lane0(pos[0].w)};
  };
  if constexpr (MODE == ROWS_STRIDED_X) positions(xpos, XV, xr);
  if constexpr (MODE == ROWS_GATHERED_DY) {
    positions(ypos, YV, yr);
    // the column lies in one tap (kk is a multiple of 8): offset of the tap within the output grid
    int t = y_ok ? (k0 + yc) / p.kk : 0;
    const int cc = y_ok ? k0 + yc - t * p.kk : 0;
    const int tw = t % p.stride[2]; t /= p.stride[2];
    const int th = t % p.stride[1];
    y_tap = (unsigned)(((((t / p.stride[1]) * p.osp[1] + th) * p.osp[2] + tw) * p.kk + cc) * 2);
  }

  const unsigned lds0 = (unsigned)(uintptr_t)lds_rows + g * 2 * T::BUF;          // this group's pair of buffers
  const unsigned lds_w = __builtin_amdgcn_readfirstlane(lds0 + wq * 1024);
  // block `r * G + g` of the split into buffer `buf`; rows from hi on lie beyond the buffers
  auto fetch = [&](int r, int buf) {
    const long long r0 = lo + (long long)(r * G + g) * PB;
    const long long left = r0 < hi ? hi - r0 : 0;
    const unsigned dst = lds_w + buf * T::BUF;
    long long big0 = 0;
    if constexpr (MODE != ROWS_PLAIN) {
      big0 = big_row(first);
      row_step(first, p.step, small);
    }
    if constexpr (MODE == ROWS_STRIDED_X) {
      const v4u rs = buffer_rsrc(p.X + big0 * p.cx, 0x7fffffff);
#pragma unroll
      for (int j = 0; j < XV; ++j) {
        const unsigned o = (unsigned)((big_row(xpos[j]) - big0) * p.cx * 2) + (unsigned)((c0 + xc) * 2);
        load_lds16(rs, dst + j * T::GT * 16, x_ok && xr + j * XRS < left ? o : DMA_OOB, 0);
        row_step(xpos[j], p.step, small);
      }
    } else {
      const v4u rs = buffer_rsrc(p.X + r0 * p.cx, left * p.cx * 2);
#pragma unroll
      for (int j = 0; j < XV; ++j) load_lds16(rs, dst + j * T::GT * 16, x_off + (unsigned)(j * XRS * p.cx * 2), 0);
    }
    if constexpr (MODE == ROWS_GATHERED_DY) {
      const v4u rs = buffer_rsrc(p.DY + big0 * p.kk, 0x7fffffff);
#pragma unroll
      for (int j = 0; j < YV; ++j) {
        const unsigned o = (unsigned)((big_row(ypos[j]) - big0) * p.kk * 2) + y_tap;
        load_lds16(rs, dst + T::X_BYTES + j * T::GT * 16, y_ok && yr + j * YRS < left ? o : DMA_OOB, 0);
        row_step(ypos[j], p.step, small);
      }
    } else {
      const v4u rs = buffer_rsrc(p.DY + r0 * p.ky, left * p.ky * 2);
#pragma unroll
      for (int j = 0; j < YV; ++j) load_lds16(rs, dst + T::X_BYTES + j * T::GT * 16, y_off + (unsigned)(j * YRS * p.ky * 2), 0);
    }
  };

  // ---- LDS read addresses: lane's row of a transpose read and its 8 bytes of a 64-byte block ----
  const int rd_row = 8 * (lg >> 1) + (li >> 2), rd_in = 32 * (lg & 1) + 8 * (li & 3);
  int x_rd[2], y_rd[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    x_rd[i] = rd_row * TC * 2 + (((wc / 32 + i) ^ rows_swz<TC>(rd_row)) << 6) + rd_in;
    y_rd[i] = T::X_BYTES + rd_row * TK * 2 + (((wk / 32 + i) ^ rows_swz<TK>(rd_row)) << 6) + rd_in;
  }

  f32x16 acc[2][2], cs[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc[i][0][v] = 0.f; acc[i][1][v] = 0.f; cs[i][v] = 0.f; }
  const bool cs_on = CS && ct == 0 && wc == 0;                // uniform over the wave
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.f;

  auto multiply = [&](const unsigned char* t) {
    constexpr int NKS = PB / 16;
    bf16x8 af[2][2], bfr[2][2];
    auto load = [&](int ks) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const unsigned char* a = t + x_rd[i] + ks * 16 * TC * 2;
        const unsigned char* q = t + y_rd[i] + ks * 16 * TK * 2;
        af[ks & 1][i] = tr_frag8(a, a + 4 * TC * 2);
        bfr[ks & 1][i] = tr_frag8(q, q + 4 * TK * 2);
      }
    };
    load(0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      if (ks + 1 < NKS) load(ks + 1);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks & 1][i], bfr[ks & 1][j], acc[i][j], 0, 0, 0);
      if (cs_on) {
#pragma unroll
        for (int j = 0; j < 2; ++j) cs[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, bfr[ks & 1][j], cs[j], 0, 0, 0);
      }
    }
  };

  if (rounds > 0) fetch(0, 0);
  const unsigned char* ring = lds_rows + g * 2 * T::BUF;
  for (int r = 0; r < rounds; r += 2) {
    wait_barrier<0>();                                        // the block of this round has landed, the other buffer is free
    if (r + 1 < rounds) fetch(r + 1, 1);
    multiply(ring);
    if (r + 1 < rounds) {
      wait_barrier<0>();
      if (r + 2 < rounds) fetch(r + 2, 0);
      multiply(ring + T::BUF);
    }
  }

  // ---- the groups' sums meet in LDS; every group adds its share of the entries, in the order of the groups, and stores it (group 0
  // alone adding and storing all of them cost small layers 1.5 us) ----
  constexpr int SHARE = 16 / G;
  float* sums = reinterpret_cast<float*>(lds_rows);
  float* out = p.part + (long long)split * p.cx * p.ky;
  auto own = [&](int q) {
    const f32x16& a = acc[q >> 3][(q >> 2) & 1];
    return make_float4(a[4 * (q & 3)], a[4 * (q & 3) + 1], a[4 * (q & 3) + 2], a[4 * (q & 3) + 3]);
  };
  auto slot = [&](int grp, int q) { return reinterpret_cast<float4*>(sums + grp * (TC * TK) + (wq * 16 + q) * 256 + lane * 4); };
  auto put = [&](int q, const float4& t) {
    const int c = c0 + wc + 32 * (q >> 3) + 8 * (q & 3) + 4 * (lane >> 5), k = k0 + wk + 32 * ((q >> 2) & 1) + (lane & 31);
    const float v[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < p.cx && k < p.ky) out[(long long)(c + e) * p.ky + k] = v[e];
  };
  auto plus = [](const float4& t, const float4& u) { return make_float4(t.x + u.x, t.y + u.y, t.z + u.z, t.w + u.w); };
  __syncthreads();
  if constexpr (G == 2) {                                     // a group keeps its own half
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (g != q / SHARE) *slot(g, q) = own(q);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (g == q / SHARE) put(q, plus(q < SHARE ? own(q) : *slot(0, q), q < SHARE ? *slot(1, q) : own(q)));
  } else {
#pragma unroll
    for (int q = 0; q < 16; ++q) *slot(g, q) = own(q);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SHARE; ++r) {
      const int q = g * SHARE + r;
      float4 t = *slot(0, q);
#pragma unroll
      for (int grp = 1; grp < G; ++grp) t = plus(t, *slot(grp, q));
      put(q, t);
    }
  }
  if (CS && ct == 0) {
    __syncthreads();                                          // the sums above have been read
    if (wc == 0 && lane < 32) {                               // every row of the product with ones is the sum: row 0
#pragma unroll
      for (int j = 0; j < 2; ++j) sums[g * TK + wk + 32 * j + lane] = cs[j][0];
    }
    __syncthreads();
    if (tid < TK && k0 + tid < p.ky) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < G; ++i) t += sums[i * TK + tid];
      p.cs_part[(long long)split * p.ky + k0 + tid] = t;
    }
  }
}

typedef RowsTile<128, 128, 64> Rows128;
typedef RowsTile<256, 64, 64> Rows256x64;
typedef RowsTile<64, 256, 64> Rows64x256;
typedef RowsTile<64, 128, 32> Rows64x128;
typedef RowsTile<128, 64, 32> Rows128x64;
typedef RowsTile<64, 64, 32> Rows64;

struct RowsPlan { int shape, ctiles, ktiles, splits, rows_per_split; };

RowsPlan rows_plan(long long rows, int cx, int ky) {
  // The shape with the least traffic: x is read once per k-tile, dy once per c-tile, mostly out of the L2 (counted at 0.7 of a
  // byte; 0.4 and 0.55 lose up to 10 % on long reductions), and every split writes a partial filter that is read again.
  // Long reductions take wide tiles, short ones under large filters narrow tiles with more groups of waves and fewer
  // splits (both gradients, us, by operand reads alone / this rule: 256 x 256 at 7680 rows 16.2 / 10.8, 1024 x 256 at 3136 16.0 / 13.3,
  // transposed convolution 256 -> 128 at 16^3 19.3 / 16.6 and 64 -> 32 at 32^3 22.3 / 13.9; 48 x 72 at 4096 8.8 / 9.5).
  static const int shapes[6][3] = {{64, 64, 256}, {64, 128, 128}, {128, 64, 128}, {128, 128, 128}, {256, 64, 128}, {64, 256, 128}};   // third: positions of a round
  RowsPlan best{};
  double best_cost = -1;
  for (int i = 0; i < 6; ++i) {
    const int ct = (cx + shapes[i][0] - 1) / shapes[i][0], kt = (ky + shapes[i][1] - 1) / shapes[i][1];
    const long long tiles = (long long)ct * kt, round = shapes[i][2];
    // at most one work-group of eight waves per CU, all that its LDS holds: 260 of them (432 x 616 at 10920 rows) took
    // 31 us, 240 20
    long long splits = 256 / tiles;
    const long long blocks = (rows + round - 1) / round;
    if (splits > blocks) splits = blocks;
    if (splits < 1) splits = 1;
    const long long per = ((blocks + splits - 1) / splits) * round;
    splits = (rows + per - 1) / per;
    if (splits < 1) splits = 1;
    // more tiles than compute units: whole rounds of them
    const double rounds = tiles > 256 ? (double)((tiles + 255) / 256) * 256. / (double)tiles : 1.;
    const double cost = 0.7 * rounds * 2. * (double)rows * ((double)cx * kt + (double)ky * ct) + 8. * (double)splits * cx * ky;
    if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = RowsPlan{i, ct, kt, (int)splits, (int)per}; }
  }
  return best;
}

template <typename T, int MODE, bool CS>
hipError_t launch_rows_t(WRowsP p, hipStream_t s) {
  const int* small = MODE == ROWS_GATHERED_DY ? p.asp : p.osp;
  p.step = row_pos(T::G * T::PB, small);
  p.vstep = row_pos(T::GT / ((MODE == ROWS_GATHERED_DY ? T::TK : T::TC) / 8), small);
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(wgrad_rows_kernel<T, MODE, CS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((wgrad_rows_kernel<T, MODE, CS>), dim3((unsigned)xcd_grid((long long)p.ctiles * p.ktiles * p.splits)), dim3(RT), T::LDS_BYTES, s, p);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_rows(const WRowsP& p, int mode, hipStream_t s) {
  if (mode == ROWS_GATHERED_DY) return launch_rows_t<T, ROWS_GATHERED_DY, false>(p, s);
  if (p.cs_part) return mode == ROWS_STRIDED_X ? launch_rows_t<T, ROWS_STRIDED_X, true>(p, s) : launch_rows_t<T, ROWS_PLAIN, true>(p, s);
  return mode == ROWS_STRIDED_X ? launch_rows_t<T, ROWS_STRIDED_X, false>(p, s) : launch_rows_t<T, ROWS_PLAIN, false>(p, s);
}
hipError_t launch_rows_shape(const WRowsP& p, int shape, int mode, hipStream_t s) {
  switch (shape) {
    case 0: return launch_rows<Rows64>(p, mode, s);
    case 1: return launch_rows<Rows64x128>(p, mode, s);
    case 2: return launch_rows<Rows128x64>(p, mode, s);
    case 3: return launch_rows<Rows128>(p, mode, s);
    case 4: return launch_rows<Rows256x64>(p, mode, s);
    default: return launch_rows<Rows64x256>(p, mode, s);
  }
}

}  // namespace

// Rows of the wider grid that a block of 64 positions may span, times its channels, and the 64 rows of the other operand: 32-bit
// offsets from the first one.
static bool rows_span_ok(const int* big, const int* stride, long long channels, long long other) {
  return 64 * other < 0x3fffffffLL && (64LL * stride[0] * stride[1] * stride[2] + 2LL * stride[0] * big[1] * big[2] + 2LL * stride[1] * big[2]) * channels < 0x3fffffffLL;
}

bool wgrad_rows_eligible(int cx, int ky, const int* asp, const int* filt, const int* stride, const int* pad) {
  if (getenv("LMS_NO_WGRAD_ROWS")) return false;
  for (int i = 0; i < 3; ++i)
    if (filt[i] != 1 || stride[i] < 1 || pad[i] != 0) return false;
  return (cx & 7) == 0 && (ky & 7) == 0 && cx >= 48 && ky >= 48 && rows_span_ok(asp, stride, cx, ky);
}

int wgrad_rows_splits(long long rows, int cx, int ky) { return rows_plan(rows, cx, ky).splits; }

hipError_t launch_wgrad_rows(const uint16_t* X, const uint16_t* DY, float* part, long long rows, int cx, int ky, const int* asp,
                             const int* osp, const int* stride, float* cs_part, hipStream_t s) {
  const RowsPlan pl = rows_plan(rows, cx, ky);
  if ((long long)pl.ctiles * pl.ktiles * pl.splits > 0x7fffff00LL || rows >= 0x7fffff00LL) return hipErrorInvalidValue;
  WRowsP p{};
  p.X = X; p.DY = DY; p.part = part; p.rows = rows; p.cx = cx; p.ky = ky; p.cs_part = cs_part;
  p.ctiles = pl.ctiles; p.ktiles = pl.ktiles; p.splits = pl.splits; p.rows_per_split = pl.rows_per_split;
  bool strided = false;
  for (int i = 0; i < 3; ++i) {
    p.asp[i] = asp[i]; p.osp[i] = osp[i]; p.stride[i] = stride[i];
    strided = strided || stride[i] != 1;
  }
  return launch_rows_shape(p, pl.shape, strided ? ROWS_STRIDED_X : ROWS_PLAIN, s);
}

// Weight gradient of a transposed convolution whose window equals its stride (1 or 2 per axis): every output
// position belongs to one tap, so dw[t][c][k] = sum over x-positions m of x[m][c] * dy[stride * m + t][k] is a
// pointwise weight gradient whose second operand has taps * kk virtual channels.  Partial results are
// [split][c][taps * kk]; the caller sums them into [t][c][k].
bool wgrad_rows_tconv_eligible(int cx, int kk, const int* osp, const int* filt, const int* stride) {
  if (getenv("LMS_NO_WGRAD_ROWS")) return false;
  long long taps = 1;
  for (int i = 0; i < 3; ++i) {
    if (filt[i] != stride[i] || stride[i] < 1 || stride[i] > 2) return false;
    taps *= filt[i];
  }
  return (cx & 7) == 0 && (kk & 7) == 0 && cx >= 48 && taps * kk >= 48 && rows_span_ok(osp, stride, kk, cx);
}

hipError_t launch_wgrad_rows_tconv(const uint16_t* X, const uint16_t* DY, float* part, long long rows, int cx, int kk, const int* asp,
                                   const int* osp, const int* stride, hipStream_t s) {
  const int ky = stride[0] * stride[1] * stride[2] * kk;
  const RowsPlan pl = rows_plan(rows, cx, ky);
  if ((long long)pl.ctiles * pl.ktiles * pl.splits > 0x7fffff00LL || rows >= 0x7fffff00LL) return hipErrorInvalidValue;
  WRowsP p{};
  p.X = X; p.DY = DY; p.part = part; p.rows = rows; p.cx = cx; p.ky = ky; p.kk = kk;
  p.ctiles = pl.ctiles; p.ktiles = pl.ktiles; p.splits = pl.splits; p.rows_per_split = pl.rows_per_split;
  for (int i = 0; i < 3; ++i) { p.asp[i] = asp[i]; p.osp[i] = osp[i]; p.stride[i] = stride[i]; }
  return launch_rows_shape(p, pl.shape, ROWS_GATHERED_DY, s);
}

}  // namespace lms
