// Weight gradient of first layers (2-D) whose stride times channels is six: the 7x7 stride-2 stem on 3 channels and smaller filters.
//
// dw[(tap, channel)][k] = sum over positions of x * dy.  Neighbouring positions start six elements further in an input row, so the
// row is staged in LDS in groups of six elements padded to eight (16 bytes): the elements that the taps of a filter row read at a
// position are then `span` whole groups from the position's own on, every position at a 16-byte step, and the LDS transpose
// read delivers them as MFMA operands, 8 * span (padded) elements of the reduction's other side per filter row, with nothing
// gathered (what bounds wgrad_small.hip).  The first padding element of a group is 1: its row of the product is the
// column sum of dy, the bias / shift gradient, for nothing.  dy goes straight to LDS (buffer loads that write it).  Positions of a
// tile's last group of 16 that are none of its row's would meet dy = 0 with real pixels, which makes NaN of infinite ones: where tiles
// do not fill rows and maps in whole groups (RAGGED) their x is masked, and rows below the last are left out.
//
// A work-group of eight waves, one per compute unit, owns the whole filter gradient and a run of tiles of up to 256 positions; a wave
// takes 32 output channels (all rows of the product) and every fourth 16 positions; dy of the next two tiles and x of the next
// are on their way while one is multiplied.  The waves' sums meet in LDS.
//
// 64 images of 224 x 224, with both final sums: 90 -> 47 us against 21 for the 122 MB at the rate of a large copy; 64 images of 48 x 48 30 -> 16, 4 of
// them 16 -> 15 (the ends of a work-group: addresses, sums, partial filter).  At 256 images of 224 x 224 it moves 498 MB at 3.5 TB/s with the
// matrix pipes busy 26 % of the cycles and LDS active in 20 %: one work-group a compute unit, whose eight waves meet at a barrier per tile.
#include <hip/hip_runtime.h>

#include <cstdlib>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"

namespace lms {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int WT_NT = 512, WT_NX = 3;                 // threads; groups of x a thread stages per tile
constexpr int WT_PIX = 256, WT_PIX_B = 128;          // positions of a tile, bytes of one of dy (64 channels)
constexpr int WT_X = WT_NX * WT_NT * 16, WT_Y = WT_PIX * WT_PIX_B;
constexpr int WT_LDS = 2 * WT_X + 3 * WT_Y;
constexpr int WT_YV = WT_PIX * 8 / WT_NT;            // loads of dy per thread and tile

__device__ __forceinline__ v2u wt_tr(const unsigned char* q) {
  return __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)q));
}
__device__ __forceinline__ bf16x8 wt_frag(const unsigned char* a, const unsigned char* b) {
  const v2u u = wt_tr(a), v = wt_tr(b);
  return __builtin_bit_cast(bf16x8, v4u{u[0], u[1], v[0], v[1]});
}

// JT: 32-row tiles of the padded (filter row, element) index.
template <int JT, bool RAGGED>
__global__ __launch_bounds__(WT_NT, 2) void wgrad_stem_kernel(StemGradPlan p) {
  extern __shared__ __attribute__((aligned(256))) unsigned char lds_st[];
  const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = wave8 & 1, g = wave8 >> 1;                       // 32 output channels; turn among the groups of 16 positions
  const int row_el = p.W * p.cx;

  // ---- this thread's groups of x and vectors of dy in a tile: row, and byte offset from the tile's first (outside its columns:
  // beyond every buffer).  Offsets change with the tile's column only. ----
  const int begin = (int)blockIdx.x * p.tiles_per_split, end = begin + p.tiles_per_split < p.tiles ? begin + p.tiles_per_split : p.tiles;
  const int y_ch = ((((tid & 7) >> 1) ^ ((tid >> 4) & 3)) << 1 | (tid & 1)) * 8;      // 16-byte slot tid % 8: pairs permuted as the transpose read wants them
  int x_row[WT_NX], y_row[WT_YV];
  unsigned x_off[WT_NX][3], y_off[WT_YV];
#pragma unroll
  for (int i = 0; i < WT_NX; ++i) x_row[i] = (int)((unsigned)(tid + i * WT_NT) * p.gw_magic >> 20);
#pragma unroll
  for (int j = 0; j < WT_YV; ++j) y_row[j] = (int)((unsigned)((tid >> 3) + 64 * j) * p.pix_magic >> 20);
  auto columns = [&](int ow0) {
    const int e0 = ow0 * 6 - p.pad_w * p.cx - p.lead, tw = p.OW - ow0 < p.tw ? p.OW - ow0 : p.tw;
#pragma unroll
    for (int i = 0; i < WT_NX; ++i) {
      const int e = (tid + i * WT_NT - x_row[i] * p.gw) * 6;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        x_off[i][k] = tid + i * WT_NT < p.groups && (unsigned)(e0 + e + 2 * k) < (unsigned)row_el ? (unsigned)(x_row[i] * row_el + e + 2 * k) * 2u : DMA_OOB;
    }
#pragma unroll
    for (int j = 0; j < WT_YV; ++j) {
      const int c = (tid >> 3) + 64 * j - y_row[j] * p.gpr * 16;
      y_off[j] = y_ch < p.ky && c < tw && y_row[j] < p.th ? (unsigned)(((y_row[j] * p.OW + c) * p.ky + y_ch) * 2) : DMA_OOB;
    }
  };
  const unsigned lds_y = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)lds_st + 2 * WT_X + wave8 * 1024);
  // the tile asked for next
  int nw = begin % p.tiles_w, nh = begin / p.tiles_w % p.tiles_h, nn = begin / p.tiles_w / p.tiles_h;
  columns(nw * p.tw);
  typedef unsigned XRegs[WT_NX][3];
  XRegs xr0, xr1;                                                 // x of two tiles: even and odd ones
  auto fetch = [&](XRegs& xr, int buf) {
    const int oh0 = nh * p.th, ow0 = nw * p.tw, ih0 = oh0 * p.stride - p.pad_h;
    const long long row0 = ((long long)nn * p.OH + oh0) * p.OW + ow0;
    const v4u ry = buffer_rsrc(p.DY + row0 * p.ky, 0x7fffffff);       // positions outside the tile are never asked for
    const uint16_t* x0 = p.X + ((long long)nn * p.H + ih0) * row_el + ow0 * 6 - p.pad_w * p.cx - p.lead;
    const auto rx = __builtin_amdgcn_make_buffer_rsrc((void*)x0, 0, 0x7fffffff, 0x00020000);
    const bool y_all = oh0 + p.th <= p.OH, x_all = ih0 >= 0 && ih0 + p.rows <= p.H;     // uniform
#pragma unroll
    for (int j = 0; j < WT_YV; ++j)
      load_lds16(ry, lds_y + buf * WT_Y + j * 64 * WT_PIX_B, y_all || oh0 + y_row[j] < p.OH ? y_off[j] : DMA_OOB, 0);
#pragma unroll
    for (int i = 0; i < WT_NX; ++i) {
      const bool ok = x_all || (unsigned)(ih0 + x_row[i]) < (unsigned)p.H;
#pragma unroll
      for (int k = 0; k < 3; ++k) xr[i][k] = __builtin_amdgcn_raw_buffer_load_b32(rx, (int)(ok ? x_off[i][k] : DMA_OOB), 0, 0);
    }
    if (++nw == p.tiles_w) { nw = 0; if (++nh == p.tiles_h) { nh = 0; ++nn; } }
    if (p.tiles_w > 1) columns(nw * p.tw);
  };

  // ---- LDS read addresses ----
  const int li = lane & 15, lg = lane >> 4, row = (lg >> 1) * 8 + (li >> 2), x_pitch = p.gw * 16;
  int xa[JT];
#pragma unroll
  for (int j = 0; j < JT; ++j) {
    const int v = j * 32 + 16 * (lg & 1) + 4 * (li & 3), kh = (int)((unsigned)(v >> 3) * p.span_magic >> 20), e = v - kh * p.span * 8;
    xa[j] = (kh < p.filt ? kh * x_pitch + e * 2 : 0) + row * 16;      // rows beyond the filter: any elements, nobody stores them
  }
  const int pair = kq * 2 + (lg & 1);
  int ya[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = row + 4 * i;
    ya[i] = r * WT_PIX_B + ((pair ^ ((r >> 1) & 3)) << 5) + (li & 3) * 8;
  }

  f32x16 acc[JT];
#pragma unroll
  for (int j = 0; j < JT; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;

  // 16 positions: operands, read one turn ahead of their products
  struct Frag { bf16x8 y, x[JT]; int left; };                     // left (RAGGED): positions from the first of the 16 to the end of the row
  int tw_at = begin % p.tiles_w, th_at = begin / p.tiles_w % p.tiles_h;      // the tile that is multiplied
  if (begin < end) {
    fetch(xr0, 0);
    if (begin + 1 < end) fetch(xr1, 1);
  }
  int ybuf = 0;
  auto tile = [&](int t, XRegs& xr, int xbuf) {
    // one barrier a tile: x alternates between two buffers, so what is written here was last read before the barrier of the tile
    // before; the buffer of dy that is filled behind the barrier was read in the tile before
#pragma unroll
    for (int i = 0; i < WT_NX; ++i)
      *reinterpret_cast<uint4*>(lds_st + xbuf * WT_X + (tid + i * WT_NT) * 16) = make_uint4(xr[i][0], xr[i][1], xr[i][2], 0x00003f80u);
    if (t + 1 < end) wait_barrier<3 * WT_NX>();                   // dy of this tile is older than x of the next
    else wait_barrier<0>();
    if (t + 2 < end) fetch(xr, ybuf == 0 ? 2 : ybuf - 1);
    const unsigned char* sx = lds_st + xbuf * WT_X;
    const unsigned char* sy = lds_st + 2 * WT_X + ybuf * WT_Y;
    int row_len = p.tw, rows_in = p.th;
    if constexpr (RAGGED) {
      if (p.OW - tw_at * p.tw < row_len) row_len = p.OW - tw_at * p.tw;
      if (p.OH - th_at * p.th < rows_in) rows_in = p.OH - th_at * p.th;
      if (++tw_at == p.tiles_w) { tw_at = 0; if (++th_at == p.tiles_h) th_at = 0; }
    }
    const int turns = (rows_in * p.gpr - g + 3) / 4;              // of this wave
    int r = 0, c = g;                                             // row and group of 16 of the next turn
    while (c >= p.gpr) { c -= p.gpr; ++r; }
    auto load = [&](Frag& f) {
      const unsigned char* xq = sx + r * p.stride * x_pitch + c * 256;
      const unsigned char* yq = sy + (r * p.gpr + c) * 16 * WT_PIX_B;
      if constexpr (RAGGED) f.left = row_len - c * 16;
      f.y = wt_frag(yq + ya[0], yq + ya[1]);
#pragma unroll
      for (int j = 0; j < JT; ++j) f.x[j] = wt_frag(xq + xa[j], xq + xa[j] + 64);
      c += 4;
      while (c >= p.gpr) { c -= p.gpr; ++r; }
    };
    auto mul = [&](Frag& f) {
      if constexpr (RAGGED) {
        if (f.left < 16) {                                          // uniform
          const int n = f.left - 8 * (lane >> 5);
          v4u m;
#pragma unroll
          for (int w = 0; w < 4; ++w) m[w] = (2 * w < n ? 0xffffu : 0u) | (2 * w + 1 < n ? 0xffff0000u : 0u);
#pragma unroll
          for (int j = 0; j < JT; ++j) f.x[j] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(v4u, f.x[j]) & m);
        }
      }
#pragma unroll
      for (int j = 0; j < JT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.x[j], f.y, acc[j], 0, 0, 0);
    };
    Frag fa, fb;
    if (turns > 0) load(fa);
#pragma unroll 1
    for (int i = 0; i < turns; i += 2) {
      if (i + 1 < turns) load(fb);
      mul(fa);
      if (i + 1 < turns) {
        if (i + 2 < turns) load(fa);
        mul(fb);
      }
    }
    ybuf = ybuf == 2 ? 0 : ybuf + 1;
  };
#pragma unroll 1
  for (int t = begin; t < end; t += 2) {
    tile(t, xr0, 0);
    if (t + 1 < end) tile(t + 1, xr1, 1);
  }

  // ---- the waves' sums: turns 2 and 3 to 0 and 1, then 1 to 0 ----
  float4* sums = reinterpret_cast<float4*>(lds_st);
  auto slot = [&](int w, int j, int q) -> float4& { return sums[((w * JT + j) * 4 + q) * 64 + lane]; };
#pragma unroll
  for (int half = 2; half >= 1; half >>= 1) {
    __syncthreads();
    if (g >= half && g < 2 * half) {
#pragma unroll
      for (int j = 0; j < JT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) slot(wave8 - 2 * half, j, q) = make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
    }
    __syncthreads();
    if (g < half) {
#pragma unroll
      for (int j = 0; j < JT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 o = slot(wave8, j, q);
          acc[j][4 * q] += o.x; acc[j][4 * q + 1] += o.y; acc[j][4 * q + 2] += o.z; acc[j][4 * q + 3] += o.w;
        }
    }
  }
  if (g > 0) return;
  const int k = kq * 32 + (lane & 31);
  // rows that are padding, and columns beyond the last, go beyond the buffer
  const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(p.part + (long long)blockIdx.x * p.filt * p.run * p.ky, 0, p.filt * p.run * p.ky * 4, 0x00020000);
  const int i0 = 4 * (lane >> 5);
  const unsigned col = k < p.ky ? (unsigned)(k * 4) : DMA_OOB;
  int kh = 0, e0 = -p.lead;                                       // filter row and first element of the group
#pragma unroll
  for (int j = 0; j < JT; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int e = e0 + i0 + v;
        const bool ok = i0 + v < 6 && (unsigned)e < (unsigned)p.run && kh < p.filt;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[j][4 * q + v]), out, (int)(ok ? col + (unsigned)((kh * p.run + e) * p.ky * 4) : DMA_OOB), 0, 0);
      }
      e0 += 6;
      if (e0 >= p.span * 6 - p.lead) { e0 = -p.lead; ++kh; }      // uniform
    }
  // row 6 of the product, the first group's ones: lanes 32 and on, their third value
  if (p.cs_part && lane >= 32 && k < p.ky) p.cs_part[(long long)blockIdx.x * p.ky + k] = acc[0][2];
}

template <int JT, bool RAGGED>
hipError_t launch_stem_t(const StemGradPlan& p, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(wgrad_stem_kernel<JT, RAGGED>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, WT_LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((wgrad_stem_kernel<JT, RAGGED>), dim3((unsigned)p.splits), dim3(WT_NT), WT_LDS, s, p);
  return hipGetLastError();
}

}  // namespace

bool wgrad_stem_plan(StemGradPlan& p, long long rows, int cx, int ky, const int* asp, const int* osp, const int* filt, const int* stride, const int* pad) {
  static const bool off = getenv("LMS_NO_WGRAD_STEM") != nullptr;     // tuning aid
  if (off || cx < 1 || cx > 4 || stride[2] * cx != 6 || asp[0] != 1 || osp[0] != 1 || filt[0] != 1 || pad[0] != 0 || ky > 64 || (ky & 7) != 0) return false;
  if ((asp[2] * cx & 1) != 0 || 2LL * asp[1] * asp[2] * cx >= 0x7fffffffLL) return false;
  p.cx = cx; p.ky = ky; p.H = asp[1]; p.W = asp[2]; p.OH = osp[1]; p.OW = osp[2];
  p.filt = filt[1]; p.stride = stride[1]; p.pad_h = pad[1]; p.pad_w = pad[2];
  p.run = filt[2] * cx;
  p.lead = (pad[2] * cx) & 1;
  p.span = (p.lead + p.run + 5) / 6;
  if (p.filt * p.span * 8 > 224) return false;
  // the row split evenly into tiles of up to 128 positions, as many rows as fit
  p.tiles_w = (p.OW + 127) / 128;
  p.tw = (p.OW + p.tiles_w - 1) / p.tiles_w;
  p.gpr = (p.tw + 15) / 16;
  p.gw = p.gpr * 16 + p.span - 1;
  int th = WT_PIX / (p.gpr * 16), fit = (WT_NX * WT_NT / p.gw - p.filt) / p.stride + 1;
  if (WT_NX * WT_NT / p.gw < p.filt) return false;
  if (fit < th) th = fit;
  if (th > p.OH) th = p.OH;
  const long long images = rows / ((long long)p.OH * p.OW);
  while (th > 1 && images * ((p.OH + th - 1) / th) * p.tiles_w < 128) th = (th + 1) / 2;
  p.th = th;
  p.gw_magic = (unsigned)(((1 << 20) + p.gw - 1) / p.gw);
  p.pix_magic = (unsigned)(((1 << 20) + p.gpr * 16 - 1) / (p.gpr * 16));
  p.span_magic = (unsigned)(((1 << 20) + p.span - 1) / p.span);
  p.rows = (th - 1) * p.stride + p.filt;
  p.groups = p.rows * p.gw;
  p.tiles_h = (p.OH + th - 1) / th;
  const long long tiles = images * p.tiles_h * p.tiles_w;
  if (tiles > 0x3fffffffLL || rows >= 0x7fffffffLL || 2LL * WT_PIX * p.OW * ky >= 0x7fffffffLL || 2LL * (p.rows + 1) * p.W * cx >= 0x7fffffffLL) return false;
  p.tiles = (int)tiles;
  // no more partial filters than wgrad_small.hip leaves, which the workspace has room for
  long long splits = wgrad_small_splits(rows, osp);
  if (splits > 256) splits = 256;
  if (splits > tiles) splits = tiles;
  if (splits < 1) splits = 1;
  p.tiles_per_split = (int)((tiles + splits - 1) / splits);
  p.splits = (int)((tiles + p.tiles_per_split - 1) / p.tiles_per_split);
  return tiles > 0;
}

hipError_t launch_wgrad_stem(StemGradPlan p, const uint16_t* X, const uint16_t* DY, float* part, float* cs_part, hipStream_t s) {
  p.X = X; p.DY = DY; p.part = part; p.cs_part = cs_part;
  const int jt = (p.filt * p.span * 8 + 31) / 32;
  const bool ragged = p.tw % 16 != 0 || p.tw * p.tiles_w != p.OW || p.th * p.tiles_h != p.OH;
  if (jt <= 2) return ragged ? launch_stem_t<2, true>(p, s) : launch_stem_t<2, false>(p, s);
  if (jt <= 4) return ragged ? launch_stem_t<4, true>(p, s) : launch_stem_t<4, false>(p, s);
  return ragged ? launch_stem_t<7, true>(p, s) : launch_stem_t<7, false>(p, s);
}

}  // namespace lms
