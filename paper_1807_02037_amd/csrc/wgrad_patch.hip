// Weight gradient of 3x3 / 3x3x3 stride-1 convolutions, patch-tiled.
//
// A work-group owns 32 input channels x 32 output channels of the filter gradient and walks over a
// range of spatial patches (128 output positions: 2-D 8x16, 3-D 4x4x8).  Per patch it brings the input
// patch with its halo (32 channels) and the output-gradient patch (32 channels) into LDS exactly as they
// lie in memory (position-major, channels contiguous); every filter tap is then a row offset into the
// same input tile.  The reduction runs over positions, so the MFMA operands must hold 8 consecutive
// positions per lane: they are read with the gfx950 LDS transpose read (ds_read_b64_tr_b16), which hands
// lane i of a 16-lane group the element (i % 4) of the four 8-byte rows addressed by lanes i/4, i/4+4,
// i/4+8, i/4+12 (layout checked on the device).  The 9 / 27 taps are dealt to the four waves; each wave
// keeps one 32x32 accumulator per tap.  Partial gradients per work-group go to the split buffer and are
// summed in a fixed order by the reduction kernel.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"
#include "wgrad_patch.hpp"

namespace lms {

namespace {

// CS: the work-groups of input-channel tile 0 also add up the gradient vectors they stage (every position of dy lies in
// exactly one patch): the bias / shift gradient without another pass over dy (two launches less; 64 -> 64 channels at
// 64^3 16 us, 256 -> 256 at 16^3 10 us).
template <int P3D, bool CS>
__global__ __launch_bounds__(NTHREADS, 2) void wgrad_patch_kernel(WPatchP p) {
  typedef WPatch<P3D> PT;
  constexpr int XV = (PT::MAXPIX * 4 + NTHREADS - 1) / NTHREADS;   // input-tile vectors per thread
  constexpr int YV = 128 * 4 / NTHREADS;                           // gradient-tile vectors per thread
  __shared__ __attribute__((aligned(16))) uint16_t sX[(PT::MAXPIX + 4) * LDX];     // the 12-position reads of the last halo row run 2 pixels over
  __shared__ __attribute__((aligned(16))) uint16_t sY[128 * LDX];

  int b = blockIdx.x;
  const int cc = b % p.cchunks; b /= p.cchunks;
  const int kt = b % p.ktiles; b /= p.ktiles;
  const int split = b;
  const int c0 = cc * 32, k0 = kt * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int hd = PT::TD + p.filt[0] - 1;
  const int halo_pix = hd * PT::HH * PT::HW;

  // this lane as a source of the transpose reads: position offset i/4 within a group of four, channels 16*(g&1) + 4*(i&3)
  const int li = lane & 15, lg = lane >> 4;
  const int src_off = (li >> 2) * LDX + 16 * (lg & 1) + 4 * (li & 3);
  const int half = lg >> 1;                                   // which 8 of the 16 positions of a k-step

  // halo coordinates of this thread's input vectors (relative to the patch origin)
  int xj[XV][3];
  bool x_valid[XV];
#pragma unroll
  for (int j = 0; j < XV; ++j) {
    const int pix = (tid + j * NTHREADS) >> 2;
    x_valid[j] = pix < halo_pix;
    unsigned t = x_valid[j] ? (unsigned)pix : 0u;
    xj[j][2] = (int)(t % PT::HW); t /= PT::HW;
    xj[j][1] = (int)(t % PT::HH); t /= PT::HH;
    xj[j][0] = (int)t;
  }
  int yj[YV][3];
#pragma unroll
  for (int j = 0; j < YV; ++j) {
    const int q = (tid + j * NTHREADS) >> 2;
    yj[j][2] = q % PT::TW; yj[j][1] = (q / PT::TW) % PT::TH; yj[j][0] = q / (PT::TW * PT::TH);
  }
  const int vch = (tid & 3) * 8;                               // channel offset of this thread's vectors
  const bool xc_ok = c0 + vch < p.cx, yc_ok = k0 + vch < p.ky;
  const bool x_vec = (p.cx & 7) == 0;

  const int pbegin = split * p.patches_per_split;
  const int pend = (pbegin + p.patches_per_split < p.patches) ? pbegin + p.patches_per_split : p.patches;

  // 32-bit offsets of this thread's vectors relative to the patch origin (input: origin - pad)
  int x_rel[XV], y_rel[YV];
#pragma unroll
  for (int j = 0; j < XV; ++j) x_rel[j] = ((xj[j][0] * p.asp[1] + xj[j][1]) * p.asp[2] + xj[j][2]) * p.cx + c0 + vch;
#pragma unroll
  for (int j = 0; j < YV; ++j) y_rel[j] = ((yj[j][0] * p.osp[1] + yj[j][1]) * p.osp[2] + yj[j][2]) * p.ky + k0 + vch;

  uint4 rx[XV], ry[YV];
  // patch coordinates advance one patch at a time (no divisions in the loop)
  int tw, th, td;
  long long nb;
  {
    unsigned t = (unsigned)pbegin;
    tw = (int)(t % (unsigned)p.tiles[2]); t /= (unsigned)p.tiles[2];
    th = (int)(t % (unsigned)p.tiles[1]); t /= (unsigned)p.tiles[1];
    td = (int)(t % (unsigned)p.tiles[0]); t /= (unsigned)p.tiles[0];
    nb = t;
  }
  auto advance = [&]() {
    if (++tw == p.tiles[2]) { tw = 0; if (++th == p.tiles[1]) { th = 0; if (++td == p.tiles[0]) { td = 0; ++nb; } } }
  };
  // With 8-channel vectors and tensors below 2 GiB, memory is read through buffer descriptors: an offset beyond the
  // tensor returns zeros, so padding and ragged patches need no branches and no 64-bit address arithmetic.
  const bool use_buf = x_vec && p.x_bytes != 0;
  constexpr int OOB = (int)0x80000000;
  const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.X), 0, (int)p.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.DY), 0, (int)p.y_bytes, 0x00020000);
  auto fetch = [&]() {
    const int o0[3] = {td * PT::TD, th * PT::TH, tw * PT::TW};
    const int i0[3] = {o0[0] - p.pad[0], o0[1] - p.pad[1], o0[2] - p.pad[2]};
    if (use_buf) {
      const int xb = (((((int)nb * p.asp[0] + i0[0]) * p.asp[1] + i0[1]) * p.asp[2] + i0[2]) * p.cx) * 2;
      const int yb = (((((int)nb * p.osp[0] + o0[0]) * p.osp[1] + o0[1]) * p.osp[2] + o0[2]) * p.ky) * 2;
#pragma unroll
      for (int j = 0; j < XV; ++j) {
        const bool ok = x_valid[j] && xc_ok && (unsigned)(i0[0] + xj[j][0]) < (unsigned)p.asp[0] &&
                        (unsigned)(i0[1] + xj[j][1]) < (unsigned)p.asp[1] && (unsigned)(i0[2] + xj[j][2]) < (unsigned)p.asp[2];
        rx[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, ok ? xb + 2 * x_rel[j] : OOB, 0, 0));
      }
#pragma unroll
      for (int j = 0; j < YV; ++j) {
        const bool ok = yc_ok && o0[0] + yj[j][0] < p.osp[0] && o0[1] + yj[j][1] < p.osp[1] && o0[2] + yj[j][2] < p.osp[2];
        ry[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_y, ok ? yb + 2 * y_rel[j] : OOB, 0, 0));
      }
      return;
    }
    const uint16_t* xb = p.X + (((nb * p.asp[0] + i0[0]) * p.asp[1] + i0[1]) * p.asp[2] + i0[2]) * p.cx;
    const uint16_t* yb = p.DY + (((nb * p.osp[0] + o0[0]) * p.osp[1] + o0[1]) * p.osp[2] + o0[2]) * p.ky;
#pragma unroll
    for (int j = 0; j < XV; ++j) {
      const int id = i0[0] + xj[j][0], ih = i0[1] + xj[j][1], iw = i0[2] + xj[j][2];
      rx[j] = make_uint4(0, 0, 0, 0);
      if (x_valid[j] && xc_ok && (unsigned)id < (unsigned)p.asp[0] && (unsigned)ih < (unsigned)p.asp[1] &&
          (unsigned)iw < (unsigned)p.asp[2]) {
        const uint16_t* src = xb + x_rel[j];
        if (x_vec) rx[j] = *reinterpret_cast<const uint4*>(src);
        else {        // channel count not a multiple of 8 (first layer): element by element
          uint32_t w4[4] = {0, 0, 0, 0};
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (c0 + vch + e < p.cx) w4[e >> 1] |= (uint32_t)src[e] << ((e & 1) * 16);
          rx[j] = make_uint4(w4[0], w4[1], w4[2], w4[3]);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < YV; ++j) {
      const int od = o0[0] + yj[j][0], oh = o0[1] + yj[j][1], ow = o0[2] + yj[j][2];
      ry[j] = make_uint4(0, 0, 0, 0);
      if (yc_ok && od < p.osp[0] && oh < p.osp[1] && ow < p.osp[2]) ry[j] = *reinterpret_cast<const uint4*>(yb + y_rel[j]);
    }
  };

  f32x16 acc[PT::MAXT];
#pragma unroll
  for (int j = 0; j < PT::MAXT; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;

  float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};     // channels k0 + vch .. + 7 of all this thread's vectors
  const bool cs_on = CS && cc == 0;
  if (pbegin < pend) fetch();
  for (int patch = pbegin; patch < pend; ++patch) {
    if (cs_on) {
#pragma unroll
      for (int j = 0; j < YV; ++j) {
        const uint32_t w[4] = {ry[j].x, ry[j].y, ry[j].z, ry[j].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) csum[e] += __uint_as_float((e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16));
      }
    }
    __syncthreads();                       // previous patch fully consumed
#pragma unroll
    for (int j = 0; j < XV; ++j) {
      const int v = tid + j * NTHREADS;
      if ((v >> 2) < PT::MAXPIX) *reinterpret_cast<uint4*>(sX + (v >> 2) * LDX + (v & 3) * 8) = rx[j];
    }
#pragma unroll
    for (int j = 0; j < YV; ++j) {
      const int v = tid + j * NTHREADS;
      *reinterpret_cast<uint4*>(sY + (v >> 2) * LDX + (v & 3) * 8) = ry[j];
    }
    __syncthreads();
    if (patch + 1 < pend) { advance(); fetch(); }
    switch (wave) {
      case 0: wgrad_patch_mma<P3D, 0>(sX, sY, acc, src_off, half, nullptr, 0, [](int) {}); break;
      case 1: wgrad_patch_mma<P3D, 1>(sX, sY, acc, src_off, half, nullptr, 0, [](int) {}); break;
      case 2: wgrad_patch_mma<P3D, 2>(sX, sY, acc, src_off, half, nullptr, 0, [](int) {}); break;
      default: wgrad_patch_mma<P3D, 3>(sX, sY, acc, src_off, half, nullptr, 0, [](int) {}); break;
    }
  }
  const int tap_lo = p.taps * wave / 4, tap_n = p.taps * (wave + 1) / 4 - tap_lo;
#pragma unroll
  for (int j = 0; j < PT::MAXT; ++j) {
    const int t = tap_lo + j;
    if (j >= tap_n) continue;
    float* out = p.part + ((long long)split * p.taps + t) * p.cx * p.ky;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int c = c0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      const int k = k0 + (lane & 31);
      if (c < p.cx && k < p.ky) out[(long long)c * p.ky + k] = acc[j][v];
    }
  }
  if (cs_on) {
    // threads tid, tid + 4, ... hold the same channels: lanes of a wave by shuffles, then the four waves in order
#pragma unroll
    for (int e = 0; e < 8; ++e)
      for (int dist = 4; dist < 64; dist <<= 1) csum[e] += __shfl_xor(csum[e], dist, 64);
    float* sh = reinterpret_cast<float*>(sY);
    __syncthreads();                       // the last patch is fully consumed
    if (lane < 4) {
#pragma unroll
      for (int e = 0; e < 8; ++e) sh[wave * 32 + lane * 8 + e] = csum[e];
    }
    __syncthreads();
    if (tid < 32 && k0 + tid < p.ky) p.cs_part[(long long)split * p.ky + k0 + tid] = (sh[tid] + sh[32 + tid]) + (sh[64 + tid] + sh[96 + tid]);
  }
}


// The same tile (32 x 32 channels, all taps) for input channel counts that are multiples of 8, eight waves: two groups of
// four that take every second patch each, into sums of their own that meet in LDS at the end.  Patches go from memory
// straight to LDS (buffer loads that write LDS, outside the tensors zeros), one patch ahead in a pair of buffers per group.
// What bounds the small layers is not the products but the partial filters, written by every work-group and read
// again: with the groups' sums added first there is one per compute unit instead of two (27 x 32 x 32 filters: 28 MB each
// way instead of 56).  Both parameter gradients, us: 64 -> 64 at 64^3 77 -> 74, 32 -> 32 38 -> 33,
// 128 -> 128 at 32^3 52 -> 46, 256 -> 256 at 16^3 37 -> 33.
template <int P3D>
struct GPatch {
  typedef WPatch<P3D> PT;
  static constexpr int XV = (PT::MAXPIX + 4 + 63) / 64;           // input loads per thread of a group and patch
  static constexpr int YV = 2;
  static constexpr int X_BYTES = XV * 64 * 64, Y_BYTES = 128 * 64, BUF = X_BYTES + Y_BYTES;
  static constexpr int TAPS = P3D ? 27 : 9;
  static constexpr int SUMS = TAPS * 4096;
  static constexpr int LDS_BYTES = 4 * BUF > SUMS ? 4 * BUF : SUMS;
};

template <int P3D, bool CS>
__global__ __launch_bounds__(GP_NT, 2) void wgrad_patch_group_kernel(WPatchP p) {
  typedef WPatch<P3D> PT;
  typedef GPatch<P3D> GP;
  constexpr int XV = GP::XV, YV = GP::YV;
  extern __shared__ __attribute__((aligned(256))) unsigned char lds_gp[];
  int b = blockIdx.x;
  const int cc = b % p.cchunks; b /= p.cchunks;
  const int kt = b % p.ktiles; b /= p.ktiles;
  const int split = b;
  const int c0 = cc * 32, k0 = kt * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = wave8 >> 2, wave = wave8 & 3, gt = tid & 255;
  const int hd = PT::TD + p.filt[0] - 1;
  const int halo_pix = hd * PT::HH * PT::HW;
  const int li = lane & 15, lg = lane >> 4;
  const int src_off = (li >> 2) * LDX + 16 * (lg & 1) + 4 * (li & 3);
  const int half = lg >> 1;

  // this thread's vectors of a patch: position relative to the patch origin (input: origin - pad), byte offset from it
  const int vch = (gt & 3) * 8;
  const bool xc_ok = c0 + vch < p.cx, yc_ok = k0 + vch < p.ky;
  int xj[XV], yj[YV];                                             // coordinates, 8 bits each
  unsigned x_off[XV], y_off[YV];
#pragma unroll
  for (int j = 0; j < XV; ++j) {
    const int pix = (gt >> 2) + j * 64;
    const int w = pix % PT::HW, h = (pix / PT::HW) % PT::HH, d = pix / (PT::HW * PT::HH);
    xj[j] = w | h << 8 | d << 16;
    x_off[j] = pix < halo_pix && xc_ok ? (unsigned)((((d * p.asp[1] + h) * p.asp[2] + w) * p.cx + c0 + vch) * 2) : DMA_OOB;
  }
#pragma unroll
  for (int j = 0; j < YV; ++j) {
    const int q = (gt >> 2) + j * 64;
    const int w = q % PT::TW, h = (q / PT::TW) % PT::TH, d = q / (PT::TW * PT::TH);
    yj[j] = w | h << 8 | d << 16;
    y_off[j] = yc_ok ? (unsigned)((((d * p.osp[1] + h) * p.osp[2] + w) * p.ky + k0 + vch) * 2) : DMA_OOB;
  }

  const int pbegin = split * p.patches_per_split;
  const int pend = (pbegin + p.patches_per_split < p.patches) ? pbegin + p.patches_per_split : p.patches;
  const int rounds = pend > pbegin ? (pend - pbegin + 1) / 2 : 0;
  int tw, th, td, nb;                                             // the group's next patch (uniform)
  {
    unsigned t = (unsigned)(pbegin + g);
    tw = (int)(t % (unsigned)p.tiles[2]); t /= (unsigned)p.tiles[2];
    th = (int)(t % (unsigned)p.tiles[1]); t /= (unsigned)p.tiles[1];
    td = (int)(t % (unsigned)p.tiles[0]);
    nb = (int)(t / (unsigned)p.tiles[0]);
  }
  auto advance = [&]() {
    if (++tw == p.tiles[2]) { tw = 0; if (++th == p.tiles[1]) { th = 0; if (++td == p.tiles[0]) { td = 0; ++nb; } } }
  };
  const unsigned lds_w = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)lds_gp + g * 2 * GP::BUF + wave * 1024);
  auto fetch = [&](int round, int buf) {
    const bool in = pbegin + 2 * round + g < pend;
    const int o0[3] = {td * PT::TD, th * PT::TH, tw * PT::TW};
    const int i0[3] = {o0[0] - p.pad[0], o0[1] - p.pad[1], o0[2] - p.pad[2]};
    const v4u rx = buffer_rsrc(p.X + (((long long)nb * p.asp[0] + i0[0]) * p.asp[1] + i0[1]) * (long long)p.asp[2] * p.cx + (long long)i0[2] * p.cx, in ? 0x7fffffff : 0);
    const v4u ry = buffer_rsrc(p.DY + (((long long)nb * p.osp[0] + o0[0]) * p.osp[1] + o0[1]) * (long long)p.osp[2] * p.ky + (long long)o0[2] * p.ky, in ? 0x7fffffff : 0);
#pragma unroll
    for (int j = 0; j < XV; ++j) {
      const bool ok = (unsigned)(i0[0] + (xj[j] >> 16)) < (unsigned)p.asp[0] && (unsigned)(i0[1] + ((xj[j] >> 8) & 255)) < (unsigned)p.asp[1] &&
                      (unsigned)(i0[2] + (xj[j] & 255)) < (unsigned)p.asp[2];
      load_lds16(rx, lds_w + buf * GP::BUF + j * 4096, ok ? x_off[j] : DMA_OOB, 0);
    }
#pragma unroll
    for (int j = 0; j < YV; ++j) {
      const bool ok = o0[0] + (yj[j] >> 16) < p.osp[0] && o0[1] + ((yj[j] >> 8) & 255) < p.osp[1] && o0[2] + (yj[j] & 255) < p.osp[2];
      load_lds16(ry, lds_w + buf * GP::BUF + GP::X_BYTES + j * 4096, ok ? y_off[j] : DMA_OOB, 0);
    }
    advance();
    advance();
  };

  // Everything from the sums on is written once per wave of a group: with one loop around a switch over the waves, the
  // sums of its four branches had to be moved into the same registers (250 of them, and spills).
  auto run = [&](auto wave_c) {
    constexpr int W = decltype(wave_c)::value;
    constexpr int TAP_LO = GP::TAPS * W / 4, TAP_N = GP::TAPS * (W + 1) / 4 - TAP_LO;
    f32x16 acc[PT::MAXT], cs;
#pragma unroll
    for (int j = 0; j < PT::MAXT; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) cs[v] = 0.f;
    if (rounds > 0) fetch(0, 0);
#pragma unroll 1
    for (int r = 0; r < rounds; ++r) {
      wait_barrier<0>();                                          // this round's patches have landed, the other buffers are free
      if (r + 1 < rounds) fetch(r + 1, (r + 1) & 1);
      const uint16_t* sX = reinterpret_cast<const uint16_t*>(lds_gp + (g * 2 + (r & 1)) * GP::BUF);
      wgrad_patch_mma<P3D, W, CS && W == 0>(sX, sX + GP::X_BYTES / 2, acc, src_off, half, &cs, 0, [](int) {});
    }
    // ---- group 1 leaves its sums in LDS, group 0 adds them and writes ----
    float4* sums = reinterpret_cast<float4*>(lds_gp);
    __syncthreads();
    if (g == 1) {
#pragma unroll
      for (int j = 0; j < TAP_N; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          sums[((TAP_LO + j) * 4 + q) * 64 + lane] = make_float4(acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]);
    }
    __syncthreads();
    if (g == 0) {
#pragma unroll
      for (int j = 0; j < TAP_N; ++j) {
        float* out = p.part + ((long long)split * p.taps + TAP_LO + j) * p.cx * p.ky;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 t = sums[((TAP_LO + j) * 4 + q) * 64 + lane];
          const float v[4] = {acc[j][4 * q] + t.x, acc[j][4 * q + 1] + t.y, acc[j][4 * q + 2] + t.z, acc[j][4 * q + 3] + t.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int c = c0 + 8 * q + 4 * (lane >> 5) + e, k = k0 + (lane & 31);
            if (c < p.cx && k < p.ky) out[(long long)c * p.ky + k] = v[e];
          }
        }
      }
    }
    if (CS && cc == 0) {
      float* sh = reinterpret_cast<float*>(lds_gp);
      __syncthreads();                                            // the sums above have been read
      if (W == 0 && lane < 32) sh[g * 32 + lane] = cs[0];         // every row of the product with ones is the sum
      __syncthreads();
      if (tid < 32 && k0 + tid < p.ky) p.cs_part[(long long)split * p.ky + k0 + tid] = sh[tid] + sh[32 + tid];
    }
  };
  switch (wave) {
    case 0: run(std::integral_constant<int, 0>{}); break;
    case 1: run(std::integral_constant<int, 1>{}); break;
    case 2: run(std::integral_constant<int, 2>{}); break;
    default: run(std::integral_constant<int, 3>{}); break;
  }
}

// 2-D variant with a 64 x 64 channel tile per work-group, for what wgrad_run.hip does not take (other paddings, rows of more
// than 126 positions, tensors that do not start on 16 bytes): every wave owns one 32 x 32 quadrant with all nine
// taps (nine accumulators), so an input patch and a gradient patch are read from memory once for 64 x 64
// filter entries instead of once per 32 x 32.
constexpr int LDW = 72;    // LDS row pitch: 64 channels + 8 (144 bytes)
constexpr int WGRAD64_LDS_BYTES = 2 * (10 * 18 + 128) * LDW * 2;

// CS: the work-groups of input-channel tile 0 also add up the gradient vectors they stage (every position of dy
// lies in exactly one patch): the bias / shift gradient without another pass over dy.
// PK: feature maps at most 7 wide and 8 high (the last stage of ResNet-50: 7 x 7), where one image fills 49 of a
// patch's 128 positions.  A patch then holds two images side by side, image g of the pair in columns 8 g .. 8 g + 6:
// column 7 (and 15) stays zero and is the padding between them, to the left of the second image as much as to the
// right of the first, so the nine taps read what they would read in each image alone.
template <bool CS, bool PK>
__global__ __launch_bounds__(NTHREADS, 1) void wgrad_patch64_kernel(WPatchP p) {
  constexpr int TH = 8, TW = 16, HH = TH + 2, HW = TW + 2, PIX = HH * HW;
  constexpr int XV = (PIX * 8 + NTHREADS - 1) / NTHREADS;        // 6 input vectors per thread
  constexpr int YV = 128 * 8 / NTHREADS;                         // 4 gradient vectors per thread
  // two buffers of (input halo tile, gradient tile): one is multiplied while the next patch is written
  extern __shared__ __attribute__((aligned(16))) uint16_t lds64[];
  constexpr int BUF = (PIX + 128) * LDW;
  static_assert(2 * BUF * 2 == WGRAD64_LDS_BYTES, "launch passes the LDS size");

  int b = blockIdx.x;
  const int cc = b % p.cchunks; b /= p.cchunks;
  const int kt = b % p.ktiles; b /= p.ktiles;
  const int split = b;
  const int c0 = cc * 64, k0 = kt * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ch = (wave & 1) * 32, kh = (wave >> 1) * 32;       // this wave's quadrant

  const int li = lane & 15, lg = lane >> 4;
  const int src_off = (li >> 2) * LDW + 16 * (lg & 1) + 4 * (li & 3);
  const int half = lg >> 1;

  int xh[XV], xw[XV], x_rel[XV];
  bool x_valid[XV];
  const int vch = (tid & 7) * 8;
#pragma unroll
  for (int j = 0; j < XV; ++j) {
    const int pix = (tid + j * NTHREADS) >> 3;
    x_valid[j] = pix < PIX && c0 + vch < p.cx;
    const int t = pix < PIX ? pix : 0;
    xw[j] = t % HW; xh[j] = t / HW;
    x_rel[j] = (xh[j] * p.asp[2] + xw[j]) * p.cx + c0 + vch;
    if (PK) {
      const int vc = xw[j] - p.pad[2];                       // column of the pair: image vc / 8, its column vc % 8
      const int g = vc >= 8;
      xw[j] = g;                                             // from here on: which image of the pair
      x_valid[j] = x_valid[j] && vc >= 0 && vc < TW && vc - 8 * g < p.asp[2];
      x_rel[j] = ((g * p.asp[1] + xh[j]) * p.asp[2] + vc - 8 * g) * p.cx + c0 + vch;
    }
  }
  int yh[YV], yw[YV], y_rel[YV];
  const bool yc_ok = k0 + vch < p.ky;
#pragma unroll
  for (int j = 0; j < YV; ++j) {
    const int q = (tid + j * NTHREADS) >> 3;
    yw[j] = q % TW; yh[j] = q / TW;
    y_rel[j] = (yh[j] * p.osp[2] + yw[j]) * p.ky + k0 + vch;
    if (PK) {
      const int g = yw[j] >= 8, x = yw[j] - 8 * g;
      y_rel[j] = ((g * p.osp[1] + yh[j]) * p.osp[2] + x) * p.ky + k0 + vch;
      yw[j] = x < p.osp[2] ? g : 2;                          // which image of the pair; 2: the padding column
    }
  }

  const int pbegin = split * p.patches_per_split;
  const int pend = (pbegin + p.patches_per_split < p.patches) ? pbegin + p.patches_per_split : p.patches;

  uint4 rxa[XV], rya[YV];
  auto fetch = [&](int patch, uint4 (&rx)[XV], uint4 (&ry)[YV]) {
    unsigned t = (unsigned)patch;
    const int tw = (int)(t % (unsigned)p.tiles[2]); t /= (unsigned)p.tiles[2];
    const int th = (int)(t % (unsigned)p.tiles[1]); t /= (unsigned)p.tiles[1];
    const long long nb = PK ? 2LL * patch : (long long)t;       // PK: one patch per pair of images
    const int oh0 = PK ? 0 : th * TH, ow0 = PK ? 0 : tw * TW;
    const int ih0 = oh0 - p.pad[1], iw0 = PK ? 0 : ow0 - p.pad[2];
    const uint16_t* xb = p.X + ((nb * p.asp[1] + ih0) * p.asp[2] + iw0) * p.cx;
    const uint16_t* yb = p.DY + ((nb * p.osp[1] + oh0) * p.osp[2] + ow0) * p.ky;
#pragma unroll
    for (int j = 0; j < XV; ++j) {
      rx[j] = make_uint4(0, 0, 0, 0);
      const bool col_ok = PK ? nb + xw[j] < p.batch : (unsigned)(iw0 + xw[j]) < (unsigned)p.asp[2];
      if (x_valid[j] && (unsigned)(ih0 + xh[j]) < (unsigned)p.asp[1] && col_ok)
        rx[j] = *reinterpret_cast<const uint4*>(xb + x_rel[j]);
    }
#pragma unroll
    for (int j = 0; j < YV; ++j) {
      ry[j] = make_uint4(0, 0, 0, 0);
      const bool col_ok = PK ? (yw[j] < 2 && nb + yw[j] < p.batch) : ow0 + yw[j] < p.osp[2];
      if (yc_ok && oh0 + yh[j] < p.osp[1] && col_ok) ry[j] = *reinterpret_cast<const uint4*>(yb + y_rel[j]);
    }
  };

  f32x16 acc[9];
#pragma unroll
  for (int j = 0; j < 9; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;

  float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};     // channels k0 + vch .. + 7 of all this thread's vectors
  const bool cs_on = CS && cc == 0;
  auto stage = [&](uint16_t* sX, const uint4 (&rx)[XV], const uint4 (&ry)[YV]) {
    uint16_t* sY = sX + PIX * LDW;
    if (cs_on) {
#pragma unroll
      for (int j = 0; j < YV; ++j) {
        const uint32_t w[4] = {ry[j].x, ry[j].y, ry[j].z, ry[j].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) csum[e] += __uint_as_float((e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16));
      }
    }
#pragma unroll
    for (int j = 0; j < XV; ++j) {
      const int v = tid + j * NTHREADS;
      if ((v >> 3) < PIX) *reinterpret_cast<uint4*>(sX + (v >> 3) * LDW + (v & 7) * 8) = rx[j];
    }
#pragma unroll
    for (int j = 0; j < YV; ++j) {
      const int v = tid + j * NTHREADS;
      *reinterpret_cast<uint4*>(sY + (v >> 3) * LDW + (v & 7) * 8) = ry[j];
    }
  };
  auto multiply = [&](const uint16_t* sX) {
    const uint16_t* sY = sX + PIX * LDW;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      // one k-step is one row of the patch; the tap (r, s) reads the halo tile r rows down and s columns right
      const int q0 = ks * 16 + 8 * half;
      const int pw = q0 % TW, ph = q0 / TW;
      const uint16_t* yb = sY + q0 * LDW + src_off + kh;
      const bf16x8 bfr = tr_frag(yb, yb + 4 * LDW);
      const uint16_t* xb0 = sX + (ph * HW + pw) * LDW + src_off + ch;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const uint16_t* xb = xb0 + ((t / 3) * HW + (t % 3)) * LDW;
        const bf16x8 af = tr_frag(xb, xb + 4 * LDW);
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr, acc[t], 0, 0, 0);
      }
    }
  };

  if (pbegin < pend) {
    fetch(pbegin, rxa, rya);
    stage(lds64, rxa, rya);
    if (pbegin + 1 < pend) fetch(pbegin + 1, rxa, rya);
  }
  __syncthreads();
  int cur = 0;
  for (int patch = pbegin; patch < pend; ++patch) {
    if (patch + 1 < pend) {
      stage(lds64 + (cur ^ 1) * BUF, rxa, rya);          // the other buffer was last read before the barrier below
      if (patch + 2 < pend) fetch(patch + 2, rxa, rya);
    }
    multiply(lds64 + cur * BUF);
    __syncthreads();
    cur ^= 1;
  }
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    float* out = p.part + ((long long)split * 9 + t) * p.cx * p.ky;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int c = c0 + ch + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      const int k = k0 + kh + (lane & 31);
      if (c < p.cx && k < p.ky) out[(long long)c * p.ky + k] = acc[t][v];
    }
  }
  if (cs_on) {
    // threads tid, tid + 8, ... hold the same channels: add them in a fixed order (the loop ended with a barrier,
    // or never ran, so LDS is free)
    float* sh = reinterpret_cast<float*>(lds64);
#pragma unroll
    for (int e = 0; e < 8; ++e) sh[tid * 9 + e] = csum[e];
    __syncthreads();
    if (tid < 64 && k0 + tid < p.ky) {
      float t = 0.f;
      for (int i = 0; i < NTHREADS / 8; ++i) t += sh[((tid >> 3) + i * 8) * 9 + (tid & 7)];
      p.cs_part[(long long)split * p.ky + k0 + tid] = t;
    }
  }
}

// 64 x 64 channel tile: 2-D filters with at least 48 channels on both sides
bool wide_tile(const int* filt, int cx, int ky) {
  static const bool off = getenv("LMS_NO_WGRAD_WIDE") != nullptr;     // tuning aid
  return !off && filt[0] == 1 && cx >= 48 && ky >= 48 && (cx & 7) == 0;
}

// Two images per patch (the PK form of the 64 x 64 kernel): same-size 3 x 3 convolution on maps at most 7 wide and 8 high.
bool pair_packed(const int* asp, const int* osp, const int* filt, const int* pad, int cx, int ky) {
  static const bool off = getenv("LMS_NO_WGRAD_PAIRS") != nullptr;    // tuning aid
  return !off && wide_tile(filt, cx, ky) && osp[2] <= 7 && osp[1] <= 8 && asp[1] == osp[1] && asp[2] == osp[2] && pad[2] == 1;
}

// Channel counts whose rows are 16-byte vectors take the kernel with two groups of waves; it addresses a patch (six input
// planes of ten rows at most, four of dy and eight rows) with 31 bits.
bool grouped(const int* asp, const int* osp, int cx, int ky) {
  return (cx & 7) == 0 && 2LL * ((5LL * asp[1] + 10) * asp[2] + 18) * cx < 0x7fffffffLL && 2LL * ((3LL * osp[1] + 8) * osp[2] + 16) * ky < 0x7fffffffLL;
}

// On the small layers an XCD for the tiles of a split gains where they run alone (64 -> 64 at 32^3 25.3 / 23.4 us) and loses inside a step, where what
// they read has just been written (the U-Net step at 64^3, all layers of at most eight patches, 574.7 / 578.6).
template <int P3D, bool CS>
hipError_t launch_grouped(const WPatchP& p, hipStream_t s) {
  if (P3D && wgrad_ring_wins(p)) return launch_wgrad_ring(p, s);
  constexpr int LDS = GPatch<P3D>::LDS_BYTES;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(wgrad_patch_group_kernel<P3D, CS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((wgrad_patch_group_kernel<P3D, CS>), dim3((unsigned)(p.cchunks * p.ktiles * p.splits)), dim3(GP_NT), LDS, s, p);
  return hipGetLastError();
}

struct PatchGrid { int tiles[3]; long long patches; int splits, per_split; bool pairs; };
PatchGrid patch_grid(long long batch, const int* asp, const int* osp, const int* filt, const int* pad, int cx, int ky) {
  PatchGrid g;
  const bool p3d = filt[0] == 3;
  const int td = p3d ? 4 : 1, th = p3d ? 4 : 8, tw = p3d ? 8 : 16;
  g.tiles[0] = (osp[0] + td - 1) / td;
  g.tiles[1] = (osp[1] + th - 1) / th;
  g.tiles[2] = (osp[2] + tw - 1) / tw;
  g.patches = batch * g.tiles[0] * g.tiles[1] * g.tiles[2];
  g.pairs = pair_packed(asp, osp, filt, pad, cx, ky);
  if (g.pairs) g.patches = (batch + 1) / 2;
  const int tile = wide_tile(filt, cx, ky) ? 64 : 32;
  const long long wg = (long long)((cx + tile - 1) / tile) * ((ky + tile - 1) / tile);
  // partial sums cost 4 bytes x filter size per work-group, written and read again: two work-groups per compute unit
  // (32 x 32 tiles) measured 5 % faster on the 3D U-Net step than four; with two groups of waves in one that is one, and
  // no more than one, which is what its LDS leaves room for (240 x 80 at 29 x 25 x 27: 264 of them 65 us, 240 47)
  const bool one = tile == 32 && grouped(asp, osp, cx, ky);
  static const char* const wgs = getenv("LMS_WGRAD_PATCH_WGS");       // tuning aid
  const long long target = wgs ? atoll(wgs) : tile == 64 || one ? 256 : 512;
  long long splits = one ? target / wg : (target + wg - 1) / wg;
  if (splits > g.patches) splits = g.patches;
  if (splits < 1) splits = 1;
  g.per_split = (int)((g.patches + splits - 1) / splits);
  g.splits = (int)((g.patches + g.per_split - 1) / g.per_split);
  return g;
}

}  // namespace

bool wgrad_patch_eligible(int cx, int ky, const int* filt, const int* stride) {
  for (int i = 0; i < 3; ++i)
    if (stride[i] != 1) return false;
  if (filt[1] != 3 || filt[2] != 3 || (filt[0] != 1 && filt[0] != 3)) return false;
  (void)cx;                       // any input channel count: odd counts are gathered element by element
  return (ky & 7) == 0;
}

int wgrad_patch_splits(long long batch, const int* asp, const int* osp, const int* filt, const int* pad, int cx, int ky) {
  return patch_grid(batch, asp, osp, filt, pad, cx, ky).splits;
}

hipError_t launch_wgrad_patch(const uint16_t* X, const uint16_t* DY, float* part, long long batch, const int* asp,
                              const int* osp, const int* filt, const int* pad, int cx, int ky, float* cs_part, hipStream_t s) {
  WPatchP p{};
  p.X = X; p.DY = DY; p.part = part; p.cs_part = cs_part;
  p.batch = (int)batch;
  for (int i = 0; i < 3; ++i) { p.asp[i] = asp[i]; p.osp[i] = osp[i]; p.filt[i] = filt[i]; p.pad[i] = pad[i]; }
  p.cx = cx; p.ky = ky; p.taps = filt[0] * filt[1] * filt[2];
  p.cchunks = (cx + 31) / 32; p.ktiles = (ky + 31) / 32;
  const PatchGrid g = patch_grid(batch, asp, osp, filt, pad, cx, ky);
  if (g.patches > 0x7fffff00LL) return hipErrorInvalidValue;
  for (int i = 0; i < 3; ++i) p.tiles[i] = g.tiles[i];
  p.patches = (int)g.patches; p.splits = g.splits; p.patches_per_split = g.per_split;
  const long long xb = batch * asp[0] * asp[1] * asp[2] * cx * 2, yb = batch * osp[0] * osp[1] * osp[2] * ky * 2;
  if (xb < 0x7fffff00LL && yb < 0x7fffff00LL) { p.x_bytes = (unsigned)xb; p.y_bytes = (unsigned)yb; }
  if (wide_tile(filt, cx, ky)) {
    p.cchunks = (cx + 63) / 64; p.ktiles = (ky + 63) / 64;
    auto run = [&](auto kernel) -> hipError_t {
      const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, WGRAD64_LDS_BYTES);
      if (attr != hipSuccess) return attr;
      const dim3 grid((unsigned)(p.cchunks * p.ktiles * p.splits));
      hipLaunchKernelGGL(kernel, grid, dim3(NTHREADS), WGRAD64_LDS_BYTES, s, p);
      return hipGetLastError();
    };
    if (g.pairs) return cs_part ? run(wgrad_patch64_kernel<true, true>) : run(wgrad_patch64_kernel<false, true>);
    return cs_part ? run(wgrad_patch64_kernel<true, false>) : run(wgrad_patch64_kernel<false, false>);
  }
  const long long blocks = (long long)p.cchunks * p.ktiles * p.splits;
  if (grouped(asp, osp, cx, ky) && aligned16(X, DY)) {
    if (filt[0] == 3) return cs_part ? launch_grouped<1, true>(p, s) : launch_grouped<1, false>(p, s);
    return cs_part ? launch_grouped<0, true>(p, s) : launch_grouped<0, false>(p, s);
  }
  auto run = [&](auto kernel) -> hipError_t {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(NTHREADS), 0, s, p);
    return hipGetLastError();
  };
  if (filt[0] == 3) return cs_part ? run(wgrad_patch_kernel<1, true>) : run(wgrad_patch_kernel<1, false>);
  return cs_part ? run(wgrad_patch_kernel<0, true>) : run(wgrad_patch_kernel<0, false>);
}

}  // namespace lms
