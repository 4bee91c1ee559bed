// Weight gradient of 3x3x3 stride-1 convolutions, patch-tiled as in wgrad_patch.hip, for large volumes: the two groups of waves take turns at 16 positions of one patch, and three more patches
// are on their way, a load at a time between the products, for a patch and its halo in 64-byte pieces of lines take 3 us to arrive and 0.9 to multiply.
// The tiles of a split run on one XCD: they read the same patches, half lines each, and neighbouring splits their halos.  Both parameter
// gradients, us, wgrad_patch_group_kernel / this one (and the mapping to XCDs): 64 -> 64 at 64^3 71.6 / 65.4, batch 2 130 / 118; 96 -> 96 at 40^3 48.7 / 43.8;
// 64 -> 32 at 80^3 76 / 68.  Where it runs and where it loses: wgrad_ring_wins.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_dma.hpp"
#include "wgrad_patch.hpp"

namespace lms {

namespace {

struct RPatch {
  typedef WPatch<1> PT;
  static constexpr int PIX = GP_NT / 4;                           // pixels a load
  static constexpr int XV = (PT::MAXPIX + 4 + PIX - 1) / PIX, YV = 128 / PIX;        // loads per thread and patch
  static constexpr int X_BYTES = XV * PIX * 64, Y_BYTES = 128 * 64, BUF = X_BYTES + Y_BYTES, RING = 4;
  static constexpr int TAPS = 27;
  static constexpr int SUMS = TAPS * 4096;
  static constexpr int LDS_BYTES = RING * BUF > SUMS ? RING * BUF : SUMS;
  static_assert(XV + YV <= 8 / 2, "a load behind each 16 positions of a group, and the waits count them all");
  static_assert(LDS_BYTES <= 163840, "what a compute unit has");
};

template <bool CS>
__global__ __launch_bounds__(GP_NT, 2) void wgrad_patch_ring_kernel(WPatchP p) {
  typedef WPatch<1> PT;
  typedef RPatch GP;
  constexpr int XV = GP::XV, YV = GP::YV, RING = GP::RING;
  extern __shared__ __attribute__((aligned(256))) unsigned char lds_gp[];
  int b = xcd_order(p.cchunks * p.ktiles * p.splits);
  if (b < 0) return;
  const int cc = b % p.cchunks; b /= p.cchunks;
  const int kt = b % p.ktiles; b /= p.ktiles;
  const int split = b;
  const int c0 = cc * 32, k0 = kt * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = wave8 >> 2, wave = wave8 & 3;
  const int hd = PT::TD + p.filt[0] - 1;
  const int halo_pix = hd * PT::HH * PT::HW;
  const int li = lane & 15, lg = lane >> 4;
  const int src_off = (li >> 2) * LDX + 16 * (lg & 1) + 4 * (li & 3);
  const int half = lg >> 1;

  // this thread's vectors of a patch: position relative to the patch origin (input: origin - pad), byte offset from it
  const int vch = (tid & 3) * 8;
  const bool xc_ok = c0 + vch < p.cx, yc_ok = k0 + vch < p.ky;
  int xj[XV], yj[YV];                                             // coordinates, 8 bits each
  unsigned x_off[XV], y_off[YV];
#pragma unroll
  for (int j = 0; j < XV; ++j) {
    const int pix = (tid >> 2) + j * GP::PIX;
    const int w = pix % PT::HW, h = (pix / PT::HW) % PT::HH, d = pix / (PT::HW * PT::HH);
    xj[j] = w | h << 8 | d << 16;
    x_off[j] = pix < halo_pix && xc_ok ? (unsigned)((((d * p.asp[1] + h) * p.asp[2] + w) * p.cx + c0 + vch) * 2) : DMA_OOB;
  }
#pragma unroll
  for (int j = 0; j < YV; ++j) {
    const int q = (tid >> 2) + j * GP::PIX;
    const int w = q % PT::TW, h = (q / PT::TW) % PT::TH, d = q / (PT::TW * PT::TH);
    yj[j] = w | h << 8 | d << 16;
    y_off[j] = yc_ok ? (unsigned)((((d * p.osp[1] + h) * p.osp[2] + w) * p.ky + k0 + vch) * 2) : DMA_OOB;
  }

  const int pbegin = split * p.patches_per_split;
  const int pend = (pbegin + p.patches_per_split < p.patches) ? pbegin + p.patches_per_split : p.patches;
  const int rounds = pend > pbegin ? pend - pbegin : 0;
  int tw, th, td, nb;                                             // the next patch (uniform)
  {
    unsigned t = (unsigned)pbegin;
    tw = (int)(t % (unsigned)p.tiles[2]); t /= (unsigned)p.tiles[2];
    th = (int)(t % (unsigned)p.tiles[1]); t /= (unsigned)p.tiles[1];
    td = (int)(t % (unsigned)p.tiles[0]);
    nb = (int)(t / (unsigned)p.tiles[0]);
  }
  auto advance = [&]() {
    if (++tw == p.tiles[2]) { tw = 0; if (++th == p.tiles[1]) { th = 0; if (++td == p.tiles[0]) { td = 0; ++nb; } } }
  };
  const unsigned lds_w = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)lds_gp + wave8 * 1024);
  struct Fetch { v4u rx, ry; int o0[3], i0[3]; };                 // what the loads of a patch share
  auto fetch_patch = [&]() __attribute__((always_inline)) {
    Fetch f;
    const int o[3] = {td * PT::TD, th * PT::TH, tw * PT::TW};
#pragma unroll
    for (int i = 0; i < 3; ++i) { f.o0[i] = o[i]; f.i0[i] = o[i] - p.pad[i]; }
    f.rx = buffer_rsrc(p.X + (((long long)nb * p.asp[0] + f.i0[0]) * p.asp[1] + f.i0[1]) * (long long)p.asp[2] * p.cx + (long long)f.i0[2] * p.cx, 0x7fffffff);
    f.ry = buffer_rsrc(p.DY + (((long long)nb * p.osp[0] + o[0]) * p.osp[1] + o[1]) * (long long)p.osp[2] * p.ky + (long long)o[2] * p.ky, 0x7fffffff);
    advance();
    return f;
  };
  auto load_one = [&](const Fetch& f, int r, int j) __attribute__((always_inline)) {
    const unsigned lds = lds_w + (r % RING) * GP::BUF;
    if (j < XV) {
      const bool ok = (unsigned)(f.i0[0] + (xj[j] >> 16)) < (unsigned)p.asp[0] && (unsigned)(f.i0[1] + ((xj[j] >> 8) & 255)) < (unsigned)p.asp[1] &&
                      (unsigned)(f.i0[2] + (xj[j] & 255)) < (unsigned)p.asp[2];
      load_lds16(f.rx, lds + j * (GP::PIX * 64), ok ? x_off[j] : DMA_OOB, 0);
    } else {
      const int y = yj[j - XV];
      const bool ok = f.o0[0] + (y >> 16) < p.osp[0] && f.o0[1] + ((y >> 8) & 255) < p.osp[1] && f.o0[2] + (y & 255) < p.osp[2];
      load_lds16(f.ry, lds + GP::X_BYTES + (j - XV) * (GP::PIX * 64), ok ? y_off[j - XV] : DMA_OOB, 0);
    }
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
    constexpr int LOADS = XV + YV;
    auto fetch = [&](int r) {
      const Fetch f = fetch_patch();
      unrolled<LOADS>([&](auto j) { load_one(f, r, decltype(j)::value); });
    };
#pragma unroll 1
    for (int r = 0; r < RING - 1 && r < rounds; ++r) fetch(r);
    auto patch = [&](int r, auto&& between) {
      const uint16_t* sX = reinterpret_cast<const uint16_t*>(lds_gp + (r % RING) * GP::BUF);
      wgrad_patch_mma<1, W, CS && W == 0, 2>(sX, sX + GP::X_BYTES / 2, acc, src_off, half, &cs, g, between);
    };
    // this patch has landed, and the one before it, whose place the next loads take, has been read
    int r = 0;
#pragma unroll 1
    for (; r + RING - 1 < rounds; ++r) {
      wait_barrier<(RING - 2) * LOADS>();
      const Fetch f = fetch_patch();
      patch(r, [&](int i) { if (i < LOADS) load_one(f, r + RING - 1, i); });
    }
#pragma unroll 1
    for (int left = (rounds < RING - 1 ? rounds : RING - 1) - 1; left >= 0; --left) {     // the last ones
      if (left == 0) wait_barrier<0>();
      else if (left == 1) wait_barrier<LOADS>();
      else wait_barrier<(RING - 2) * LOADS>();
      patch(rounds - 1 - left, [](int) {});
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

template <bool CS>
hipError_t launch_ring(const WPatchP& p, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(wgrad_patch_ring_kernel<CS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, RPatch::LDS_BYTES);
  if (attr != hipSuccess) return attr;
  const long long wgs = (long long)p.cchunks * p.ktiles * p.splits;
  hipLaunchKernelGGL((wgrad_patch_ring_kernel<CS>), dim3((unsigned)xcd_grid(wgs)), dim3(GP_NT), RPatch::LDS_BYTES, s, p);
  return hipGetLastError();
}

}  // namespace

// The ring pays where the patches come from beyond the L2s: 800 layers of 9 to 60 patches a work-group, time against the group kernel: from 20 MB of x and dy on with
// two chunks of input channels that are mostly there, and from 32 MB on with any two tiles, 0.78 to 1.01 (mean 0.92 of 438); the others 0.87 to 1.28, 99
// of them would gain (us, 128 -> 152 at 22^3, 6 MB 30.4 / 38.9; 96 -> 160 at 29 x 29 x 30, 13 MB 40.3 / 41.5; 48 -> 176 at 27^3 28.6 / 33.5; of one
// tile 16 -> 16 at 78^3, batch 2, 61 MB 52.8 / 55.3).
bool wgrad_ring_wins(const WPatchP& p) {
  const double bytes = 2.0 * p.batch * ((double)p.asp[0] * p.asp[1] * p.asp[2] * p.cx + (double)p.osp[0] * p.osp[1] * p.osp[2] * p.ky);
  return p.patches_per_split > 8 && ((p.cx > 52 && bytes >= 20e6) || (p.cx >= 24 && p.cchunks * p.ktiles > 1 && bytes >= 32e6));
}

hipError_t launch_wgrad_ring(const WPatchP& p, hipStream_t s) { return p.cs_part ? launch_ring<true>(p, s) : launch_ring<false>(p, s); }

}  // namespace lms
