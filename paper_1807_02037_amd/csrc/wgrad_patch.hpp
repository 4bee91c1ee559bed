// What the patch-tiled weight-gradient kernels share (wgrad_patch.hip, wgrad_ring.hip; internal).
#pragma once
#include "conv_dma.hpp"

namespace lms {

struct WPatchP {
  const uint16_t* X;
  const uint16_t* DY;
  float* part;
  int batch;
  int asp[3], osp[3], filt[3], pad[3];
  int cx, ky, taps;
  int cchunks, ktiles, splits;
  int tiles[3];
  int patches;             // batch * tiles (pairs of images in the packed form of the 64 x 64 kernel)
  int patches_per_split;
  unsigned x_bytes, y_bytes;   // tensor sizes if both are below 2 GiB (32-bit buffer offsets), else 0
  float* cs_part;              // partial column sums of dy [split][ky] on the side, or null
};

// The kernel with a ring of patches (wgrad_ring.hip): whether it is the faster one, and its launch (P3D, input channels in 16-byte vectors).
bool wgrad_ring_wins(const WPatchP& p);
hipError_t launch_wgrad_ring(const WPatchP& p, hipStream_t s);

namespace {

constexpr int GP_NT = 512; // threads of the kernels with two groups of four waves
constexpr int LDX = 32;    // LDS row pitch in bf16 elements: 64 bytes = 16 banks, so the four rows of a transpose read cover all 64 banks (no conflicts measured)

template <int P3D>
struct WPatch {
  static constexpr int TD = P3D ? 4 : 1, TH = P3D ? 4 : 8, TW = P3D ? 8 : 16;
  static constexpr int HH = TH + 2, HW = TW + 2;
  static constexpr int MAXPIX = (TD + (P3D ? 2 : 0)) * HH * HW;
  static constexpr int MAXT = P3D ? 7 : 3;          // taps per wave at most
};

// Wave w owns the contiguous taps [TAPS*w/4, TAPS*(w+1)/4).  The taps kw = 0, 1, 2 of one filter row (kd, kh) read
// the positions p .. p+9 of one halo row: where a wave has several of them, the 12 positions p .. p+11 are fetched
// once (three transpose reads) and the fragments of the three taps are cut out in registers.
// CS: also ones x dy, the column sums (wave 0, which has one tap less than the others).
// G groups of waves take turns at 16 positions; g: this one.  between(i): after the products of the group's i-th 16 positions.
template <int P3D, int W, bool CS = false, int G = 1, typename F>
__device__ __forceinline__ void wgrad_patch_mma(const uint16_t* sX, const uint16_t* sY, f32x16 (&acc)[WPatch<P3D>::MAXT], int src_off,
                                                int half, f32x16* cs, int g, F&& between) {
  typedef WPatch<P3D> PT;
  constexpr int TAPS = P3D ? 27 : 9;
  constexpr int LO = TAPS * W / 4, HI = TAPS * (W + 1) / 4;
#pragma unroll
  for (int i = 0; i < 8 / G; ++i) {
    // positions q0 .. q0+7 of this lane's half: one row (or half row) of the patch, contiguous in the halo tile
    const int q0 = (i * G + g) * 16 + 8 * half;
    const int pw = q0 % PT::TW, ph = (q0 / PT::TW) % PT::TH, pd = q0 / (PT::TW * PT::TH);
    const uint16_t* xb = sX + ((pd * PT::HH + ph) * PT::HW + pw) * LDX + src_off;
    const uint16_t* yb = sY + q0 * LDX + src_off;
    const bf16x8 bfr = tr_frag(yb, yb + 4 * LDX);
    if constexpr (CS) {
      const __bf16 o = (__bf16)1.f;
      const bf16x8 ones = {o, o, o, o, o, o, o, o};
      *cs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, bfr, *cs, 0, 0, 0);
    }
#pragma unroll
    for (int row = LO / 3; row <= (HI - 1) / 3; ++row) {
      const int k_lo = (LO > row * 3 ? LO : row * 3) - row * 3, k_hi = (HI < row * 3 + 3 ? HI : row * 3 + 3) - row * 3;   // kw range
      const uint16_t* xr = xb + ((row / 3) * PT::HH + (row % 3)) * PT::HW * LDX;
      if (k_hi - k_lo == 1) {
        const bf16x8 af = tr_frag(xr + k_lo * LDX, xr + (k_lo + 4) * LDX);
        acc[row * 3 + k_lo - LO] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr, acc[row * 3 + k_lo - LO], 0, 0, 0);
      } else {
        const v2u r0 = tr_read(xr);
        const v2u r1 = tr_read(xr + 4 * LDX);
        const v2u r2 = tr_read(xr + 8 * LDX);
        const unsigned u[6] = {r0[0], r0[1], r1[0], r1[1], r2[0], r2[1]};     // two positions per word
#pragma unroll
        for (int kw = k_lo; kw < k_hi; ++kw) {
          v4u f;
          if (kw == 0) f = v4u{u[0], u[1], u[2], u[3]};
          else if (kw == 2) f = v4u{u[1], u[2], u[3], u[4]};
          else f = v4u{__builtin_amdgcn_alignbit(u[1], u[0], 16), __builtin_amdgcn_alignbit(u[2], u[1], 16),
                       __builtin_amdgcn_alignbit(u[3], u[2], 16), __builtin_amdgcn_alignbit(u[4], u[3], 16)};
          acc[row * 3 + kw - LO] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f), bfr, acc[row * 3 + kw - LO], 0, 0, 0);
        }
      }
    }
    between(i);
  }
}

}  // namespace
}  // namespace lms
