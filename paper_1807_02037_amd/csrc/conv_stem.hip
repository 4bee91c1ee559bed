// Forward convolution of first layers (2-D, 1 to 4 input channels) whose stride times channels is even: the 7x7 stride-2 stem on
// 3 channels, 3x3 and 5x5 stride-2 stems, any filter on 2 or 4 channels.
//
// The taps of one filter row read one contiguous run of filt[2] * channels elements of an input row, and neighbouring positions
// start stride * channels elements further, an even number: a run can be read from the input rows as they lie in LDS with
// 4-byte alignment, eight elements a lane, which is an MFMA operand.  So a reduction of filt[1] runs, each padded to a multiple of
// eight with zero weights, takes the place of the patch matrix that conv_small.hip gathers element by element (what bounds it).
// A tile is up to four output rows by up to 128 positions, its positions numbered through, 32 to a product; the filter
// stays in registers (both halves of 64 outputs), the input rows of the next tile are on their way while one is multiplied, and
// results leave through wave_epilogue.
//
// The elements under a run's zero weights are pixels beside the window, and zero times an infinity or a NaN is a NaN.  A sum that is
// finite met no such value; 32 positions with one that is not are multiplied again with those elements masked, so that an
// infinity or a NaN reaches the outputs whose window contains it and no others (the look at the sums: 45.6 -> 46.6 us at 64 images of
// 224 x 224; at the input rows on their way to LDS, before the next ones are asked for, 47.4).
//
// 64 images of 224 x 224: 87 -> 46 us against 21 for its 122 MB at the rate of a large copy; 64 images of 48 x 48 24 -> 10.  At 256 images of
// 224 x 224 it moves 535 MB at 3.3 TB/s with the matrix pipes busy 18 % of the cycles and LDS active in 25 %: what bounds it is the chain of a
// tile (rows to LDS, barrier, products, epilogue: 16 other vector instructions per product) on two work-groups a compute unit.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "conv_common.hpp"
#include "conv_tile.hpp"

namespace lms {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef unsigned v4ua __attribute__((ext_vector_type(4), aligned(4)));

constexpr int ST_NI = 4, ST_NH = 7;                  // rows a wave stages, dwords a lane has of each
constexpr int ST_ROWS = 4 * ST_NI, ST_PD = 64 * ST_NH;    // staged rows and dwords of one at most
constexpr int ST_UNITS = 4;                          // groups of 32 positions a wave takes per tile
constexpr int ST_LDW = 96;                           // pitch of the staged filter rows (192 bytes)
constexpr int ST_EPI = 4 * epi_wave_bytes(64);

struct StemP {
  IgemmP g;
  int lead;                    // zero weight before a run: its first element is then at an even offset
  int rc, chunks;              // groups of eight elements of a run, of the reduction
  int th, tw;                  // tile: output rows, positions
  int tiles_h, tiles_w, tiles;
  int rows, pd, pitch;         // staged input rows, their dwords, and those rounded up to a wave's 64
  unsigned tw_magic;           // u / tw = u * tw_magic >> 20
};

__device__ __forceinline__ bf16x8 st_tr_frag(const uint16_t* p0, const uint16_t* p1) {
  const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p0);
  const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p1);
  const v8s r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// KS: reduction steps of 16 elements, two groups of eight
template <int KS>
__global__ __launch_bounds__(NTHREADS, 2) void conv_stem_kernel(StemP sp) {
  __shared__ __attribute__((aligned(16))) unsigned raw[ST_ROWS * ST_PD];
  __shared__ __attribute__((aligned(16))) unsigned char epi[ST_EPI];
  static_assert(KS * 16 * ST_LDW * 2 <= ST_EPI, "the filter is staged where the results go later");
  const IgemmP& p = sp.g;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4, half = lane >> 5;
  const int c = p.red, run = p.filt[2] * c, row_el = p.asp[2] * c;

  // ---- the filter: row 8 g + i of LDS holds element i of group g, zeros outside the run; then both halves as fragments ----
  uint16_t* sW = reinterpret_cast<uint16_t*>(epi);
  for (int v = tid; v < KS * 16 * 8; v += NTHREADS) {
    const int j = v >> 3, cv = v & 7, grp = j >> 3, kh = grp / sp.rc, e = (grp - kh * sp.rc) * 8 + (j & 7) - sp.lead;
    uint4 w = make_uint4(0, 0, 0, 0);
    if (grp < sp.chunks && e >= 0 && e < run && cv * 8 < p.nout) w = *reinterpret_cast<const uint4*>(p.B + (long long)(kh * run + e) * p.nout + cv * 8);
    *reinterpret_cast<uint4*>(sW + j * ST_LDW + cv * 8) = w;
  }
  __syncthreads();
  bf16x8 wf[KS][2];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint16_t* q = sW + (ks * 16 + 8 * half + (li >> 2)) * ST_LDW + j * 32 + 16 * (lg & 1) + 4 * (li & 3);
      wf[ks][j] = st_tr_frag(q, q + 4 * ST_LDW);
    }
  // ---- where this lane's group of each step lies in the staged rows, bytes from its position's first element ----
  int g_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int grp = 2 * ks + half, kh = grp / sp.rc;
    g_off[ks] = grp < sp.chunks ? kh * sp.pitch * 4 + (grp - kh * sp.rc) * 16 : 0;      // zero weights: any elements (masked where a sum is not finite)
  }

  // ---- input rows: wave w stages rows w, w + 4, ..., a lane every 64th dword ----
  unsigned next[ST_NI][ST_NH];
  const int step = (int)gridDim.x;
  auto place = [&](int t, int& n, int& oh0, int& ow0) {
    const int tw = t % sp.tiles_w, r = t / sp.tiles_w;
    ow0 = tw * sp.tw;
    oh0 = r % sp.tiles_h * sp.th;
    n = r / sp.tiles_h;
  };
  const long long img_el = (long long)p.asp[1] * row_el;
  auto load = [&](int t) {
    int n, oh0, ow0;
    place(t, n, oh0, ow0);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(p.A + n * img_el), 0, (int)(img_el * 2), 0x00020000);
    const int e0 = (ow0 * p.stride[2] - p.pad[2]) * c - sp.lead, ih0 = oh0 * p.stride[1] - p.pad[1];
    unsigned off[ST_NH];
#pragma unroll
    for (int h = 0; h < ST_NH; ++h) {
      const int e = e0 + 2 * (lane + 64 * h);
      off[h] = (unsigned)e < (unsigned)row_el && lane + 64 * h < sp.pd ? (unsigned)e * 2u : DMA_OOB;
    }
#pragma unroll
    for (int i = 0; i < ST_NI; ++i) {
      const int r = wave + 4 * i, ih = ih0 + r;
      const bool ok = r < sp.rows && (unsigned)ih < (unsigned)p.asp[1];               // uniform
      const unsigned base = ok ? (unsigned)(ih * row_el * 2) : DMA_OOB;
#pragma unroll
      for (int h = 0; h < ST_NH; ++h) next[i][h] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(ok ? off[h] + base : DMA_OOB), 0, 0);
    }
  };

  const int cg = (lane & 7) * 8, er = lane >> 3;                  // this lane's vector of eight outputs, its row of eight
  const unsigned col = cg < p.nout ? (unsigned)(cg * 2) : DMA_OOB;
  int t = (int)blockIdx.x;
  if (t < sp.tiles) load(t);
  for (; t < sp.tiles; t += step) {
    __syncthreads();                                              // the rows (and the filter) have been read
#pragma unroll
    for (int i = 0; i < ST_NI; ++i)
#pragma unroll
      for (int h = 0; h < ST_NH; ++h)
        if (wave + 4 * i < sp.rows && 64 * h < sp.pd) raw[(wave + 4 * i) * sp.pitch + lane + 64 * h] = next[i][h];
    int n, oh0, ow0;
    place(t, n, oh0, ow0);
    if (t + step < sp.tiles) load(t + step);
    wait_barrier<63>();                                           // the stores to LDS; the loads stay in flight
    const int tw = p.osp[2] - ow0 < sp.tw ? p.osp[2] - ow0 : sp.tw, th = p.osp[1] - oh0 < sp.th ? p.osp[1] - oh0 : sp.th;
    const long long row0 = ((long long)n * p.osp[1] + oh0) * p.osp[2] + ow0;
    const EpiBuffers eb(p, row0, (p.M - row0) * p.nout * 2);
#pragma unroll 1
    for (int i = 0; i < ST_UNITS; ++i) {
      const int u0 = (wave + 4 * i) * 32;
      if (u0 >= sp.th * sp.tw) break;                             // uniform
      auto at = [&](int u, int& dr, int& dc) {                    // position u of the tile; false: outside the image
        dr = (int)((unsigned)u * sp.tw_magic >> 20);
        dc = u - dr * sp.tw;
        return dr < th && dc < tw;
      };
      int dr, dc;
      const bool in = at(u0 + (lane & 31), dr, dc);
      const unsigned char* x = reinterpret_cast<const unsigned char*>(raw) + (in ? dr * p.stride[1] * sp.pitch * 4 + dc * p.stride[2] * c * 2 : 0);
      f32x16 acc[1][2];
      auto products = [&](auto masked_c) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[0][j][v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          v4ua q = *reinterpret_cast<const v4ua*>(x + g_off[ks]);
          if constexpr (decltype(masked_c)::value) {
            int off = g_off[ks], first = sp.lead, end = run + sp.lead;      // elements of the run in this group: first to end
            asm volatile("" : "+v"(off));                         // worked out here: eleven steps' masks do not fit the registers
            const int gi = sp.rc > 16 ? off >> 4 : off >> 4 & 15; // a row is whole 256 bytes, and one of more than 16 groups the only one
            first -= gi * 8;
            end = 2 * ks + half < sp.chunks ? end - gi * 8 : 0;
#pragma unroll
            for (int w = 0; w < 4; ++w)
              q[w] &= (2 * w >= first && 2 * w < end ? 0xffffu : 0u) | (2 * w + 1 >= first && 2 * w + 1 < end ? 0xffff0000u : 0u);
          }
          const bf16x8 xf = __builtin_bit_cast(bf16x8, q);
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks][j], xf, acc[0][j], 0, 0, 0);
        }
      };
      products(std::false_type{});
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(magnitude(acc[0][0], magnitude(acc[0][1], 0.f)) < __builtin_inff())) != 0, 0))
        products(std::true_type{});
      auto out_off = [&](int r) -> unsigned {                     // r: row of the 32 positions
        int d, e;
        return at(u0 + r, d, e) ? col + (unsigned)((d * p.osp[2] + e) * p.nout * 2) : DMA_OOB;
      };
      uint4 add[4], mask[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) add[q] = mask[q] = make_uint4(0, 0, 0, 0);
      if (p.add || p.mask) {                                      // uniform
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          add[q] = EpiBuffers::get(eb.add, out_off(er + q * 8));
          mask[q] = EpiBuffers::get(eb.mask, out_off(er + q * 8));
        }
      }
      wave_epilogue<64, 1, 2>(p, eb, acc, epi + wave * epi_wave_bytes(64), add, mask, cg, cg < p.nout, er, out_off);
    }
  }
}

bool stem_plan(const IgemmP& p, StemP& sp) {
  sp.g = p;
  const int c = p.red, sc = p.stride[2] * c, run = p.filt[2] * c;
  if (p.mode != 0 || c < 1 || c > 4 || p.nout > 64 || (p.nout & 7) != 0 || p.asp[0] != 1 || p.osp[0] != 1 || p.filt[0] != 1 || p.pad[0] != 0) return false;
  if ((sc & 1) != 0 || (p.asp[2] * c & 1) != 0 || 2LL * p.asp[1] * p.asp[2] * c >= 0x7fffffffLL || p.filt[1] > ST_ROWS) return false;
  sp.lead = (p.pad[2] * c) & 1;
  sp.rc = (sp.lead + run + 7) / 8;
  sp.chunks = p.filt[1] * sp.rc;
  if (sp.chunks > 22 || sp.rc * 8 > 2 * ST_PD) return false;
  // up to four rows, up to 128 positions (the row split evenly)
  sp.th = (ST_ROWS - p.filt[1]) / p.stride[1] + 1;
  if (sp.th > 4) sp.th = 4;
  if (sp.th > p.osp[1]) sp.th = p.osp[1];
  int most = (2 * ST_PD - sp.rc * 8) / sc + 1;
  if (most > 128) most = 128;
  sp.tiles_w = (p.osp[2] + most - 1) / most;
  sp.tw = (p.osp[2] + sp.tiles_w - 1) / sp.tiles_w;
  const long long images = p.M / ((long long)p.osp[1] * p.osp[2]);
  while (sp.th > 1 && images * ((p.osp[1] + sp.th - 1) / sp.th) * sp.tiles_w < 192) sp.th = (sp.th + 1) / 2;
  while (sp.th > 1 && 2LL * sp.th * p.osp[2] * p.nout >= 0x7fffffffLL) --sp.th;      // 31-bit offsets within the output rows of a tile
  sp.tiles_h = (p.osp[1] + sp.th - 1) / sp.th;
  sp.rows = (sp.th - 1) * p.stride[1] + p.filt[1];
  sp.pd = ((sp.tw - 1) * sc + sp.rc * 8 + 1) / 2;
  sp.pitch = (sp.pd + 63) / 64 * 64;
  sp.tw_magic = (unsigned)(((1u << 20) + sp.tw - 1) / sp.tw);
  const long long tiles = images * sp.tiles_h * sp.tiles_w;
  if (tiles > 0x3fffffffLL || p.M >= 0x7fffffffLL) return false;
  sp.tiles = (int)tiles;
  return true;
}

}  // namespace

bool conv_stem_eligible(const IgemmP& p) {
  static const bool off = getenv("LMS_NO_CONV_STEM") != nullptr;      // tuning aid
  StemP sp{};
  return !off && ((uintptr_t)p.A & 3) == 0 && aligned16(p.B, p.out, p.add, p.mask) && stem_plan(p, sp);
}

hipError_t launch_conv_stem(IgemmP& p, hipStream_t s) {
  StemP sp{};
  if (!stem_plan(p, sp)) return hipErrorInvalidValue;
  if (sp.tiles <= 0) return hipSuccess;
  const dim3 grid((unsigned)(sp.tiles < 512 ? sp.tiles : 512));       // two work-groups per compute unit
  const int ks = (sp.chunks + 1) / 2;
  if (ks <= 4) hipLaunchKernelGGL(conv_stem_kernel<4>, grid, dim3(NTHREADS), 0, s, sp);
  else if (ks <= 7) hipLaunchKernelGGL(conv_stem_kernel<7>, grid, dim3(NTHREADS), 0, s, sp);
  else hipLaunchKernelGGL(conv_stem_kernel<11>, grid, dim3(NTHREADS), 0, s, sp);
  return hipGetLastError();
}

}  // namespace lms
