// Barrier and epilogue of the convolution kernels that move operands and results through buffers and LDS (internal).
#pragma once
#include <type_traits>

#include "conv_common.hpp"

namespace lms {
namespace {

constexpr unsigned DMA_OOB = 0x80000000u;        // a buffer offset outside every buffer

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef short v4s __attribute__((ext_vector_type(4)));

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<N, I + 1>(f);
  }
}

// Eight values of a column as an operand: two LDS transpose reads, of the four rows at q0 and the four at q1 of this lane's half.
__device__ __forceinline__ v2u tr_read(const void* q) {
  return __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)q));
}
__device__ __forceinline__ bf16x8 tr_frag(const void* q0, const void* q1) {
  const v2u a = tr_read(q0), b = tr_read(q1);
  return __builtin_bit_cast(bf16x8, v4u{a[0], a[1], b[0], b[1]});
}

// At most N of this wave's memory loads may still be in flight, and its LDS reads have come back; then every wave of the
// work-group has got here.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Nothing of this wave's loads to LDS is in flight.  A __syncthreads() behind it, and not a wait_barrier, tells the compiler that the loads it
// knows have come back: without that it waits for each where it is used, and with it for the stores before it.
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// LDS bytes that wave_epilogue needs per wave: 32 positions x WTN channels of fp32, rows 16 bytes apart modulo 256.
constexpr int epi_wave_bytes(int wtn) { return 32 * (wtn + 4) * 4; }

// The tensors of the epilogue as the rows of one tile see them: buffers that start at the tile's first row, so that offsets
// have 32 bits and everything beyond them (rows past the last, columns past the last, a tensor that is not there) reads
// zeros and drops writes.  No branch: behind one the compiler waits for every older load before the next, and
// the 16 vectors of a thread came one latency after the other.
struct EpiBuffers {
  __amdgpu_buffer_rsrc_t add, mask, out;
  __device__ __forceinline__ EpiBuffers(const IgemmP& p, long long row0, long long bytes) {
    const int n = (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff);
    const long long at = row0 * p.nout;
    add = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.add ? p.add + at : p.out), 0, p.add ? n : 0, 0x00020000);
    mask = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.mask ? p.mask + at : p.out), 0, p.mask ? n : 0, 0x00020000);
    out = __builtin_amdgcn_make_buffer_rsrc(p.out + at, 0, n, 0x00020000);
  }
  __device__ __forceinline__ static uint4 get(__amdgpu_buffer_rsrc_t rs, unsigned off) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
  }
  __device__ __forceinline__ void put(unsigned off, const uint4& d) const {            // 2: nontemporal, around the L2s
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, d), out, (int)off, 0, 2);
  }
};

// Epilogue of a wave's TM x TN transposed accumulators (lane l of a 32 x 32 one holds position l % 32, channels
// 8 * (v / 4) + 4 * (l / 32) + v % 4): 32 positions at a time go through the wave's own LDS (in order: no barrier) and leave
// as 8-channel vectors, WTN / 8 lanes to a position.  n: this lane's first channel (n_ok: it exists); er: tile row of the
// lane's first vector; add / mask: the vectors of those rows, fetched ahead; off(r): byte offset of the lane's vector in
// row r of the tile.
template <int WTN, int TM, int TN, typename Off>
__device__ __forceinline__ void wave_epilogue(const IgemmP& p, const EpiBuffers& eb, const f32x16 (&acc)[TM][TN], unsigned char* lds, const uint4* add,
                                              const uint4* mask, int n, bool n_ok, int er, Off&& off) {
  constexpr int LDC = WTN + 4, LPR = WTN / 8, RPI = 64 / LPR, QV = 32 / RPI;
  const int lane = threadIdx.x & 63, half = lane >> 5, cg = (lane % LPR) * 8;
  float* sC = reinterpret_cast<float*>(lds);
  EpiCoef coef;
  if (n_ok) epilogue_coef(p, n, 8, coef);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        *reinterpret_cast<float4*>(sC + (lane & 31) * LDC + j * 32 + 8 * v + 4 * half) =
            make_float4(acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]);
#pragma unroll
    for (int q = 0; q < QV; ++q) {
      const float* row = sC + (lane / LPR + q * RPI) * LDC + cg;
      const float4 lo = *reinterpret_cast<const float4*>(row), hi = *reinterpret_cast<const float4*>(row + 4);
      const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      eb.put(off(er + i * 32 + q * RPI), epilogue_pack8(p, coef, v, add[i * QV + q], mask[i * QV + q]));
    }
  }
}

}  // namespace
}  // namespace lms
