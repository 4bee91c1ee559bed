// Loads from memory straight to LDS, for the convolution kernels built on them (internal).
#pragma once
#include "conv_tile.hpp"

namespace lms {
namespace {

// 16 bytes per lane from buffer offset voff + soff to LDS bytes lds + 16 * lane (lds: the same for the whole wave; offsets
// outside the buffer write zeros).  Written in assembly because the compiler, seeing such a load, waits for all of
// them before any LDS transpose read; it has no register output, and wait_barrier does the waiting.  The compiler does not
// know that a load is in here and adds no wait states: of the five between a vector instruction that writes a scalar
// register and a load that reads it (rsrc, soff), two are here; that the code around keeps the distance is tested on the
// assembly (all five here: 0.7 % slower).  m0 is a reserved register, which clang warns about; the clobber keeps its
// initialisations from being merged across.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lds16(v4u rsrc, unsigned lds, unsigned voff, unsigned soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ v4u buffer_rsrc(const void* base, long long bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  return v4u{(unsigned)a, (unsigned)(a >> 32) & 0xffffu, (unsigned)(bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00020000u};
}

}  // namespace
}  // namespace lms
