// What the BP team kernels (bp_chunk.hip, bp_stream.hip) share on the device:
// the 12-byte state of a check (or part of one) and its messages, and access to
// their arguments.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "decoder.h"

namespace tmcs {
namespace dec {

// State {n1, n2, word}.  n1, n2: the two smallest |q|, times alpha.  word: the
// sign of the message to edge j in bit 31 - j, s_c in bit 5, and in bits 0..4 the
// edge that holds the minimum (31: none here).
constexpr int PART_MAX_DEG = 26;            // sign bits 31..6
constexpr uint32_t W_SIGNS = 0xFFFFFFC0u;
constexpr uint32_t W_SC = 0x20u;
constexpr uint32_t W_POS = 0x1Fu;

__device__ __forceinline__ uint32_t gload(const uint32_t* p) { return *(const TMCS_GLOBAL_AS uint32_t*)p; }

__device__ __forceinline__ float with_sign(float mag, uint32_t s) {
  return __uint_as_float(__float_as_uint(mag) ^ (s & 0x80000000u));
}

// The launch's arguments (kernel arguments, or an item's entry of a multi
// launch's table) are read through the scalar cache where they are used: held in
// registers all at once they would not fit beside the passes' own scalars.
#define TMCS_CONST_AS __attribute__((address_space(4)))
// The same pointer, opaque to the compiler, so that what is read through it is
// read here and not at the start of the kernel.
template <typename P>
__device__ __forceinline__ P reread(P p) {
  asm volatile("" : "+s"(p));
  return p;
}
template <typename T>
__device__ __forceinline__ T at_byte(const T* base, uint32_t byte) {
  return gload((const T*)((const char*)base + byte));
}

}  // namespace dec
}  // namespace tmcs
