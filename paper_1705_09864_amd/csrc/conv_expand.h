// Bits to FP4 (E2M1) operands for the matrix-core convolutions, see conv_mfma.hip.
#pragma once
#include "bmx_internal.h"

namespace bmx {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v8i widen(v4i e) {
  v8i x;
#pragma unroll
  for (int d = 0; d < 4; ++d) x[d] = e[d];
#pragma unroll
  for (int d = 4; d < 8; ++d) x[d] = 0;
  return x;
}

// The four bit planes of a dword as the four operand dwords of an MFMA step (nibble i of dword
// d = bit 4 i + d).  The pixel side leaves planes 0 to 2 where they stand in their nibbles
// (E2M1 codes 1, 2, 4 = 0.5, 1, 2) and shifts only the plane under the nibble's sign bit: five
// VALU instructions instead of seven, in a kernel whose VALU work outweighs its MFMA time.  The
// filter side, expanded once per workgroup, carries the reciprocal magnitudes (2, 1, 0.5, 2)
// with the sign of the filter value (bit set: +, bit clear: -, the nibble's sign bit being
// the inverted filter bit), so that a set pixel bit contributes +1 or -1 and a clear one nothing.
__device__ __forceinline__ v4i expand_pixel(uint32_t w) {
  v4i e;
  e[0] = (int)(w & 0x11111111u);
  e[1] = (int)(w & 0x22222222u);
  e[2] = (int)(w & 0x44444444u);
  e[3] = (int)((w >> 3) & 0x11111111u);
  return e;
}
__device__ __forceinline__ v4i expand_filter(uint32_t w) {
  const uint32_t nw = ~w;
  v4i e;
  e[0] = (int)(((nw << 3) & 0x88888888u) | 0x44444444u);
  e[1] = (int)(((nw << 2) & 0x88888888u) | 0x22222222u);
  e[2] = (int)(((nw << 1) & 0x88888888u) | 0x11111111u);
  e[3] = (int)((nw & 0x88888888u) | 0x44444444u);
  return e;
}

}  // namespace
}  // namespace bmx
