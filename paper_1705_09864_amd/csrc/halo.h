// The halo of a packed image, written by the kernels that write the image.
#pragma once
#include "bmx_internal.h"

namespace bmx {

// Halo pixels first, first + step, .. of `images` images of H x W pixels and `pad` more beyond each edge (pad > 0; less than 2^31
// pixels in all), Cw words each: their word cw is +1 (the sign of the next layer's zero padding) for every real one of C
// channels and 0 bits for missing ones.  In the order of the padded image a halo pixel k is pixel k as far as the first interior
// row, then what is right of an interior row and left of the next in one run, then the rest: two divisions a word.
// (They are left to the compiler, which keeps the reciprocals out of the loop; constants from the host would be six more scalar
// registers, which the convolution of 49 and 50 words, its offsets in them, does not have.)
__device__ __forceinline__ void write_halo(uint64_t* image, int images, int H, int W, int pad, int C, int Cw, int cw,
                                           uint32_t first, uint32_t step) {
  const uint64_t ones = (cw == Cw - 1 && (C & 63)) ? (((uint64_t)1 << (C & 63)) - 1) : ~(uint64_t)0;
  const uint32_t side = 2 * pad, padded = (uint32_t)(H + side) * (uint32_t)(W + side), inside = (uint32_t)H * (uint32_t)W;
  const uint32_t lead = (uint32_t)pad * (uint32_t)(W + side + 1), last_row = H - 1, per_image = padded - inside;
  for (uint32_t i = first; i < per_image * (uint32_t)images; i += step) {
    const uint32_t n = i / per_image, k = i - n * per_image;
    uint32_t at = n * padded + k;
    if (k >= lead) at += (uint32_t)W * (min((k - lead) / side, last_row) + 1);
    image[(int64_t)at * Cw + cw] = ones;
  }
}

}  // namespace bmx
