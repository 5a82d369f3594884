// Where the 16-byte loads of a product's operand rows lie (gemm_fp4.hip, gemm_block.hip), and which segments of an im2col row hold a piece
// of two kernel rows.  Plain arithmetic, on the host too: the tests walk every row length and check what is read.
#pragma once
#include <stdint.h>

namespace bmx {

// A row of `dwords` data dwords is fetched in segments of four pieces of 16 bytes.  A piece that the row ends in, and those behind it,
// are the row's last 16 bytes, so that nothing behind the row is read, which may be where the buffer ends; rows of less than 16 bytes
// are whole pieces and stand 16 bytes apart.  By how many bytes piece `piece` of segment `segment` is moved back for that, 0 for whole
// pieces: up to 12 bytes in front of the segment.
__host__ __device__ __forceinline__ uint32_t piece_back(int segment, int piece, int dwords) {
  const int over = 16 * segment + 4 * piece + 4 - (dwords > 4 ? dwords : 4);
  return over > 0 ? 4u * (uint32_t)over : 0u;
}

// Whether a piece of segment `segment` of an im2col row, whose kernel rows are runs of `run` words, holds words of two runs, or the row's
// last word alone: an odd multiple of an odd run lies among the segment's eight words.  two_runs(x) is x / (2 run).
template <class Div>
__host__ __device__ __forceinline__ bool runs_meet(uint32_t run, Div two_runs, int segment) {
  const uint32_t end = 8u * (uint32_t)segment + 7u;
  if (!(run & 1u) || end < run) return false;
  return run * (2u * two_runs(end - run) + 1u) >= 8u * (uint32_t)segment;
}

}  // namespace bmx
