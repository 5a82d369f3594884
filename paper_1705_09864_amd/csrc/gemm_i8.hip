// k-bit products on the int8 matrix cores (Sec. 2.1, Eq. 1; arbitrary bit widths after DoReFa-Net):
// S[m][n] = sum_k q[m][k] * v[n][k] with q the level of the activation and v the weight's odd
// integer (sign for one bit, 2 q_w - L_w above).
//
// Taken for every pair of bit widths, large products of 1 or 2 by 1 bits aside (gemm_fp4.hip).  Walked plane by plane with AND +
// popcount, such a product costs bits_a * bits_w passes over K on the vector ALU (4 x 4 bits, 500 x
// 1000 x 2304: 67 us, and a 16 MB array of per-plane results to add up afterwards, 5 us).  As whole
// numbers it is one pass on the matrix cores, whatever the bits.
//
// Up to four bits on both sides, two values share a byte of the operands' copies (see `ahead`): the product waits for its
// operands' way from L2.  us a call, a value a byte / two: 500 x 1000 x 2304 of 4 x 4 bits 12.4 / 10.1, 415 x 832 x 1152 of 4 x 2
// 8.1 / 6.5, 871 x 369 x 7304 of 4 x 1 19.8 / 16.0.
//
// Eight-bit levels do not fit a signed byte: q - 128 and q_w - 128 do, and the sums of the operands'
// rows, counted from the words a lane loads anyway (v_dot4), put the difference right:
//   S = scale * (sum a' v' + ca * sum_k v') + rs * (sum_k a' + ca * K),  a' = q - ca,
//   v' = v, scale = 1, rs = 0  (up to 7 weight bits)  or  v' = q_w - 128, scale = 2, rs = 1  (8 bits),
// in 32-bit wrap-around arithmetic (the result itself fits, the launcher's caller has checked).
//
// Layout.  A dot product does not care about the order of k, and both operands are written by
// quant_tiles_kernel for this kernel alone, so they are stored the way the MFMA wants them: tile
// (row block of 32, k step of 32; of 64 with two values a byte) is 1 KiB, lane l of a wave taking bytes [16 l, 16 l + 16): row
// l % 32, half l / 32 of the step.  Every operand load is one contiguous KiB, no LDS, no
// transposition.  K is zero padded to whole blocks of 256, rows to whole blocks of 32.
#include "bmx_internal.h"

#include <algorithm>
#include <type_traits>

namespace bmx {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// ---- quantise + tile.  A workgroup turns 32 rows x 256 k of one operand into eight tiles: a wave
// reads its rows, 1 KiB of each (all loads in flight), a lane quantises its four values into one
// dword, and the tiles leave through LDS as whole KiB.  Bound by the fp32
// operand's way in.
constexpr int kTileRow = 132;  // dwords per half tile in LDS: 128 + 4, so that a row's 16 half tiles start on different banks

struct QuantOperand {
  const float* x;
  int64_t ld;
  int rows;
  int sign;  // 1-bit weights: the sign of x
  // else the level q = round(L * clamp(x * s + c)), s, c = 1, 0 for activations, 0.5, 0.5 for weights in [-1, 1], and the byte
  float s, c, L;
  int odd;        // 2 q - L for weights of this many bits (2 to 7),
  uint32_t flip;  // or (odd = 0) q exclusive-or this: 0, or the top bits where q - 128 is wanted
  uint4* tiles;
};

// The levels of four values as four bytes, the first lowest.  Five instructions a value; with the byte made in fp32 (truncate,
// multiply, add, convert) they were eight, and that is what the kernels below waited for where the values come from a cache.
__device__ __forceinline__ uint32_t level_bytes(float s, float c, float L, float x, float y, float z, float w) {
#pragma clang fp contract(off)  // (the rest of the rounded product L * u, not of the exact one, decides a tie)
  const float v[4] = {x, y, z, w};
  uint32_t q[4];
  // Rounding half away from zero of u >= 0 is trunc(u + (0.5 - 2^-25)) in fp32: with 0.5 itself the
  // one value 0.5 - 2^-25 would round up.  (x + 1) / 2 is the fused x / 2 + 1 / 2: halving rounds nothing.
#pragma unroll
  for (int e = 0; e < 4; ++e)
    q[e] = (uint32_t)(__builtin_amdgcn_fmed3f(__builtin_fmaf(v[e], s, c), 0.0f, 1.0f) * L + 0x1.fffffep-2f);
  return (q[0] | q[1] << 8) | (q[2] | q[3] << 8) << 16;
}
// 2 q - L of four levels q of `bits` (2 to 7) bits: of 2 q + 1 the low bits, and above them the sign, bit `bits` inverted.
__device__ __forceinline__ uint32_t odd_bytes(uint32_t q, int bits) {
  const uint32_t top = 0x01010101u << bits, x2 = q << 1 | 0x01010101u, minus = ~x2 & top;
  return (x2 & (top - 0x01010101u)) | ((minus << (8 - bits)) - minus);
}
__device__ __forceinline__ uint32_t sign_bytes(float x, float y, float z, float w) {
  return (x >= 0.0f ? 1u : 255u) | (y >= 0.0f ? 1u : 255u) << 8 | (z >= 0.0f ? 1u : 255u) << 16 | (w >= 0.0f ? 1u : 255u) << 24;
}
// a / b, correctly rounded as the IEEE division is, for a whole number b and y = 1 / b rounded: the remainder of a product that
// is off by its rounding is exact, and so is the sum rounded once (P. Markstein, IBM J. Res. Dev. 34, 1990; no
// result here is near the ends of the range).  Three instructions for ten.
__device__ __forceinline__ float quotient(float a, float b, float y) {
  const float q = a * y;
  return __builtin_fmaf(__builtin_fmaf(-q, b, a), y, q);
}
// Bytes of a dword that lie inside a row with `left` elements to go.
__device__ __forceinline__ uint32_t byte_mask(int left) {
  return left >= 4 ? 0xffffffffu : (left <= 0 ? 0u : (1u << (8 * left)) - 1u);
}
// Four floats at any 4-byte aligned address in one load.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

struct QuantTilesParams {
  QuantOperand op[2];
  int K, kblocks;      // blocks of 256
  FastDiv div_kblocks;
  int blocks0;         // workgroups of operand 0
};

// (four waves of eight rows: what a wave does beside its values is as many instructions as for two rows of them)
constexpr int kTileWaves = 4, kTileRows = 32 / kTileWaves;  // rows of the block per wave

template <bool NIB>
__global__ void __launch_bounds__(64 * kTileWaves)
quant_tiles_kernel(const QuantTilesParams p) {
  __shared__ uint32_t t[16 * kTileRow];
  // (all arguments named at the top: fetched in one batch, one trip to memory instead of one per group)
  asm volatile("" ::"s"(p.blocks0), "s"(p.div_kblocks.mul), "s"(p.div_kblocks.sh1), "s"(p.div_kblocks.sh2), "s"(p.kblocks), "s"(p.K));
  const bool second = (int)blockIdx.x >= p.blocks0;
  QuantOperand o = p.op[0], o1 = p.op[1];
  // (both operands' fields in registers before one is taken: the compiler would load the one that is taken, behind the choice)
  asm volatile("" : "+s"(o.x), "+s"(o.ld), "+s"(o.rows), "+s"(o.sign), "+s"(o.s), "+s"(o.c), "+s"(o.L), "+s"(o.odd), "+s"(o.flip));
  asm volatile("" : "+s"(o1.x), "+s"(o1.ld), "+s"(o1.rows), "+s"(o1.sign), "+s"(o1.s), "+s"(o1.c), "+s"(o1.L), "+s"(o1.odd), "+s"(o1.flip));
  if (second) o = o1;
  const int b = (int)blockIdx.x - (second ? p.blocks0 : 0);
  const int rb = (int)__builtin_amdgcn_readfirstlane(fast_div((uint32_t)b, p.div_kblocks)), kb = b - rb * p.kblocks;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k0 = kb * 256 + 4 * lane;
  // A row is read as a buffer of K floats: what lies past it reads as zero, and is masked below.  (Rows past the matrix repeat
  // its last: their results are never stored.)
  v4f_any v[kTileRows];
  const int row0 = rb * 32 + wave * kTileRows, last = o.rows - 1;
  const float* at = o.x + (int64_t)min(row0, last) * o.ld;
#pragma unroll
  for (int j = 0; j < kTileRows; ++j) {
    const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc((void*)at, 0, 4 * p.K, 0x00020000);
    v[j] = __builtin_bit_cast(v4f_any, __builtin_amdgcn_raw_buffer_load_b128(row, 4 * k0, 0, 0));
    at += row0 + j < last ? o.ld : 0;
  }
  const uint32_t mask = byte_mask(p.K - k0);
  uint32_t* const dst = &t[(lane >> 2) * kTileRow + wave * (4 * kTileRows) + (lane & 3)];
  if constexpr (NIB) {  // a for activations; s of the odd integer 2 s + 1 for weights, whatever k is past the row's end
    if (o.sign) {
#pragma unroll
      for (int j = 0; j < kTileRows; ++j) dst[4 * j] = sign_bytes(v[j][0], v[j][1], v[j][2], v[j][3]) >> 1 & 0x0f0f0f0fu;
    } else {
      const uint32_t add = o.odd ? (16u - (1u << o.odd >> 1)) * 0x01010101u : 0u, keep = o.odd ? 0x0f0f0f0fu : mask;
#pragma unroll
      for (int j = 0; j < kTileRows; ++j) dst[4 * j] = (level_bytes(o.s, o.c, o.L, v[j][0], v[j][1], v[j][2], v[j][3]) + add) & keep;
    }
  } else if (o.sign) {
#pragma unroll
    for (int j = 0; j < kTileRows; ++j) dst[4 * j] = sign_bytes(v[j][0], v[j][1], v[j][2], v[j][3]) & mask;
  } else if (o.odd) {
#pragma unroll
    for (int j = 0; j < kTileRows; ++j)
      dst[4 * j] = odd_bytes(level_bytes(o.s, o.c, o.L, v[j][0], v[j][1], v[j][2], v[j][3]), o.odd) & mask;
  } else {
#pragma unroll
    for (int j = 0; j < kTileRows; ++j) dst[4 * j] = (level_bytes(o.s, o.c, o.L, v[j][0], v[j][1], v[j][2], v[j][3]) ^ o.flip) & mask;
  }
  __syncthreads();
  // half tile 2 s + h of the block is t[(2 s + h) * kTileRow ...]: row r at dword 4 r
  if constexpr (NIB) {  // k and k + 128 in a byte
    static_assert(kTileWaves == 4, "a piece a thread");
    const uint32_t* const half = &t[(threadIdx.x >> 5) * kTileRow + (threadIdx.x & 31) * 4];
    const uint4 lo = *(const uint4*)half, hi = *(const uint4*)(half + 8 * kTileRow);
    o.tiles[(int64_t)b * 256 + threadIdx.x] = uint4{lo.x | hi.x << 4, lo.y | hi.y << 4, lo.z | hi.z << 4, lo.w | hi.w << 4};
    return;
  }
  uint4* out = o.tiles + (int64_t)b * 512;
#pragma unroll
  for (int i = 0; i < 8 / kTileWaves; ++i) {
    const int c = threadIdx.x + 64 * kTileWaves * i;  // 16-byte piece: half tile c / 32, row c % 32
    out[c] = *(const uint4*)&t[(c >> 5) * kTileRow + (c & 31) * 4];
  }
}

// ---- the product.  TM x TN blocks of 32 x 32 per wave, K split over the S waves of a workgroup
// (partial tiles added through LDS once) where there are too few tiles to fill the chip.  What
// bounds it at the sizes of a layer is latency: operand loads of two groups of k steps are in flight
// while one is multiplied.  Beyond that the L1 path (64 B per clock and CU against 1 KiB per 32-clock
// MFMA and SIMD) holds it at half the matrix rate.
struct I8Params {
  const uint4 *A, *B;  // tiles of the activations and of the weights
  int M, N, nk;        // nk: k steps, of 32 or (two values a byte) 64
  int mblocks, nblocks;
  int tiles_m, tiles_n, tiles_per_xcd;
  int S;
  int ca, scale, rs, Kreal;
  float denom, inv;  // inv = 1 / denom
  int32_t* C_i32;
  float* C_f32;
  int64_t ldc;
  int s_base, s_rem;  // k steps per wave: s_base, the first s_rem waves one more
  // tile order, see tile_of: 2^lg_bands bands of `band` rows of tiles
  int lg_bands, band;
  FastDiv div_band;
};

// Workgroup b sits on XCD b % 8.  Band i has the rows of tiles i, i + bands, i + 2 bands and so on, and each of its XCDs a run of
// its tiles, down the rows first: what an XCD's L2 fetches of the operands is a band's rows and its run's columns.
__device__ __forceinline__ bool tile_of(const I8Params& p, int* tile_m, int* tile_n) {
  const int xcd = (int)(blockIdx.x & 7), lg = p.lg_bands;
  const int at = (xcd >> lg) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  *tile_n = (int)__builtin_amdgcn_readfirstlane(fast_div((uint32_t)at, p.div_band));
  *tile_m = (xcd & ((1 << lg) - 1)) + ((at - *tile_n * p.band) << lg);
  return *tile_m < p.tiles_m && *tile_n < p.tiles_n;
}

// Where both operands have at most four bits (NIB), a step is of 64 k: a byte of its tile holds a level of the activations, or
// s of the weight 2 s + 1, for k and for k + 128 of a block of 256.  A weight is multiplied as the byte 16 s + 8, one instruction
// from where s lies in the upper half, two from the lower; the sums are eight times the result's.  Half the bytes from L2,
// which is what the product of bytes waits for (above).
constexpr int ahead(bool nib) { return nib ? 3 : 4; }  // steps per group of loads

template <int TM, int TN, bool NIB>
struct Group {
  v4i a[ahead(NIB)][TM], b[ahead(NIB)][TN];
};

// The tile's end: operand sums of the two half-waves, the partial tiles of the S waves of a workgroup
// through LDS (S > 1, at most MAXS), the 8-bit correction, stores.
template <int TM, int TN, bool SUMS, bool NIB, int MAXS>
__device__ __forceinline__ void finish_tile(const I8Params& p, const v16i (&acc)[TM][TN], int (&sa)[TM], int (&sb)[TN],
                                            int* red, int lane, int wave, int tile_m, int tile_n) {
  constexpr int kGroups = TM * TN * 4;
  const int r = lane & 31, h = lane >> 5, S = p.S;
  if (SUMS) {  // a lane summed its half of every k step
#pragma unroll
    for (int i = 0; i < TM; ++i) sa[i] += __shfl_xor(sa[i], 32);
#pragma unroll
    for (int j = 0; j < TN; ++j) sb[j] += __shfl_xor(sb[j], 32);
  }

  // Register v of lane (r, h) in block (i, j) is C[32 i + 8 (v / 4) + 4 h + v % 4][32 j + r];
  // group g = (i * TN + j) * 4 + v / 4: four rows of one column.
  auto finish = [&](int g, const int (&d)[4], const int (&ra)[4], int cb) {
    const int blk = g >> 2, i = blk / TN, j = blk % TN;
    const int n = (tile_n * TN + j) * 32 + r;
    if (n >= p.N) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = (tile_m * TM + i) * 32 + 8 * (g & 3) + 4 * h + e;
      if (m >= p.M) continue;
      int sv = NIB ? d[e] >> 3 : d[e];
      if (SUMS)
        sv = (int)((uint32_t)p.scale * ((uint32_t)d[e] + (uint32_t)p.ca * (uint32_t)cb) +
                   (uint32_t)p.rs * ((uint32_t)ra[e] + (uint32_t)p.ca * (uint32_t)p.Kreal));
      const int64_t idx = (int64_t)m * p.ldc + n;
      if (p.C_i32) p.C_i32[idx] = sv;
      if (p.C_f32) p.C_f32[idx] = quotient((float)sv, p.denom, p.inv);
    }
  };
  if (S == 1) {
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      const int i = (g >> 2) / TN, j = (g >> 2) % TN, q = g & 3;
      int d[4], ra[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        d[e] = acc[i][j][4 * q + e];
        ra[e] = SUMS ? __shfl(sa[i], 8 * q + 4 * h + e) : 0;
      }
      finish(g, d, ra, sb[j]);
    }
    return;
  }
  v4i* part = (v4i*)red;                       // [S][kGroups][64]
  int* sums = red + S * kGroups * 64 * 4;      // [S][32 (TM + TN)]
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v4i d;
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = acc[i][j][4 * q + e];
        part[(wave * kGroups + (i * TN + j) * 4 + q) * 64 + lane] = d;
      }
  if (SUMS && h == 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i) sums[wave * 32 * (TM + TN) + 32 * i + r] = sa[i];
#pragma unroll
    for (int j = 0; j < TN; ++j) sums[wave * 32 * (TM + TN) + 32 * (TM + j) + r] = sb[j];
  }
  __syncthreads();
  for (int g = wave; g < kGroups; g += S) {
    v4i t[MAXS];
#pragma unroll
    for (int s = 0; s < MAXS; ++s) t[s] = part[(min(s, S - 1) * kGroups + g) * 64 + lane];
    int d[4] = {}, ra[4] = {}, cb = 0;
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) d[e] += s < S ? t[s][e] : 0;
    if (SUMS) {
      const int i = (g >> 2) / TN, j = (g >> 2) % TN;
#pragma unroll 1
      for (int s0 = 0; s0 < S; s0 += 4) {  // (four waves' sums in flight at a time)
        int wc[4];
        v4i wr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int* w = sums + min(s0 + u, S - 1) * 32 * (TM + TN);
          wc[u] = w[32 * (TM + j) + r];
          wr[u] = *(const v4i*)(w + 32 * i + 8 * (g & 3) + 4 * h);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          cb += s0 + u < S ? wc[u] : 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) ra[e] += s0 + u < S ? wr[u][e] : 0;
        }
      }
    }
    finish(g, d, ra, cb);
  }
}

template <int TM, int TN, bool SUMS, bool NIB>
__global__ void __launch_bounds__(512)
gemm_i8_kernel(const I8Params p) {
  extern __shared__ int red[];
  // (all arguments named at the top: fetched in one batch, one trip to memory instead of one per group)
  asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.M), "s"(p.N), "s"(p.nk), "s"(p.S), "s"(p.mblocks), "s"(p.nblocks),
               "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.tiles_per_xcd), "s"(p.s_base), "s"(p.s_rem), "s"(p.lg_bands), "s"(p.band),
               "s"(p.div_band.mul), "s"(p.div_band.sh1), "s"(p.div_band.sh2));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tile_m, tile_n;
  if (!tile_of(p, &tile_m, &tile_n)) return;  // (the whole workgroup)
  const int k_lo = wave * p.s_base + min(wave, p.s_rem), k_hi = k_lo + p.s_base + (wave < p.s_rem ? 1 : 0);

  const uint4 *arow[TM], *brow[TN];  // (blocks past the matrix repeat its last one)
#pragma unroll
  for (int i = 0; i < TM; ++i) arow[i] = p.A + (int64_t)min(tile_m * TM + i, p.mblocks - 1) * p.nk * 64 + lane;
#pragma unroll
  for (int j = 0; j < TN; ++j) brow[j] = p.B + (int64_t)min(tile_n * TN + j, p.nblocks - 1) * p.nk * 64 + lane;

  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;
  int sa[TM] = {}, sb[TN] = {};

  static_assert(!(SUMS && NIB), "8 bits do not fit half a byte");
  constexpr int kAhead = ahead(NIB);
  auto load = [&](Group<TM, TN, NIB>& g, int k) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      const int kk = min(k + d, k_hi - 1) * 64;  // (a group's steps past the range repeat its last)
#pragma unroll
      for (int i = 0; i < TM; ++i) g.a[d][i] = *(const v4i*)(arow[i] + kk);
#pragma unroll
      for (int j = 0; j < TN; ++j) g.b[d][j] = *(const v4i*)(brow[j] + kk);
    }
  };
  auto multiply = [&](const Group<TM, TN, NIB>& g, int k) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      if (k + d >= k_hi) break;  // wave-uniform
      if constexpr (NIB) {
        constexpr int kLow = 0x0f0f0f0f, kHigh = (int)0xf0f0f0f0u, kHalf = 0x08080808;
        v4i a[2][TM], b[2][TN];  // of the lower halves, of the upper
#pragma unroll
        for (int i = 0; i < TM; ++i) a[0][i] = g.a[d][i] & kLow, a[1][i] = (g.a[d][i] >> 4) & kLow;
#pragma unroll
        for (int j = 0; j < TN; ++j) b[0][j] = ((g.b[d][j] << 4) & kHigh) | kHalf, b[1][j] = (g.b[d][j] & kHigh) | kHalf;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[u][i], b[u][j], acc[i][j], 0, 0, 0);
        continue;
      }
      if (SUMS) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) sa[i] = __builtin_amdgcn_sdot4(g.a[d][i][e], 0x01010101, sa[i], false);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) sb[j] = __builtin_amdgcn_sdot4(g.b[d][j][e], 0x01010101, sb[j], false);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(g.a[d][i], g.b[d][j], acc[i][j], 0, 0, 0);
    }
  };
  if (k_lo < k_hi) {
    Group<TM, TN, NIB> g0, g1;
    load(g0, k_lo);
    for (int k = k_lo; k < k_hi; k += 2 * kAhead) {
      if (k + kAhead < k_hi) load(g1, k + kAhead);
      multiply(g0, k);
      if (k + 2 * kAhead < k_hi) load(g0, k + 2 * kAhead);
      multiply(g1, k + kAhead);
    }
  }
  finish_tile<TM, TN, SUMS, NIB, 8>(p, acc, sa, sb, red, lane, wave, tile_m, tile_n);
}

// The same product with 16 x 16 of C per workgroup, for results of few tiles.  There a CU waits for its one tile's operands, 64 bytes a
// clock: a quarter of the tile has half of the bytes, and four times the CUs work on it.  The operands lie as above; a step of 64 k
// (NIB: 128) is two of their tiles, whose four half tiles are the four quarters of the MFMA's K: a lane's 16 bytes are those of its
// row, in runs of 256.  us a call in a graph, 32 x 32 / 16 x 16: 56 x 122 x 5294 of 3 x 8 bits 9.7 / 7.6, 297 x 64 x 4672 of 1 x 8 10.1 /
// 8.6, 55 x 22 x 4359 of 3 x 2 6.8 / 5.8, 83 x 88 x 3058 of 1 x 2 6.4 / 5.4.
template <bool SUMS, bool NIB>
__global__ void __launch_bounds__(512)
gemm_i8_16_kernel(const I8Params p) {
  extern __shared__ int red[];
  asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.M), "s"(p.N), "s"(p.nk), "s"(p.S), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.tiles_per_xcd), "s"(p.s_base), "s"(p.s_rem),
               "s"(p.lg_bands), "s"(p.band),
               "s"(p.div_band.mul), "s"(p.div_band.sh1), "s"(p.div_band.sh2));
  static_assert(!(SUMS && NIB), "8 bits do not fit half a byte");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tile_m, tile_n;
  if (!tile_of(p, &tile_m, &tile_n)) return;  // (the whole workgroup)
  const int k_lo = wave * p.s_base + min(wave, p.s_rem), k_hi = k_lo + p.s_base + (wave < p.s_rem ? 1 : 0);
  const int at = (lane >> 4) * 32 + (lane & 15);
  const uint4* const arow = p.A + (int64_t)(tile_m >> 1) * p.nk * 64 + (tile_m & 1) * 16 + at;
  const uint4* const brow = p.B + (int64_t)(tile_n >> 1) * p.nk * 64 + (tile_n & 1) * 16 + at;

  v4i acc = {0, 0, 0, 0};
  int sa = 0, sb = 0;
  constexpr int kAhead = 4;
  v4i a[2][kAhead], b[2][kAhead];
  auto load = [&](int i, int k) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      const int kk = min(k + d, k_hi - 1) * 128;  // (a group's steps past the range repeat its last)
      a[i][d] = *(const v4i*)(arow + kk);
      b[i][d] = *(const v4i*)(brow + kk);
    }
  };
  auto multiply = [&](int i, int k) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      if (k + d >= k_hi) break;  // wave-uniform
      const v4i x = a[i][d], y = b[i][d];
      if constexpr (NIB) {
        constexpr int kLow = 0x0f0f0f0f, kHigh = (int)0xf0f0f0f0u, kHalf = 0x08080808;
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(x & kLow, ((y << 4) & kHigh) | kHalf, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8((x >> 4) & kLow, (y & kHigh) | kHalf, acc, 0, 0, 0);
      } else {
        if (SUMS) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sa = __builtin_amdgcn_sdot4(x[e], 0x01010101, sa, false);
            sb = __builtin_amdgcn_sdot4(y[e], 0x01010101, sb, false);
          }
        }
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, y, acc, 0, 0, 0);
      }
    }
  };
  if (k_lo < k_hi) {
    load(0, k_lo);
    for (int k = k_lo; k < k_hi; k += 2 * kAhead) {
      if (k + kAhead < k_hi) load(1, k + kAhead);
      multiply(0, k);
      if (k + 2 * kAhead < k_hi) load(0, k + 2 * kAhead);
      multiply(1, k + kAhead);
    }
  }
  if (SUMS) {  // of row and column lane % 16
    sa += __shfl_xor(sa, 16), sb += __shfl_xor(sb, 16);
    sa += __shfl_xor(sa, 32), sb += __shfl_xor(sb, 32);
  }
  // the waves' sums meet: [wave][register][lane], and with SUMS [wave][row of a, of b] behind them; a thread a result
  int* const sums = red + p.S * 256;
#pragma unroll
  for (int e = 0; e < 4; ++e) red[wave * 256 + 64 * e + lane] = acc[e];
  if (SUMS && lane < 16) sums[wave * 32 + lane] = sa, sums[wave * 32 + 16 + lane] = sb;
  __syncthreads();
  for (int o = threadIdx.x; o < 256; o += 64 * p.S) {
    const int row = 4 * ((o & 63) >> 4) + (o >> 6), col = o & 15;
    int d = 0, ra = 0, cb = 0;
#pragma unroll 4
    for (int s = 0; s < p.S; ++s) {
      d += red[s * 256 + o];
      if (SUMS) ra += sums[s * 32 + row], cb += sums[s * 32 + 16 + col];
    }
    if (NIB) d >>= 3;
    if (SUMS)
      d = (int)((uint32_t)p.scale * ((uint32_t)d + (uint32_t)p.ca * (uint32_t)cb) + (uint32_t)p.rs * ((uint32_t)ra + (uint32_t)p.ca * (uint32_t)p.Kreal));
    const int m = tile_m * 16 + row, n = tile_n * 16 + col;
    if (m >= p.M || n >= p.N) continue;
    const int64_t idx = (int64_t)m * p.ldc + n;
    if (p.C_i32) p.C_i32[idx] = d;
    if (p.C_f32) p.C_f32[idx] = quotient((float)d, p.denom, p.inv);
  }
}

// ---- the whole product in one launch, for problems small enough that a second launch costs more
// than quantising a row once per tile of results.  Up to 16 waves split the K of a T x T tile.  Of a step of KS = 1024 / T k a
// wave fetches T rows of both operands, KS / 4 lanes to a row's 4 KS bytes (16 bytes straight into the
// MFMA's layout would touch 64 lines per load: 202 x 192 x 437 7.7 us), quantises four values per lane and
// load into a dword of bytes, and turns those into the MFMA's layout (a lane: 16 bytes of a row)
// through 2 KB of LDS of its own, where its partial sums go in the end.
// What bounds it is what one CU has to take in and to quantise for its 2 T rows: 64 bytes a clock and five vector instructions a
// value.  So 16 x 16 of the result per workgroup as long as the CUs are not full of them.
struct QuantSmallParams {
  const float *a, *w;
  int64_t lda, ldw;
  int M, N, K;
  int tiles_m, S, s_base, s_rem;  // k steps per wave: s_base, the first s_rem waves one more
  FastDiv div_tiles_m;
  float La, Lw;
  uint32_t flip_a;
  int odd;  // bits of the weights (2 to 7; 8: levels - 128)
  int ca, scale, rs;
  float denom, inv;
  int32_t* C_i32;
  float* C_f32;
  int64_t ldc;
};

constexpr int kSignW = 1, kOddW = 2, kLevelW = 3;  // weights of one bit, of 2 to 7, of 8

template <bool SUMS, int WK, int T>
__global__ void __launch_bounds__(1024)
quant_small_kernel(const QuantSmallParams p) {
  extern __shared__ int red[];
  asm volatile("" ::"s"(p.a), "s"(p.w), "s"(p.lda), "s"(p.ldw), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.tiles_m), "s"(p.S), "s"(p.s_base),
               "s"(p.s_rem), "s"(p.div_tiles_m.mul), "s"(p.div_tiles_m.sh1), "s"(p.div_tiles_m.sh2), "s"(p.La), "s"(p.Lw), "s"(p.flip_a),
               "s"(p.odd), "s"(p.ca), "s"(p.denom), "s"(p.C_i32), "s"(p.C_f32), "s"(p.ldc));
  constexpr int KS = 1024 / T, kLanes = KS / 4;             // k per step; lanes that share a row of a load
  constexpr int NR = T * T / 64;                            // results per lane
  constexpr int kWave = (NR > 8 ? NR : 8) * 64;             // ints of LDS per wave: both operands of a step, then its sums
  typedef int acc_t __attribute__((ext_vector_type(NR)));
  typedef v4i __attribute__((may_alias)) v4i_alias;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile_n = (int)__builtin_amdgcn_readfirstlane(fast_div(blockIdx.x, p.div_tiles_m));
  const int tile_m = (int)blockIdx.x - tile_n * p.tiles_m;
  const int k_lo = wave * p.s_base + min(wave, p.s_rem), k_hi = k_lo + p.s_base + (wave < p.s_rem ? 1 : 0);
  // byte offsets of row 256 / KS * t + lane / kLanes (rows past a matrix repeat its last; their results are never stored)
  const __amdgpu_buffer_rsrc_t a_rows = __builtin_amdgcn_make_buffer_rsrc((void*)p.a, 0, (int)0xffffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t w_rows = __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, (int)0xffffffff, 0x00020000);
  uint32_t arow[4], wrow[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int row = T / 4 * t + lane / kLanes;
    arow[t] = (uint32_t)min(tile_m * T + row, p.M - 1) * ((uint32_t)p.lda * 4u);
    wrow[t] = (uint32_t)min(tile_n * T + row, p.N - 1) * ((uint32_t)p.ldw * 4u);
  }
  const int c = 4 * (lane & (kLanes - 1));
  acc_t acc;
#pragma unroll
  for (int e = 0; e < NR; ++e) acc[e] = 0;
  int sa = 0, sb = 0;
  v4f_any va[2][4], vw[2][4];
  auto load = [&](int i, int k) {
    // four values past the row's end are its last four instead; those that the piece before has are masked
    // below (of both operands: what remains still meets its partner, and K has no order)
    const uint32_t off = 4u * (uint32_t)min(KS * k + c, p.K - 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      va[i][t] = __builtin_bit_cast(v4f_any, __builtin_amdgcn_raw_buffer_load_b128(a_rows, arow[t] + off, 0, 0));
      vw[i][t] = __builtin_bit_cast(v4f_any, __builtin_amdgcn_raw_buffer_load_b128(w_rows, wrow[t] + off, 0, 0));
    }
  };
  uint32_t* const turn = (uint32_t*)red + wave * kWave;  // [operand][row][KS / 4 dwords]
  auto multiply = [&](int i, int k) {
    const uint32_t mask = ~byte_mask(KS * k + c + 4 - p.K);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const v4f_any x = va[i][t], y = vw[i][t];
      turn[64 * t + lane] = (level_bytes(1.0f, 0.0f, p.La, x[0], x[1], x[2], x[3]) ^ (SUMS ? p.flip_a : 0u)) & mask;
      uint32_t v;
      if constexpr (WK == kSignW) v = sign_bytes(y[0], y[1], y[2], y[3]);
      else v = level_bytes(0.5f, 0.5f, p.Lw, y[0], y[1], y[2], y[3]);
      if constexpr (WK == kOddW) v = odd_bytes(v, p.odd);
      if constexpr (WK == kLevelW) v ^= 0x80808080u;
      turn[256 + 64 * t + lane] = v & mask;
    }
    const int at = (lane & (T - 1)) * kLanes + 4 * (lane / T);
    const v4i a = *(const v4i_alias*)(turn + at), b = *(const v4i_alias*)(turn + 256 + at);
    if (SUMS) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sa = __builtin_amdgcn_sdot4(a[e], 0x01010101, sa, false);
        sb = __builtin_amdgcn_sdot4(b[e], 0x01010101, sb, false);
      }
    }
    if constexpr (T == 32) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
    else acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, acc, 0, 0, 0);
  };
  load(0, k_lo);
  for (int k = k_lo; k < k_hi; k += 2) {
    if (k + 1 < k_hi) load(1, k + 1);
    multiply(0, k);
    if (k + 1 >= k_hi) break;
    if (k + 2 < k_hi) load(0, k + 2);
    multiply(1, k + 1);
  }

  if (SUMS) {  // of row and column lane % T
    if (T == 16) sa += __shfl_xor(sa, 16), sb += __shfl_xor(sb, 16);
    sa += __shfl_xor(sa, 32), sb += __shfl_xor(sb, 32);
  }
  auto row_of = [](int e, int l) { return T == 32 ? 8 * (e >> 2) + 4 * (l >> 5) + (e & 3) : 4 * (l >> 4) + e; };  // register e of lane l of the MFMA's result
  auto store = [&](int row, int col, int d, int ra, int cb) {
    if (SUMS)
      d = (int)((uint32_t)p.scale * ((uint32_t)d + (uint32_t)p.ca * (uint32_t)cb) + (uint32_t)p.rs * ((uint32_t)ra + (uint32_t)p.ca * (uint32_t)p.K));
    const int m = tile_m * T + row, n = tile_n * T + col;
    if (m >= p.M || n >= p.N) return;
    const int64_t idx = (int64_t)m * p.ldc + n;
    if (p.C_i32) p.C_i32[idx] = d;
    if (p.C_f32) p.C_f32[idx] = quotient((float)d, p.denom, p.inv);
  };
  // Nothing to meet: from the registers (through LDS as below: 2100 x 2100 x 24 of 4 x 4 bits 12.0 / 8.9 us, 200 x 200 x 40 3.2 / 2.8;
  // not expected, so that it lies behind: ahead of the code below it cost that a percent)
  if (__builtin_expect(p.S == 1, 0)) {
#pragma unroll
    for (int e = 0; e < NR; ++e) {
      const int row = row_of(e, lane);
      store(row, lane & (T - 1), acc[e], SUMS ? __shfl(sa, row) : 0, sb);
    }
    return;
  }
  // ---- the waves' sums meet: [wave][register][lane], and with SUMS [wave][row of a, of w] behind them; a thread a result
  int* const sums = red + p.S * kWave;
#pragma unroll
  for (int e = 0; e < NR; ++e) red[wave * kWave + 64 * e + lane] = acc[e];
  if (SUMS && lane < T) sums[wave * 2 * T + lane] = sa, sums[wave * 2 * T + T + lane] = sb;
  __syncthreads();
  for (int o = threadIdx.x; o < T * T; o += 64 * p.S) {
    const int row = row_of(o >> 6, o & 63), col = o & (T - 1);
    int d = 0, ra = 0, cb = 0;
#pragma unroll 4
    for (int s = 0; s < p.S; ++s) {
      d += red[s * kWave + o];
      if (SUMS) ra += sums[s * 2 * T + row], cb += sums[s * 2 * T + T + col];
    }
    store(row, col, d, ra, cb);
  }
}

template <int TM, int TN, bool SUMS, bool NIB>
hipError_t launch_i8(const I8Params& p, hipStream_t s) {
  auto kern = gemm_i8_kernel<TM, TN, SUMS, NIB>;
  const size_t lds = p.S > 1 ? (size_t)p.S * (TM * TN * 4 * 1024 + 128 * (TM + TN)) : 0;
  static std::atomic<bool> asked[64];
  const hipError_t e = allow_lds((const void*)kern, lds, asked);
  if (e != hipSuccess) return e;
  note_kernel("gemm_i8_kernel<%d,%d%s> grid %d x %d, K split %d, bands %d", TM, TN, SUMS ? ",sums" : NIB ? ",halves" : "", 8 * p.tiles_per_xcd, 64 * p.S, p.S,
              1 << p.lg_bands);
  launch_kernel(kern, dim3((unsigned)(8 * p.tiles_per_xcd)), dim3(64 * p.S), lds, s, p);
  return launch_error();
}

template <bool SUMS, bool NIB>
hipError_t launch_i8_16(const I8Params& p, hipStream_t s) {
  note_kernel("gemm_i8_kernel<16 x 16%s> (gemm_i8_16_kernel) grid %d x %d, K split %d, bands %d", SUMS ? ",sums" : NIB ? ",halves" : "",
              8 * p.tiles_per_xcd, 64 * p.S, p.S, 1 << p.lg_bands);
  launch_kernel(gemm_i8_16_kernel<SUMS, NIB>, dim3((unsigned)(8 * p.tiles_per_xcd)), dim3(64 * p.S), (size_t)p.S * (1024 + (SUMS ? 128 : 0)), s, p);
  return launch_error();
}

int64_t tile_bytes(int64_t rows, int64_t K) { return ceil_div(rows, 32) * 32 * ceil_div(K, 256) * 256; }

}  // namespace

// Activations of 1 or 2 bits by weights of 1: as planes (gemm_fp4.hip), or here with two values a byte.  The planes' pack and their
// splits of K have coarse pieces, the bytes' way from L2 grows with the product: 4674 products on both forms, planes' time over
// this one's: operands of up to a million values 1.4 to 1.8, one to three million 1.3 to 1.6, three to six 1.1 to 1.25; above the
// line 0.71 to 1.05.  The choice is 0.04 % behind the better one (16 % at most).  Whole rounds of 4096 values, from the second on,
// the planes' pieces fit: 16 x 200 x 16384 of 1 x 1 bits 11.4 / 14.1, 300 x 300 x 8192 11.9 / 13.4, of 2 x 1 13.4 / 13.3, 16 x 2048 x 8192
// 17.5 / 18.1.  us a call, planes / here: 302 x 1536 x 1726 of 2 x 1 11.4 /
// 9.2, 690 x 128 x 2605 9.8 / 7.8, 852 x 256 x 1558 of 1 x 1 9.1 / 7.1; 1803 x 512 x 3844 of 1 x 1 14.0 / 19.2.
static bool halves_pay(int64_t M, int64_t N, int64_t K, int bits_a) {
  if (K % 4096 == 0 && K >= 8192) return false;
  return K < (1 << 20) && M * N <= 1000000000 && M * N * K < 1200000000 * (int64_t)bits_a;
}
// Workspace of the two tiled operands (0: not taken).  Taken: a result that fills a quarter of a 32 x 32 block (below that the
// padding of the tiles is most of what is moved).  (More than few bits keep a byte a value, what callers were told before two
// shared one: the query is part of the interface.)
size_t quant_i8_workspace(int64_t M, int64_t N, int64_t K, int bits_a, int bits_w) {
  if (M * N < 256 || (quant_few_bits(bits_a, bits_w) && !halves_pay(M, N, K, bits_a))) return 0;
  const int64_t a = tile_bytes(M, K), b = tile_bytes(N, K);
  const int64_t tiles = ceil_div(M, 32) * ceil_div(N, 32);
  if (a >= ((int64_t)1 << 40) || b >= ((int64_t)1 << 40) || tiles >= ((int64_t)1 << 30) ||
      ceil_div(M, 32) * ceil_div(K, 256) + ceil_div(N, 32) * ceil_div(K, 256) >= ((int64_t)1 << 30))
    return 0;
  return (size_t)(a + b) / (quant_few_bits(bits_a, bits_w) ? 2 : 1);
}

namespace {

void fill_operands(QuantOperand (&op)[2], const float* a, int64_t lda, int bits_a, const float* w, int64_t ldw, int bits_w,
                   int M, int N) {
  const int La = (1 << bits_a) - 1, Lw = (1 << bits_w) - 1;
  op[0] = {a, lda, M, 0, 1.0f, 0.0f, (float)La, 0, bits_a == 8 ? 0x80808080u : 0u, nullptr};
  op[1] = {w, ldw, N, bits_w == 1 ? 1 : 0, 0.5f, 0.5f, (float)Lw, bits_w > 1 && bits_w < 8 ? bits_w : 0, bits_w == 8 ? 0x80808080u : 0u, nullptr};
}

void fill_product(I8Params& p, int bits_a, int bits_w, int M, int N, int K, int32_t* S_out, float* out_f32, int64_t ldo) {
  p.A = p.B = nullptr;
  p.M = M;
  p.N = N;
  p.mblocks = (int)ceil_div(M, 32);
  p.nblocks = (int)ceil_div(N, 32);
  p.ca = bits_a == 8 ? 128 : 0;
  p.scale = bits_w == 8 ? 2 : 1;
  p.rs = bits_w == 8 ? 1 : 0;
  p.Kreal = K;
  p.denom = (float)(((1 << bits_a) - 1) * ((1 << bits_w) - 1));
  p.inv = 1.0f / p.denom;
  p.C_i32 = S_out;
  p.C_f32 = out_f32;
  p.ldc = ldo;
}

}  // namespace

static void set_split(I8Params& p) {
  p.s_base = p.nk / p.S;
  p.s_rem = p.nk % p.S;
}

// One, two, four or eight bands, whichever has an XCD fetch the fewest rows of the operands where that is a fifth less than with one, and
// 192 KB (1256 x 1024 x 366 of 2 x 2 bits, 147 KB less, 7.65 / 8.1 us).
// (A band that is a row short leaves its XCDs idle for it: not where a CU then has a tile more than it would, which may be one more
// than it holds at once: 1750 x 1472 x 552 of 2 x 8 bits 15.2 / 16.3 us.)
// us a call in a graph, three sets of inputs in turn, one band / as here: 1472 x 64 x 1361 of 8 x 2 bits 9.7 / 7.6, 1045 x 61 x 3520 of 8 x 1 13.8 /
// 10.95, 922 x 53 x 5376 of 3 x 1 11.9 / 10.1, 1575 x 82 x 2944 of 3 x 8 14.6 / 12.45; of 160 drawn products with more than one 1.07 in the mean
// (two bands 1.02, four 1.03, eight 1.12).
static void set_tile_order(I8Params& p, int tile_rows, int tile_cols) {
  p.lg_bands = 0;
  p.band = p.tiles_m;
  const int most = (int)ceil_div(p.tiles_m * p.tiles_n, 8);
  p.tiles_per_xcd = most;
  const float one = (float)(p.tiles_m * tile_rows) + 0.125f * (float)(p.tiles_n * tile_cols);
  float least = std::min(0.8f * one, one - 196608.0f / (32.0f * (float)p.nk));  // (a step is 32 bytes of a row)
  for (int lg = 1; lg <= 3 && p.tiles_m >> lg; ++lg) {
    const int band = (p.tiles_m + (1 << lg) - 1) >> lg, per = (band * p.tiles_n + (8 >> lg) - 1) >> (3 - lg);
    const float fetched = (float)(band * tile_rows) + 0.125f * (float)((p.tiles_n * tile_cols) << lg);
    if (fetched >= least || (per + 31) / 32 > (most + 31) / 32) continue;
    least = fetched;
    p.lg_bands = lg;
    p.band = band;
    p.tiles_per_xcd = per;
  }
  p.div_band = make_fast_div((uint32_t)p.band);
}

// The one-launch form, for any pair of bit widths; false when the problem is too large for it.
bool launch_quant_small(const float* a, int64_t lda, int bits_a, const float* w, int64_t ldw, int bits_w, int M, int N,
                        int K, int32_t* S_out, float* out_f32, int64_t ldo, bool pair, hipStream_t s, hipError_t* err) {
  if (gemm_engine != 0) return false;
  const bool sums = bits_a == 8 || bits_w == 8;
  const int64_t t32 = ceil_div(M, 32) * ceil_div(N, 32), t16 = ceil_div(M, 16) * ceil_div(N, 16);
  // 16 x 16 of the result per workgroup while a CU has one of them, or two or more of few steps (3600 products of both: time as
  // 32 x 32 over that as 16 x 16, up to 256 tiles of 16 x 16 1.24 to 1.37; 257 to 512 1.08 to 1.26 up to a K of 512, 0.90 beyond; 513
  // to 2048 1.08 to 1.17 up to 128, 0.8 beyond).
  const bool small = t16 <= 256 || (t16 <= 512 && K <= 512) || (t16 <= 2048 && K <= 128);
  // Where 16 x 16 of the result per workgroup are one a CU and the pair of launches can be had: fitted to 900 products of 10 to 128 steps of
  // 64 k, in us in a graph, in the mean of one set of inputs and three in turn (operands that the L2s still hold, and others): a wave's
  // steps and what the workgroups read (a row once per tile) on one side, the operands' way in once and a wave's steps on the other.  By
  // them the choice is 0.2 (two values a byte) and 0.4 % behind the better form.  As calls the pair takes 6.1 to 7.2 us whatever its
  // size, process by process, which is what the host needs to make its launches: it has to be worth 6.65 and 6.8 (0.2 and 0.25 % behind with
  // three sets, 0.6 and 0.5 with one; 6.4 0.3 to 1.0, 7.2 0.4).  What decides most of what is left is where the operands are, which nobody
  // knows here (a call, one launch / two, three sets and one: 139 x 256 x 2432 of 8 x 1 bits 7.9 / 6.5 and 5.8 / 6.5, two; 407 x 125 x 1792 6.2 /
  // 6.4 and 4.9 / 6.4, one).
  // Of more steps, where the fit ends, two launches (16 x 1408 x 10000 of 8 x 1 20.7 / 18.4; of 150 products of 128 to 512 steps one launch was
  // ahead of two once, by 5 %).
  const bool halves = bits_a <= 4 && bits_w <= 4;
  const int64_t steps = small ? ceil_div(K, 64) : ceil_div(K, 32) * ceil_div(t32, 256);
  if (t16 <= 256 && pair) {
    const double read = 128e-6 * (double)t16 * K, input = 4e-6 * ((double)M + N) * K;  // MB
    const double one = halves ? 2.46 + 0.0756 * steps + 0.0375 * read : 2.67 + 0.0808 * steps + 0.0366 * read;
    const double two = halves ? 4.71 + 0.012 * steps + 0.145 * input : 4.81 + 0.0228 * steps + 0.196 * input;
    if (steps > 128 || (one > two && (one > (halves ? 6.65 : 6.8) || capturing(s)))) return false;
  } else {
    // Steps of K per CU up to which one launch is ahead of the better pair of launches: 16 x 16 44; 32 x 32, a tile a CU or less, 20 to 28
    // 1.11 in a graph and 1.36 as calls, 28 to 36 1.00 and 1.15 (8 bits at 256 tiles 0.9: 486 x 512 x 990 of 3 x 8 8.8 / 7.1), 36 to 40
    // 0.91 and 1.02; more tiles, 16 to 24 1.02 and 1.12, 24 to 32 0.87 and 0.98.  us a call, before two values shared a byte and
    // tiles were of 32 x 32 alone / now: 36 x 346 x 1062 of 1 x 1 bits 5.9 / 3.8, 213 x 256 x 818 of 8 x 1 8.0 / 4.1, 58 x 320 x 870 of 2
    // x 4 5.8 / 3.6, 202 x 192 x 437 5.0 / 3.4.
    if (steps > (small ? 44 : t32 > 256 ? 24 : sums ? 28 : 32)) return false;
    // In a graph the host's part is not paid on replay, and the lines stand lower: where the GPU's part of both forms is level, rows of
    // whole lines or not (a tile reads its own rows, each for itself; 287 x 256 x 789 of 2 x 1 bits: one launch 6.9 us, two 5.5).
    // (Up to four steps of K over many tiles stay: two launches 1.03 to 1.05, 1125 x 1216 x 128 of 8 x 1 bits 7.8 / 8.8.)
    const bool ragged = (lda | ldw) % 32 != 0;
    const int64_t graph_steps = small ? 44 : t32 > 256 ? (K <= 128 ? 24 : 18) : t32 > 128 ? (ragged ? 18 : 22) : (ragged ? 22 : 28);
    if (steps > graph_steps && capturing(s)) return false;
  }
  if (K < 4 || (int64_t)M * lda * 4 >= ((int64_t)1 << 32) || (int64_t)N * ldw * 4 >= ((int64_t)1 << 32)) return false;
  const int T = small ? 16 : 32, nk = (int)ceil_div(K, 1024 / T);
  QuantSmallParams p;
  p.a = a;
  p.w = w;
  p.lda = lda;
  p.ldw = ldw;
  p.M = M;
  p.N = N;
  p.K = K;
  p.tiles_m = (int)ceil_div(M, T);
  p.div_tiles_m = make_fast_div((uint32_t)p.tiles_m);
  const int tiles = p.tiles_m * (int)ceil_div(N, T);
  // waves per tile: a step of K each while the chip has room for them (two steps each: 10 % slower; 15: 64 KB of LDS)
  p.S = std::min({sums && T == 32 ? 15 : 16, std::max(1, (T == 32 ? 4096 : 8192) / tiles), nk});
  p.s_base = nk / p.S;
  p.s_rem = nk % p.S;
  I8Params g;
  fill_product(g, bits_a, bits_w, M, N, K, S_out, out_f32, ldo);
  p.La = (float)((1 << bits_a) - 1);
  p.Lw = (float)((1 << bits_w) - 1);
  p.flip_a = bits_a == 8 ? 0x80808080u : 0u;
  p.odd = bits_w;
  p.ca = g.ca;
  p.scale = g.scale;
  p.rs = g.rs;
  p.denom = g.denom;
  p.inv = g.inv;
  p.C_i32 = S_out;
  p.C_f32 = out_f32;
  p.ldc = ldo;
  const size_t lds = (size_t)p.S * ((T == 32 ? 4096 : 2048) + (sums ? 8 * T : 0));
  note_kernel("quant_small_kernel%s<%d> grid %d x %d", sums ? "<sums>" : "", T, tiles, 64 * p.S);
  auto go = [&](auto kern) { launch_kernel(kern, dim3((unsigned)tiles), dim3(64 * p.S), lds, s, p); };
  auto pick = [&](auto sums_tag, auto wk) {
    if (T == 32) go(quant_small_kernel<decltype(sums_tag)::value, decltype(wk)::value, 32>);
    else go(quant_small_kernel<decltype(sums_tag)::value, decltype(wk)::value, 16>);
  };
  using std::integral_constant;
  if (bits_w == 8) pick(std::true_type{}, integral_constant<int, kLevelW>{});
  else if (bits_w == 1) sums ? pick(std::true_type{}, integral_constant<int, kSignW>{}) : pick(std::false_type{}, integral_constant<int, kSignW>{});
  else sums ? pick(std::true_type{}, integral_constant<int, kOddW>{}) : pick(std::false_type{}, integral_constant<int, kOddW>{});
  *err = launch_error();
  return true;
}

bool launch_quant_i8(const float* a, int64_t lda, int bits_a, const float* w, int64_t ldw, int bits_w, int M, int N,
                     int K, int32_t* S_out, float* out_f32, int64_t ldo, void* workspace, size_t workspace_bytes, hipStream_t s,
                     hipError_t* err) {
  const size_t need = quant_i8_workspace(M, N, K, bits_a, bits_w);
  if (gemm_engine == 1 || need == 0) return false;
  // (few bits: an engine of the plane form is pinned, or there is room for the planes alone)
  if (quant_few_bits(bits_a, bits_w) && (gemm_engine != 0 || workspace_bytes < need)) return false;
  QuantTilesParams q;
  fill_operands(q.op, a, lda, bits_a, w, ldw, bits_w, M, N);
  // (a sum is at most 15 * 120 K, and so within 32 bits)
  const bool halves = bits_a <= 4 && bits_w <= 4 && K < (1 << 20);
  q.op[0].tiles = (uint4*)workspace;
  q.op[1].tiles = (uint4*)((char*)workspace + tile_bytes(M, K) / (halves ? 2 : 1));
  q.K = K;
  q.kblocks = (int)ceil_div(K, 256);
  q.div_kblocks = make_fast_div((uint32_t)q.kblocks);
  I8Params p;
  fill_product(p, bits_a, bits_w, M, N, K, S_out, out_f32, ldo);
  q.blocks0 = p.mblocks * q.kblocks;
  launch_kernel(halves ? quant_tiles_kernel<true> : quant_tiles_kernel<false>, dim3((unsigned)(q.blocks0 + p.nblocks * q.kblocks)), dim3(64 * kTileWaves), 0, s, q);
  *err = launch_error();
  if (*err != hipSuccess) return true;
  p.A = q.op[0].tiles;
  p.B = q.op[1].tiles;
  p.nk = q.kblocks * (halves ? 4 : 8);
  // C per wave: 32 x 32 while K is short (many waves, each with little to fetch before its first product), 32 x 64, and 64 x 64
  // where K is long, each with tiles for half the CUs.  K is split over as many waves as leave the workgroups of
  // a CU resident at once (the registers hold 24, 12 and 8 waves, rounded as below), a power of two of them so that its
  // SIMDs stay level.  us a call, before (2048 waves in all, 64 x 64 and 32 x 64 once they fill the chip) and now: 994 x 551 x
  // 2226, 288 tiles of 32 x 64, where the second workgroup of seven waves had to wait for the first, 18.8 and 15.3; 721
  // x 1438 x 681 14.2 and 11.4; 1650 x 1566 x 103 16.8 and 12.2; 1098 x 1728 x 265 12.1 and 11.3.  Over 150
  // products 8.7 % and 1.8 % behind the best of all splits and forms.
  // (With two values a byte the same lines and splits are 0.5 % behind the best of all over 414 products.)
  const bool sums = bits_a == 8 || bits_w == 8;
  // 16 x 16 of C per workgroup up to one and a half of them a CU (250 products, the time of the calls over that with 32 x 32 and 32 x 64:
  // up to 64 tiles 0.78 to 0.82, 65 to 128 0.81 to 0.85, 129 to 256 0.88, 257 to 384 0.98 of two values a byte and 0.96 of one,
  // 385 to 512 0.99 and 1.01, beyond 1.04 to 1.16; sixteen waves of K are level with eight, four behind them to 256 tiles).
  const int64_t t16 = ceil_div(M, 16) * ceil_div(N, 16);
  if (t16 <= 384) {
    p.tiles_m = (int)ceil_div(M, 16);
    p.tiles_n = (int)ceil_div(N, 16);
    set_tile_order(p, 16, 16);
    const int steps = p.nk / 2;
    p.S = std::min(8, steps);
    p.s_base = steps / p.S;
    p.s_rem = steps % p.S;
    *err = halves ? launch_i8_16<false, true>(p, s) : sums ? launch_i8_16<true, false>(p, s) : launch_i8_16<false, false>(p, s);
    return true;
  }
  const int64_t t12 = ceil_div(M, 32) * ceil_div(N, 64), t22 = ceil_div(M, 64) * ceil_div(N, 64);
  const int TM = K >= 5000 && t22 >= 128 ? 2 : 1, TN = TM == 2 || (K > 1100 && t12 >= 128) ? 2 : 1;
  p.tiles_m = (int)ceil_div(M, 32 * TM);
  p.tiles_n = (int)ceil_div(N, 32 * TN);
  set_tile_order(p, 32 * TM, 32 * TN);
  const int64_t room = (TM * TN == 4 ? 8 : TM * TN == 2 ? 12 : 24) / ceil_div((int64_t)p.tiles_m * p.tiles_n, 256);  // waves a workgroup
  p.S = room >= 8 ? 8 : room >= 4 ? 4 : room >= 2 ? 2 : 1;
  while (p.S > 1 && p.S > 2 * q.kblocks) p.S /= 2;  // (each with 128 k at least)
  set_split(p);
  auto form = [&](auto tm, auto tn) {
    constexpr int M_ = decltype(tm)::value, N_ = decltype(tn)::value;
    return halves ? launch_i8<M_, N_, false, true>(p, s) : sums ? launch_i8<M_, N_, true, false>(p, s) : launch_i8<M_, N_, false, false>(p, s);
  };
  using One = std::integral_constant<int, 1>;
  using Two = std::integral_constant<int, 2>;
  if (TM == 2) *err = form(Two{}, Two{});
  else if (TN == 2) *err = form(One{}, Two{});
  else *err = form(One{}, One{});
  return true;
}

}  // namespace bmx
