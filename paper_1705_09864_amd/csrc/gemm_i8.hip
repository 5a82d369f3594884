// k-bit products on the int8 matrix cores (Sec. 2.1, Eq. 1; arbitrary bit widths after DoReFa-Net):
// S[m][n] = sum_k q[m][k] * v[n][k] with q the level of the activation and v the weight's odd
// integer (sign for one bit, 2 q_w - L_w above).
//
// Taken where an operand has more bits than the FP4 form of gemm_fp4.hip folds into a nibble (more
// than two for the activations, more than one for the weights), and for small products of any.  Walked plane by plane with AND +
// popcount, such a product costs bits_a * bits_w passes over K on the vector ALU (4 x 4 bits, 500 x
// 1000 x 2304: 67 us, and a 16 MB array of per-plane results to add up afterwards, 5 us).  As bytes
// it is one pass on the matrix cores, whatever the bits.
//
// Eight-bit levels do not fit a signed byte: q - 128 and q_w - 128 do, and the sums of the operands'
// rows, counted from the words a lane loads anyway (v_dot4), put the difference right:
//   S = scale * (sum a' v' + ca * sum_k v') + rs * (sum_k a' + ca * K),  a' = q - ca,
//   v' = v, scale = 1, rs = 0  (up to 7 weight bits)  or  v' = q_w - 128, scale = 2, rs = 1  (8 bits),
// in 32-bit wrap-around arithmetic (the result itself fits, the launcher's caller has checked).
//
// Layout.  A dot product does not care about the order of k, and both operands are written by
// quant_tiles_kernel for this kernel alone, so they are stored the way the MFMA wants them: tile
// (row block of 32, k step of 32) is 1 KiB, lane l of a wave taking bytes [16 l, 16 l + 16): row
// l % 32, half l / 32 of the step.  Every operand load is one contiguous KiB, no LDS, no
// transposition.  K is zero padded to whole blocks of 256, rows to whole blocks of 32.
#include "bmx_internal.h"

#include <algorithm>

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
  int sign;  // 1-bit weights: the sign; else the byte is mul * q + add - 128 of the level q
  // q = round(L * clamp((x + c0) * c1)): c0, c1 = 0, 1 for activations, 1, 0.5 for weights in [-1, 1]
  float c0, c1, L;
  float mul, add;
  uint4* tiles;
};

// Four values of an operand as four bytes, the first lowest.
__device__ __forceinline__ uint32_t quant_bytes(const QuantOperand& o, float x, float y, float z, float w) {
#pragma clang fp contract(off)  // (the rest of the rounded product L * u, not of the exact one, decides a tie)
  const float v[4] = {x, y, z, w};
  uint32_t d = 0;
  // Rounding half away from zero of u >= 0 is trunc(u + (0.5 - 2^-25)) in fp32: with 0.5 itself the
  // one value 0.5 - 2^-25 would round up.  The byte is made in fp32 (whole numbers up to 255) with
  // 128 added, so that it is never negative, and the 128 goes again as the flip of its top bit.
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float u = fminf(fmaxf((v[e] + o.c0) * o.c1, 0.0f), 1.0f) * o.L;
    d = __builtin_amdgcn_cvt_pk_u8_f32(truncf(u + 0x1.fffffep-2f) * o.mul + o.add, e, d);
  }
  return d ^ 0x80808080u;
}
__device__ __forceinline__ uint32_t sign_bytes(float x, float y, float z, float w) {
  return (x >= 0.0f ? 1u : 255u) | (y >= 0.0f ? 1u : 255u) << 8 | (z >= 0.0f ? 1u : 255u) << 16 | (w >= 0.0f ? 1u : 255u) << 24;
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

constexpr int kTileWaves = 8, kTileRows = 32 / kTileWaves;  // rows of the block per wave

__global__ void __launch_bounds__(64 * kTileWaves)
quant_tiles_kernel(const QuantTilesParams p) {
  __shared__ uint32_t t[16 * kTileRow];
  // (all arguments named at the top: fetched in one batch, one trip to memory instead of one per group)
  asm volatile("" ::"s"(p.blocks0), "s"(p.div_kblocks.mul), "s"(p.op[0].x), "s"(p.op[0].ld), "s"(p.op[0].L), "s"(p.op[0].tiles),
               "s"(p.op[1].x), "s"(p.op[1].ld), "s"(p.op[1].L), "s"(p.op[1].tiles), "s"(p.K));
  const bool second = (int)blockIdx.x >= p.blocks0;
  QuantOperand o = p.op[0];
  if (second) o = p.op[1];
  const int b = (int)blockIdx.x - (second ? p.blocks0 : 0);
  const int rb = (int)fast_div((uint32_t)b, p.div_kblocks), kb = b - rb * p.kblocks;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k0 = kb * 256 + 4 * lane;
  float v[kTileRows][4];
  // (rows past the matrix repeat its last: their results are never stored)
  const int row0 = rb * 32 + wave * kTileRows;
  const float* const x = o.x + k0;
  const int64_t ld = o.ld;
  const int last = o.rows - 1;
  if (kb * 256 + 256 <= p.K) {  // workgroup-uniform
#pragma unroll
    for (int j = 0; j < kTileRows; ++j) {
      const v4f_any f = *(const v4f_any*)(x + (int64_t)min(row0 + j, last) * ld);
      v[j][0] = f[0], v[j][1] = f[1], v[j][2] = f[2], v[j][3] = f[3];
    }
  } else {
#pragma unroll
    for (int j = 0; j < kTileRows; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)  // (elements past the row read its last and are masked below)
        v[j][e] = o.x[(int64_t)min(row0 + j, last) * ld + min(k0 + e, p.K - 1)];
  }
  const uint32_t mask = byte_mask(p.K - k0);
  uint32_t* const dst = &t[(lane >> 2) * kTileRow + wave * (4 * kTileRows) + (lane & 3)];
  if (o.sign) {
#pragma unroll
    for (int j = 0; j < kTileRows; ++j) dst[4 * j] = sign_bytes(v[j][0], v[j][1], v[j][2], v[j][3]) & mask;
  } else {
#pragma unroll
    for (int j = 0; j < kTileRows; ++j) dst[4 * j] = quant_bytes(o, v[j][0], v[j][1], v[j][2], v[j][3]) & mask;
  }
  __syncthreads();
  // half tile 2 s + h of the block is t[(2 s + h) * kTileRow ...]: row r at dword 4 r
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
  int M, N, nk;        // nk: k steps of 32
  int mblocks, nblocks;
  int tiles_m, tiles, tiles_per_xcd;
  int S;
  int ca, scale, rs, Kreal;
  float denom;
  int32_t* C_i32;
  float* C_f32;
  int64_t ldc;
  int s_base, s_rem;  // k steps per wave: s_base, the first s_rem waves one more
  FastDiv div_tiles_m;
};

constexpr int kAhead = 4;  // k steps per group of loads

template <int TM, int TN>
struct Group {
  v4i a[kAhead][TM], b[kAhead][TN];
};

// The tile's end: operand sums of the two half-waves, the partial tiles of the S waves of a workgroup
// through LDS (S > 1, at most MAXS), the 8-bit correction, stores.
template <int TM, int TN, bool SUMS, int MAXS>
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
      int sv = d[e];
      if (SUMS)
        sv = (int)((uint32_t)p.scale * ((uint32_t)d[e] + (uint32_t)p.ca * (uint32_t)cb) +
                   (uint32_t)p.rs * ((uint32_t)ra[e] + (uint32_t)p.ca * (uint32_t)p.Kreal));
      const int64_t idx = (int64_t)m * p.ldc + n;
      if (p.C_i32) p.C_i32[idx] = sv;
      if (p.C_f32) p.C_f32[idx] = (float)sv / p.denom;
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

template <int TM, int TN, bool SUMS>
__global__ void __launch_bounds__(512)
gemm_i8_kernel(const I8Params p) {
  extern __shared__ int red[];
  // (all arguments named at the top: fetched in one batch, one trip to memory instead of one per group)
  asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.M), "s"(p.N), "s"(p.nk), "s"(p.S), "s"(p.mblocks), "s"(p.nblocks), "s"(p.tiles_m),
               "s"(p.tiles), "s"(p.tiles_per_xcd), "s"(p.s_base), "s"(p.s_rem), "s"(p.div_tiles_m.mul), "s"(p.div_tiles_m.sh1),
               "s"(p.div_tiles_m.sh2));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup b sits on XCD b % 8: every XCD gets a contiguous run of tiles, rows of C fastest
  const int lin = (int)(blockIdx.x & 7) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  if (lin >= p.tiles) return;  // (the whole workgroup)
  const int tile_n = (int)__builtin_amdgcn_readfirstlane(fast_div((uint32_t)lin, p.div_tiles_m)), tile_m = lin - tile_n * p.tiles_m;
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

  auto load = [&](Group<TM, TN>& g, int k) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      const int kk = min(k + d, k_hi - 1) * 64;  // (a group's steps past the range repeat its last)
#pragma unroll
      for (int i = 0; i < TM; ++i) g.a[d][i] = *(const v4i*)(arow[i] + kk);
#pragma unroll
      for (int j = 0; j < TN; ++j) g.b[d][j] = *(const v4i*)(brow[j] + kk);
    }
  };
  auto multiply = [&](const Group<TM, TN>& g, int k) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      if (k + d >= k_hi) break;  // wave-uniform
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
    Group<TM, TN> g0, g1;
    load(g0, k_lo);
    for (int k = k_lo; k < k_hi; k += 2 * kAhead) {
      if (k + kAhead < k_hi) load(g1, k + kAhead);
      multiply(g0, k);
      if (k + 2 * kAhead < k_hi) load(g0, k + 2 * kAhead);
      multiply(g1, k + kAhead);
    }
  }
  finish_tile<TM, TN, SUMS, 8>(p, acc, sa, sb, red, lane, wave, tile_m, tile_n);
}

// ---- the whole product in one launch, for problems small enough that a second launch costs more
// than quantising a row once per tile of results.  Up to 16 waves split a tile's K.  Of a step of 32 k a
// wave fetches 32 rows of both operands, eight lanes to a row's 128 bytes (16 bytes straight into the
// MFMA's layout would touch 64 lines per load: 202 x 192 x 437 7.7 us), quantises four values per lane and
// load into a dword of bytes, and turns those into the MFMA's layout (lane (r, h): 16 bytes of row r)
// through 2 KB of LDS of its own, where its partial sums go in the end.
struct QuantSmallParams {
  I8Params g;
  QuantOperand a, w;
};

template <bool SUMS, bool SIGN>
__global__ void __launch_bounds__(1024)
quant_small_kernel(const QuantSmallParams p) {
  extern __shared__ int red[];
  asm volatile("" ::"s"(p.a.x), "s"(p.a.ld), "s"(p.a.L), "s"(p.a.mul), "s"(p.a.add), "s"(p.w.x), "s"(p.w.ld), "s"(p.w.L),
               "s"(p.w.mul), "s"(p.w.add), "s"(p.g.M), "s"(p.g.N), "s"(p.g.Kreal), "s"(p.g.tiles_m), "s"(p.g.S), "s"(p.g.s_base),
               "s"(p.g.s_rem), "s"(p.g.div_tiles_m.mul), "s"(p.g.div_tiles_m.sh1), "s"(p.g.div_tiles_m.sh2));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5, c = lane & 7;
  const int tile_n = (int)__builtin_amdgcn_readfirstlane(fast_div(blockIdx.x, p.g.div_tiles_m));
  const int tile_m = (int)blockIdx.x - tile_n * p.g.tiles_m;
  const int k_lo = wave * p.g.s_base + min(wave, p.g.s_rem), k_hi = k_lo + p.g.s_base + (wave < p.g.s_rem ? 1 : 0);
  const int K = p.g.Kreal;
  // byte offsets of row 8 t + lane / 8 (rows past a matrix repeat its last; their results are never stored)
  uint32_t arow[4], wrow[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int row = 8 * t + (lane >> 3);
    arow[t] = (uint32_t)min(tile_m * 32 + row, p.g.M - 1) * (uint32_t)p.a.ld * 4u;
    wrow[t] = (uint32_t)min(tile_n * 32 + row, p.g.N - 1) * (uint32_t)p.w.ld * 4u;
  }
  v16i acc[1][1];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[0][0][e] = 0;
  int sa[1] = {}, sb[1] = {};
  QuantOperand oa = p.a, ow = p.w;
  oa.sign = 0;
  ow.sign = SIGN ? 1 : 0;
  v4f_any va[2][4], vw[2][4];
  auto load = [&](int i, int k) {
    // four values past the row's end are its last four instead; those that the piece before has are masked
    // below (of both operands: what remains still meets its partner, and K has no order)
    const uint32_t off = 4u * (uint32_t)min(32 * k + 4 * c, K - 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      va[i][t] = *(const v4f_any*)((const char*)p.a.x + (arow[t] + off));
      vw[i][t] = *(const v4f_any*)((const char*)p.w.x + (wrow[t] + off));
    }
  };
  uint32_t* const turn = (uint32_t*)red + wave * 1024;  // [operand][row][8 dwords]
  auto multiply = [&](int i, int k) {
    const uint32_t mask = ~byte_mask(32 * k + 4 * c + 4 - K);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const v4f_any x = va[i][t], y = vw[i][t];
      turn[64 * t + lane] = quant_bytes(oa, x[0], x[1], x[2], x[3]) & mask;
      turn[256 + 64 * t + lane] = (SIGN ? sign_bytes(y[0], y[1], y[2], y[3]) : quant_bytes(ow, y[0], y[1], y[2], y[3])) & mask;
    }
    typedef v4i __attribute__((may_alias)) v4i_alias;
    const v4i a = *(const v4i_alias*)(turn + 8 * r + 4 * h), b = *(const v4i_alias*)(turn + 256 + 8 * r + 4 * h);
    if (SUMS) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sa[0] = __builtin_amdgcn_sdot4(a[e], 0x01010101, sa[0], false);
        sb[0] = __builtin_amdgcn_sdot4(b[e], 0x01010101, sb[0], false);
      }
    }
    acc[0][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc[0][0], 0, 0, 0);
  };
  if (k_lo < k_hi) {
    load(0, k_lo);
    for (int k = k_lo; k < k_hi; k += 2) {
      if (k + 1 < k_hi) load(1, k + 1);
      multiply(0, k);
      if (k + 1 >= k_hi) break;
      if (k + 2 < k_hi) load(0, k + 2);
      multiply(1, k + 1);
    }
  }
  finish_tile<1, 1, SUMS, 16>(p.g, acc, sa, sb, red, lane, wave, tile_m, tile_n);
}

template <int TM, int TN, bool SUMS>
hipError_t launch_i8(const I8Params& p, hipStream_t s) {
  auto kern = gemm_i8_kernel<TM, TN, SUMS>;
  const size_t lds = p.S > 1 ? (size_t)p.S * (TM * TN * 4 * 1024 + 128 * (TM + TN)) : 0;
  static std::atomic<bool> asked[64];
  const hipError_t e = allow_lds((const void*)kern, lds, asked);
  if (e != hipSuccess) return e;
  note_kernel("gemm_i8_kernel<%d,%d%s> grid %d x %d, K split %d", TM, TN, SUMS ? ",sums" : "", 8 * p.tiles_per_xcd, 64 * p.S, p.S);
  launch_kernel(kern, dim3((unsigned)(8 * p.tiles_per_xcd)), dim3(64 * p.S), lds, s, p);
  return launch_error();
}

int64_t tile_bytes(int64_t rows, int64_t K) { return ceil_div(rows, 32) * 32 * ceil_div(K, 256) * 256; }

}  // namespace

// Workspace of the two tiled operands, and whether the problem is taken: an operand of more bits than
// the FP4 form holds, or a product of few bits where bytes cost less than the plane pack and its GEMM; and a result that
// fills a quarter of a 32 x 32 block (below that the padding of the tiles is most of what is moved, and the plane
// kernels' workspace is smaller).
// Few bits (1 or 2 by 1): the byte form writes its tiles and reads them again and multiplies a byte a value; the plane
// form multiplies once per activation bit, and its pack and its splits of K have coarser pieces, so that a round of 4096
// values that is not full costs much of a full one.  The line below fits 518 products on
// both forms (chosen form over the better one: 0.5 % on average, 18 % at most; bytes always 5.5 %, planes always 15 %).  us a
// call, bytes / planes: 572 x 896 x 1293 of 1 x 1 bits 10.3 / 14.3, 496 x 1408 x 640 9.4 / 12.7, 418 x 1024 x 605
// of 2 x 1 8.1 / 12.1; 612 x 384 x 3968 15.4 / 12.0, 361 x 64 x 8115 15.1 / 12.1, 1744 x 256 x 2234 16.8 / 13.4.
static bool bytes_pay(int64_t M, int64_t N, int64_t K, int bits_a) {
  if (M * N >= 1000000000) return false;  // (the products below stay in range)
  const int64_t bytes = tile_bytes(M, K) + tile_bytes(N, K) + M * N * K / 1000 * 20 + 100 * K;
  const int64_t planes = 14000000 * (bits_a - 1) + (K % 1024 ? 4000000 : 0) + 5500 * (ceil_div(K, 4096) * 4096 - K);
  return bytes < planes;
}

bool quant_i8_takes(int64_t M, int64_t N, int64_t K, int bits_a, int bits_w, size_t* bytes) {
  if (bits_a <= 2 && bits_w == 1 && !bytes_pay(M, N, K, bits_a)) return false;
  if (M * N < 256) return false;
  const int64_t a = tile_bytes(M, K), b = tile_bytes(N, K);
  *bytes = (size_t)(a + b);
  const int64_t tiles = ceil_div(M, 32) * ceil_div(N, 32);
  return a < ((int64_t)1 << 40) && b < ((int64_t)1 << 40) && tiles < ((int64_t)1 << 30) &&
         ceil_div(M, 32) * ceil_div(K, 256) + ceil_div(N, 32) * ceil_div(K, 256) < ((int64_t)1 << 30);
}

namespace {

void fill_operands(QuantOperand (&op)[2], const float* a, int64_t lda, int bits_a, const float* w, int64_t ldw, int bits_w,
                   int M, int N) {
  const int La = (1 << bits_a) - 1, Lw = (1 << bits_w) - 1;
  op[0] = {a, lda, M, 0, 0.0f, 1.0f, (float)La, 1.0f, bits_a == 8 ? 0.0f : 128.0f, nullptr};
  op[1] = {w, ldw, N, bits_w == 1 ? 1 : 0, 1.0f, 0.5f, (float)Lw, bits_w == 8 ? 1.0f : 2.0f,
           bits_w == 8 ? 0.0f : 128.0f - (float)Lw, nullptr};
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
  p.C_i32 = S_out;
  p.C_f32 = out_f32;
  p.ldc = ldo;
}

}  // namespace

static void set_split(I8Params& p) {
  p.s_base = p.nk / p.S;
  p.s_rem = p.nk % p.S;
  p.div_tiles_m = make_fast_div((uint32_t)p.tiles_m);
}

// The one-launch form, for any pair of bit widths; false when the problem is too large for it.
bool launch_quant_small(const float* a, int64_t lda, int bits_a, const float* w, int64_t ldw, int bits_w, int M, int N,
                        int K, int32_t* S_out, float* out_f32, int64_t ldo, hipStream_t s, hipError_t* err) {
  if (gemm_engine != 0) return false;
  const int64_t tiles = ceil_div(M, 32) * ceil_div(N, 32), nk = ceil_div(K, 32);
  // Steps of K per CU up to which one launch is ahead (us a call: 202 x 192 x 437 5.0 against 8.1, 1735 x 64 x 768
  // 6.3 / 7.6, 83 x 64 x 1152 6.4 / 7.8, 245 x 773 x 1792 10.8 / 8.0, 748 x 448 x 512, two tiles on a CU, 8.5 / 7.8,
  // 104 x 697 x 1045, 88 tiles, 9.0 / 8.2;
  // with 8 bits on a side and so the operands' sums 674 x 64 x 896 7.5 / 8.0, 230 x 64 x 1142 8.2 / 8.2).
  if (nk * ceil_div(tiles, 256) > (tiles > 256 ? 24 : tiles > 48 || bits_a == 8 || bits_w == 8 ? 28 : 36)) return false;
  if (K < 4 || (int64_t)M * lda * 4 >= ((int64_t)1 << 32) || (int64_t)N * ldw * 4 >= ((int64_t)1 << 32)) return false;
  QuantSmallParams p;
  QuantOperand op[2];
  fill_operands(op, a, lda, bits_a, w, ldw, bits_w, M, N);
  p.a = op[0];
  p.w = op[1];
  fill_product(p.g, bits_a, bits_w, M, N, K, S_out, out_f32, ldo);
  p.g.nk = (int)nk;
  p.g.tiles_m = p.g.mblocks;
  p.g.tiles = (int)tiles;
  p.g.tiles_per_xcd = 0;
  // waves per tile: a step or two of K each while the chip has room for them
  const bool sums = bits_a == 8 || bits_w == 8;
  const int64_t S = std::min<int64_t>(sums ? 15 : 16, std::max<int64_t>(1, 4096 / tiles));  // (15: 64 KB of LDS)
  p.g.S = (int)std::min(S, nk);
  set_split(p.g);
  const size_t lds = (size_t)p.g.S * (4096 + (sums ? 256 : 0));
  note_kernel("quant_small_kernel%s grid %lld x %d", sums ? "<sums>" : "", (long long)tiles, 64 * p.g.S);
  auto go = [&](auto kern) { launch_kernel(kern, dim3((unsigned)tiles), dim3(64 * p.g.S), lds, s, p); };
  if (bits_w == 1) sums ? go(quant_small_kernel<true, true>) : go(quant_small_kernel<false, true>);
  else sums ? go(quant_small_kernel<true, false>) : go(quant_small_kernel<false, false>);
  *err = launch_error();
  return true;
}

bool launch_quant_i8(const float* a, int64_t lda, int bits_a, const float* w, int64_t ldw, int bits_w, int M, int N,
                     int K, int32_t* S_out, float* out_f32, int64_t ldo, void* workspace, hipStream_t s, hipError_t* err) {
  size_t need;
  if (gemm_engine == 1 || !quant_i8_takes(M, N, K, bits_a, bits_w, &need)) return false;
  if (gemm_engine != 0 && bits_a <= 2 && bits_w == 1) return false;  // (an engine of the plane form is pinned)
  QuantTilesParams q;
  fill_operands(q.op, a, lda, bits_a, w, ldw, bits_w, M, N);
  q.op[0].tiles = (uint4*)workspace;
  q.op[1].tiles = (uint4*)((char*)workspace + tile_bytes(M, K));
  q.K = K;
  q.kblocks = (int)ceil_div(K, 256);
  q.div_kblocks = make_fast_div((uint32_t)q.kblocks);
  I8Params p;
  fill_product(p, bits_a, bits_w, M, N, K, S_out, out_f32, ldo);
  q.blocks0 = p.mblocks * q.kblocks;
  launch_kernel(quant_tiles_kernel, dim3((unsigned)(q.blocks0 + p.nblocks * q.kblocks)), dim3(64 * kTileWaves), 0, s, q);
  *err = launch_error();
  if (*err != hipSuccess) return true;
  p.A = q.op[0].tiles;
  p.B = q.op[1].tiles;
  p.nk = q.kblocks * 8;
  // C per wave: 32 x 32 while K is short (many waves, each with little to fetch before its first product), 32 x 64, and 64 x 64
  // where K is long, each with tiles for half the CUs.  K is split over as many waves as leave the workgroups of
  // a CU resident at once (the registers hold 24, 12 and 8 waves, rounded as below), a power of two of them so that its
  // SIMDs stay level.  us a call, before (2048 waves in all, 64 x 64 and 32 x 64 once they fill the chip) and now: 994 x 551 x
  // 2226, 288 tiles of 32 x 64, where the second workgroup of seven waves had to wait for the first, 18.8 and 15.3; 721
  // x 1438 x 681 14.2 and 11.4; 1650 x 1566 x 103 16.8 and 12.2; 1098 x 1728 x 265 12.1 and 11.3.  Over 150
  // products 8.7 % and 1.8 % behind the best of all splits and forms.
  const int64_t t12 = ceil_div(M, 32) * ceil_div(N, 64), t22 = ceil_div(M, 64) * ceil_div(N, 64);
  const int TM = K >= 5000 && t22 >= 128 ? 2 : 1, TN = TM == 2 || (K > 1100 && t12 >= 128) ? 2 : 1;
  p.tiles_m = (int)ceil_div(M, 32 * TM);
  p.tiles = (int)(p.tiles_m * ceil_div(N, 32 * TN));
  p.tiles_per_xcd = (int)ceil_div(p.tiles, 8);
  const int64_t room = (TM * TN == 4 ? 8 : TM * TN == 2 ? 12 : 24) / ceil_div(p.tiles, 256);  // waves a workgroup
  p.S = room >= 8 ? 8 : room >= 4 ? 4 : room >= 2 ? 2 : 1;
  while (p.S > 1 && p.S > p.nk / kAhead) p.S /= 2;  // (each with at least one group of k steps)
  set_split(p);
  const bool sums = bits_a == 8 || bits_w == 8;
  if (TM == 2) *err = sums ? launch_i8<2, 2, true>(p, s) : launch_i8<2, 2, false>(p, s);
  else if (TN == 2) *err = sums ? launch_i8<1, 2, true>(p, s) : launch_i8<1, 2, false>(p, s);
  else *err = sums ? launch_i8<1, 1, true>(p, s) : launch_i8<1, 1, false>(p, s);
  return true;
}

}  // namespace bmx
