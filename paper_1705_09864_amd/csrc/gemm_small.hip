// xnor GEMM for small problems: 32 x 32 of C per workgroup, K split over its 1 to 16 waves.
// Paper: Sec. 2.2.1 / Sec. 2.2.2 (Eq. 2): C[m][n] = K - 2 * popcount(A[m] xor B[n]).
//
// A launch of this size is a chain: arguments, operands, multiply, sum over the waves, results, and the
// code itself, which the instruction cache does not hold when a kernel starts.  So: one trip to memory
// (a wave requests all its words, up to four steps of 256 bits, before it uses the first), rows read
// straight into the MFMA's layout (lane (r, h) takes 16 bytes of row r: an access per lane pair, which
// does not matter at this size, and no transposition through LDS), one barrier, and a short kernel per
// kind of result and number of waves (4 to 6 KB each, where the general one has 12).
//
// Arithmetic as in gemm_fp4.hip: C = K - 2 pc(a) - 2 pc(b) + 4 * sum a b, one MFMA per nibble plane of
// the four dwords a lane holds (which bits share a place in K does not matter as long as both operands
// agree).  Rows may start on any dword and may hold an odd number of them.
//
// Measured, us per launch in a graph, against the general kernels: 46 x 430 x 875 2.8 / 4.7, 250 x 250 x 250
// 3.1 / 4.8, 703 x 143 x 384 3.1 / 5.5, 18 x 128 x 2624 2.9 / 4.4, 1000 x 300 x 2000 3.8 / 6.1, 64 x 4289 x 3633
// 4.2 / 7.1, 32 x 4096 x 9216 5.0 / 6.7, 365 x 4117 x 516 5.6 / 8.0.
#include <type_traits>

#include "bmx_internal.h"

namespace bmx {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kF32 = 0, kI32 = 1, kBits = 2;

struct SmallGemmParams {
  const char* A;
  const char* B;
  uint32_t lda, ldb;  // bytes
  int M, N, Kd, Kreal;  // Kd dwords of data per row, zero bits behind the K-th
  int tiles_n, s_base, s_rem;  // steps of eight dwords per wave: s_base, the first s_rem waves one more
  FastDiv div_tiles_n;
  const float* alpha;  // per column, or null
  const float* thr;    // packed bits: per column threshold, or null (0)
  void* C;             // fp32, int32, or packed bits in dwords
  int ldc;             // elements per row (packed bits: dwords)
  int as_count;
  int per_xcd;         // tiles in a row that every XCD takes (RUNS)
};

__device__ __forceinline__ v8i plane(const v4u& w, int n) {
  v8i e;
#pragma unroll
  for (int d = 0; d < 4; ++d) e[d] = (int)(n == 3 ? (w[d] >> 3) & 0x11111111u : w[d] & (0x11111111u << n));
#pragma unroll
  for (int d = 4; d < 8; ++d) e[d] = 0;
  return e;
}

// RUNS: a run of tiles per XCD, else in the grid's order.  (A kernel of its own: as a choice in one kernel the others, whose first addresses
// wait for it, lost 0.8 % in the mean and 2.7 % at 3 us.)
template <int OUT, int S, bool RUNS>
__global__ void __launch_bounds__(64 * S)
gemm_small_kernel(const SmallGemmParams p) {
  __shared__ float sums[S > 1 ? S : 1][17][64];  // a wave's sixteen sums per lane and its popcounts
  asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.lda), "s"(p.ldb), "s"(p.M), "s"(p.N), "s"(p.Kd), "s"(p.tiles_n), "s"(p.s_base),
               "s"(p.s_rem), "s"(p.div_tiles_n.mul), "s"(p.div_tiles_n.sh1), "s"(p.div_tiles_n.sh2), "s"(p.alpha), "s"(p.thr));
  if (RUNS) asm volatile("" ::"s"(p.per_xcd));
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int wave = S > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const int tile = RUNS ? (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int tile_m = (int)__builtin_amdgcn_readfirstlane(fast_div((uint32_t)tile, p.div_tiles_n));
  const int m0 = tile_m * 32, n0 = (tile - tile_m * p.tiles_n) * 32;
  if (RUNS && m0 >= p.M) return;  // (the whole workgroup)
  const int col = n0 + r, ncol = min(col, p.N - 1);
  // (rows past a matrix repeat its last; their results are not stored)
  const uint32_t arow = (uint32_t)min(m0 + r, p.M - 1) * p.lda, brow = (uint32_t)ncol * p.ldb;
  const int s0 = wave * p.s_base + min(wave, p.s_rem), s1 = s0 + p.s_base + (wave < p.s_rem ? 1 : 0);

  // A piece that reaches past the row's end is fetched from the row's last 16 bytes instead; `trim` then
  // clears the dwords that the piece before it already has (of both operands: what remains still
  // meets its partner, and K has no order).
  v4u a[4], b[4];
  const int last = p.Kd - 4;
  auto fetch = [&](int i, int s) {
    const uint32_t off = 4u * (uint32_t)min(8 * s + 4 * h, last);
    b[i] = *(const v4u_any*)(p.B + (brow + off));
    a[i] = *(const v4u_any*)(p.A + (arow + off));
  };
  auto trim = [&](int s, v4u& x, v4u& y) {
    if (8 * s + 8 <= p.Kd) return;  // wave-uniform
#pragma unroll
    for (int d = 0; d < 4; ++d)
      if (last + d < 8 * s + 4 * h) x[d] = y[d] = 0u;
  };
  if (p.Kd >= 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (s0 + i < s1) fetch(i, s0 + i);
  } else {  // rows of 1 to 3 dwords, all in the lower half-wave's piece of the only step
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t off = 4u * (uint32_t)min(d, p.Kd - 1);
      b[0][d] = *(const uint32_t*)(p.B + (brow + off));
      a[0][d] = *(const uint32_t*)(p.A + (arow + off));
      if (h || d >= p.Kd) a[0][d] = b[0][d] = 0u;
    }
  }
  const float al = (OUT != kI32 && p.alpha) ? p.alpha[ncol] : 1.0f;
  const float th = (OUT == kBits && p.thr) ? p.thr[ncol] : 0.0f;

  v16f acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
  int pa = 0, pb = 0;
  for (int s = s0; s < s1; s += 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (s + i >= s1) break;  // wave-uniform
      v4u x = a[i], y = b[i];
      if (s + i + 4 < s1) fetch(i, s + i + 4);
      if (p.Kd >= 4) trim(s + i, x, y);
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        pa += __builtin_popcount(x[d]);
        pb += __builtin_popcount(y[d]);
      }
#pragma unroll
      for (int n = 0; n < 4; ++n) {  // (planes 0 and 3 hold 0.5, plane 1 holds 1, plane 2 holds 2)
        const int sc = n == 1 ? 127 : (n == 2 ? 126 : 128);
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(plane(x, n), plane(y, n), acc, 4, 4, 0, sc, 0, sc);
      }
    }
  }
  // row r's count in lane (r, 0), column r's in lane (r, 1): a lane counted its half of K
  const int other = __shfl_xor(h ? pa : pb, 32);
  float cnt = (float)((h ? pb : pa) + other);
  constexpr int kOwn = 16 / S;
  if (S > 1) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sums[wave][v][lane] = acc[v];
    sums[wave][16][lane] = cnt;
    __syncthreads();
    cnt = 0.0f;
#pragma unroll
    for (int w = 0; w < S; ++w) cnt += sums[w][16][lane];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      acc[i] = 0.0f;
#pragma unroll
      for (int w = 0; w < S; ++w) acc[i] += sums[w][wave * kOwn + i][lane];
    }
  }
  const float base = (float)p.Kreal - 2.0f * __shfl(cnt, 32 + r);
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    const int v = S > 1 ? wave * kOwn + i : i;
    const int mi = 8 * (v >> 2) + (v & 3) + 4 * h, m = m0 + mi;
    const float dot = fmaf(4.0f, acc[i], base - 2.0f * __shfl(cnt, mi));  // exact: whole numbers below 2^24
    const bool in = m < p.M && col < p.N;
    if (OUT == kBits) {
      // the 64-lane mask of the decision: its low half is 32 columns of row m, its high half those of the
      // row four below
      const uint64_t mask = __ballot(col < p.N && al * dot >= th);
      if (r == 0 && m < p.M) ((uint32_t*)p.C)[(uint32_t)(m * p.ldc + (n0 >> 5))] = h ? (uint32_t)(mask >> 32) : (uint32_t)mask;
    } else if (in) {
      const uint32_t at = (uint32_t)(m * p.ldc + col);
      if (OUT == kI32) ((int32_t*)p.C)[at] = p.as_count ? ((int)dot + p.Kreal) >> 1 : (int)dot;
      else ((float*)p.C)[at] = al * dot;
    }
  }
}

template <int OUT>
void launch_kind(const SmallGemmParams& p, int S, int64_t blocks, hipStream_t s) {
  auto of = [&](auto runs) {
    constexpr bool R = decltype(runs)::value;
    return S == 1 ? gemm_small_kernel<OUT, 1, R> : S == 2 ? gemm_small_kernel<OUT, 2, R> : S == 4 ? gemm_small_kernel<OUT, 4, R>
         : S == 8 ? gemm_small_kernel<OUT, 8, R> : gemm_small_kernel<OUT, 16, R>;
  };
  auto kern = of(std::false_type{});
  if constexpr (OUT != kBits) {
    if (p.per_xcd) kern = of(std::true_type{});
  }
  launch_kernel(kern, dim3((unsigned)blocks), dim3(64 * S), 0, s, p);
}

}  // namespace

int gemm_small = 0;  // 1 = never (measurements and tests of the general kernels)

bool launch_gemm_small(const void* A, int64_t lda_bytes, const void* B, int64_t ldb_bytes, int M, int N, int K, int dwords,
                       const float* alpha, int32_t* C_i32, float* C_f32, uint64_t* C_bits, const float* thr, int64_t ldc,
                       bool as_count, hipStream_t s, hipError_t* err) {
  if (gemm_small == 1 || gemm_engine || gemm_mfma_ksplit || gemm_mfma_tile || gemm_fp4_split || gemm_fp4_half || gemm_fp4_band ||
      gemm_block > 1)
    return false;
  if (K >= (1 << 24)) return false;
  const int64_t lim = (int64_t)1 << 31;
  if (M * lda_bytes >= lim || N * ldb_bytes >= lim || ((int64_t)M + 32) * ldc * (C_bits ? 2 : 1) >= lim) return false;
  const int64_t tiles_n = C_bits ? ceil_div(N, 64) * 2 : ceil_div(N, 32);  // (both halves of the last word)
  const int64_t tiles = ceil_div(M, 32) * tiles_n;
  const int steps = (dwords + 7) / 8;
  // Against the kernels of 64 x 64 tiles and more, from 2500 products of 64 to 1300 such tiles and 1500 to 16000 tile steps of 32 x 32 x 256
  // (their time over this kernel's, in a graph).  Up to 28 words, where gemm_fp4_kernel does not divide K over four waves, up to 12288
  // steps (8000 to 9000 1.10, 10000 to 13000 1.01 to 1.04).  Beyond: below 128 of its tiles up to 8192 (7000 to 8000 1.09, then 0.92), to
  // 255 up to 7000 (5000 to 7000 1.0 to 1.05, then 0.95 to 0.8), to 511 up to 8192 (0.99, then 0.88).
  // 12288 too where that kernel does not take the product; of a K of more than four steps for each of
  // sixteen waves only few (200 x 300 x 30000 12.1 / 10.4); and 4096 tiles, where the results outweigh the rest.
  // From some hundred tiles of 64 x 64 on, where that kernel has work for most SIMDs (this one's time over its, 2100 products of 64 to 1100
  // tiles and 2 to 20 words, in a graph and as calls): packed bits from 352 (300 to 351 1.00, 0.98; 352 to 399 1.02, 1.00), of one step of K
  // from 256 (200 to 255 1.09, 0.97; 256 to 319 1.11, 1.01); int32 and fp32 results by which tiles there are whole, stored without bounds.
  // All: int32 from 400 (350 to 399 1.02, 0.97; 400 to 447 1.02, 1.01), fp32 and one step of K from 512 (fp32 448 to 511 0.97, 0.97; 512 to
  // 599 1.06, 1.07; int32 of one step 400 to 447 0.93, 0.90, 512 to 599 1.04, 1.00).  All but the last rows': from 512 (int32 448 to 511
  // 0.98, 0.97, 512 to 599 1.06, 1.06; fp32 0.93, 0.93, then 1.03, 1.03), of one step from 800 (int32 700 to 799 0.97, 0.96, 800 to 1023 1.04,
  // 1.02).  Columns that end inside a tile: from 700 (int32 600 to 699 0.98, 0.97, 700 to 799 1.00, 1.00; fp32 0.95, 0.95, then 0.99, 0.99), of
  // one step none (800 to 1023 0.93, 0.91).  The choice is 0.5 % behind the better kernel (0.9 % without the case of whole columns), packed bits
  // 0.8 % in a graph and 0.2 as calls; 1.7 and 2.2 % while int32 had 256 to 448, drawn before tiles side by side shared an XCD.  From 21 words on, where that kernel
  // divides K over three waves or four, from 512 (652 x 2512 x 1472 as bits 6.9 / 6.4).
  const int64_t work = tiles * steps, tiles64 = ceil_div(M, 64) * ceil_div(N, 64);
  const bool apart = !((lda_bytes | ldb_bytes) & 15) && !(((uintptr_t)A | (uintptr_t)B) & 15);  // (launch_gemm_fp4)
  const bool pays = (dwords >= 4 || apart) && gemm_fp4_pays(M, N, lda_bytes, ldb_bytes, ldc, C_bits != nullptr);
  const int64_t most = steps > 64                                ? 2048
                       : !pays || (dwords <= 56 && tiles64 < 512) ? 12288
                                                                  : (tiles64 >= 128 && tiles64 < 256 ? 7000 : 8192);
  const bool cols = N % 64 == 0, whole = cols && M % 64 == 0;
  const int64_t below = dwords > 40 ? 512
                      : C_bits      ? (steps == 1 ? 256 : 352)
                      : whole       ? (C_f32 || steps == 1 ? 512 : 400)
                      : cols        ? (steps == 1 ? 800 : 512)
                                    : (steps == 1 ? lim : 700);
  // (Packed bits of rows of less than 16 bytes that the next begins in, whatever the size: gemm_fp4.hip does not take them, and gemm_mfma.hip, which
  // would, is behind.  us in a graph there / here: 3000 x 2001 x 64 14.4 / 8.3, 4096 x 4096 26.1 / 17.1, 60000 x 300 33.3 / 18.6, 8192 x 8192
  // 88.9 / 52.7; dword by dword through registers gemm_fp4_kernel once took 9.6, 17.3, 22.4 and 61.2.)
  if ((work > most || tiles > 4096) && !(C_bits && dwords < 4 && !apart)) return false;
  if (pays && tiles64 >= below) return false;
  int S = 1;
  while (S < 16 && 2 * S <= steps && 2 * S * tiles <= (work > 8192 ? 8192 : 4096)) S *= 2;
  SmallGemmParams p;
  p.A = (const char*)A;
  p.B = (const char*)B;
  p.lda = (uint32_t)lda_bytes;
  p.ldb = (uint32_t)ldb_bytes;
  p.M = M;
  p.N = N;
  p.Kd = dwords;
  p.Kreal = K;
  p.tiles_n = (int)tiles_n;
  // Workgroup b sits on XCD b % 8.  Where tiles side by side write parts of one line they go to one XCD, whose L2 puts the line together
  // (int32 results in a graph, in the grid's order / so: 576 x 2934 x 64 5.0 / 4.4 us, 5760 x 238 x 1011 5.9 / 5.4; 100 drawn ones 1.03 with 257 to
  // 512 tiles, 1.05 to 1200, 1.08 beyond; with fewer, and of whole lines, 0.99).
  p.per_xcd = !C_bits && ldc % 32 != 0 && tiles > 256 ? (int)ceil_div(tiles, 8) : 0;
  const int64_t blocks = p.per_xcd ? 8 * (int64_t)p.per_xcd : tiles;
  p.s_base = steps / S;
  p.s_rem = steps % S;
  p.div_tiles_n = make_fast_div((uint32_t)tiles_n);
  p.alpha = alpha;
  p.thr = thr;
  p.C = C_bits ? (void*)C_bits : C_i32 ? (void*)C_i32 : (void*)C_f32;
  p.ldc = (int)(C_bits ? 2 * ldc : ldc);
  p.as_count = as_count ? 1 : 0;
  note_kernel("gemm_small_kernel<%s> grid %lld x %d", C_bits ? "bits" : C_i32 ? "i32" : "f32", (long long)blocks, 64 * S);
  if (C_bits) launch_kind<kBits>(p, S, blocks, s);
  else if (C_i32) launch_kind<kI32>(p, S, blocks, s);
  else launch_kind<kF32>(p, S, blocks, s);
  *err = launch_error();
  return true;
}

}  // namespace bmx
