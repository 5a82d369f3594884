// xnor GEMM on the matrix cores (FP4 form by default, int8 form beside it).
// Paper: Sec. 2.2.1 / Sec. 2.2.2 (Eq. 2): C[m][n] = K - 2 * popcount(A[m] xor B[n]).
//
// With a, b in {0, 1}:  a xor b = a + b - 2ab, so
//     C[m][n] = K - 2 * pc(A[m]) - 2 * pc(B[n]) + 4 * sum_k a[m][k] * b[n][k],
// and the last sum is an integer matrix product.  The operands stay bit-packed in memory and
// in the loads (that is what keeps the traffic 32x below fp32, Sec. 1); a lane turns its
// bits into 0/1 bytes in registers right before v_mfma_i32_32x32x32_i8 consumes them (or
// into FP4 nibbles for v_mfma_scale_f32_32x32x64_f8f6f4: see plane4 below).
// Expansion (int8 form): for a 32-bit word w, (w >> j) & 0x01010101 puts bits j, j+8, j+16, j+24 into the
// four bytes of a dword, so eight shift/and pairs give the 32 bytes two MFMA steps take.
// Which bit lands in which byte does not matter as long as both operands use the same order:
// a dot product is invariant under a permutation of k applied to both.
//
// Layout facts of the instruction (established on the hardware with a 32 x 32 x 64 tile
// against a CPU count): operand A: lane l supplies row l % 32, operand B: lane l supplies
// column l % 32, both the 16 bytes of k-half l / 32; result register v of lane l is
// D[8 * (v / 4) + 4 * (l / 32) + v % 4][l % 32].  Lanes therefore run along n (the B
// operand = weight rows), and stores are two 128-byte runs per instruction.
//
// A wave owns a (32 * TM) x (32 * TN) tile of C and a range of K; per row and "macro step"
// of 1024 bits a lane ends up with its 64 bytes (one half of a 128-byte line, the other
// half-wave holds the rest; how they get there is described at load_rows_coalesced), counts
// their ones (pc(A[m]), pc(B[n]) come for free this way), and feeds 16 (FP4) or 32 (int8)
// MFMA steps.  The S waves of a workgroup split K and add their partial results in LDS.
//
// The k-bit activations of the quantised GEMM (Sec. 2.1, Eq. 1) ride the same kernel: the A
// byte becomes the quantised value itself, q = sum_p 2^p * plane_p, assembled from the bit
// planes during the expansion, the B byte stays the weight bit, and one pass gives
// sum_k q * wb for all planes at once; S = 2 * that - rowsum as in the plane-by-plane form.
//
// Convolution (Sec. 3.1: M = filters, N = batch * output pixels, K = kh * kw * C): operand A
// is the packed filter matrix, operand B the im2col row of a pixel, gathered word by word
// from the halo-padded packed image (word w of the row is channel word w % Cw of tap w / Cw);
// lanes run along pixels, so the NCHW stores stay coalesced, and alpha is per row.
#include "bmx_internal.h"

namespace bmx {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

template <bool F4> struct AccOf { typedef v16i type; };
template <> struct AccOf<true> { typedef v16f type; };

struct MfmaParams {
  const uint64_t* A;  // [M][lda] words, tail bits zero
  const uint64_t* B;  // [N][ldb] words
  int64_t lda, ldb;   // in words, even (16-byte aligned rows)
  int M, N, Kw, Kreal;  // Kw data words per row
  int nsteps;           // piece steps in all: 4 per whole macro step + those of the last one
  int tail_half;        // words per half-wave in the last macro step (8 when it is whole)
  int tiles_n;
  const float* alpha;  // per column n, or null
  int as_count;        // int32 GEMM output: the xnor count (dot + K) / 2 instead of the dot product
  const float* thr;    // packed-bit output: per column n threshold of the sign decision, or null (0)
  const int32_t* rowsum;  // plane mode: sum_k q[m][k]
  float levels;           // plane mode: 2^bits - 1
  // convolution mode: B is the packed image, column n is output pixel n (flat over images)
  int HoWo, Wo, Hp, Wpp, Cw, stride, KWid;
  FastDiv div_howo, div_wo, div_cw, div_kw;
  int32_t* C_i32;
  float* C_f32;
  uint32_t* C_bits;  // packed sign bits, addressed in 32-bit halves of the output words
  int64_t ldc;       // elements per row (C_bits: 64-bit words per row)
};

// Sixteen bytes of a row whose start is only a multiple of 8 (rows of an odd number of words, as
// binarize_pack leaves them for such K): one global load all the same.
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(8)));

// A macro step covers up to 16 words (1024 bits) of every row: half h of the wave takes
// words h * half .. h * half + half - 1 of it (half = 8 except in a shorter last step), in
// pieces of two words; piece step q is words h * half + 2q, + 1.  One piece step of all rows
// feeds eight MFMA steps, and piece steps are the unit in which K is split over waves.
//
// Loading.  The layout the MFMA wants (lane = row) makes every lane of a load touch a
// different cache line, and the vector memory pipeline then spends one access per lane: it,
// not the matrix cores, set the pace (11 M cache accesses for 0.2 M load instructions on a
// convolution).  So the 32 rows x 128 bytes of a block are loaded the coalesced way (eight
// consecutive lanes read the eight 16-byte pieces of one row) and turned into the MFMA layout
// through a 4 KiB LDS tile private to the wave.  Piece p of row w lives in slot p ^ (w & 7),
// which makes both the row-wise writes and the column-wise reads conflict free.
__device__ __forceinline__ void load_rows_coalesced(const uint64_t* mat, int64_t ld, int row0, int nrows, int planes,
                                                    int pl, int mac, int Kw, bool whole, int lane,
                                                    uint4 (&r)[4]) {
  const int pp = lane & 7;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int row = min(row0 + 8 * t + (lane >> 3), nrows - 1);  // rows past the matrix repeat its last
    const uint64_t* src = mat + ((int64_t)row * planes + pl) * ld + mac * 16 + 2 * pp;
    if (whole) {
      const v4u_any v = *(const v4u_any*)src;
      r[t] = make_uint4(v[0], v[1], v[2], v[3]);
    } else {
      const int w = mac * 16 + 2 * pp;
      const uint64_t lo = w < Kw ? src[0] : 0;
      const uint64_t hi = w + 1 < Kw ? src[1] : 0;
      r[t] = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
  }
}

// Coalesced layout (r[t] = piece lane % 8 of row 8t + lane / 8) -> MFMA layout (r[q] = piece
// h * half / 2 + q of row lane % 32), pieces outside [qlo, qhi) zero.
__device__ __forceinline__ void to_mfma_layout(uint4* tile, int lane, int half, int qlo, int qhi, uint4 (&r)[4]) {
  const int pp = lane & 7;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int row = 8 * t + (lane >> 3);
    tile[row * 8 + (pp ^ (row & 7))] = r[t];
  }
  const int row = lane & 31, c0 = (lane >> 5) * (half >> 1);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q >= qlo && q < qhi) r[q] = tile[row * 8 + (((c0 + q) & 7) ^ (row & 7))];
    else r[q] = make_uint4(0, 0, 0, 0);
  }
}

// The same pieces of an im2col row: word w sits at the pixel's base + tab[w], the offset of
// its tap and channel word (a table the workgroup builds once in LDS).  With an even number
// of channel words per pixel a piece never straddles two taps and is one 16-byte load.
__device__ __forceinline__ void load_im2col(const uint64_t* base, int w0, const MfmaParams& p, const int* tab,
                                            int qlo, int qhi, uint4 (&r)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int w = w0 + 2 * q;
    r[q] = make_uint4(0, 0, 0, 0);
    if (q < qlo || q >= qhi) continue;
    if ((p.Cw & 1) == 0) {
      if (w < p.Kw) r[q] = *(const uint4*)(base + tab[w]);
    } else {
      const uint64_t lo = w < p.Kw ? base[tab[w]] : 0;
      const uint64_t hi = w + 1 < p.Kw ? base[tab[w + 1]] : 0;
      r[q] = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
  }
}

__device__ __forceinline__ int popcount_row(const uint4 (&r)[4]) {
  int pc = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    pc += __builtin_popcount(r[q].x) + __builtin_popcount(r[q].y) + __builtin_popcount(r[q].z) +
          __builtin_popcount(r[q].w);
  return pc;
}

__device__ __forceinline__ uint32_t dword_of(const uint4& v, int d) {
  return d == 0 ? v.x : (d == 1 ? v.y : (d == 2 ? v.z : v.w));
}

__device__ __forceinline__ v4i expand(uint32_t w, int s) {
  v4i e;
#pragma unroll
  for (int j = 0; j < 4; ++j) e[j] = (int)((w >> (4 * s + j)) & 0x01010101u);
  return e;
}

// The FP4 form (v_mfma_scale_f32_32x32x64_f8f6f4 with both operands E2M1): an element is a
// nibble, and the E2M1 codes 0, 1, 2, 3, 4 are the values 0, 0.5, 1, 1.5, 2.  A bit left where it
// stands in its nibble is therefore worth 0.5, 1 or 2 (the nibble's top bit is the sign and
// carries no value), and the E8M0 block scale of the instruction, one per lane and MFMA,
// brings every product back to 1: one MFMA takes one nibble plane n of four dwords,
//   n = 0: w & 0x11111111, scale 2     n = 1: w & 0x22222222, scale 1
//   n = 2: w & 0x44444444, scale 1/2   n = 3: (w >> 3) & 0x11111111, scale 2
// on both operands (five VALU instructions per dword and operand instead of the seven of
// shifting every plane down to bit 0; the four MFMAs of a 16-byte piece are K = 4 x 64 as
// before).  Products and fp32 sums are exact integers below 2^24.  A k-bit operand (planes
// p = 0, 1 of a quantised value q) has to sit at the bottom of the nibble, where the codes
// 0..3 are q/2: its planes are shifted down and keep the scale of 2, the 1-bit operand beside
// it still takes the cheap form.  (Checked on the hardware against a CPU count before use,
// like the int8 layout.)
__device__ __forceinline__ v8i plane4(const uint4& v, int n) {
  v8i e;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t w = dword_of(v, s);
    e[s] = (int)(n == 3 ? (w >> 3) & 0x11111111u : w & (0x11111111u << n));
  }
#pragma unroll
  for (int s = 4; s < 8; ++s) e[s] = 0;
  return e;
}
// nibble plane n of plane pl of a k-bit value, at nibble bit pl
__device__ __forceinline__ v8i plane4_low(const uint4& v, int n, int pl) {
  v8i e;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t w = dword_of(v, s);
    const int sh = n - pl;
    e[s] = (int)((sh >= 0 ? (w >> sh) : (w << -sh)) & (0x11111111u << pl));
  }
#pragma unroll
  for (int s = 4; s < 8; ++s) e[s] = 0;
  return e;
}
__device__ __forceinline__ v8i or8(v8i a, v8i b) {
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] |= b[s];
  return a;
}

// Plane pl of a k-bit value: the same bits as expand(), shifted to bit pl of every byte.
__device__ __forceinline__ v4i expand_plane(uint32_t w, int s, int pl, v4i e) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int sh = 4 * s + j - pl;  // (w >> (4s + j)) << pl
    const uint32_t x = sh >= 0 ? (w >> sh) : (w << -sh);
    e[j] |= (int)(x & (0x01010101u << pl));
  }
  return e;
}

// One macro step of a wave's tile: load the pieces, count their ones (XNOR form only),
// expand and multiply.  PL bit planes make up the A operand.
template <int TM, int TN, int PL, bool XNOR, bool CONV, bool F4, bool ALL>
__device__ __forceinline__ void macro_step(int m0, int n0, const uint64_t* (&brow)[TN], int mac, int half,
                                           bool whole, int qlo, int qhi, const MfmaParams& p,
                                           const int* tab, uint4* tile, int lane,
                                           typename AccOf<F4>::type (&acc)[TM][TN], int (&pa)[TM],
                                           int (&pb)[TN]) {
  uint4 ra[TM][PL][4], rb[TN][4];
  // every block's loads first, then the blocks through the tile one after the other
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int pl = 0; pl < PL; ++pl)
      load_rows_coalesced(p.A, p.lda, m0 + 32 * i, p.M, PL, pl, mac, p.Kw, whole, lane, ra[i][pl]);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    if (CONV) load_im2col(brow[j], mac * 16 + (lane >> 5) * half, p, tab, qlo, qhi, rb[j]);
    else load_rows_coalesced(p.B, p.ldb, n0 + 32 * j, p.N, 1, 0, mac, p.Kw, whole, lane, rb[j]);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) to_mfma_layout(tile, lane, half, qlo, qhi, ra[i][pl]);
  if (!CONV) {
#pragma unroll
    for (int j = 0; j < TN; ++j) to_mfma_layout(tile, lane, half, qlo, qhi, rb[j]);
  }
  if (XNOR) {
#pragma unroll
    for (int i = 0; i < TM; ++i) pa[i] += popcount_row(ra[i][0]);
#pragma unroll
    for (int j = 0; j < TN; ++j) pb[j] += popcount_row(rb[j]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (!ALL && (q < qlo || q >= qhi)) continue;
    if constexpr (F4) {
      // one MFMA per nibble plane n of the piece's four dwords (see plane4)
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        v8i ea[TM], eb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          if constexpr (PL == 1) {
            ea[i] = plane4(ra[i][0][q], n);
          } else {
            ea[i] = plane4_low(ra[i][0][q], n, 0);
#pragma unroll
            for (int pl = 1; pl < PL; ++pl) ea[i] = or8(ea[i], plane4_low(ra[i][pl][q], n, pl));
          }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) eb[j] = plane4(rb[j][q], n);
        // plane 1 holds 1.0 and plane 2 holds 2.0 where planes 0 and 3 hold 0.5
        const int sb = n == 1 ? 127 : (n == 2 ? 126 : 128);
        const int sa = PL == 1 ? sb : 128;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ea[i], eb[j], acc[i][j], 4, 4, 0, sa, 0, sb);
      }
    } else {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          v4i ea[TM], eb[TN];
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            ea[i] = expand(dword_of(ra[i][0][q], d), s);
#pragma unroll
            for (int pl = 1; pl < PL; ++pl) ea[i] = expand_plane(dword_of(ra[i][pl][q], d), s, pl, ea[i]);
          }
#pragma unroll
          for (int j = 0; j < TN; ++j) eb[j] = expand(dword_of(rb[j][q], d), s);
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ea[i], eb[j], acc[i][j], 0, 0, 0);
        }
      }
    }
  }
}

template <int TM, int TN, int PL, bool XNOR, bool CONV, bool F4>
__global__ void __launch_bounds__(512)
gemm_mfma_kernel(const MfmaParams p) {
  extern __shared__ int red[];  // [TM * TN * 16][64] partial results when K is split
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int S = blockDim.x >> 6;
  const int r = lane & 31, h = lane >> 5;
  const int tile_n = blockIdx.x % p.tiles_n, tile_m = blockIdx.x / p.tiles_n;
  const int m0 = tile_m * (32 * TM), n0 = tile_n * (32 * TN);
  // LDS: a 4 KiB transposition tile per wave; once the main loop is over the same memory holds
  // the partial results of a K split; behind both, the convolution's table of im2col offsets
  uint4* tile = (uint4*)red + wave * 256;
  const int red_ints = S > 1 ? TM * TN * 16 * 64 : 0;
  int* tab = red + (S * 1024 > red_ints ? S * 1024 : red_ints);
  // ... and the per-row constants of the epilogue (a convolution's alpha, the plane form's row
  // sums), fetched once here instead of once per stored value; the per-column alpha of the
  // GEMM sits in a register per column block
  int* rowk = tab + (CONV ? p.Kw : 0);
  float aln[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
    aln[j] = (XNOR && !CONV && p.alpha) ? p.alpha[min(n0 + 32 * j + (lane & 31), p.N - 1)] : 1.0f;
  float thn[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
    thn[j] = (XNOR && !CONV && p.C_bits && p.thr) ? p.thr[min(n0 + 32 * j + (lane & 31), p.N - 1)] : 0.0f;
  if (wave == 0 && (CONV || !XNOR)) {
    for (int i = lane; i < 32 * TM; i += 64) {
      const int m = min(m0 + i, p.M - 1);
      rowk[i] = !XNOR ? p.rowsum[m] : (p.alpha ? __float_as_int(p.alpha[m]) : __float_as_int(1.0f));
    }
  }
  if (CONV) {
    for (int w = threadIdx.x; w < p.Kw; w += blockDim.x) {
      const uint32_t tap = fast_div((uint32_t)w, p.div_cw);
      const uint32_t kh = fast_div(tap, p.div_kw);
      tab[w] = (int)((kh * (uint32_t)p.Wpp + (tap - kh * (uint32_t)p.KWid)) * (uint32_t)p.Cw +
                     ((uint32_t)w - tap * (uint32_t)p.Cw));
    }
    __syncthreads();
  }

  // rows past the matrix repeat its last row; their results are never stored
  // (plane pl of row m is row m * PL + pl of A; the row addresses are formed per load)
  const uint64_t* brow[TN];
  uint32_t pix_img[TN], pix_rem[TN];  // convolution: image and pixel within it of column n
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = min(n0 + 32 * j + r, p.N - 1);
    if (CONV) {
      pix_img[j] = fast_div((uint32_t)n, p.div_howo);
      pix_rem[j] = (uint32_t)n - pix_img[j] * (uint32_t)p.HoWo;
      const uint32_t ho = fast_div(pix_rem[j], p.div_wo);
      const uint32_t wo = pix_rem[j] - ho * (uint32_t)p.Wo;
      brow[j] = p.B + (((int64_t)pix_img[j] * p.Hp + ho * p.stride) * p.Wpp + wo * p.stride) * p.Cw;
    } else {
      pix_img[j] = pix_rem[j] = 0;
      brow[j] = p.B + (int64_t)n * p.ldb;
    }
  }

  typename AccOf<F4>::type sum[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) sum[i][j][e] = 0;
  int pa[TM], pb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) pa[i] = 0;
#pragma unroll
  for (int j = 0; j < TN; ++j) pb[j] = 0;

  // this wave's piece steps [ps0, ps1); step ps is piece ps % 4 of macro step ps / 4
  const int ps0 = (int)((int64_t)wave * p.nsteps / S), ps1 = (int)((int64_t)(wave + 1) * p.nsteps / S);
  const int last_mac = (p.nsteps - 1) >> 2;
  for (int mac = ps0 >> 2; mac <= ((ps1 - 1) >> 2) && ps0 < ps1; ++mac) {
    const int qlo = max(ps0 - 4 * mac, 0), qhi = min(ps1 - 4 * mac, 4);
    const bool whole = mac < last_mac || (p.tail_half == 8 && (p.Kw & 15) == 0);  // wave-uniform
    const int half = mac < last_mac ? 8 : p.tail_half;
    // the common case (a whole macro step, all of it this wave's) without the piece tests
    if (whole && qlo == 0 && qhi == 4)
      macro_step<TM, TN, PL, XNOR, CONV, F4, true>(m0, n0, brow, mac, 8, true, 0, 4, p, tab, tile, lane, sum, pa,
                                                   pb);
    else
      macro_step<TM, TN, PL, XNOR, CONV, F4, false>(m0, n0, brow, mac, half, whole, qlo, qhi, p, tab, tile, lane,
                                                    sum, pa, pb);
  }

  // the sums as integers (the fp32 sums of the FP4 form are exact integers)
  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = (int)sum[i][j][e];

  // ---- this wave's share of C - K:  4 * and_count - 2 * pc(A row) - 2 * pc(B row), all over
  // the wave's K range.  A lane holds the counts of row / column r for its k-half; the other
  // half sits 32 lanes away.  (The plane form keeps the plain sums: its row term is the
  // given rowsum, applied once at the end.)
  if (XNOR) {
    // (waited for here, not before each of the stores below, which would wait for the stores before it as well)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(aln[j]), "+v"(thn[j]));
#pragma unroll
    for (int i = 0; i < TM; ++i) pa[i] += __shfl_xor(pa[i], 32);
#pragma unroll
    for (int j = 0; j < TN; ++j) pb[j] += __shfl_xor(pb[j], 32);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row_in_block = 8 * (v / 4) + 4 * h + (v % 4);
        const int pai = __shfl(pa[i], row_in_block);
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j][v] = 4 * acc[i][j][v] - 2 * pai - 2 * pb[j];
      }
  }

  auto store = [&](int i, int j, int v, int t) {  // called by whole waves only
    const int mi = 32 * i + 8 * (v / 4) + 4 * h + (v % 4);
    const int m = m0 + mi;
    const int n = n0 + 32 * j + r;
    if (!XNOR) {
      const int sv = 2 * t - rowk[mi];
      if (m < p.M && n < p.N) {
        const int64_t idx = (int64_t)m * p.ldc + n;
        if (p.C_i32) p.C_i32[idx] = sv;
        if (p.C_f32) p.C_f32[idx] = (float)sv / p.levels;
      }
      return;
    }
    const int dot = p.Kreal + t;
    if (CONV) {
      const float al = __int_as_float(rowk[mi]);
      if (m < p.M && n < p.N) {  // NCHW: plane m of the pixel's image
        const int64_t idx = ((int64_t)pix_img[j] * p.M + m) * p.HoWo + pix_rem[j];
        if (p.C_i32) p.C_i32[idx] = dot;
        else p.C_f32[idx] = al * (float)dot;
      }
      return;
    }
    const float al = (TN > 1 && j == 1) ? aln[TN - 1] : aln[0];
    if (p.C_bits) {
      // the 64-lane mask of (scaled result >= 0): its low half is 32 columns of row m as seen
      // by lanes 0..31, its high half the same columns of the row four below
      const float th = (TN > 1 && j == 1) ? thn[TN - 1] : thn[0];
      const uint64_t mask = __ballot(n < p.N && al * (float)dot >= th);
      if (r == 0 && m < p.M)
        p.C_bits[(int64_t)m * (2 * p.ldc) + (n >> 5)] = h ? (uint32_t)(mask >> 32) : (uint32_t)mask;
    } else if (m < p.M && n < p.N) {
      const int64_t idx = (int64_t)m * p.ldc + n;
      if (p.C_i32) p.C_i32[idx] = p.as_count ? (dot + p.Kreal) >> 1 : dot;
      else p.C_f32[idx] = al * (float)dot;
    }
  };

  if (S == 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) store(i, j, v, acc[i][j][v]);
    return;
  }

  // ---- K split: wave 0 writes its share, the others add theirs, then the entries are
  // finished and stored by the waves in turn
  __syncthreads();  // every wave is done with its transposition tile (same memory)
  if (wave == 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[((i * TN + j) * 16 + v) * 64 + lane] = acc[i][j][v];
  }
  __syncthreads();
  if (wave != 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) atomicAdd(&red[((i * TN + j) * 16 + v) * 64 + lane], acc[i][j][v]);
  }
  __syncthreads();
  // (four entries per trip: their LDS reads go out together)
  for (int e0 = wave; e0 < TM * TN * 16; e0 += 4 * S) {
    int t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = red[min(e0 + k * S, TM * TN * 16 - 1) * 64 + lane];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = e0 + k * S;
      if (e < TM * TN * 16) store((e >> 4) / TN, (e >> 4) % TN, e & 15, t[k]);
    }
  }
}

}  // namespace

// 0 = automatic, 1 = xor/popcount kernel, 2 = int8 matrix cores, 3 = FP4 matrix cores (either
// kernel), 4 = FP4 on this file's kernel, 5 = FP4 on the 64 x 64 per wave kernel whatever the size
int gemm_engine = 0;
int gemm_mfma_ksplit = 0;
int gemm_mfma_tile = 0;  // 1 forces the 32 x 32 per wave variant, 2 the 64 x 64 one

namespace {

template <int TM, int TN, int PL, bool XNOR, bool CONV>
void launch_engine(const MfmaParams& p, bool f4, int64_t tiles, int S, size_t lds, hipStream_t s) {
  note_kernel("gemm_mfma_kernel<%d,%d,%d,%s,%s,%s> grid %lld x %d", TM, TN, PL, XNOR ? "xnor" : "planes",
              CONV ? "conv" : "gemm", f4 ? "fp4" : "int8", (long long)tiles, 64 * S);
  if (f4)
    launch_kernel((gemm_mfma_kernel<TM, TN, PL, XNOR, CONV, true>), dim3((unsigned)tiles), dim3(64 * S), lds,
                       s, p);
  else
    launch_kernel((gemm_mfma_kernel<TM, TN, PL, XNOR, CONV, false>), dim3((unsigned)tiles), dim3(64 * S), lds,
                       s, p);
}

// FP4 unless told otherwise or the sums could leave the exact range of fp32
bool use_fp4(int64_t max_sum) { return gemm_engine != 2 && max_sum < ((int64_t)1 << 24); }

void set_k_steps(MfmaParams& p, int K) {
  p.Kw = (int)words_for(K);
  p.Kreal = K;
  const int span = p.Kw - (int)((p.Kw - 1) / 16) * 16;    // words of the last macro step, 1..16
  p.tail_half = (int)ceil_div(ceil_div(span, 2), 2) * 2;  // per half-wave, whole pieces
  p.nsteps = (int)((p.Kw - 1) / 16) * 4 + p.tail_half / 2;
}

// transposition tiles (4 KiB per wave) and, in the same memory, the partial results of a K
// split (16 x 64 ints per 32 x 32 block of the wave tile)
size_t lds_bytes(int S, int blocks) {
  const size_t tiles = (size_t)S * 4096, red = S > 1 ? (size_t)blocks * 16 * 64 * 4 : 0;
  return (tiles > red ? tiles : red) + 64 * 4;  // + the table of row constants (up to 64 rows)
}

int choose_split(int64_t tiles, int nsteps) {
  int S = gemm_mfma_ksplit;
  if (S <= 0) {
    S = (int)ceil_div(2048, tiles);  // about two waves per SIMD
    // a third where every wave still keeps a long run of K (12 piece steps = 3072 bits):
    // 256 x 4096 x 9216 10.7 against 12.1 us; shorter runs lose to the reduction
    const int S3 = (int)(3072 / tiles);
    if (S3 > S && S3 <= 8 && nsteps / S3 >= 12) S = S3;
  }
  if (S > 8) S = 8;
  if (S > nsteps) S = nsteps;
  return S < 1 ? 1 : S;
}

}  // namespace

bool launch_xnor_gemm_dwords(const uint32_t* A, int64_t lda_dw, const uint32_t* B, int64_t ldb_dw, int M, int N, int K,
                             int32_t* C, int64_t ldc, hipStream_t s, hipError_t* err) {
  const int dwords = (int)ceil_div(K, 32);
  return launch_gemm_small(A, lda_dw * 4, B, ldb_dw * 4, M, N, K, dwords, nullptr, C, nullptr, nullptr, nullptr, ldc, false, s,
                           err) ||
         launch_gemm_block(A, lda_dw * 4, B, ldb_dw * 4, M, N, K, dwords, nullptr, C, nullptr, ldc, false, s, err) ||
         launch_gemm_fp4(A, lda_dw * 4, 1, nullptr, B, ldb_dw * 4, M, N, K, dwords, nullptr, C, nullptr, nullptr, nullptr, ldc,
                         false, s, err);
}

bool launch_xnor_gemm_mfma(const uint64_t* A, int64_t lda_w, const uint64_t* B, int64_t ldb_w, int M,
                           int N, int K, const float* alpha_n, int32_t* C_i32, float* C_f32,
                           uint64_t* C_bits, const float* thr_n, int64_t ldc, hipStream_t s, hipError_t* err,
                           bool as_count) {
  if (gemm_engine == 1) return false;
  if (launch_gemm_small(A, lda_w * 8, B, ldb_w * 8, M, N, K, 2 * (int)words_for(K), alpha_n, C_i32, C_f32, C_bits, thr_n, ldc,
                        as_count, s, err))
    return true;
  if (!C_bits && launch_gemm_block(A, lda_w * 8, B, ldb_w * 8, M, N, K, 2 * (int)words_for(K), alpha_n, C_i32, C_f32, ldc, as_count, s, err))
    return true;
  if (launch_gemm_fp4(A, lda_w * 8, 1, nullptr, B, ldb_w * 8, M, N, K, 2 * (int)words_for(K), alpha_n, C_i32, C_f32, C_bits, thr_n, ldc, as_count,
                      s, err))
    return true;
  MfmaParams p;
  p.A = A;
  p.B = B;
  p.lda = lda_w;
  p.ldb = ldb_w;
  p.M = M;
  p.N = N;
  set_k_steps(p, K);
  p.alpha = alpha_n;
  p.rowsum = nullptr;
  p.levels = 1.0f;
  p.C_i32 = C_i32;
  p.C_f32 = C_f32;
  p.C_bits = (uint32_t*)C_bits;
  p.thr = thr_n;
  p.as_count = as_count ? 1 : 0;
  p.ldc = ldc;
  // 64 x 64 per wave; 32 x 32 while that grid has at most four tiles per CU (measured:
  // 256 x 4096 x 4096 8.0 against 10.1 us, 2048 x 2048 x 1024 9.7 against 12.6 us,
  // 2048 x 2048 x 4096 18.7 against 19.5 us; 4096 x 2048 x 4096 28.7 against 25.5 us)
  const bool small = gemm_mfma_tile ? gemm_mfma_tile == 1 : ceil_div(M, 64) * ceil_div(N, 64) <= 1024;
  const int T = small ? 1 : 2;
  const int tiles_m = (int)ceil_div(M, 32 * T);
  // (packed output: both 32-bit halves of the last word of a row get a block that writes them)
  p.tiles_n = C_bits ? (int)(ceil_div(N, 64) * (2 / T)) : (int)ceil_div(N, 32 * T);
  const int64_t tiles = (int64_t)tiles_m * p.tiles_n;
  const int S = choose_split(tiles, p.nsteps);
  const size_t lds = lds_bytes(S, T * T);
  const bool f4 = use_fp4(K);
  if (small)
    launch_engine<1, 1, 1, true, false>(p, f4, tiles, S, lds, s);
  else
    launch_engine<2, 2, 1, true, false>(p, f4, tiles, S, lds, s);
  *err = launch_error();
  return true;
}

// S = 2 * sum_k q[m][k] * wb[n][k] - rowsum[m] with q assembled from `bits` planes (1 or 2).
bool launch_plane_gemm_mfma(const uint64_t* planes_rows, int64_t lda_w, int bits, const int32_t* rowsum,
                            const uint64_t* Wb, int64_t ldb_w, int M, int N, int K, int32_t* S_out,
                            float* out_f32, int64_t ldo, hipStream_t s, hipError_t* err) {
  if (gemm_engine == 1 || bits > 2) return false;
  if (launch_gemm_fp4(planes_rows, lda_w * 8, bits, rowsum, Wb, ldb_w * 8, M, N, K, 2 * (int)words_for(K), nullptr, S_out, out_f32, nullptr, nullptr,
                      ldo, false, s, err))
    return true;
  MfmaParams p;
  p.A = planes_rows;
  p.B = Wb;
  p.lda = lda_w;
  p.ldb = ldb_w;
  p.M = M;
  p.N = N;
  set_k_steps(p, K);
  p.alpha = nullptr;
  p.rowsum = rowsum;
  p.levels = (float)((1u << bits) - 1u);
  p.C_i32 = S_out;
  p.C_f32 = out_f32;
  p.C_bits = nullptr;
  p.thr = nullptr;
  p.as_count = 0;
  p.ldc = ldo;
  // 32 rows x 64 columns per wave: the two planes of a row double the A registers
  const int tiles_m = (int)ceil_div(M, 32);
  p.tiles_n = (int)ceil_div(N, 64);
  const int64_t tiles = (int64_t)tiles_m * p.tiles_n;
  const int S = choose_split(tiles, p.nsteps);
  const size_t lds = lds_bytes(S, 2);
  const bool f4 = use_fp4((int64_t)K * ((1 << bits) - 1));
  if (bits == 1)
    launch_engine<1, 2, 1, false, false>(p, f4, tiles, S, lds, s);
  else
    launch_engine<1, 2, 2, false, false>(p, f4, tiles, S, lds, s);
  *err = launch_error();
  return true;
}

static inline int64_t Wpp_host(int W, int pad) { return (int64_t)W + 2 * pad; }

// The convolution on the matrix cores; Xp, Wp as for launch_binary_conv2d.
bool launch_conv_mfma(const uint64_t* Xp, int Nimg, int C, int H, int W, const uint64_t* Wp, int O, int KH,
                      int KW, int stride, int pad, const float* alpha, int32_t* out_i32, float* out_f32,
                      hipStream_t s, hipError_t* err) {
  if (gemm_engine == 1) return false;
  const int Ho = (H + 2 * pad - KH) / stride + 1;
  const int Wo = (W + 2 * pad - KW) / stride + 1;
  const int Cw = (int)words_for(C);
  const int kwords = KH * KW * Cw;
  const int64_t ld_words = conv_weight_row_words(kwords);
  const int64_t P = (int64_t)Nimg * Ho * Wo;
  if ((ld_words & 1) || ((uintptr_t)Wp & 15) || ((uintptr_t)Xp & 15) || P >= ((int64_t)1 << 31)) return false;
  if ((int64_t)KH * Wpp_host(W, pad) * Cw >= ((int64_t)1 << 31)) return false;
  MfmaParams p;
  p.A = Wp;
  p.B = Xp;
  p.lda = ld_words;
  p.ldb = 0;
  p.M = O;
  p.N = (int)P;
  set_k_steps(p, 64 * kwords);
  p.Kreal = C * KH * KW;
  p.alpha = alpha;
  p.rowsum = nullptr;
  p.levels = 1.0f;
  p.C_i32 = out_i32;
  p.C_f32 = out_f32;
  p.C_bits = nullptr;
  p.thr = nullptr;
  p.as_count = 0;
  p.ldc = 0;
  p.HoWo = Ho * Wo;
  p.Wo = Wo;
  p.Hp = H + 2 * pad;
  p.Wpp = W + 2 * pad;
  p.Cw = Cw;
  p.stride = stride;
  p.KWid = KW;
  p.div_howo = make_fast_div((uint32_t)(Ho * Wo));
  p.div_wo = make_fast_div((uint32_t)Wo);
  p.div_cw = make_fast_div((uint32_t)Cw);
  p.div_kw = make_fast_div((uint32_t)KW);
  // (32 x 32 tiles further up than in the GEMM: 15.7 against 19.0 us at 784 tiles of 64 x 64)
  const bool small = gemm_mfma_tile ? gemm_mfma_tile == 1 : ceil_div(O, 64) * ceil_div(P, 64) < 2048;
  const int T = small ? 1 : 2;
  const int tiles_m = (int)ceil_div(O, 32 * T);
  p.tiles_n = (int)ceil_div(P, 32 * T);
  const int64_t tiles = (int64_t)tiles_m * p.tiles_n;
  if (tiles >= ((int64_t)1 << 31)) return false;
  const int S = choose_split(tiles, p.nsteps);
  const size_t lds = lds_bytes(S, T * T) + (size_t)kwords * 4;
  if (lds > 64 * 1024) return false;
  const bool f4 = use_fp4(64 * (int64_t)kwords);
  if (small)
    launch_engine<1, 1, 1, true, true>(p, f4, tiles, S, lds, s);
  else
    launch_engine<2, 2, 1, true, true>(p, f4, tiles, S, lds, s);
  *err = launch_error();
  return true;
}

}  // namespace bmx
