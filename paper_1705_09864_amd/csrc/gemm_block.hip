// xnor GEMM on the FP4 matrix cores for problems of many tiles: operand rows staged once per workgroup.
// Paper: Sec. 2.2.1 / Sec. 2.2.2 (Eq. 2): C[m][n] = K - 2 * popcount(A[m] xor B[n]).
//
// Arithmetic as in gemm_fp4.hip: K - 2 pc(a) - 2 pc(b) + 4 * sum_k a * b, a bit stays where it stands
// in its nibble and the MFMA's block scale makes it worth 1; but every fourth value, whose bit is the nibble's sign, is
// multiplied as the sign itself and needs no popcount: sum_k s(a) s(b).  An operand takes 4 instructions a word and plane
// then and not 5 (8192^3, all bits clear, where the power does not bound it, 152.4 -> 147.8 us; random bits, where it does,
// 182.4 -> 178.2 in the first millisecond, level once the clock has settled: 376 -> 361 thousand clocks, at a lower rate; 69 x 64 x 19 x 21 -> 406 in three packed layers 64.9 -> 64.1; 4531 x 1600 x 4096 16.8 -> 16.4).
//
// There every wave fetches the rows of its own tile, waits for its own reads of a segment before it may request
// the next, and turns all of a segment's bits into operands before it multiplies.  With the chip full that
// leaves the matrix cores half idle: 8192^3 took 202 us, of which its products are 109 at 2.4 GHz.  Here:
//   - Four waves, two by two, share the rows of a workgroup's tile of C: 256 x 128 (128 x 64 per wave, 244
//     registers, two workgroups on a CU) or 128 x 128 (64 x 64 per wave, 146 registers, three).  Rows cross the
//     L2 once per workgroup.  Several workgroups per CU rather than one large one, so that one's results leave
//     while the others multiply: as one of 256 x 256 the same loop was 5 % slower.
//   - Segments of 64 bytes of K go from memory to LDS past the registers, into two stages in turn.  A wave holds
//     segment s in registers when the barrier in the middle of its products passes; everyone's segment s + 1 has
//     then landed, and s + 2 is requested into the stage of s.  One barrier per segment of 4096 (2048) clocks.
//   - The operands of the next plane of bits are made between the products of this one (sched_barrier: left to
//     itself the compiler makes them all at once, and then multiplies with the vector ALU idle).
//   - Two waves share every block of rows; each counts the bits of half its blocks.
//   - Rows may start on any dword, which is all that loads of 16 bytes need (dword by dword, four times the loads, 4224 x
//     4736 x 1600 took 23.8 us, now 22.8).
//   - The convolution form gathers the im2col rows of 128 (256) pixels from the packed image, 16 bytes at a
//     time (a dword in segments that hold a piece of two runs of an odd number of words), once for 128 (64) filters; where the patches start stands in LDS.  Its results are fp32, int32 or
//     the next convolution's packed image, halo included.
//   (Three and four stages in flight changed nothing, at 8192^3 or with one workgroup per CU: it is issue and, with
//   one wave on a SIMD, the chain of its own instructions that bounds the loop, not the memory behind it.)
// What bounds it, from counters at 8192^3 as 256 x 128: the matrix pipe is busy in 73 % of
// the clocks, a SIMD issues an instruction in 75 % of them (4.6 of the vector ALU for every MFMA), a wave waits for data or a barrier
// in 13 % of its time; and the clock stands at 2.0 to 2.15 GHz under that load, by the power that the products take: the same launch on
// zeros is a fifth faster.  The same launch back to back takes 178 us in the first millisecond, 244
// in the fourth, 181 after 15 and 171 to 174 from 30 on; the clocks that it needs stay 361 thousand.
// Measured, us a call, gemm_fp4.hip / here: 8192^3 202 / 173, 8192 x 8192 x 1024 75 / 50, 4096^3 33 / 28, 3008 x 1471
// x 5184 25.6 / 23.1.  Convolutions of packed
// images: 11 x 320 x 49 x 49 -> 334, 3 x 3, 26.3 / 21.2, 40 x 192 x 28 x 28 -> 128, 5 x 5, 21.6 / 16.0; as packed bits, a channel pack of
// the fp32 result behind them before: 26411 pixels, 334 filters, 45 words 33.2 / 20.1, 13500, 332, 72 24.0 / 17.6.
#include <algorithm>
#include <type_traits>

#include "bmx_internal.h"
#include "halo.h"
#include "row_pieces.h"

namespace bmx {

namespace block {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f_alias __attribute__((ext_vector_type(4), may_alias));
typedef float f_alias __attribute__((may_alias));
typedef uint32_t u_alias __attribute__((may_alias));

struct BlockParams {
  const char* A;
  const char* B;
  uint32_t lda, ldb;  // bytes from row to row
  int M, N;
  int Kd, nseg;  // data dwords per row, segments of 16
  int tiles_m, tiles_n, tiles_per_xcd;
  int band, per_band, last_band, last_rows;
  FastDiv div_per_band, div_band, div_last;
  const float* alpha;                 // per column, or null
  float row_const, row_mul, tot_mul;  // result = row_const + row_mul * (pc(a) + pc(b)) + tot_mul * sum
  void* C;
  int ldc, nt;
  // Convolution form (Sec. 3.1): A is the filter matrix, column n of B the im2col row of output pixel n in the halo-padded
  // packed image B: runs of `run` words, row_bytes from run to run.  alpha and thr are per row m.  C is NCHW, or (packed bits)
  // the next convolution's image of oHp x oWp x oCw words with a halo of opad.
  int HoWo, Wo, Ho, Hp, Wpp, Cw, stride, Nimg;
  uint32_t run, row_bytes;
  FastDiv div_howo, div_wo, div_run, div_two_runs;
  const float* thr;
  int opad, oHp, oWp, oCw;
};

constexpr int kF32 = 0, kI32 = 1, kBits = 2;

// Plane n of four words as an operand: bit 4 i + n of a dword in nibble i.  Planes 0 to 2 as they stand, worth 0.5, 1 or 2 (a
// clear bit nothing); plane 3, whose bit is the nibble's sign, as 1 with that sign: one instruction a dword like the others, where
// a bit shifted down to 0.5 would take two.
__device__ __forceinline__ v4i plane(const uint4& w, int n) {
  const uint32_t m = 0x11111111u << n;
  if (n == 3) {
    // (v & 8s | 2s, named as the one instruction that it is: from the operators the compiler makes two, as if the constant could not
    // stay in a register; written as asm it would not know to keep two wait states between it and the MFMA that reads it)
    auto sign = [](uint32_t v) { return (int)__builtin_amdgcn_bitop3_b32(v, 0x88888888u, 0x22222222u, 0xf0 & 0xcc | 0xaa); };
    return v4i{sign(w.x), sign(w.y), sign(w.z), sign(w.w)};
  }
  return v4i{(int)(w.x & m), (int)(w.y & m), (int)(w.z & m), (int)(w.w & m)};
}

__device__ __forceinline__ v8i wide(const v4i& e) { return v8i{e[0], e[1], e[2], e[3], 0, 0, 0, 0}; }

// acc + popcount of planes 0 to 2 of four words
__device__ __forceinline__ int add_popcount4(int acc, const uint4& w) {
  auto add = [&](uint32_t v) { asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"(v & 0x77777777u)); };
  add(w.x), add(w.y), add(w.z), add(w.w);
  return acc;
}

// How many bytes the operands' addresses are lower than the operands (see the loads).
constexpr uint32_t lowered(bool conv, int lw) { return conv || lw == 4 ? 0u : 16u; }

// WM x 4 / WM waves of TM x TN blocks of 32 x 32 each.  A stage holds blocks of 32 rows x 64 bytes, A's, then B's, in the
// layout of gemm_fp4.hip: piece c of row r of a block at 16-byte place 64 (r / 16) + 4 (r % 16) + (c xor ((r / 2) & 3)).
// LW: bytes a lane fetches per load: 16, and 4 where rows are less than that and not that far apart, or (convolution form) for the
// patches in segments that hold a piece of two runs of an odd number of words.
template <int WM, int TM, int TN, int OUT, int LW, bool CONV>
__global__ void __launch_bounds__(256, TM * TN >= 8 ? 2 : 3)
gemm_fp4_kernel(const BlockParams p) {
  extern __shared__ uint4 lds[];
  constexpr int WN = 4 / WM, NBA = WM * TM, NB = NBA + WN * TN;
  constexpr int HA = NBA / 2, HB = (NB - NBA) / 2;  // half blocks of A and of B that a wave fetches
  constexpr int LWA = CONV ? 16 : LW;
  constexpr int kStage = NB * 128;  // uint4 per stage
  asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.lda), "s"(p.ldb), "s"(p.M), "s"(p.N), "s"(p.Kd), "s"(p.nseg), "s"(p.tiles_m),
               "s"(p.tiles_n), "s"(p.tiles_per_xcd), "s"(p.band), "s"(p.per_band), "s"(p.last_band), "s"(p.last_rows),
               "s"(p.div_per_band.mul), "s"(p.div_per_band.sh1), "s"(p.div_per_band.sh2), "s"(p.div_band.mul),
               "s"(p.div_band.sh1), "s"(p.div_band.sh2), "s"(p.div_last.mul), "s"(p.div_last.sh1), "s"(p.div_last.sh2));
  if constexpr (CONV)
    asm volatile("" ::"s"(p.HoWo), "s"(p.Wo), "s"(p.Hp), "s"(p.Wpp), "s"(p.Cw), "s"(p.stride), "s"(p.run), "s"(p.row_bytes),
                 "s"(p.div_howo.mul), "s"(p.div_howo.sh1), "s"(p.div_howo.sh2), "s"(p.div_wo.mul), "s"(p.div_wo.sh1),
                 "s"(p.div_wo.sh2), "s"(p.div_run.mul), "s"(p.div_run.sh1), "s"(p.div_run.sh2));
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lin = (int)(blockIdx.x & 7) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  if (lin >= p.tiles_m * p.tiles_n) return;
  const int bnd = (int)fast_div((uint32_t)lin, p.div_per_band), within = lin - bnd * p.per_band;
  const bool lastb = bnd == p.last_band;
  const int tile_n = (int)fast_div((uint32_t)within, lastb ? p.div_last : p.div_band);
  const int tile_m = bnd * p.band + (within - tile_n * (lastb ? p.last_rows : p.band));
  const int m0 = tile_m * (32 * NBA), n0 = tile_n * (32 * (NB - NBA));

  // ---- loads.  A half block (16 rows) is one load of 16 bytes a lane or four of 4 bytes.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  const bool tail = (p.Kd & 15) != 0;
  // What differs from lane to lane: LW 16: row lane / 4 of the half block and a piece; LW 4: row 4 u + lane / 16 in load u and
  // dword d[u & 1] of the segment.  over: how far that lies behind the row's end in the last segment.
  const int piece16 = (lane & 3) ^ ((lane >> 3) & 3);
  const int dw4[2] = {4 * (((lane & 15) >> 2) ^ (lane >> 5)) + (lane & 3), 4 * (((lane & 15) >> 2) ^ (2 + (lane >> 5))) + (lane & 3)};
  const int last0 = 16 * (p.nseg - 1) - (p.Kd - 1);
  // (Rows of a product: A and B are 16 bytes lower than the operands and all offsets 16 more, so that none is negative.  Filters of a
  // convolution are whole pieces.)
  constexpr uint32_t kLower = lowered(CONV, LW);
  const bool part_pieces = !CONV && LW == 16 && p.Kd >= 4;
  const uint32_t sub16 = CONV ? (last0 + 4 * piece16 > 0 ? 16u * piece16 : 0u)
                              : piece_back(p.nseg - 1, piece16, p.Kd);
  const uint32_t sub4[2] = {last0 + dw4[0] > 0 ? 4u * (last0 + dw4[0]) : 0u, last0 + dw4[1] > 0 ? 4u * (last0 + dw4[1]) : 0u};
  // offset of the lane's first load of each half block in segment 0 (LW 4: of its first two loads; the other two are eight rows on)
  uint32_t va[HA][2], vb[CONV ? 1 : HB][2];
  auto offsets = [&](uint32_t (&v)[2], int lw, int row0, uint32_t ld, int rows) {
    if (lw == 16) {
      v[0] = (uint32_t)min(row0 + (lane >> 2), rows - 1) * ld + 16u * piece16 + kLower;
    } else {
      v[0] = (uint32_t)(row0 + (lane >> 4)) * ld + 4u * dw4[0];
      v[1] = (uint32_t)(row0 + 4 + (lane >> 4)) * ld + 4u * dw4[1];
    }
  };
#pragma unroll
  for (int k = 0; k < HA; ++k) offsets(va[k], LWA, m0 + 16 * (wave * HA + k), p.lda, p.M);
  if constexpr (!CONV) {
#pragma unroll
    for (int k = 0; k < HB; ++k) offsets(vb[k], LW, n0 + 16 * (wave * HB + k), p.ldb, p.N);
  }
  // (As asm: the compiler would wait for every load of this kind before every LDS read.  m0 is the load's LDS address;
  // nothing else here uses it.)
  auto load16 = [&](uint32_t to, const char* base, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory");
  };
  auto load4 = [&](uint32_t to, const char* base, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory");
  };
  auto load_rows = [&](uint32_t to, const char* base, const uint32_t (&v)[2], int lw, uint32_t ld, int rows, bool last) {
    if (lw == 16) {
      load16(to, base, v[0] - (last ? sub16 : 0u));
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // (rows past the last repeat it)
        const uint32_t off = min(v[u & 1] + (uint32_t)(u >> 1) * 8u * ld, 4u * dw4[u & 1] + (uint32_t)(rows - 1) * ld);
        load4(to + 256u * u, base, off - (last ? sub4[u & 1] : 0u));
      }
    }
  };
  // convolution form: where the patches of the tile's pixels start in the image (pixels past the last repeat it)
  uint32_t* const patch = (uint32_t*)(lds + 2 * kStage);
  if constexpr (CONV) {
    for (int i = threadIdx.x; i < 32 * (NB - NBA); i += 256) {
      const uint32_t n = (uint32_t)min(n0 + i, p.N - 1);
      const uint32_t img = fast_div(n, p.div_howo), rem = n - img * (uint32_t)p.HoWo;
      const uint32_t ho = fast_div(rem, p.div_wo), wo = rem - ho * (uint32_t)p.Wo;
      patch[i] = (((img * (uint32_t)p.Hp + ho * (uint32_t)p.stride) * (uint32_t)p.Wpp + wo * (uint32_t)p.stride) * (uint32_t)p.Cw) * 8u;
    }
    __syncthreads();
  }
  uint32_t vp[CONV ? HB : 1];
  if constexpr (CONV) {
#pragma unroll
    for (int k = 0; k < HB; ++k) vp[k] = patch[16 * (wave * HB + k) + (lane >> 2)];
  }
  // dword d of a patch
  auto in_patch = [&](uint32_t d) {
    const uint32_t w = d >> 1, run = fast_div(w, p.div_run);
    return run * p.row_bytes + (w - run * p.run) * 8u + (d & 1u) * 4u;
  };
  auto meet = [&](int seg) { return runs_meet(p.run, [&](uint32_t x) { return fast_div(x, p.div_two_runs); }, seg); };
  // Requests segment seg of the wave's half blocks into stage buf.
  auto issue = [&](int seg, int buf) {
    const bool last = tail && seg + 1 == p.nseg;
    const uint32_t to = lds0 + (uint32_t)(buf * kStage) * 16u;
#pragma unroll
    for (int k = 0; k < HA; ++k)
      load_rows(to + 1024u * (uint32_t)(wave * HA + k), p.A + (uint32_t)seg * 64u, va[k], LWA, p.lda, p.M, last);
    const uint32_t tob = to + 2048u * NBA + 1024u * (uint32_t)(wave * HB);
    if constexpr (!CONV) {
#pragma unroll
      for (int k = 0; k < HB; ++k) load_rows(tob + 1024u * k, p.B + (uint32_t)seg * 64u, vb[k], LW, p.ldb, p.N, last);
    } else if (LW == 16 || !meet(seg)) {
      const uint32_t d = 16u * (uint32_t)seg + 4u * piece16;
      const uint32_t at = in_patch(d < (uint32_t)p.Kd ? d : 16u * (uint32_t)seg);
#pragma unroll
      for (int k = 0; k < HB; ++k) load16(tob + 1024u * k, p.B, vp[k] + at);
    } else {
      uint32_t at[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) at[t] = in_patch(min(16u * (uint32_t)seg + dw4[t], (uint32_t)p.Kd - 1u));
#pragma unroll
      for (int k = 0; k < HB; ++k)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          load4(tob + 1024u * k + 256u * u, p.B, patch[16 * (wave * HB + k) + 4 * u + (lane >> 4)] + at[u & 1]);
    }
  };
  // What the loads left behind the row's last dword counts as zero; of a piece that the row ends in (sub16), what stands in front of
  // its last dwords, which the piece before it has.  (In two loops: with the bounds of both asked of every dword 4320 x 7136 x 3157 took
  // 49.6 us and not 48.6.)
  auto zero_tail = [&](int buf) {
    u_alias* const d = (u_alias*)(lds + buf * kStage);
    const int valid = p.Kd & 15, rest = part_pieces ? valid & 3 : 0, part = valid - rest;
    const int front = rest ? 4 - rest : 0, behind = rest ? part + 4 : valid;
    for (int row = threadIdx.x; row < 32 * NB; row += 256) {
      const int base = (row >> 4) * 256 + (row & 15) * 16, x = (row >> 1) & 3;
      for (int k = 0; k < front; ++k) d[base + (((part >> 2) ^ x) << 2) + k] = 0u;
      for (int k = behind; k < 16; ++k) d[base + (((k >> 2) ^ x) << 2) + (k & 3)] = 0u;
    }
  };

  // ---- products.  Waves side by side share blocks; each takes its blocks in an order of its own (block i of the registers is
  // block i xor xa of the wave's) and counts the first half of those that it shares.
  const int wm = WM == 2 ? wave >> 1 : 0, wn = WM == 2 ? wave & 1 : wave;
  constexpr int CA = TM / 2, CB = WM == 2 ? TN / 2 : TN;
  const int xa = (wn & 1) * CA, xb = WM == 2 ? wm * CB : 0;
  int rd[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) rd[g] = (r >> 4) * 64 + (r & 15) * 4 + ((2 * g + h) ^ ((r >> 1) & 3));
  uint4 wa[2][TM], wb[2][TN];
  auto read = [&](int g, int buf) {
#pragma unroll
    for (int j = 0; j < TN; ++j) wb[g][j] = lds[buf * kStage + (NBA + wn * TN + (j ^ xb)) * 128 + rd[g]];
#pragma unroll
    for (int i = 0; i < TM; ++i) wa[g][i] = lds[buf * kStage + (wm * TM + (i ^ xa)) * 128 + rd[g]];
  };
  v16f acc[TM][TN];
  int pa[CA], pb[CB];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
#pragma unroll
  for (int i = 0; i < CA; ++i) pa[i] = 0;
#pragma unroll
  for (int j = 0; j < CB; ++j) pb[j] = 0;
  // The products of group g, a plane of the bits at a time; between them the next plane's operands (after the last
  // plane the other group's first) and the popcounts.
  v4i ea[2][TM], eb[2][TN];
  auto expand = [&](int set, int g, int n, int b) {
    if (b < TN) eb[set][b] = plane(wb[g][b], n);
    else if (b < TN + TM) ea[set][b - TN] = plane(wa[g][b - TN], n);
  };
  auto count = [&](int g, int b) {
    if (b < CB) pb[b] = add_popcount4(pb[b], wb[g][b]);
    else if (b < CB + CA) pa[b - CB] = add_popcount4(pa[b - CB], wa[g][b - CB]);
  };
  auto multiply = [&](int g) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int sc = n == 1 ? 127 : n == 0 ? 128 : 126;  // block scales that make a product worth 1, of signs a quarter
#pragma unroll
      for (int k = 0; k < TM * TN; ++k) {
        const int i = k / TN, j = k % TN;
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wide(ea[n & 1][i]), wide(eb[n & 1][j]), acc[i][j], 4, 4, 0, sc, 0, sc);
        if (n < 3) expand((n + 1) & 1, g, n + 1, k);
        else expand(0, g ^ 1, 0, k);
        if (k == TM * TN - 1) count(g, n);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // (what multiply computes stays where it is: left to itself the compiler moves it behind the barrier)
  auto stay = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));
      asm volatile("" : "+v"(ea[0][i]));
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(eb[0][j]));
#pragma unroll
    for (int i = 0; i < CA; ++i) asm volatile("" : "+v"(pa[i]));
#pragma unroll
    for (int j = 0; j < CB; ++j) asm volatile("" : "+v"(pb[j]));
  };

  // the epilogue's constants, requested first of all: alpha of the lane's columns, or alpha and threshold of row m0 + thread
  float al[TN], al_row = 1.0f, th_row = 0.0f;
#pragma unroll
  for (int j = 0; j < TN; ++j)
    al[j] = (!CONV && OUT == kF32 && p.alpha) ? p.alpha[min(n0 + 32 * (wn * TN + (j ^ xb)) + r, p.N - 1)] : 1.0f;
  if (CONV && OUT != kI32) {
    const int m = min(m0 + (int)threadIdx.x, p.M - 1);
    if (p.alpha) al_row = p.alpha[m];
    if (OUT == kBits && p.thr) th_row = p.thr[m];
  }
  issue(0, 0);
  if (p.nseg > 1) issue(1, 1);
  if constexpr (OUT == kBits) {
    // the tile's words of the output image's halo, spread over the tiles of this row of tiles
    for (int cw = m0 >> 6; p.opad > 0 && cw < min(p.oCw, (m0 >> 6) + WM); ++cw)
      write_halo((uint64_t*)p.C, p.Nimg, p.Ho, p.Wo, p.opad, p.M, p.oCw, cw, tile_n * 256 + threadIdx.x, p.tiles_n * 256);
  }
  if (p.nseg > 1) {
    constexpr int kLoads = HA * (LWA == 16 ? 1 : 4) + HB * (LW == 16 ? 1 : 4);  // a wave's loads of segment 1
    if (CONV && LW == 4 && !meet(1)) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(HA + HB) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kLoads) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (tail) {
      zero_tail(0);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
  }
  read(0, 0);
#pragma unroll
  for (int b = 0; b < TM + TN; ++b) expand(0, 0, 0, b);
  for (int s = 0; s < p.nseg; ++s) {
    read(1, s & 1);
    multiply(0);
    stay();
    if (s + 1 < p.nseg) {
      // segment s + 1 has landed, and everyone holds segment s in registers
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (s + 2 < p.nseg) {
        issue(s + 2, s & 1);
      } else if (tail) {
        zero_tail((s + 1) & 1);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      }
      read(0, (s + 1) & 1);
    }
    if (16 * s + 8 < p.Kd) {
      multiply(1);
      stay();
    }
  }

  // ---- epilogue.  Row and column terms of the whole tile meet in the stage that nobody reads any more.
  f_alias* const rt = (f_alias*)(lds + (p.nseg & 1) * kStage);
  f_alias* const ct = rt + 32 * NBA;
#pragma unroll
  for (int i = 0; i < CA; ++i) {
    pa[i] += __shfl_xor(pa[i], 32);
    if (h == 0) rt[32 * (wm * TM + (i ^ xa)) + r] = fmaf(p.row_mul, (float)pa[i], p.row_const);
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    pb[j] += __shfl_xor(pb[j], 32);
    if (h == 0) ct[32 * (wn * TN + (j ^ xb)) + r] = p.row_mul * (float)pb[j];
  }
  f_alias *const alr = ct + 32 * (NB - NBA), *const thr = alr + 32 * NBA;
  if (CONV && OUT != kI32 && threadIdx.x < 32 * NBA) {
    alr[threadIdx.x] = al_row;
    if (OUT == kBits) thr[threadIdx.x] = th_row;
  }
  const int mw = m0 + 32 * TM * wm, nw = n0 + 32 * TN * wn;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  float cb[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) cb[j] = ct[32 * (wn * TN + (j ^ xb)) + r];
  // (waited for here: in the stores of an edge tile, each under its own condition, every use of it would wait for the
  // stores before it; 649 x 3816 x 1024 in a layer 14.3 us so, now 10.1)
  if (!CONV && OUT == kF32) {
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(al[j]));
  }
  uint32_t img[TN], rem[TN];  // convolution form: image and pixel of the lane's columns
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const uint32_t n = (uint32_t)min(nw + 32 * (j ^ xb) + r, p.N - 1);
    img[j] = CONV ? fast_div(n, p.div_howo) : 0u;
    rem[j] = CONV ? n - img[j] * (uint32_t)p.HoWo : n;
  }
  if constexpr (OUT == kBits) {
    static_assert(TM == 2 && TN == 2, "a wave holds a word of 64 pixels");
    uint32_t half[TN][TM];  // of pixel block j: filters of block i
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) half[j][i] = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int mi = 32 * (i ^ xa) + 8 * q, at = 32 * wm * TM + mi + 4 * h;
        const v4f_alias rc = *(const v4f_alias*)(rt + at), a4 = *(const v4f_alias*)(alr + at), t4 = *(const v4f_alias*)(thr + at);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const float dot = fmaf(p.tot_mul, acc[i][j][4 * q + e], rc[e] + cb[j]);
            if (mw + mi + 4 * h + e < p.M && a4[e] * dot >= t4[e]) half[j][i] |= 1u << (8 * q + 4 * h + e);
          }
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) half[j][i] |= (uint32_t)__shfl_xor((int)half[j][i], 32);
    }
    // lane (r, h) stores the word of pixel r of block h of the registers
    const uint32_t lo = xa ? (h ? half[1][1] : half[0][1]) : (h ? half[1][0] : half[0][0]);
    const uint32_t hi = xa ? (h ? half[1][0] : half[0][0]) : (h ? half[1][1] : half[0][1]);
    if (nw + 32 * (h ^ xb) + r < p.N && mw < p.M) {
      const uint32_t im = h ? img[1] : img[0], re = h ? rem[1] : rem[0];
      const uint32_t ho = fast_div(re, p.div_wo), wo = re - ho * (uint32_t)p.Wo;
      const uint32_t word = ((im * (uint32_t)p.oHp + ho + (uint32_t)p.opad) * (uint32_t)p.oWp + wo + (uint32_t)p.opad) * (uint32_t)p.oCw + (uint32_t)(mw >> 6);
      ((uint64_t*)p.C)[word] = (uint64_t)hi << 32 | lo;
    }
    return;
  }
  const int ldr = CONV ? p.HoWo : p.ldc;  // elements from row to row
  uint32_t at[TN];                        // byte offset of the lane's results in row 0 of each column block
#pragma unroll
  for (int j = 0; j < TN; ++j) at[j] = ((img[j] * (uint32_t)p.M + 4u * h) * (uint32_t)ldr + (CONV ? rem[j] : (uint32_t)(32 * (j ^ xb) + r))) * 4u;
  char* const cbase = (char*)p.C + ((size_t)mw * ldr + (CONV ? 0 : nw)) * 4;
  auto store = [&](auto inside_tag, auto nt_tag) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int mi = 32 * (i ^ xa) + 8 * q;
        const v4f_alias rc = *(const v4f_alias*)(rt + 32 * wm * TM + mi + 4 * h);
        v4f_alias a4 = {1.0f, 1.0f, 1.0f, 1.0f};
        if (CONV && OUT == kF32) a4 = *(const v4f_alias*)(alr + 32 * wm * TM + mi + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          char* const row = cbase + (size_t)(uint32_t)((mi + e) * ldr) * 4;
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const float dot = fmaf(p.tot_mul, acc[i][j][4 * q + e], rc[e] + cb[j]);  // exact: see exact_k
            const int v = OUT == kI32 ? (int)dot : __builtin_bit_cast(int, (CONV ? a4[e] : al[j]) * dot);
            if constexpr (decltype(inside_tag)::value) {
              if constexpr (decltype(nt_tag)::value)
                asm volatile("global_store_dword %0, %1, %2 nt" ::"v"(at[j]), "v"(v), "s"(row) : "memory");
              else
                asm volatile("global_store_dword %0, %1, %2" ::"v"(at[j]), "v"(v), "s"(row) : "memory");
            } else if (mw + mi + 4 * h + e < p.M && nw + 32 * (j ^ xb) + r < p.N) {
              *(int*)(row + at[j]) = v;
            }
          }
        }
      }
  };
  if (mw + 32 * TM <= p.M && nw + 32 * TN <= p.N) {
    if (p.nt) store(std::true_type{}, std::true_type{});
    else store(std::true_type{}, std::false_type{});
  } else {
    store(std::false_type{}, std::false_type{});
  }
}

// Sums exact in fp32.  Planes 0 to 2 add 0 or 1 a value, plane 3 +-1/4: sums are multiples of 1/4 up to 13/16 K, which fp32 holds
// below 2^22.  The results, 4 times the sum and the terms of row and column, are whole numbers; none of the three is above 13/4 K.
bool exact_k(int64_t K) { return K < (1 << 22); }

// K, less the values of plane 3 in K (whose products of signs count themselves) and those among the zero bits behind it up to
// a whole group of 256, which count one each: together every value of plane 3 of the groups multiplied.  (For Eq. 2's count, half.)
float row_const(int K, int dwords, bool as_count) {
  const int plane3 = (int)ceil_div(dwords, 8) * 64;
  return as_count ? (float)(K - plane3 / 2) : (float)(K - plane3);
}

template <int WM, int TM, int TN, int OUT, int LW, bool CONV>
hipError_t go(BlockParams& p, hipStream_t s) {
  constexpr int NBA = WM * TM, NBB = 4 / WM * TN;
  constexpr size_t lds = 2 * (NBA + NBB) * 2048 + (CONV ? 128 * NBB : 0);
  static_assert(lds <= 64 * 1024, "within the LDS a kernel may use without asking");
  p.tiles_m = (int)ceil_div(p.M, 32 * NBA);
  p.tiles_n = (int)ceil_div(p.N, 32 * NBB);
  p.band = std::min(32 / NBA, p.tiles_m);  // 1024 rows of C, as in gemm_fp4.hip
  p.per_band = p.band * p.tiles_n;
  p.last_band = (p.tiles_m - 1) / p.band;
  p.last_rows = p.tiles_m - p.last_band * p.band;
  p.div_per_band = make_fast_div((uint32_t)p.per_band);
  p.div_band = make_fast_div((uint32_t)p.band);
  p.div_last = make_fast_div((uint32_t)p.last_rows);
  p.tiles_per_xcd = (int)ceil_div((int64_t)p.tiles_m * p.tiles_n, 8);
  p.A -= lowered(CONV, LW);
  p.B -= lowered(CONV, LW);
  const unsigned blocks = 8u * (unsigned)p.tiles_per_xcd;
  note_kernel("block::gemm_fp4_kernel<%d,%d,1,xnor,%s,%sblock%s%s> grid %u x 256, K split 1, fp4", TM, TN,
              OUT == kI32 ? "i32" : OUT == kBits ? "bits" : "f32", CONV ? "conv," : "", LW != 4 ? "" : CONV ? " of odd runs" : " of dwords",
              WM == 1 ? " one high" : "", blocks);
  launch_kernel((gemm_fp4_kernel<WM, TM, TN, OUT, LW, CONV>), dim3(blocks), dim3(256), lds, s, p);
  return launch_error();
}

}  // namespace
}  // namespace block

int gemm_block = 0;  // 1 = never, 2 = 256 x 128 and 3 = 128 x 128 of C per workgroup whatever the size

bool launch_gemm_block(const void* A, int64_t lda_bytes, const void* B, int64_t ldb_bytes, int M, int N, int K, int dwords,
                       const float* alpha, int32_t* C_i32, float* C_f32, int64_t ldc, bool as_count, hipStream_t s,
                       hipError_t* err) {
  if (gemm_block == 1 || gemm_engine == 1 || gemm_engine == 2 || gemm_engine == 4) return false;
  if (gemm_block == 0 && (gemm_engine || gemm_fp4_split || gemm_fp4_half || gemm_fp4_band)) return false;
  // rows of less than 16 bytes that the next begins in: dword by dword
  const bool short_rows = dwords < 4 && ((lda_bytes & 15) || (ldb_bytes & 15) || ((uintptr_t)A & 15) || ((uintptr_t)B & 15));
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, 128), tiles64 = ceil_div(M, 64) * ceil_div(N, 64);
  const bool lines = ldc % 32 == 0 && (((uintptr_t)C_i32 | (uintptr_t)C_f32) & 127) == 0;
  // Against gemm_fp4.hip by its tiles of 64 x 64, from 1400 products of 700 to 2700 of them and 8 to 128 words, rows on any word (the
  // time there over the time here, in a graph; the choice by this rule is 0.37 % off the best, where it was 0.90 % with all of up to 512
  // tiles of 128 x 128 left there: 4480 x 1792 x 5343 20.9 there, 19.6 here):
  //   - to 1280 K is divided over a CU's waves there (0.75 to 0.87), or a SIMD has one undivided tile (769 to 1024 0.91).
  //   - to 2048, undivided and up to two a SIMD, here from 70 words on, with fp32 results, scaled behind there as the waves finish one
  //     by one, from 50 (int32 of 20 to 39 words 0.97, 40 to 59 0.98, 60 to 89 1.02, 90 on 1.05; fp32 0.99, 1.01, 1.03, 1.06; the lines
  //     where two in a hundred lose more than 2 %), but not past 512 tiles of 128 x 128, two workgroups a CU (513 to 540 0.88).
  // Beyond, the products have to outweigh the results' way out, which takes longer where rows of C are parts of lines and
  // a tile of 64 x 64 is a better piece of it (whole lines: 8 to 19 words 0.98, 20 to 39 1.01, 40 on 1.04 to 1.12; parts: 0.87, 0.97,
  // 1.04 to 1.12).  What that kernel does not take (rows of less than 16 bytes, whose results are the time, and results that its
  // 32-bit indices do not reach) is this one's whatever K, where gemm_small.hip does not take it and from 512 of those tiles on: gemm_mfma.hip,
  // which would get it, takes 28.5 us for 2048 x 2560 x 4096, rows 1048576 apart, 15.1 here; x 256 15.3 / 6.9; of 21 dwords, widened first,
  // 28.7 / 7.6; 1800 x 1300 x 960 9.3 / 7.5, x 16384 34.7 / 28.8; 100 tiles, 640 x 640 x 640 5.4 / 5.2, but x 8192 9.1 / 15.0.
  // The larger of the two shapes (us as 128 x 128 / as 256 x 128, each held for 50 ms): its waves read LDS and expand less for a
  // product, which shows once the chip's power has settled, where the results leave in whole lines and fill many rounds:
  // 8192 x 8192 x 8192 186 / 177, x 4096 106 / 102; 8192 x 12288 x 8192 277 / 263, 16384 x 8192 x 8192 370 / 352, 10240 x 10240 x
  // 8192 289 / 278, 16384 x 4096 x 8192 187 / 176, 8130 x 8192 x 8192 187 / 178; in bursts of 2.5 ms 0 to 6 % behind to 3 % ahead.
  // Rows of C that are no whole lines: 8150 x 8130 x 8192 204 / 212, 8192 x 8130 x 8192 205 / 208, 9000 x 9000 x 6000 201 / 202, 5000
  // x 15000 x 9000 261 / 262.  Below 4096 tiles it depends on the last round: 8192 x 6144 x 8192 143 / 132, but 5120 x 5120 x 8192
  // 78 / 85, 6144 x 6144 x 4096 60.5 / 62.4, 7168 x 7168 x 4096 83.5 / 84.3 (in bursts 77 / 86); 8192 x 8192 x 1024 50 / 54.
  if (gemm_block == 0) {
    if (short_rows || !gemm_fp4_pays(M, N, lda_bytes, ldb_bytes, ldc, false)) {  // (gemm_fp4.hip does not take it)
      if (tiles64 < 512) return false;
    } else if (dwords < 22 || tiles64 <= 1280 || (tiles64 <= 2048 ? tiles > 512 || dwords < (C_f32 ? 100 : 140) : dwords < (lines ? 38 : 64))) {
      return false;
    }
  }
  // (32-bit offsets, rows of the last tile past the last row counted, of C within a tile)
  const int64_t lim = (int64_t)1 << 32;
  if (!block::exact_k(K) || ((int64_t)M + 256) * lda_bytes >= lim || ((int64_t)N + 256) * ldb_bytes >= lim) return false;
  if (ldc >= (1 << 22) || ((uintptr_t)A & 3) || ((uintptr_t)B & 3)) return false;
  block::BlockParams p;
  p.A = (const char*)A;
  p.B = (const char*)B;
  p.lda = (uint32_t)lda_bytes;
  p.ldb = (uint32_t)ldb_bytes;
  p.M = M;
  p.N = N;
  p.Kd = dwords;
  p.nseg = (int)ceil_div(dwords, 16);
  p.alpha = alpha;
  p.row_const = block::row_const(K, dwords, as_count);
  p.row_mul = as_count ? -1.0f : -2.0f;
  p.tot_mul = as_count ? 2.0f : 4.0f;
  p.C = C_i32 ? (void*)C_i32 : (void*)C_f32;
  p.ldc = (int)ldc;
  p.nt = lines;
  p.HoWo = p.Wo = p.Ho = p.Hp = p.Wpp = p.Cw = p.stride = p.Nimg = 1;
  p.run = p.row_bytes = 1;
  p.div_howo = p.div_wo = p.div_run = p.div_two_runs = make_fast_div(1);
  p.thr = nullptr;
  p.opad = p.oHp = p.oWp = p.oCw = 0;
  const bool large = !short_rows && (gemm_block ? gemm_block == 2 : tiles >= 4096 && K >= 4096 && p.nt);
  using namespace block;
  if (large) *err = C_i32 ? go<2, 4, 2, kI32, 16, false>(p, s) : go<2, 4, 2, kF32, 16, false>(p, s);
  else if (short_rows) *err = C_i32 ? go<2, 2, 2, kI32, 4, false>(p, s) : go<2, 2, 2, kF32, 4, false>(p, s);
  else *err = C_i32 ? go<2, 2, 2, kI32, 16, false>(p, s) : go<2, 2, 2, kF32, 16, false>(p, s);
  return true;
}

int conv_block = 0;  // 1 = never, 2 = 128 filters x 128 pixels and 3 = 64 x 256 per workgroup whatever the size

// Fitted to 361 convolutions of 8 to 392 words measured on each (us, fp32 results and packed bits; the choice by it is 0.16 %
// off the best, 10 % at most; 0.66 % and 21 % while the terms were those of the kernels before their last change: 68175 pixels, 128 filters, 72
// words 26.6 us in gemm_fp4.hip, 22.0 here).  gemm_fp4.hip divides K of a 64 x 64 tile over a CU's waves: by its tiles per CU.
// Here by workgroups per CU; one alone on a CU takes more than half as long for a segment as two together.  With runs of an odd
// number of words, where the segments that two of them meet in take longer: of 400 such convolutions of 45 to 343 words the choice is
// 0.08 % off the best, 6 % at most.
double conv_long_us(int64_t P, int O, int kwords, bool odd, int* form) {
  const double K = kwords;
  const double n = (double)ceil_div(ceil_div(P, 64) * ceil_div(O, 64), 256);
  const double high = (double)ceil_div(ceil_div(P, 128) * ceil_div(O, 128), 256), mh = std::max(1.3, high);
  const double wide = (double)ceil_div(ceil_div(P, 256) * ceil_div(O, 64), 256), mw = std::max(1.3, wide);
  const double there = odd ? 3.65 + n * (0.78 + 0.0216 * K) : 3.6 + n * (0.87 + 0.0195 * K);
  const double us2 = odd ? 5.65 + 1.08 * high + 0.0759 * mh * K : 5.25 + 0.99 * high + 0.0718 * mh * K;
  const double us3 = odd ? 6.1 + 1.0 * wide + 0.0821 * mw * K : 4.5 + 1.14 * wide + 0.0783 * mw * K;
  *form = std::min(us2, us3) >= there ? 0 : us2 <= us3 ? 2 : 3;
  return std::min(there, std::min(us2, us3));
}

bool launch_conv_block(const uint64_t* Xp, int Nimg, int C, int H, int W, const uint64_t* Wp, int O, int KH, int KW, int stride,
                       int pad, const float* alpha, int32_t* out_i32, float* out_f32, uint64_t* out_bits, const float* thr,
                       int out_pad, hipStream_t s, hipError_t* err) {
  if (conv_block == 1 || conv_path || gemm_engine || conv_filters_per_wave || conv_ws_x4 || gemm_fp4_split || gemm_fp4_half ||
      gemm_fp4_band)
    return false;
  const int Ho = (H + 2 * pad - KH) / stride + 1, Wo = (W + 2 * pad - KW) / stride + 1;
  const int Cw = (int)words_for(C), kwords = KH * KW * Cw, Hp = H + 2 * pad, Wpp = W + 2 * pad;
  const int64_t P = (int64_t)Nimg * Ho * Wo, ld_words = conv_weight_row_words(kwords);
  const int64_t lim = (int64_t)1 << 32;
  if ((ld_words & 1) || ((uintptr_t)Wp & 15) || !block::exact_k((int64_t)C * KH * KW)) return false;
  // (32-bit byte offsets throughout, and counts of pixels, halo words and tiles)
  if ((int64_t)Nimg * Hp * Wpp * Cw * 8 >= lim || ((int64_t)O + 256) * ld_words * 8 >= lim || P >= lim / 4) return false;
  if (((int64_t)Nimg * O + 256) * Ho * Wo * 4 >= lim) return false;
  if (out_bits && (int64_t)Nimg * (Ho + 2 * out_pad) * (Wo + 2 * out_pad) * words_for(O) >= lim / 4) return false;
  const bool odd = (KW * Cw) & 1;
  int form = conv_block;
  if (form == 0) {
    conv_long_us(P, O, kwords, odd, &form);
    // Short K stays with conv_mfma.hip, but for many filters over many pixels: there a pixel's words are expanded once per
    // 32 filters, here once per 128 or 64.  Of 182 of 36, 49 and 50 words, from 90000 steps of 32 x 32 x 256 on (us there /
    // here): as packed bits 27776 pixels, 448 filters, 50 words 31.8 / 20.6, 27664, 384, 36 20.1 / 15.8, 46371, 192, 49 24.1 / 20.5;
    // fp32, 22610, 384, 49 24.1 / 21.9, 40544, 192, 50 18.1 / 15.0, but level at 36 words.  64 filters: 146160 pixels,
    // 49 words 19.7 / 23.9.
    if (conv_weight_short_k(kwords)) {
      const int64_t work = ceil_div(P, 32) * ceil_div(O, 32) * ceil_div(kwords, 4);
      if (kwords < (out_bits ? 36 : 49) || O < 128 || work < 90000) return false;
      form = ceil_div(ceil_div(P, 256) * ceil_div(O, 64), 256) < ceil_div(ceil_div(P, 128) * ceil_div(O, 128), 256) ? 3 : 2;
    }
    // Fewer words than a segment: the results are the time, and they leave best where neighbouring pixels are in one place.  As packed
    // bits from 7000 tiles of 32 x 32 on (1 x 1, 87822 pixels, 128 filters 11.8 us in conv_small.hip, 8.5 here; 51200, 137 level),
    // fp32 and int32 from 44 MB (the same 15.2 in conv.hip, 12.0; 147630 pixels, 64 filters, 38 MB 11.2 / 12.1).
    if (kwords < 8) {
      if (out_bits ? ceil_div(P, 32) * ceil_div(O, 32) < 7000 : P * O * 4 < ((int64_t)44 << 20)) return false;
      if (form == 0) form = O <= 64 ? 3 : 2;
    }
    if (form == 0) return false;
  }
  block::BlockParams p;
  p.A = (const char*)Wp;
  p.B = (const char*)Xp;
  p.lda = (uint32_t)(ld_words * 8);
  p.ldb = 0;
  p.M = O;
  p.N = (int)P;
  p.Kd = 2 * kwords;
  p.nseg = (int)ceil_div(p.Kd, 16);
  p.alpha = alpha;
  p.thr = thr;
  p.row_const = block::row_const(C * KH * KW, p.Kd, false);
  p.row_mul = -2.0f;
  p.tot_mul = 4.0f;
  p.C = out_bits ? (void*)out_bits : out_i32 ? (void*)out_i32 : (void*)out_f32;
  p.ldc = 0;
  p.nt = Ho * Wo % 32 == 0 && ((uintptr_t)p.C & 127) == 0;
  p.HoWo = Ho * Wo;
  p.Wo = Wo;
  p.Ho = Ho;
  p.Hp = Hp;
  p.Wpp = Wpp;
  p.Cw = Cw;
  p.stride = stride;
  p.Nimg = Nimg;
  p.run = (uint32_t)(KW * Cw);
  p.row_bytes = (uint32_t)((int64_t)Wpp * Cw * 8);
  p.div_howo = make_fast_div((uint32_t)p.HoWo);
  p.div_wo = make_fast_div((uint32_t)Wo);
  p.div_run = make_fast_div(p.run);
  p.div_two_runs = make_fast_div(2 * p.run);
  p.opad = out_pad;
  p.oHp = Ho + 2 * out_pad;
  p.oWp = Wo + 2 * out_pad;
  p.oCw = (int)words_for(O);
  const bool one_high = form == 3;
  using namespace block;
  auto kind = [&](auto wm, auto lw) {
    constexpr int WM = decltype(wm)::value, LW = decltype(lw)::value;
    return out_bits ? go<WM, 2, 2, kBits, LW, true>(p, s) : out_i32 ? go<WM, 2, 2, kI32, LW, true>(p, s) : go<WM, 2, 2, kF32, LW, true>(p, s);
  };
  auto high = [&](auto lw) { return one_high ? kind(std::integral_constant<int, 1>{}, lw) : kind(std::integral_constant<int, 2>{}, lw); };
  *err = odd ? high(std::integral_constant<int, 4>{}) : high(std::integral_constant<int, 16>{});
  return true;
}

}  // namespace bmx
