// xnor GEMM on the FP4 matrix cores for problems of many tiles: operand rows staged once per workgroup.
// Paper: Sec. 2.2.1 / Sec. 2.2.2 (Eq. 2): C[m][n] = K - 2 * popcount(A[m] xor B[n]).
//
// Arithmetic as in gemm_fp4.hip: K - 2 pc(a) - 2 pc(b) + 4 * sum_k a * b, a bit stays where it stands
// in its nibble and the MFMA's block scale makes it worth 1.
//
// There every wave fetches the rows of its own tile, waits for its own reads of a segment before it may request
// the next, and turns all of a segment's bits into operands before it multiplies.  With the chip full that
// leaves the matrix cores half idle: 8192^3 took 202 us, where a loop of the same multiplications on bits that
// stand in LDS takes 145 (their power holds the clock at 2.1 to 2.3 GHz, and every MFMA keeps the SIMD's issue
// slot for about 16 of its 32 clocks).  Here:
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
//   - Rows that start on any dword are fetched dword by dword (global_load_lds_dword), four times the loads of a
//     sixth of the traffic, instead of through registers.
// Measured, us a call, gemm_fp4.hip / here: 8192^3 202 / 173, 8192 x 8192 x 1024 75 / 50, 4096^3 33 / 28, 3008 x 1471
// x 5184 25.6 / 23.1; rows on any dword: 4321 x 7134 x 3157 62 / 51, 1792 x 5234 x 832 17.9 / 13.3.
#include <algorithm>
#include <type_traits>

#include "bmx_internal.h"

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
  const float* alpha;
  float row_const, row_mul, tot_mul;  // result = row_const + row_mul * (pc(a) + pc(b)) + tot_mul * sum
  void* C;
  int ldc, nt;
};

constexpr int kF32 = 0, kI32 = 1;

// Plane n of four words as an operand: bit 4 i + n of a dword in nibble i, worth 0.5, 1 or 2 where it stands (planes
// 0 to 2); plane 3, whose bit would be the nibble's sign, is shifted down to 0.5.
__device__ __forceinline__ v4i plane(const uint4& w, int n) {
  const uint32_t m = n == 3 ? 0x11111111u : 0x11111111u << n;
  const int sh = n == 3 ? 3 : 0;
  return v4i{(int)((w.x >> sh) & m), (int)((w.y >> sh) & m), (int)((w.z >> sh) & m), (int)((w.w >> sh) & m)};
}

__device__ __forceinline__ v8i wide(const v4i& e) { return v8i{e[0], e[1], e[2], e[3], 0, 0, 0, 0}; }

// acc + popcount of four words
__device__ __forceinline__ int add_popcount4(int acc, const uint4& w) {
  return __builtin_popcount(w.x) + (__builtin_popcount(w.y) + (__builtin_popcount(w.z) + (__builtin_popcount(w.w) + acc)));
}

// TM x TN blocks of 32 x 32 per wave; LW: bytes a lane fetches per load (16: rows start 16-byte aligned; 4: on any
// dword).  A stage holds blocks of 32 rows x 64 bytes, A's, then B's, in the layout of gemm_fp4.hip: piece c of row r of a
// block at 16-byte place 64 (r / 16) + 4 (r % 16) + (c xor ((r / 2) & 3)).
template <int TM, int TN, int OUT, int LW>
__global__ void __launch_bounds__(256, TM * TN >= 8 ? 2 : 3)
gemm_fp4_kernel(const BlockParams p) {
  extern __shared__ uint4 lds[];
  constexpr int NBA = 2 * TM, NB = 2 * TM + 2 * TN, PW = NB / 4;  // blocks of A, of both, fetched by a wave
  constexpr int kStage = NB * 128;  // uint4 per stage
  static_assert(NB % 4 == 0 && TM % 2 == 0 && TN % 2 == 0, "a share of the blocks for each wave, half of its own to count");
  asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.lda), "s"(p.ldb), "s"(p.M), "s"(p.N), "s"(p.Kd), "s"(p.nseg), "s"(p.tiles_m),
               "s"(p.tiles_n), "s"(p.tiles_per_xcd), "s"(p.band), "s"(p.per_band), "s"(p.last_band), "s"(p.last_rows),
               "s"(p.div_per_band.mul), "s"(p.div_per_band.sh1), "s"(p.div_per_band.sh2), "s"(p.div_band.mul),
               "s"(p.div_band.sh1), "s"(p.div_band.sh2), "s"(p.div_last.mul), "s"(p.div_last.sh1), "s"(p.div_last.sh2));
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lin = (int)(blockIdx.x & 7) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  if (lin >= p.tiles_m * p.tiles_n) return;
  const int bnd = (int)fast_div((uint32_t)lin, p.div_per_band), within = lin - bnd * p.per_band;
  const bool lastb = bnd == p.last_band;
  const int tile_n = (int)fast_div((uint32_t)within, lastb ? p.div_last : p.div_band);
  const int tile_m = bnd * p.band + (within - tile_n * (lastb ? p.last_rows : p.band));
  const int m0 = tile_m * (64 * TM), n0 = tile_n * (64 * TN);

  // ---- loads
  constexpr int NL = LW == 16 ? 2 : 8;  // loads per block of 32 rows
  constexpr int RL = 32 / NL;           // rows per load
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  // LW 16: the offset of either load of a block; LW 4: of its first two loads, the others eight rows apart each,
  // held at the last row (dw: the offset of the lane's dword in its row)
  uint32_t voff[PW][2], dw[2];
  const int lr = LW == 16 ? lane >> 2 : lane >> 4;  // row of a load
  const bool tail = (p.Kd & 15) != 0;
  uint32_t tsub[2];  // taken off the offset of a lane whose piece starts past the row's last dword
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int slot = LW == 16 ? lane & 3 : (lane & 15) >> 2;
    const int piece = slot ^ (((RL * t + lr) >> 1) & 3);
    const int d = 4 * piece + (LW == 16 ? 0 : (lane & 3));
    const int over = 16 * (p.nseg - 1) + d - (p.Kd - 1);
    dw[t] = 4u * d;
    tsub[t] = over > 0 ? (LW == 16 ? 16u * piece : 4u * over) : 0u;
#pragma unroll
    for (int b = 0; b < PW; ++b) {
      const int blk = wave * PW + b;
      const bool isa = blk < NBA;
      const uint32_t ld = isa ? p.lda : p.ldb, lim = (uint32_t)(isa ? p.M : p.N) - 1u;
      const uint32_t row = (uint32_t)(isa ? m0 + 32 * blk : n0 + 32 * (blk - NBA)) + RL * t + lr;
      voff[b][t] = (LW == 16 ? min(row, lim) : row) * ld + 4u * d;
    }
  }
  // Requests segment seg of the wave's blocks into stage buf.  (As asm: the compiler would wait for every load of this kind
  // before every LDS read.  m0 is the load's LDS address; nothing else here uses it.)
  auto issue = [&](int seg, int buf) {
    const bool last = tail && seg + 1 == p.nseg;
#pragma unroll
    for (int b = 0; b < PW; ++b) {
      const int blk = wave * PW + b;
      const char* base = (blk < NBA ? p.A : p.B) + (uint32_t)seg * 64u;
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const uint32_t to = lds0 + (uint32_t)(buf * kStage + blk * 128) * 16u + (uint32_t)u * (LW == 16 ? 1024u : 256u);
        uint32_t off = voff[b][u & 1];
        if (LW == 4)
          off = blk < NBA ? min(off + (uint32_t)(u >> 1) * 8u * p.lda, dw[u & 1] + (uint32_t)(p.M - 1) * p.lda)
                          : min(off + (uint32_t)(u >> 1) * 8u * p.ldb, dw[u & 1] + (uint32_t)(p.N - 1) * p.ldb);
        off -= last ? tsub[u & 1] : 0u;
        if constexpr (LW == 16)
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory");
        else
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"(off), "s"(base) : "memory");
      }
    }
  };
  // What the loads left behind the row's last dword counts as zero.
  auto zero_tail = [&](int buf) {
    u_alias* const d = (u_alias*)(lds + buf * kStage);
    const int valid = p.Kd & 15;
    for (int row = threadIdx.x; row < 32 * NB; row += 256) {
      const int base = (row >> 4) * 256 + (row & 15) * 16, x = (row >> 1) & 3;
      for (int k = valid; k < 16; ++k) d[base + (((k >> 2) ^ x) << 2) + (k & 3)] = 0u;
    }
  };

  // ---- products.  Two waves share every block; each takes its blocks in an order of its own (block i of the registers is
  // block i xor xa of the tile) and counts the first half of them.
  const int wm = wave >> 1, wn = wave & 1;
  constexpr int CA = TM / 2, CB = TN / 2;
  const int xa = wn * CA, xb = wm * CB;
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
      const int sc = n == 1 ? 127 : (n == 2 ? 126 : 128);  // block scales that make a product worth 1
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

  issue(0, 0);
  if (p.nseg > 1) {
    issue(1, 1);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(PW * NL) : "memory");
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
  const int mw = m0 + 32 * TM * wm, nw = n0 + 32 * TN * wn;
  float cb[TN], al[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) al[j] = (OUT == kF32 && p.alpha) ? p.alpha[min(nw + 32 * (j ^ xb) + r, p.N - 1)] : 1.0f;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int j = 0; j < TN; ++j) cb[j] = ct[32 * (wn * TN + (j ^ xb)) + r];
  auto value = [&](float tot, float rc, int j) {
    const float dot = fmaf(p.tot_mul, tot, rc + cb[j]);  // exact: whole numbers below 2^24
    return OUT == kI32 ? (int)dot : __builtin_bit_cast(int, al[j] * dot);
  };
  uint32_t at[TN];  // byte offset of the lane's results in row 0 of each column block
#pragma unroll
  for (int j = 0; j < TN; ++j) at[j] = (uint32_t)(4 * h * p.ldc + 32 * (j ^ xb) + r) * 4u;
  char* const cbase = (char*)p.C + ((size_t)mw * p.ldc + nw) * 4;
  auto store = [&](auto inside_tag, auto nt_tag) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int mi = 32 * (i ^ xa) + 8 * q;
        const v4f_alias rc = *(const v4f_alias*)(rt + 32 * wm * TM + mi + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          char* const row = cbase + (size_t)(uint32_t)((mi + e) * p.ldc) * 4;
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int v = value(acc[i][j][4 * q + e], rc[e], j);
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

template <int TM, int TN, int OUT, int LW>
hipError_t go(const BlockParams& p, int64_t blocks, hipStream_t s) {
  constexpr size_t lds = 2 * (2 * TM + 2 * TN) * 2048;
  static_assert(lds <= 64 * 1024, "within the LDS a kernel may use without asking");
  note_kernel("gemm_fp4_kernel<%d,%d,1,xnor,%s,block%s> grid %lld x 256, K split 1, fp4", TM, TN, OUT == kI32 ? "i32" : "f32",
              LW == 4 ? " of dwords" : "", (long long)blocks);
  launch_kernel((gemm_fp4_kernel<TM, TN, OUT, LW>), dim3((unsigned)blocks), dim3(256), lds, s, p);
  return launch_error();
}

template <int TM, int TN>
hipError_t launch_shape(BlockParams& p, bool f32, bool dwords, hipStream_t s) {
  p.tiles_m = (int)ceil_div(p.M, 64 * TM);
  p.tiles_n = (int)ceil_div(p.N, 64 * TN);
  p.band = std::min(16 / TM, p.tiles_m);  // 1024 rows of C, as in gemm_fp4.hip
  p.per_band = p.band * p.tiles_n;
  p.last_band = (p.tiles_m - 1) / p.band;
  p.last_rows = p.tiles_m - p.last_band * p.band;
  p.div_per_band = make_fast_div((uint32_t)p.per_band);
  p.div_band = make_fast_div((uint32_t)p.band);
  p.div_last = make_fast_div((uint32_t)p.last_rows);
  p.tiles_per_xcd = (int)ceil_div((int64_t)p.tiles_m * p.tiles_n, 8);
  const int64_t blocks = 8 * (int64_t)p.tiles_per_xcd;
  if constexpr (TM * TN == 8) return f32 ? go<TM, TN, kF32, 16>(p, blocks, s) : go<TM, TN, kI32, 16>(p, blocks, s);
  else if (f32) return dwords ? go<TM, TN, kF32, 4>(p, blocks, s) : go<TM, TN, kF32, 16>(p, blocks, s);
  else return dwords ? go<TM, TN, kI32, 4>(p, blocks, s) : go<TM, TN, kI32, 16>(p, blocks, s);
}

}  // namespace
}  // namespace block

int gemm_block = 0;  // 1 = never, 2 = 256 x 128 and 3 = 128 x 128 of C per workgroup whatever the size

bool launch_gemm_block(const void* A, int64_t lda_bytes, const void* B, int64_t ldb_bytes, int M, int N, int K, int dwords,
                       const float* alpha, int32_t* C_i32, float* C_f32, int64_t ldc, bool as_count, hipStream_t s,
                       hipError_t* err) {
  if (gemm_block == 1 || gemm_engine || gemm_fp4_split || gemm_fp4_half || gemm_fp4_band || gemm_fp4_tall) return false;
  const bool any_dword = (lda_bytes & 15) || (ldb_bytes & 15) || ((uintptr_t)A & 15) || ((uintptr_t)B & 15);
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, 128), rounds = ceil_div(tiles, 256);
  // Against gemm_fp4.hip, from 220 products of up to 8192 x 8192 x 8192 measured on both (us, there / here).  Rows that
  // start on any dword pass through registers there: from 145 tiles on (512 x 4736 x 4921, 148 tiles, 16.6 / 13.1; 1036
  // x 7808 x 386, 549 tiles, 14.2 / 9.1); with fewer it goes both ways (4444 x 512 x 7119, 140 tiles, 23.8 / 16.9; 358 x 5312 x
  // 2946, 126 tiles, 9.5 / 10.9).  Others: where there is a workgroup for
  // every CU and no CU is given far more of them than another (1344 x 6016 x 3840, 517 tiles on 256 CUs, 17.7 / 21.1; 5504 x
  // 320 x 4956, 129 tiles and the K divided there, 11.3 / 13.1), and where K is long enough for the products to show in the
  // time (4560 x 731 x 582 8.0 / 9.1).  Of the two shapes the larger needs many tiles per CU and a long K (8192^3 184 as 128 x 128,
  // 173 as 256 x 128; 8192 x 8192 x 2880 level; 8192 x 8192 x 1024 50 and 54).
  if (gemm_block == 0) {
    if (any_dword ? tiles <= 144 : (tiles < 256 || 10 * tiles < 7 * 256 * rounds || K < 700)) return false;
  }
  // (32-bit offsets, rows of the last tile past the last row counted; whole numbers up to 3 K exact in fp32)
  const int64_t lim = (int64_t)1 << 32;
  if (K >= (1 << 22) || ((int64_t)M + 256) * lda_bytes >= lim || ((int64_t)N + 256) * ldb_bytes >= lim) return false;
  if (((int64_t)M + 256) * ldc * 4 >= lim || ((uintptr_t)A & 3) || ((uintptr_t)B & 3)) return false;
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
  p.row_const = (float)K;
  p.row_mul = as_count ? -1.0f : -2.0f;
  p.tot_mul = as_count ? 2.0f : 4.0f;
  p.C = C_i32 ? (void*)C_i32 : (void*)C_f32;
  p.ldc = (int)ldc;
  p.nt = ldc % 32 == 0 && ((uintptr_t)p.C & 127) == 0;
  const bool large = !any_dword && (gemm_block ? gemm_block == 2 : tiles >= 4096 && K >= 4096);
  *err = large ? block::launch_shape<4, 2>(p, !C_i32, false, s) : block::launch_shape<2, 2>(p, !C_i32, any_dword, s);
  return true;
}

}  // namespace bmx
