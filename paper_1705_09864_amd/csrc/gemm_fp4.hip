// xnor GEMM and bit-plane GEMM on the FP4 matrix cores: 64 x 64 of C per wave, operands staged
// through LDS by the load unit itself, K split over the waves of a workgroup.
// Paper: Sec. 2.2.1 / Sec. 2.2.2 (Eq. 2): C[m][n] = K - 2 * popcount(A[m] xor B[n]); Sec. 2.1
// (Eq. 1) for the k-bit activations of the plane form.
//
// Arithmetic (as in gemm_mfma.hip): with bits a, b in {0, 1},
//     K - 2 * pc(a xor b) = K - 2 * pc(a) - 2 * pc(b) + 4 * sum_k a * b,
// the sum on v_mfma_f32_32x32x64_f8f6f4 with both operands FP4 (E2M1).  Every fourth bit of a 32-bit
// word of bits makes one of the four 8-nibble operand dwords of four MFMAs: a bit stays where it
// stands in its nibble (worth 0.5, 1 or 2 there) or is shifted by two, in A and B so that every
// product is worth 1: five VALU instructions a dword of A, six of B.  Products and
// fp32 sums are exact integers below 2^24.  The two bit planes of a 2-bit activation are staged
// as separate rows and folded into one operand while being expanded: a nibble then holds the
// 2-bit value itself (E2M1 codes 0 to 3 = 0, 0.5, 1, 1.5), and block scales bring the products to 1.
//
// What bounds this kernel is not the matrix core but everything around it: the issue of the
// instructions that turn bits into nibbles, the loads, and fixed costs of a few-microsecond launch.
// (A SIMD issues a vector instruction in 4 clocks, this MFMA in 11, with block scales in 17: the 16 MFMAs
// and 104 other vector instructions of four words take 590 clocks of issue and 512 of the matrix core;
// interleaving them by hand and reading a segment ahead, in twice the registers, measured level.)  Hence:
//   - 2 x 2 blocks of 32 x 32 per wave: an expanded operand block serves two MFMAs, 5.5 VALU
//     instructions of expansion and 1 of row popcount per MFMA (a 32 x 32 tile needs 13).
//   - Operands travel global memory -> LDS without passing registers (global_load_lds_dwordx4:
//     lane i of the instruction writes LDS bytes [16 i, 16 i + 16) of its destination).  A load
//     covers 16 rows x 64 bytes, 4 lanes per row: whole 64-byte runs, so the memory pipeline
//     works at its coalesced rate, where the MFMA layout (lane = row) costs an access per lane.
//     Which 16-byte piece a lane fetches is permuted (piece = slot xor ((row >> 1) & 3)), so
//     that the MFMA-layout reads, lane (r, h) <- piece 2 g + h of row r, fall on all banks.  Rows may start on any
//     dword: these loads need no more (rows of an odd number of words went through registers once: 2947 x 6975 x 2624
//     as packed bits 48.5 -> 39.2 us, with a word a lane at its end 31.0; 3318 x 778 x 3264, fp32, 12.1 -> 9.2, 2212 x 2496 x 1472 of 32-bit words
//     9.8 -> 8.9).
//   - A wave owns its staging area and its range of K: no barrier in the main loop.  The words
//     of a 64-byte segment are read into registers, the next segment's loads are issued into
//     the same area once those reads have completed, and the 32 MFMAs of the segment run with
//     those loads in flight.
//   - Skinny problems (the fully connected layers: 256 rows) have too few 64 x 64 tiles to
//     fill the chip, so the S waves of a workgroup split K and add their partial tiles through
//     LDS once: every wave writes its 64 registers, then finishes 1/S of the tile (sum of S
//     partials, the popcount terms, scale, store).  Fat problems run four tiles per workgroup
//     and no split.
//   - The way from the sums to the stores is a third of a launch of 5 us: its instructions are few
//     (addresses are scalar, parts of a sum are added in pairs of 16 bits, rows of results leave in 16-byte
//     stores), its arguments and constants are there before it starts.  Against index arithmetic,
//     bounds and dword stores per result: 2240 x 539 x 1799 7.6 -> 5.3 us, 787 x 2112 x 5568 10.8 -> 8.6,
//     256 x 9216 -> 4096 -> 4096 with its packs 20.1 -> 18.8, 1024 x 1024 x 4096 of 2 x 1 bits 13.9 -> 12.6.
//   - Workgroups are numbered so that tiles sharing operand rows sit on one XCD and run back
//     to back (workgroup b runs on XCD b % 8): every XCD gets a contiguous run of tiles, walked
//     in bands of 8 or 16 rows of tiles.
//   - The convolution form gathers the B operand (im2col rows) from the halo-padded packed
//     image, 16 bytes per lane, through the same loads.  Where runs have an odd number of words only the segments that two of them
//     meet in pass registers (all did once; us in a graph, before and now: 21600 pixels, 128 filters, 45 words, 678 tiles 12.9 -> 10.2;
//     24 x 192 x 47 x 49 -> 64, 5 x 5, 17.6 -> 14.7; 22 x 192 x 42 x 42 -> 64, 7 x 7, as packed bits 20.1 -> 16.7; of 400 drawn ones
//     1.07 in the mean, 1.2 to 1.3 between 513 and 768 tiles.  Those segments dword by dword straight to LDS: 1.05).
#include <algorithm>
#include <type_traits>

#include "bmx_internal.h"
#include "halo.h"
#include "row_pieces.h"

namespace bmx {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v4i_alias __attribute__((ext_vector_type(4), may_alias));
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u_alias __attribute__((may_alias));
typedef uint16_t u16_alias __attribute__((may_alias));
typedef uint8_t u8_alias __attribute__((may_alias));

// v_writelane_b32, which this compiler knows by no builtin: `old` with `value` (uniform) in lane `lane`.
extern "C" __device__ __attribute__((const)) uint32_t write_lane(uint32_t value, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");

struct Fp4Params {
  const void* A;  // [M * PL][lda] words (plane pl of row m is row m * PL + pl), tail bits zero; products: 16 bytes in front of it
  const void* B;  // [N][ldb] words; products: 16 bytes in front of it
  uint32_t lda_bytes, ldb_bytes;  // row strides, multiples of 4
  int M, N, Kw, Kd;               // data words and dwords per row (2 Kw, or one less)
  int g_base, g_rem;  // groups of four words (256 bits = the K of four MFMAs) per wave: g_base, the first g_rem waves one more
  int tiles_m, tiles_n, tiles_per_xcd;
  // tile order: bands of `band` rows of tiles (the last band has last_rows), see the kernel
  int band, per_band, last_band, last_rows;
  FastDiv div_per_band, div_band, div_last;
  const float* alpha;     // per column n, or null
  const float* thr;       // packed-bit output: per column threshold of the sign decision, or null (0)
  const int32_t* rowsum;  // plane form: sum_k q[m][k]
  int as_count;           // int32 output holds the xnor count (dot + K) / 2
  int32_t* C_i32;
  float* C_f32;
  uint32_t* C_bits;  // packed sign bits, addressed in 32-bit halves of the output words
  int ldc;           // elements per row (C_bits: 64-bit words per row); M * ldc < 2^31
  int nt;            // result stores bypass the caches: every 32-column run is one whole 128-byte line
  // Convolution form (Sec. 3.1: M = filters, N = batch * output pixels, K = kh * kw * C): A is the
  // packed filter matrix, B the halo-padded packed image.  Column n is output pixel n (flat over
  // the images); its K words are KH runs of KW * Cw consecutive words, one run per kernel row
  // (the taps of a kernel row are neighbouring pixels, channel words innermost), so a 16-byte piece
  // of the im2col row is 16 consecutive bytes of the image, but for those that two runs of an odd number of words meet in.  alpha is per
  // row m here, and the result goes to NCHW: element (image * M + m) * HoWo + pixel.
  int HoWo, Wo, Hp, Wpp, Cw, stride;
  uint32_t run, row_bytes;  // words per run; bytes from run to run
  FastDiv div_howo, div_wo, div_run, div_two_runs;
  // packed bits of the convolution form: the next convolution's image (C_bits, 64-bit words), its size, words per pixel, halo;
  // thr is per row m
  int Nimg, Ho, opad, oHp, oWp, oCw;
  int Kreal;
};

// One nibble plane of four words of bits as the four operand dwords of one MFMA: bit 4 i + n of a dword in nibble i, worth 0.5, 1 or
// 2 where it comes to lie, in A (B_SIDE: in B) so that the product of two set bits is worth 1 in every plane and no MFMA needs block
// scales: planes 0 to 3 stand at 0.5, 1, 2 and 1 in A, at 2, 1, 0.5 and 1 in B.
template <bool B_SIDE>
__device__ __forceinline__ v8i nibble_plane(const uint4& w, int n) {
  auto at = [&](uint32_t v) {
    if (n == 1) return (int)(v & 0x22222222u);
    if (n == 3) return (int)(v >> 2 & 0x22222222u);
    if (B_SIDE) return (int)(n == 0 ? v << 2 & 0x44444444u : v >> 2 & 0x11111111u);
    return (int)(v & 0x11111111u << n);
  };
  return v8i{at(w.x), at(w.y), at(w.z), at(w.w), 0, 0, 0, 0};
}

// Two bit planes of 2-bit activations folded into values p1 * 2 + p0: those of the even bits in `even`, of the odd ones in `odd`, each
// at an even place; four instructions, and six more for the four nibble planes below (taken bit by bit from both, fourteen).
__device__ __forceinline__ void fold_planes(const uint4& p0, const uint4& p1, uint4* even, uint4* odd) {
  auto fold = [](uint32_t lo, uint32_t hi) { return (lo & 0x55555555u) | (hi & 0xaaaaaaaau); };
  *even = make_uint4(fold(p0.x, p1.x << 1), fold(p0.y, p1.y << 1), fold(p0.z, p1.z << 1), fold(p0.w, p1.w << 1));
  *odd = make_uint4(fold(p0.x >> 1, p1.x), fold(p0.y >> 1, p1.y), fold(p0.z >> 1, p1.z), fold(p0.w >> 1, p1.w));
}

// Nibble plane n of the folded planes: nibble i of a dword = the value of bit 4 i + n, worth half of itself (E2M1 codes 0 to 3 = 0,
// 0.5, 1, 1.5), and the bits of B that go with it where they stand, worth 0.5, 1, 2 and 0.5.
__device__ __forceinline__ v8i value_plane(const uint4& even, const uint4& odd, int n) {
  const uint4& w = n & 1 ? odd : even;
  auto at = [&](uint32_t v) { return (int)(v >> (n & 2) & 0x33333333u); };
  return v8i{at(w.x), at(w.y), at(w.z), at(w.w), 0, 0, 0, 0};
}
__device__ __forceinline__ v8i bit_plane(const uint4& w, int n) {
  auto at = [&](uint32_t v) { return (int)(n == 3 ? v >> 3 & 0x11111111u : v & 0x11111111u << n); };
  return v8i{at(w.x), at(w.y), at(w.z), at(w.w), 0, 0, 0, 0};
}

// acc + popcount of four words: four v_bcnt_u32_b32, each adding onto the running count (written
// as a sum of __builtin_popcount the compiler counts from zero and adds with extra instructions)
__device__ __forceinline__ int add_popcount4(int acc, const uint4& w) {
  asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"(w.x));
  asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"(w.y));
  asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"(w.z));
  asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"(w.w));
  return acc;
}

__device__ __forceinline__ bool runs_meet(const Fp4Params& p, int seg) {
  return bmx::runs_meet(p.run, [&](uint32_t x) { return fast_div(x, p.div_two_runs); }, seg);
}

// Request segment `seg` (64 bytes of every row of the wave's NB staged blocks) into the staging
// area at dst: per block two loads of 16 rows, lane i of a load writing LDS bytes [16 i, 16 i + 16)
// of its destination.  voff: a lane's byte offset of its piece in segment 0 of its row and 16 (CONV: without the 16, and for
// the B blocks, of its pixel's patch; the piece's place inside the patch is found here).  ODD: runs may be of an odd number of words;
// the segments that two of them meet in, one or two of 8 with 3 x 3 filters over 7 words, pass registers (nx, B's blocks) a word at a
// time, and the caller writes them to the same places when it gets to them.
template <int NA, int NB, bool CONV, bool ODD>
__device__ __forceinline__ void issue_segment(const Fp4Params& p, uint4* dst, const uint32_t* voff /* [NB][2] */,
                                              int piece0, int piece1, int seg, uint4* nx /* [NB - NA][2] */) {
  if constexpr (!CONV) {
    // (A and B are 16 bytes lower than the operands and voff 16 more, so that no offset is below zero, which would be one of 4 GB.
    // One set of loads for all segments: with one of its own for a row's last 2752 x 1984 x 1408 took 9.0 us and not 8.1.)
    const char* const abase = (const char*)p.A + (uint32_t)seg * 64u;
    const char* const bbase = (const char*)p.B + (uint32_t)seg * 64u;
    const uint32_t back[2] = {piece_back(seg, piece0, p.Kd), piece_back(seg, piece1, p.Kd)};
#pragma unroll
    for (int b = NB - 1; b >= 0; --b)  // (B first: its rows are the ones that come from far away)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        __builtin_amdgcn_global_load_lds((b < NA ? abase : bbase) + (voff[2 * b + t] - back[t]), (lds_ptr)(dst + b * 128 + t * 64), 16, 0, 0);
    return;
  }
  const char* abase = (const char*)p.A + (uint32_t)seg * 64u;
  const bool tail = 8 * seg + 8 > p.Kw;  // the row ends inside this segment
  const bool by_words = ODD && runs_meet(p, seg);
  uint32_t boff[2] = {0u, 0u};
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    // piece c of the im2col row, from word 2 c on: run 2 c / run (a kernel row).  A piece beyond the row's last is not fetched (the
    // reader zeroes it): its lane repeats the segment's first piece, which always exists
    uint32_t w = 8u * (uint32_t)seg + 2u * (uint32_t)(t ? piece1 : piece0);
    if (w >= (uint32_t)p.Kw) w = 8u * (uint32_t)seg;
    const uint32_t run = fast_div(w, p.div_run);
    boff[t] = run * p.row_bytes + (w - run * p.run) * 8u;
  }
#pragma unroll
  for (int b = NB - 1; b >= 0; --b)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int pc = t ? piece1 : piece0;
      uint32_t off = voff[2 * b + t];
      if (b >= NA) off += boff[t];
      // (filters) a piece that starts beyond the row's last word: repeat the segment's first
      else if (tail && 8 * seg + 2 * pc >= p.Kw) off -= 16u * pc;
      if (b < NA || !by_words)
        __builtin_amdgcn_global_load_lds((b < NA ? abase : (const char*)p.B) + off, (lds_ptr)(dst + b * 128 + t * 64), 16, 0, 0);
    }
  if (by_words) {
    // (words past the row repeat its last, the reader zeroes them)
    uint32_t woff[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t w = (uint32_t)min(8 * seg + 2 * (t ? piece1 : piece0) + e, p.Kw - 1), run = fast_div(w, p.div_run);
        woff[t][e] = run * p.row_bytes + (w - run * p.run) * 8u;
      }
#pragma unroll
    for (int b = NB - 1; b >= NA; --b)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const uint2 lo = *(const uint2*)((const char*)p.B + (voff[2 * b + t] + woff[t][0]));
        const uint2 hi = *(const uint2*)((const char*)p.B + (voff[2 * b + t] + woff[t][1]));
        nx[2 * (b - NA) + t] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
  }
}

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Four results in a row, `off` bytes behind an address that the wave shares.  NT: past the caches.  (As asm: as a builtin the
// compiler merges the hinted store with the ordinary one of the other branch, and the hint is gone.  What follows a 16-byte store
// may not write its registers in the next instruction, which the compiler sees to only where it knows of the store.)
// (BMX_FP4_STAMPS: the stamps' branches make the compiler take the wave's address for the lanes': plain stores in that build.
// With the address put back into scalar registers ahead of each, the asm would want five wait states there)
__device__ __forceinline__ void store_four(char* to, uint32_t off, const v4u& v, bool nt) {
#ifdef BMX_FP4_STAMPS
  *(v4u_any*)(to + off) = v;
  return;
#endif
  if (nt) asm volatile("global_store_dwordx4 %0, %1, %2 nt\n\ts_nop 1" ::"v"(off), "v"(v), "s"(to) : "memory");
  else asm volatile("global_store_dwordx4 %0, %1, %2\n\ts_nop 1" ::"v"(off), "v"(v), "s"(to) : "memory");
}

// The lane's two results of one row, `off0` and `off1` bytes behind an address that the wave shares (its part of the address is
// scalar work).  NT as above; MASKED: each only where `left0`, `left1` say that more than `e` rows are left of its column, an
// instruction and three scalar ones a result.
template <bool NT, bool MASKED>
__device__ __forceinline__ void store_two(char* to, uint32_t off0, uint32_t off1, int left0, int left1, int e, uint32_t v0, uint32_t v1) {
#ifdef BMX_FP4_STAMPS
  if (!MASKED || e < left0) *(uint32_t*)(to + off0) = v0;
  if (!MASKED || e < left1) *(uint32_t*)(to + off1) = v1;
  return;
#endif
  if constexpr (MASKED) {
    uint64_t all;
    asm volatile("s_mov_b64 %0, exec\n\tv_cmp_lt_i32_e32 vcc, %8, %3\n\ts_and_b64 exec, %0, vcc\n\tglobal_store_dword %1, %5, %7\n\ts_mov_b64 exec, %0\n\t"
                 "v_cmp_lt_i32_e32 vcc, %8, %4\n\ts_and_b64 exec, %0, vcc\n\tglobal_store_dword %2, %6, %7\n\ts_mov_b64 exec, %0"
                 : "=&s"(all)
                 : "v"(off0), "v"(off1), "v"(left0), "v"(left1), "v"(v0), "v"(v1), "s"(to), "n"(e)
                 : "vcc", "scc", "memory");
  } else if constexpr (NT) {
    asm volatile("global_store_dword %0, %2, %4 nt\n\tglobal_store_dword %1, %3, %4 nt" ::"v"(off0), "v"(off1), "v"(v0), "v"(v1), "s"(to) : "memory");
  } else {
    asm volatile("global_store_dword %0, %2, %4\n\tglobal_store_dword %1, %3, %4" ::"v"(off0), "v"(off1), "v"(v0), "v"(v1), "s"(to) : "memory");
  }
}

// x / 3 as division rounds it (Markstein: the quotient from the rounded reciprocal, corrected by the remainder; equal for every
// whole number below 2^24)
__device__ __forceinline__ float third(float x) {
  const float q = x * (1.0f / 3.0f);
  return fmaf(fmaf(-3.0f, q, x), 1.0f / 3.0f, q);
}

#ifdef BMX_FP4_STAMPS
// Profiling builds only: per-wave shader-clock stamps at the phase boundaries of the kernel.
}  // namespace
unsigned long long* fp4_stamps = nullptr;
namespace {
#define FP4_STAMP(k) do { if (stamps && lane == 0) stamps[(size_t)(blockIdx.x * (blockDim.x >> 6) + wave) * 8 + (k)] = __builtin_readcyclecounter(); } while (0)
// (without a split, slots 4 and 5 take the constant 100 MHz counter at the loop's ends: with the shader-clock stamps 1 and 3 that gives the clock the loop ran at)
#define FP4_REALTIME(k) do { if (!SPLIT && stamps && lane == 0) stamps[(size_t)(blockIdx.x * (blockDim.x >> 6) + wave) * 8 + (k)] = __builtin_amdgcn_s_memrealtime(); } while (0)
#else
#define FP4_REALTIME(k) do { } while (0)
#define FP4_STAMP(k) do { } while (0)
#endif

// Output kinds of the xnor form (the plane form stores S and / or S / levels as its pointers say).
constexpr int kOutF32 = 0, kOutI32 = 1, kOutBits = 2;

// TM x TN blocks of 32 x 32 per wave
constexpr int TM = 2, TN = 2;
// where the MFMA sums of HALF start: from here on the low bits of the fp32 number are the sum
constexpr float kBias = 8388608.0f;

// uint4 of a wave's partial tile: 64 rows of 32 dwords (pairs of 16-bit numbers, columns c and c + 32) or 64, behind them the
// popcounts of the columns in a row like those and of the rows in 64 dwords
constexpr int tab_row(bool half) { return half ? 8 : 16; }
constexpr int slot_size(int pl, bool split, bool half) { return std::max((TM * pl + TN) * 128, split ? 65 * tab_row(half) + 16 : 0); }

// PL bit planes per A row; XNOR: the xnor form (row popcounts from the words themselves), else the plane form (row sums given); OUT: what the
// xnor form stores; SPLIT: K split over the S waves of the workgroup (else a tile per wave);
// HALF: the partial tiles of a split cross LDS as pairs of 16-bit whole numbers (full sums up to 65535,
// which the launcher checks); CONV: the convolution form (see Fp4Params); ODD:
// its runs have an odd number of words (see issue_segment; "reg" in the kernel's name).
// One instantiation per combination keeps each kernel's code short: the instruction cache
// starts cold at every launch, and a launch lasts a few microseconds.
template <int PL, bool XNOR, int OUT, bool SPLIT, bool HALF, bool CONV, bool ODD>
__global__ void __launch_bounds__(512)
gemm_fp4_kernel(const Fp4Params p, const int S_arg
#ifdef BMX_FP4_STAMPS
                , unsigned long long* stamps
#endif
) {
  extern __shared__ uint4 lds[];
  constexpr int NA = TM * PL, NB = NA + TN;  // staged blocks of 32 rows: A's, then B's
  // LDS per wave: its staging area, overlaid after the main loop of a split by its partial tile and counts
  constexpr int kSlot = slot_size(PL, SPLIT, HALF);
  // Everything the wave needs before its first load, named in one statement at the top: the
  // compiler then fetches the kernel arguments in one batch of scalar loads with one wait instead
  // of one memory round trip per group of first uses.
  asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.lda_bytes), "s"(p.ldb_bytes), "s"(p.M), "s"(p.N), "s"(p.Kw), "s"(p.Kd), "s"(p.g_base),
               "s"(p.g_rem), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.tiles_per_xcd), "s"(p.band), "s"(p.per_band),
               "s"(p.last_band), "s"(p.last_rows), "s"(p.div_per_band.mul), "s"(p.div_per_band.sh1),
               "s"(p.div_per_band.sh2), "s"(p.div_band.mul), "s"(p.div_band.sh1), "s"(p.div_band.sh2),
               "s"(p.div_last.mul), "s"(p.div_last.sh1), "s"(p.div_last.sh2), "s"(S_arg), "s"(p.alpha), "s"(p.thr), "s"(p.rowsum));
  const int S = SPLIT ? S_arg : 1;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;
  FP4_STAMP(0);
  const int ks = SPLIT ? wave : 0;          // this wave's part of K
  const int tile_in_wg = SPLIT ? 0 : wave;  // without a split every wave has a tile of its own
  const int tiles_per_wg = SPLIT ? 1 : (int)(blockDim.x >> 6);
  // workgroup b sits on XCD b % 8: give every XCD a contiguous run of tiles, rows of C fastest
  const int lin = ((int)(blockIdx.x & 7) * p.tiles_per_xcd + (int)(blockIdx.x >> 3)) * tiles_per_wg + tile_in_wg;
  if (lin >= p.tiles_m * p.tiles_n) return;  // (a whole workgroup of a split; without one there is no barrier ahead)
  // Within an XCD's run the tiles go band by band: a band is `band` rows of tiles high, and
  // inside it the rows of C run fastest, so the few hundred tiles in flight on an XCD at any time
  // form a block about as wide as high and share their operand rows through its L2.
  // (divisions by multiply-high with constants from the host: this runs before the first load)
  const int bnd = (int)fast_div((uint32_t)lin, p.div_per_band), within = lin - bnd * p.per_band;
  const bool last = bnd == p.last_band;
  const int tile_n = (int)fast_div((uint32_t)within, last ? p.div_last : p.div_band);
  const int tile_m = bnd * p.band + (within - tile_n * (last ? p.last_rows : p.band));
  const int m0 = tile_m * (32 * TM), n0 = tile_n * (32 * TN);

  // ---- this wave's K range in groups of four words.  The first g_rem waves carry one group
  // more: waves w and w + 4 share a SIMD, so with the extras up front the SIMDs stay level (36
  // groups over 8 waves: 5 5 5 5 4 4 4 4, nine per SIMD).
  const int g_lo = ks * p.g_base + min(ks, p.g_rem), g_hi = g_lo + p.g_base + (ks < p.g_rem ? 1 : 0);
  const int seg_lo = g_lo >> 1, seg_hi = (g_hi + 1) >> 1;  // 64-byte segments [seg_lo, seg_hi) of two groups

  // ---- loader: lane i of load t of a block fetches, for local row 16 t + i / 4, the piece
  // (i % 4) xor ((row >> 1) & 3) of the segment; voff = byte offset of that piece in segment 0 (products: and 16, see issue_segment).
  uint4* const stage = lds + wave * kSlot;
  int piece[2];
  uint32_t voff[NB][2];
#pragma unroll
  for (int t = 0; t < 2; ++t) piece[t] = (lane & 3) ^ (((16 * t + (lane >> 2)) >> 1) & 3);
#pragma unroll
  for (int b = NB - 1; b >= 0; --b)  // (B first: its rows are the ones that come from far away)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int rl = 16 * t + (lane >> 2);
      if (b < NA) {  // block b = row block b / PL, plane b % PL
        const int m = min(m0 + 32 * (b / PL) + rl, p.M - 1);
        voff[b][t] = (uint32_t)(m * PL + (b % PL)) * p.lda_bytes + 16u * piece[t] + (CONV ? 0u : 16u);
      } else {
        const int n = min(n0 + 32 * (b - NA) + rl, p.N - 1);
        if (CONV) {  // byte offset of the pixel's patch: tap (0, 0), channel word 0
          const uint32_t img = fast_div((uint32_t)n, p.div_howo);
          const uint32_t rem = (uint32_t)n - img * (uint32_t)p.HoWo;
          const uint32_t ho = fast_div(rem, p.div_wo);
          const uint32_t wo = rem - ho * (uint32_t)p.Wo;
          voff[b][t] = (((img * (uint32_t)p.Hp + ho * (uint32_t)p.stride) * (uint32_t)p.Wpp + wo * (uint32_t)p.stride) *
                        (uint32_t)p.Cw) * 8u;
        } else {
          voff[b][t] = (uint32_t)n * p.ldb_bytes + 16u * piece[t] + 16u;
        }
      }
    }
  // reader: lane (r, h) takes piece 2 g + h of row r for group g of the segment
  int rd[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) rd[g] = (r >> 4) * 64 + (r & 15) * 4 + ((2 * g + h) ^ ((r >> 1) & 3));

  // The epilogue's constants are requested first of all (fetched where they are used, each would
  // put a trip to memory between the main loop and the stores; and ahead of the segments'
  // loads they do not disturb the count of loads in flight that the main loop relies on).  Alpha and the threshold of the sign
  // decision of this lane's columns: of a split columns lcol to lcol + 3 and 32 more of the tile, else r and 32 + r; per row of the
  // tile (64 of them), row m0 + l in lane l: the row sum of the plane form, alpha and threshold of the convolution form.
  // (undivided, plain variables: indexed by a run-time number an array is put into scratch memory, whose every access also waits
  // for the stores issued before it)
  const int lcol = 4 * (lane & 7);
  const bool inside_n = n0 + 64 <= p.N;
  auto of_columns = [&](const float* from, float none, v4f_any (&v)[2]) {
    v[0] = v[1] = v4f_any{none, none, none, none};
    if (!SPLIT || !from) return;
    if (inside_n) {
      v[0] = *(const v4f_any*)(from + n0 + lcol);
      v[1] = *(const v4f_any*)(from + n0 + 32 + lcol);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e >> 2][e & 3] = from[min(n0 + 32 * (e >> 2) + lcol + (e & 3), p.N - 1)];
    }
  };
  v4f_any al_c[2], th_c[2];
  constexpr bool kAlpha = XNOR && !CONV && OUT != kOutI32, kThr = XNOR && !CONV && OUT == kOutBits;
  of_columns(kAlpha ? p.alpha : nullptr, 1.0f, al_c);
  of_columns(kThr ? p.thr : nullptr, 0.0f, th_c);
  const int n_c0 = min(n0 + r, p.N - 1), n_c1 = min(n0 + 32 + r, p.N - 1);
  float aln0 = !SPLIT && kAlpha && p.alpha ? p.alpha[n_c0] : 1.0f;
  float aln1 = !SPLIT && kAlpha && p.alpha ? p.alpha[n_c1] : 1.0f;
  float thn0 = !SPLIT && kThr && p.thr ? p.thr[n_c0] : 0.0f;
  float thn1 = !SPLIT && kThr && p.thr ? p.thr[n_c1] : 0.0f;
  const int rowsum_lane = XNOR ? 0 : p.rowsum[min(m0 + lane, p.M - 1)];
  const float alpha_lane = (CONV && p.alpha) ? p.alpha[min(m0 + lane, p.M - 1)] : 1.0f;
  const float thr_lane = (CONV && OUT == kOutBits && p.thr) ? p.thr[min(m0 + lane, p.M - 1)] : 0.0f;

  uint4 nx[2 * TN];  // ODD
  if (seg_lo < seg_hi) issue_segment<NA, NB, CONV, ODD>(p, stage, &voff[0][0], piece[0], piece[1], seg_lo, nx);
  if constexpr (CONV && OUT == kOutBits) {
    // word tile_m of the output image's halo, spread over the tiles of this row of tiles
    if (p.opad > 0) {
      const int per_tile = SPLIT ? (int)blockDim.x : 64;
      write_halo((uint64_t*)p.C_bits, p.Nimg, p.Ho, p.Wo, p.opad, p.M, p.oCw, tile_m,
                 tile_n * per_tile + (SPLIT ? threadIdx.x : lane), p.tiles_n * per_tile);
    }
  }
  FP4_STAMP(1);
  FP4_REALTIME(4);

  v16f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = SPLIT && HALF ? kBias : 0.0f;
  int pa[TM], pb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) pa[i] = 0;
#pragma unroll
  for (int j = 0; j < TN; ++j) pb[j] = 0;

  for (int seg = seg_lo; seg < seg_hi; ++seg) {
    // the segment's words into registers (the compiler waits for the loads in flight: it tracks
    // LDS writes of the load unit)
    if (ODD && runs_meet(p, seg)) {
#pragma unroll
      for (int k = 0; k < 2 * TN; ++k) stage[NA * 128 + k * 64 + lane] = nx[k];
    }
    uint4 w[NB][2];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int g = 0; g < 2; ++g) w[b][g] = stage[b * 128 + rd[g]];
    if (!CONV && 16 * seg + 16 > p.Kd) {  // last segment of a row that ends inside it (see issue_segment): what stands in front of a
                                           // part piece's dwords, and all past the row, is zero
      const bool back = p.Kd >= 4;         // (in a row of less than a piece, what stands behind them)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int left = p.Kd - (16 * seg + 4 * (2 * g + h));  // dwords of this lane's piece
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          if (left < (back ? 4 : 1)) w[b][g].x = 0;
          if (left < (back ? 3 : 2)) w[b][g].y = 0;
          if (left < (back ? 2 : 3)) w[b][g].z = 0;
          if (left < (back ? 1 : 4)) w[b][g].w = 0;
        }
      }
    }
    if (CONV && 8 * seg + 8 > p.Kw) {  // words past the row are zero
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const int left = p.Kw - (8 * seg + 2 * (2 * g + h));  // valid words of this lane's piece
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          if (left < 2) w[b][g].z = w[b][g].w = 0;
          if (left < 1) w[b][g].x = w[b][g].y = 0;
        }
      }
    }
    // The next segment is requested before this one is multiplied, into the area just read.  Its
    // loads must not land on words that are still to be read, and a read that has merely been
    // issued may still wait in the LDS queue behind those of the CU's other waves when the data
    // arrives (a few hundred cycles for an L2 hit; seen as a few wrong counts in a chip-filling
    // GEMM): the reads are waited for first.  (A second area per wave used in turn, which needs
    // no wait, and two segments' loads in flight on top of that, with counted waits written out
    // because the compiler waits for every pending load of the load unit before an LDS read it
    // knows of, both measured no faster with operands that really come from HBM: 9.5 and 9.9
    // against 9.5 us on the first fully connected layer.)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#ifdef BMX_FP4_STAMPS
    if (seg == seg_lo) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); FP4_STAMP(2); }
#endif
    if (seg + 1 < seg_hi) issue_segment<NA, NB, CONV, ODD>(p, stage, &voff[0][0], piece[0], piece[1], seg + 1, nx);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int kg = 2 * seg + g;
      if (kg < g_lo || kg >= g_hi) continue;  // wave-uniform: a range may start or end mid-segment
      if (XNOR) {
#pragma unroll
        for (int i = 0; i < TM; ++i) pa[i] = add_popcount4(pa[i], w[i][g]);
#pragma unroll
        for (int j = 0; j < TN; ++j) pb[j] = add_popcount4(pb[j], w[NA + j][g]);
      }
      // One bit plane: unscaled MFMAs (with block scales one takes 17 clocks of its SIMD's issue, without 11, and the shifts that bring
      // every plane's products to 1 cost less than that).  Two: E8M0 block scales, as the 2-bit values stand at one weight only and
      // B's bits would all have to be shifted (level at 1024 x 1024 x 4096, 1.3 % behind at 1553 x 1344 x 4096).
      auto mfma = [](const v8i& x, const v8i& y, const v16f& z, int n) {
        if constexpr (PL == 1) return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, z, 4, 4, 0, 0, 0, 0);
        else return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, z, 4, 4, 0, 128, 0, n == 1 ? 127 : n == 2 ? 126 : 128);
      };
      uint4 even[TM], odd[TM];
      if constexpr (PL == 2) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fold_planes(w[2 * i][g], w[2 * i + 1][g], &even[i], &odd[i]);
      }
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        v8i eb[TN], ea[TM];
#pragma unroll
        for (int j = 0; j < TN; ++j) eb[j] = PL == 2 ? bit_plane(w[NA + j][g], n) : nibble_plane<true>(w[NA + j][g], n);
#pragma unroll
        for (int i = 0; i < TM; ++i) ea[i] = PL == 2 ? value_plane(even[i], odd[i], n) : nibble_plane<false>(w[i][g], n);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma(ea[i], eb[j], acc[i][j], n);
      }
    }
  }
  FP4_STAMP(3);
  FP4_REALTIME(5);
  // The constants requested before the loop are taken in here, in one place: met for the first
  // time in the branches of the epilogue, each would get a wait of its own there, and such a
  // wait also sits out every store issued before it.  The same for the arguments that only the epilogue
  // reads: fetched where they are used, each is a trip to memory with the stores waiting behind it.
  if constexpr (SPLIT) asm volatile("" : "+v"(al_c[0]), "+v"(al_c[1]), "+v"(th_c[0]), "+v"(th_c[1]));
  else asm volatile("" : "+v"(aln0), "+v"(aln1), "+v"(thn0), "+v"(thn1));
  int rowsum_l = rowsum_lane;
  float alpha_l = alpha_lane, thr_l = thr_lane;
  asm volatile("" : "+v"(rowsum_l), "+v"(alpha_l), "+v"(thr_l));
  const int M = p.M, N = p.N, Kreal = p.Kreal, as_count = OUT == kOutI32 ? p.as_count : 0, nt = p.nt;
  char* const C = OUT == kOutBits ? (char*)p.C_bits : XNOR && OUT == kOutI32 ? (char*)p.C_i32 : (char*)p.C_f32;
  char* const C2 = XNOR ? nullptr : (char*)p.C_i32;  // (the plane form stores either or both)

  // ---- epilogue.  Register v of lane (r, h) in block (i, j) is C[32 i + 8 (v / 4) + 4 h + v % 4][32 j + r].
  // Results are 32-bit elements, elems from row to row; row m0 of the tile (CONV: that channel of the image of the tile's first
  // pixel) is the wave's, a lane's rows and columns lie behind it by less than 2^32 bytes (the launchers see to it).
  const uint32_t elems = CONV ? (uint32_t)p.HoWo : (uint32_t)p.ldc;
  uint64_t at0 = (uint64_t)((uint32_t)m0 * elems) * 4u;
  uint32_t img0 = 0;
  if (CONV) {
    img0 = __builtin_amdgcn_readfirstlane(fast_div((uint32_t)n0, p.div_howo));
    at0 += (uint64_t)(img0 * (uint32_t)M) * elems * 4u;
  }
  auto place = [&](int row, int n, bool* whole) -> uint32_t {  // whole: columns n to n + 3 are there, in a row
    if (!CONV) {
      *whole = n + 3 < N;
      return ((uint32_t)row * elems + (uint32_t)n) * 4u;
    }
    const uint32_t m = (uint32_t)min(n, N - 1), img = fast_div(m, p.div_howo), rem = m - img * elems;
    *whole = n + 3 < N && rem + 3 < elems;
    return (((img - img0) * (uint32_t)M + (uint32_t)row) * elems + rem) * 4u;
  };
  // packed bits of the convolution form: word tile_m of pixel n0 + lane of the tile, filter m0 in its bit 0
  auto store_word = [&](uint64_t word) {
    if (n0 + lane >= N) return;
    const uint32_t img = fast_div((uint32_t)(n0 + lane), p.div_howo), rem = (uint32_t)(n0 + lane) - img * elems;
    const uint32_t ho = fast_div(rem, p.div_wo), wo = rem - ho * (uint32_t)p.Wo;
    ((uint64_t*)C)[((img * (uint32_t)p.oHp + ho + (uint32_t)p.opad) * (uint32_t)p.oWp + wo + (uint32_t)p.opad) * (uint32_t)p.oCw + (uint32_t)tile_m] = word;
  };
  // Popcounts: a lane counted its half of a group for row / column r of every block; one exchange of half waves and one addition
  // leave row l and column l of the tile with lane l.
  int row_l = 0, col_l = 0;
  if (XNOR) {
    const auto sa = __builtin_amdgcn_permlane32_swap(pa[0], pa[1], false, false);
    const auto sb = __builtin_amdgcn_permlane32_swap(pb[0], pb[1], false, false);
    row_l = (int)(sa[0] + sa[1]);
    col_l = (int)(sb[0] + sb[1]);
  }
  // A result is its row's term - its column's term + (the sum << mul).  xnor: K - 2 pc(a) - 2 pc(b) + 4 sum (the count of equal
  // bits: K - pc(a) - pc(b) + 2 sum); planes: 2 sum - the row sum of the activations.
  const int mul = XNOR ? 2 - (as_count != 0) : 1;
  auto result = [&](int d, float al) {  // what is stored for it (C)
    if (XNOR && OUT == kOutI32) return (uint32_t)d;
    if (XNOR) return __float_as_uint(al * (float)d);
    return __float_as_uint(PL == 2 ? third((float)d) : (float)d);
  };

  if constexpr (!SPLIT) {
    // The row terms of every result register first (a shuffle each: fetched one by one between the stores, each would cost an LDS
    // round trip), then arithmetic and stores, a row of 64 results at a time, tiles that lie inside C without any bounds (5248 x 384 x
    // 2048 6.95 us, masked 7.85; a store takes the load unit 16 clocks, which leaves a wave room for little else).  Through LDS for
    // stores of 16 bytes a lane, as below, they are a quarter as many, but behind a trip through LDS: 4160 x 1056 x 128 6.36 / 6.52 us,
    // 5248 x 384 x 2048 6.95 / 7.76, and rows of C that are not 16-byte aligned fall back further.
    const int row_t = XNOR ? Kreal - (row_l << (mul - 1)) : -rowsum_l;
    int ct[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) ct[j] = XNOR ? __shfl(col_l << (mul - 1), 32 * j + r) : 0;
    int rt[TM][16];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) rt[i][v] = __shfl(row_t, 32 * i + 8 * (v >> 2) + 4 * h + (v & 3));
    if constexpr (CONV && OUT == kOutBits) {
      uint32_t half[TN][TM];  // of pixel 32 j + r: filters 32 i .. 32 i + 31
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) half[j][i] = 0u;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int bit = 8 * (v >> 2) + 4 * h + (v & 3), mi = 32 * i + bit;
          const float al = __shfl(alpha_l, mi), th = __shfl(thr_l, mi);
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const float dot = (float)(rt[i][v] - ct[j] + ((int)acc[i][j][v] << mul));
            if (m0 + mi < M && al * dot >= th) half[j][i] |= 1u << bit;
          }
        }
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) half[j][i] |= (uint32_t)__shfl_xor((int)half[j][i], 32);
      store_word((uint64_t)(h ? half[1][1] : half[0][1]) << 32 | (h ? half[1][0] : half[0][0]));
    } else if constexpr (OUT == kOutBits) {
      // The 64-lane mask of a sign decision: its low half is 32 columns of a row, its high half the same columns of the row four below.
      // Either goes to the lane of its row, which then has the row's word: one store a tile.  (A store of each half by a lane of its
      // own, under its own condition and with its own address, made 64 of them: 4 us of a launch of 7.9, 1844 x 448 x 192.)
      const float al0 = n0 + r < N ? aln0 : 0.0f, al1 = n0 + 32 + r < N ? aln1 : 0.0f;  // (no bit past the last column)
      const float th0 = n0 + r < N ? thn0 : 1.0f, th1 = n0 + 32 + r < N ? thn1 : 1.0f;
      uint32_t w[TN] = {0u, 0u};
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int row = 32 * i + 8 * (v >> 2) + (v & 3);
            const float dot = (float)(rt[i][v] - ct[j] + ((int)acc[i][j][v] << mul));
            const uint64_t mask = __ballot((j ? al1 : al0) * dot >= (j ? th1 : th0));
            w[j] = write_lane((uint32_t)mask, row, w[j]);
            w[j] = write_lane((uint32_t)(mask >> 32), row + 4, w[j]);
          }
      if (m0 + lane < M) ((uint64_t*)C)[(uint32_t)(m0 + lane) * elems + (uint32_t)(n0 >> 6)] = (uint64_t)w[1] << 32 | w[0];
    } else {
      bool whole;
      const uint32_t off0 = place(4 * h, n0 + r, &whole), off1 = place(4 * h, n0 + 32 + r, &whole);
      // rows of the result from the lane's first on; none where its column lies outside
      const int left0 = n0 + r < N ? M - m0 - 4 * h : 0, left1 = n0 + 32 + r < N ? M - m0 - 4 * h : 0;
      float alm[TM][16];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) alm[i][v] = CONV && OUT == kOutF32 ? __shfl(alpha_l, 32 * i + 8 * (v >> 2) + 4 * h + (v & 3)) : 1.0f;
      const uint64_t pitch = (uint64_t)elems * 4u;
      auto store_tile = [&](auto nt_tag, auto masked_tag) {
        constexpr bool NT = decltype(nt_tag)::value, MASKED = decltype(masked_tag)::value;
#pragma unroll
        for (int g = 0; g < TM * 4; ++g) {  // four rows of either half wave
          const int i = g >> 2, q = g & 3, row = 8 * g;
          if (MASKED && m0 + row >= M) break;
          char* to = C + at0 + (uint64_t)(uint32_t)row * pitch;
          char* to2 = C2 + at0 + (uint64_t)(uint32_t)row * pitch;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int v = 4 * q + e;
            const int d0 = rt[i][v] - ct[0] + ((int)acc[i][0][v] << mul), d1 = rt[i][v] - ct[1] + ((int)acc[i][1][v] << mul);
            const uint32_t v0 = result(d0, CONV ? alm[i][v] : aln0), v1 = result(d1, CONV ? alm[i][v] : aln1);
            if (XNOR || C) store_two<NT, MASKED>(to, off0, off1, left0 - row, left1 - row, e, v0, v1);
            if (!XNOR && C2) store_two<NT, MASKED>(to2, off0, off1, left0 - row, left1 - row, e, (uint32_t)d0, (uint32_t)d1);
            to += pitch;
            to2 += pitch;
          }
        }
      };
      // (Rows that are parts of lines, from several workgroups a CU at once: stored as fast as a wave can, the parts get in each
      // other's way, and the bounds' instructions are the better pace: 4000 x 4001 x 128 13.7 / 14.7 us, 3520 x 6492 x 92 17.5 / 18.7;
      // with at most one a CU 896 x 3384 x 5120 13.9 / 13.3, 640 x 3367 x 2532 9.15 / 8.6.)
      if (m0 + 32 * TM > M || n0 + 32 * TN > N || (!nt && (int)gridDim.x * tiles_per_wg > 1024)) store_tile(std::false_type{}, std::true_type{});
      else if (nt) store_tile(std::true_type{}, std::false_type{});
      else store_tile(std::false_type{}, std::false_type{});
    }
    return;
  }

  // ---- K split: every wave writes its part of every sum and its popcounts over its own staging area; a wave then finishes every
  // S-th block of eight rows, adding up S parts, a lane four columns in a row and the four 32 further on: two stores of 16 bytes a
  // lane for eight results, whole 128-byte lines, where stores from the MFMA's registers, a dword a lane, are four times as many
  // (the load unit takes one in 16 clocks).  Row 8 b + 4 h + 2 e1 + e0 of the tile stands at place 8 b + 4 e0 + 2 e1 + h, so that
  // the half waves write to different banks.
  constexpr int kRow = tab_row(HALF);
  u_alias* const tab = (u_alias*)(lds + wave * kSlot);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      u_alias* const to = tab + (32 * i + 8 * (v >> 2) + 4 * (v & 1) + 2 * ((v >> 1) & 1) + h) * (4 * kRow) + r;
      const uint32_t c0 = __float_as_uint(acc[i][0][v]), c1 = __float_as_uint(acc[i][1][v]);
      // (HALF: the sums were started at kBias: a whole number below 2^16 stands in the low half of its register)
      if constexpr (HALF) to[0] = __builtin_amdgcn_perm(c1, c0, 0x05040100u);
      else to[0] = c0, to[32] = c1;
    }
  if (XNOR) {
    if constexpr (HALF) ((u16_alias*)(tab + 64 * 4 * kRow))[2 * r + h] = (uint16_t)col_l;
    else tab[64 * 4 * kRow + lane] = (uint32_t)col_l;
    tab[65 * 4 * kRow + lane] = (uint32_t)row_l;
  }
  // this lane's places: row 8 b + mrow of the tile in block b, columns lcol + 32 k + e
  const int mrow = 4 * (lane >> 3 & 1) + 2 * (lane >> 4 & 1) + (lane >> 5);
  bool whole0 = false, whole1 = false;
  uint32_t off0 = 0, off1 = 0;
  if (OUT != kOutBits) {
    off0 = place(mrow, n0 + lcol, &whole0);
    off1 = place(mrow, n0 + lcol + 32, &whole1);
  }
  const int rows_left = M - m0 - mrow;  // of the lane's row in block 0 on
  auto put = [&](char* base, int b, const uint32_t (&v)[8]) {
    char* const to = base + at0 + (uint64_t)(uint32_t)(8 * b) * elems * 4u;
    if (8 * b >= rows_left) return;
    auto four = [&](bool whole, uint32_t off, int n, const uint32_t* d) {
      if (whole) {
        store_four(to, off, v4u{d[0], d[1], d[2], d[3]}, nt);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bool one;
          if (n + e < N) *(uint32_t*)(to + (CONV ? place(mrow, n + e, &one) : off + 4u * e)) = d[e];
        }
      }
    };
    four(whole0, off0, n0 + lcol, v);
    four(whole1, off1, n0 + lcol + 32, v + 4);
  };
  // packed bits of the convolution form: a byte per block of rows and pixel
  u8_alias* const bytes = (u8_alias*)(lds + S * kSlot);
  __syncthreads();
  FP4_STAMP(4);
  // WAVES: how many share K, 8 and 4 (the usual cases) as constants, 0: S (three where K is short), with parts past it masked out
  auto reduce = [&](auto waves_tag) {
    constexpr int WAVES = decltype(waves_tag)::value, R = WAVES ? WAVES : 8;
    auto slot = [&](int s) { return lds + (WAVES || s < S ? s : S - 1) * kSlot; };
    auto on = [&](int s, uint32_t v) { return WAVES || s < S ? v : 0u; };
    // The parts of all of a wave's blocks are requested before the first is summed (32 registers), behind the column counts, so
    // that the LDS round trips run under each other and under the sums and stores.
    constexpr int NB8 = WAVES ? 8 / WAVES : 1, NT = HALF ? 1 : 2;  // blocks; 16-byte reads a part
    uint4 cc[R][NT], part[NB8][R][NT];
    auto request = [&](uint4 (&to)[R][NT], int row) {  // row `row` of eight lanes each
#pragma unroll
      for (int s = 0; s < R; ++s)
#pragma unroll
        for (int k = 0; k < NT; ++k) to[s][k] = slot(s)[row * kRow + 8 * k + (lane & 7)];
    };
    auto row_count = [&](int b) {
      int c = 0;
#pragma unroll
      for (int s = 0; s < R; ++s) c += (int)on(s, ((const u_alias*)(slot(s) + 65 * kRow))[8 * b + mrow]);
      return c;
    };
    if (XNOR) request(cc, 64);
    if constexpr (WAVES != 0 && HALF) {
#pragma unroll
      for (int it = 0; it < NB8; ++it) request(part[it], 8 * (wave + it * R) + (lane >> 3));
    }
    // sums over the parts: eight numbers below 2^16 in four pairs, or eight fp32 numbers (whole below 2^24)
    auto total = [&](const uint4 (&from)[R][NT], bool fp, int (&to)[8]) {
      if constexpr (HALF) {
        uint32_t x = 0, y = 0, z = 0, w = 0;
#pragma unroll
        for (int s = 0; s < R; ++s) x += on(s, from[s][0].x), y += on(s, from[s][0].y), z += on(s, from[s][0].z), w += on(s, from[s][0].w);
        to[0] = x & 0xffffu, to[1] = y & 0xffffu, to[2] = z & 0xffffu, to[3] = w & 0xffffu;
        to[4] = x >> 16, to[5] = y >> 16, to[6] = z >> 16, to[7] = w >> 16;
      } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            int sum = 0;
#pragma unroll
            for (int s = 0; s < R; ++s) {
              const uint4& q = from[s][k];
              const uint32_t v = on(s, e == 0 ? q.x : e == 1 ? q.y : e == 2 ? q.z : q.w);
              sum += fp ? (int)__uint_as_float(v) : (int)v;
            }
            to[4 * k + e] = sum;
          }
        }
      }
    };
    int ct[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (XNOR) {
      total(cc, false, ct);
#pragma unroll
      for (int e = 0; e < 8; ++e) ct[e] <<= mul - 1;
    }
    auto finish = [&](const uint4 (&from)[R][NT], int b) {
      const int rt = XNOR ? Kreal - (row_count(b) << (mul - 1)) : -__shfl(rowsum_l, 8 * b + mrow);
      int d[8];
      total(from, true, d);
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = (d[e] << mul) + (rt - ct[e]);
#ifdef BMX_FP4_STAMPS
      if (b == wave) { FP4_STAMP(7); }
#endif
      const float alm = CONV && OUT != kOutI32 ? __shfl(alpha_l, 8 * b + mrow) : 1.0f;
      if constexpr (OUT == kOutBits) {
        const float thm = CONV ? __shfl(thr_l, 8 * b + mrow) : 0.0f;
        uint32_t w[2] = {0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float al = CONV ? alm : al_c[e >> 2][e & 3], th = CONV ? thm : th_c[e >> 2][e & 3];
          const int place_of = CONV ? 8 * (e & 3) + mrow : lcol + (e & 3);
          const bool there = CONV ? 8 * b < rows_left : n0 + 32 * (e >> 2) + lcol + (e & 3) < N;
          if (there && al * (float)d[e] >= th) w[e >> 2] |= 1u << place_of;
        }
        // CONV: a pixel's byte from the eight lanes of its rows; else a row's two dwords from the eight lanes of its columns
#pragma unroll
        for (int x = CONV ? 8 : 1; x < (CONV ? 64 : 8); x *= 2) {
          w[0] |= (uint32_t)__shfl_xor((int)w[0], x);
          w[1] |= (uint32_t)__shfl_xor((int)w[1], x);
        }
        if (CONV) {
          if (lane < 8) {
            *(u_alias*)(bytes + 64 * b + lcol) = w[0];
            *(u_alias*)(bytes + 64 * b + 32 + lcol) = w[1];
          }
        } else if ((lane & 7) == 0 && 8 * b < rows_left) {
          // (m * ldc words fit 32 bits: the launcher checks)
          ((uint64_t*)C)[(uint32_t)(m0 + 8 * b + mrow) * elems + (uint32_t)(n0 >> 6)] = (uint64_t)w[1] << 32 | w[0];
        }
      } else {
        uint32_t v[8], s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = result(d[e], CONV ? alm : al_c[e >> 2][e & 3]);
          s[e] = (uint32_t)d[e];
        }
        if (XNOR || C) put(C, b, v);
        if (!XNOR && C2) put(C2, b, s);
      }
    };
    if constexpr (WAVES != 0) {
#pragma unroll
      for (int it = 0; it < NB8; ++it) {
        if (!HALF) request(part[it], 8 * (wave + it * R) + (lane >> 3));
        finish(part[it], wave + it * R);
      }
    } else {
      for (int b = wave; b < 8; b += S) {
        request(part[0], 8 * b + (lane >> 3));
        finish(part[0], b);
      }
    }
  };
  if (S == 8) reduce(std::integral_constant<int, 8>{});
  else if (S == 4) reduce(std::integral_constant<int, 4>{});
  else reduce(std::integral_constant<int, 0>{});
  if constexpr (CONV && OUT == kOutBits) {
    __syncthreads();
    if (wave == 0) {
      uint64_t word = 0;
#pragma unroll
      for (int b = 0; b < 8; ++b) word |= (uint64_t)bytes[64 * b + lane] << (8 * b);
      store_word(word);
    }
  }
  FP4_STAMP(5);
#ifdef BMX_FP4_STAMPS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  FP4_STAMP(6);
#endif
}

}  // namespace
int gemm_fp4_half = 0;  // 2 = keep fp32 partials (tests of both forms)
namespace {

template <int PL, bool XNOR, int OUT, bool SPLIT, bool HALF, bool CONV, bool ODD>
hipError_t launch_tile(const Fp4Params& p, int S, int tiles_per_wg, int64_t blocks, hipStream_t s) {
  const int waves = SPLIT ? S : tiles_per_wg;
  const size_t lds = (size_t)waves * slot_size(PL, SPLIT, HALF) * 16 + (SPLIT && CONV && OUT == kOutBits ? 512 : 0);
  auto kern = gemm_fp4_kernel<PL, XNOR, OUT, SPLIT, HALF, CONV, ODD>;
  static std::atomic<bool> asked[64];
  const hipError_t e = allow_lds((const void*)kern, lds, asked);
  if (e != hipSuccess) return e;
  note_kernel("gemm_fp4_kernel<%d,%d,%d,%s,%s%s> grid %lld x %d, K split %d%s, fp4", TM, TN, PL, XNOR ? "xnor" : "planes",
              !XNOR ? "S" : (OUT == kOutF32 ? "f32" : (OUT == kOutI32 ? "i32" : "bits")), CONV ? (ODD ? ",conv,reg" : ",conv") : "",
              (long long)blocks, 64 * waves, SPLIT ? S : 1, SPLIT && HALF ? " (16-bit partials)" : "");
#ifdef BMX_FP4_STAMPS
  launch_kernel(kern, dim3((unsigned)blocks), dim3(64 * waves), lds, s, p, S, fp4_stamps);
#else
  launch_kernel(kern, dim3((unsigned)blocks), dim3(64 * waves), lds, s, p, S);
#endif
  return launch_error();
}

}  // namespace
int gemm_fp4_band = 0;  // 0 = automatic, else rows of tiles per band of the tile order
namespace {

// Rows of tiles per band: what an XCD has in flight should be about as high as wide, so that few operand rows pass its L2.
// With K undivided that is several hundred tiles, 16 high; with K divided a tile a workgroup, 32 to 64 an XCD, 8 high (graph
// times, 16 / 8: 1024 x 1024 x 4096 of 2 x 1 bits 14.3 / 14.0 us, 1852 x 384 x 6030 20.8 / 20.2, 1344 x 1325 x 5633 12.8 / 12.5; 4 and
// 6 as 8).
void set_tile_order(Fp4Params& p, int S) {
  p.band = std::min(gemm_fp4_band > 0 ? gemm_fp4_band : S > 1 ? 8 : 16, p.tiles_m);
  p.per_band = p.band * p.tiles_n;
  p.last_band = (p.tiles_m - 1) / p.band;
  p.last_rows = p.tiles_m - p.last_band * p.band;
  p.div_per_band = make_fast_div((uint32_t)p.per_band);
  p.div_band = make_fast_div((uint32_t)p.band);
  p.div_last = make_fast_div((uint32_t)p.last_rows);
}

// A full sum is at most (bits of K) x (2^planes - 1), a full count K: whether 16 bits hold them
bool fits_16_bits(int64_t K, int planes) { return K * ((1 << planes) - 1) <= 65535; }

template <int PL, bool XNOR, int OUT, bool CONV = false, bool ODD = false>
hipError_t launch_split(const Fp4Params& p, int S, int tiles_per_wg, int64_t blocks, hipStream_t s) {
  if (S <= 1) return launch_tile<PL, XNOR, OUT, false, false, CONV, ODD>(p, S, tiles_per_wg, blocks, s);
  return fits_16_bits(p.Kreal, PL) && gemm_fp4_half != 2 ? launch_tile<PL, XNOR, OUT, true, true, CONV, ODD>(p, S, tiles_per_wg, blocks, s)
                                                        : launch_tile<PL, XNOR, OUT, true, false, CONV, ODD>(p, S, tiles_per_wg, blocks, s);
}

}  // namespace

int gemm_fp4_split = 0;  // 0 = automatic; settable for sweeps and for the tests of every split

// Waves that share a tile's K.  From 350 products, 120 k-bit products and 200 convolutions measured with each, and 1500 products
// of few words since (the mean of the time over the best; graph times):
//   - eight where each has a share of two groups, up to a tile a CU (256): 61 words on (8 / 4 waves, 64 to 256 tiles: 62
//     words 0.96 to 0.97, 64 0.96, 66 0.97 to 1.01, 70 0.94, 74 0.97 to 1.02, 80 0.94 to 0.98; a whole layer of 256 tiles and 64
//     words 7.25 / 7.57 us).  Of fewer groups six or seven waves would be left of them, which four
//     beat (bit planes 1.03 / 1.00).  The patches of a convolution, whose latency
//     more waves hide, always eight (1.03 / 1.08 for four, 1.9 for one).
//   - four where each has two groups, 29 words on, up to three tiles a CU (257 to 512 tiles 1.25 / 1.00 / 1.44 for 8 / 4 / 1; 513 to
//     768 1.4 / 1.00 / 1.15; of 29 to 33 words 1.00 / 1.20, 4 / 1), and with more than one, but few, for some SIMDs (1025 to 1280: 1.45 /
//     1.00 / 1.19).  Between them a SIMD has at most one
//     undivided tile: one wave (1.5 / 1.03 / 1.00; four over one of 75 to 144 words 1.04 over 37 int32 products, 1.05 over 166 of
//     fp32).  Four and eight keep the SIMDs of a CU level where it has several tiles (390 x 3329 x 5632, 371 tiles, takes 10.4 us over four
//     waves, 15.1 over five, 12.2 over three).
//     Convolutions go on with four to 1700 tiles (45 to 72 words, time over one wave's of 200: 769 to 1024 0.88 to 0.95, 1281 to 1500 0.87 to
//     0.92, 1501 to 1700 0.97 to 1.0; of 75 words on 1.28 / 1.01 / 1.09 for 8 / 4 / 1), and from 2049 to 2350 (0.93 to 0.96; - / 1.01 / 1.10;
//     between, 1.08 to 1.14; - / 1.09 / 1.04).
//   - three of 21 to 28 words (six or seven groups), up to two tiles a CU (3 / 2 / 1 waves, to 256 tiles 1.00 / 1.14 / 1.17, to 512
//     bit planes 1.00 / 1.08 / 1.11, others 1.03 / 1.20 / 1.01; beyond, all 1.2 / 1.2 / 1.00).  Five
//     groups, 20 words, are not worth dividing (2 / 1 1.03 / 1.01 to 256 tiles, 1.24 / 1.00 to 512).
enum class Rows { direct, planes, patches };
static int choose_k_split(int64_t tiles, int kwords, Rows rows) {
  const bool patches = rows == Rows::patches;
  if (kwords < 21 && !patches) return 1;
  if (tiles <= 256 && (kwords >= 61 || patches)) return 8;
  if (kwords < 29 && !patches) return tiles <= 512 ? 3 : 1;
  if (tiles <= 512) return 4;
  if (kwords < 34 && patches) return 1;
  if (patches) return tiles <= 1700 || (tiles > 2048 && tiles <= 2350) ? 4 : 1;
  if (tiles <= 768 || (tiles > 1024 && tiles <= 1280)) return 4;
  return 1;
}

// Below 64 tiles kernels of 32 x 32 tiles: four times the waves, and there is not enough K to give these tiles to that many waves.
// (And only problems whose operands it addresses with 32-bit byte offsets, results with 32-bit element indices, rows rounded up to whole
// tiles: the kernels that leave it a problem ask for the same.)
static bool fp4_addresses(int64_t M, int64_t N, int planes, int64_t lda_bytes, int64_t ldb_bytes, int64_t ldc, bool bits) {
  return M * planes * lda_bytes < ((int64_t)1 << 32) && N * ldb_bytes < ((int64_t)1 << 32) && (M + 64) * ldc * (bits ? 2 : 1) < ((int64_t)1 << 31);
}
bool gemm_fp4_pays(int M, int N, int64_t lda_bytes, int64_t ldb_bytes, int64_t ldc, bool bits) {
  return ceil_div(M, 64) * ceil_div(N, 64) >= 64 && fp4_addresses(M, N, 1, lda_bytes, ldb_bytes, ldc, bits);
}

// Takes the problem (rows of `dwords` data dwords) when sums stay exact in fp32, the
// operands can be addressed with 32-bit byte offsets, and there are enough 64 x 64 tiles for
// the tile shape to pay; false otherwise (the caller then uses the 32 x 32 kernel).
bool launch_gemm_fp4(const void* A, int64_t lda_bytes, int planes, const int32_t* rowsum, const void* B,
                     int64_t ldb_bytes, int M, int N, int K, int dwords, const float* alpha_n, int32_t* C_i32, float* C_f32,
                     uint64_t* C_bits, const float* thr_n, int64_t ldc, bool as_count, hipStream_t s,
                     hipError_t* err) {
  if (gemm_engine == 1 || gemm_engine == 2 || gemm_engine == 4) return false;
  if (planes < 1 || planes > 2) return false;
  // rows are fetched 16 bytes at a time, the last 16 whole, and may start on any dword; shorter ones only where they are 16 bytes apart
  const bool apart = !((lda_bytes | ldb_bytes) & 15) && !(((uintptr_t)A | (uintptr_t)B) & 15);
  if (dwords < 4 && !apart) return false;
  if ((int64_t)K * ((1 << planes) - 1) >= ((int64_t)1 << 24)) return false;
  if (!fp4_addresses(M, N, planes, lda_bytes, ldb_bytes, ldc, C_bits != nullptr)) return false;
  const int tiles_m = (int)ceil_div(M, 64), tiles_n = (int)ceil_div(N, 64);
  const int64_t tiles = (int64_t)tiles_m * tiles_n;
  const int Kwords = (int)words_for(K);
  if (gemm_engine != 5 && tiles < 64) return false;
  if (tiles >= ((int64_t)1 << 28)) return false;
  Fp4Params p;
  p.A = (const char*)A - 16;
  p.B = (const char*)B - 16;
  p.lda_bytes = (uint32_t)lda_bytes;
  p.ldb_bytes = (uint32_t)ldb_bytes;
  p.Kd = dwords;
  p.M = M;
  p.N = N;
  p.Kw = Kwords;
  p.Kreal = K;
  const int ngroups = (int)ceil_div(p.Kw, 4);
  p.tiles_m = tiles_m;
  p.tiles_n = tiles_n;
  p.alpha = alpha_n;
  p.thr = thr_n;
  p.rowsum = rowsum;
  p.as_count = as_count ? 1 : 0;
  p.C_i32 = C_i32;
  p.C_f32 = C_f32;
  p.C_bits = (uint32_t*)C_bits;
  p.ldc = (int)ldc;
  p.nt = ldc % 32 == 0 && (((uintptr_t)C_i32 | (uintptr_t)C_f32) & 127) == 0;
  p.HoWo = p.Wo = p.Hp = p.Wpp = p.Cw = p.stride = 1;
  p.Nimg = p.Ho = p.opad = p.oHp = p.oWp = p.oCw = 0;
  p.run = p.row_bytes = 1;
  p.div_howo = p.div_wo = p.div_run = p.div_two_runs = make_fast_div(1);
  // (every wave of a split keeps at least one 64-byte segment)
  int S = gemm_fp4_split > 0 ? gemm_fp4_split : choose_k_split(tiles, Kwords, rowsum ? Rows::planes : Rows::direct);
  S = S > 8 ? 8 : S;
  if (S > ngroups / 2) S = ngroups / 2;
  if (S < 1) S = 1;
  set_tile_order(p, S);
  p.g_base = ngroups / S;
  p.g_rem = ngroups - p.g_base * S;
  // Undivided, a workgroup is a wave where K is short: nothing is shared, and a wave starts when there is room for it and not for four
  // (400 products, time over that with four: up to 7 words 0.96 to 1700 tiles and 0.98 beyond, 8 to 20 words 0.98; from 21 on 0.98 to 1.03,
  // and over long K, where four keep the SIMDs of a CU level, 1.06 with 1700 to 2048 tiles; planes 1.05 with 300 to 1024).
  // us in a graph: 2000 x 2048 x 320 as packed bits 5.4 / 5.1, 1462 x 1920 x 128 5.7 / 5.3.
  const int tiles_per_wg = rowsum == nullptr && Kwords < 21 ? 1 : 4;
  const int64_t wgs = S > 1 ? tiles : ceil_div(tiles, tiles_per_wg);
  p.tiles_per_xcd = (int)ceil_div(wgs, 8);
  const int64_t blocks = 8 * (int64_t)p.tiles_per_xcd;
  if (planes == 1 && rowsum == nullptr) {
    if (C_bits) *err = launch_split<1, true, kOutBits>(p, S, tiles_per_wg, blocks, s);
    else if (C_i32) *err = launch_split<1, true, kOutI32>(p, S, tiles_per_wg, blocks, s);
    else *err = launch_split<1, true, kOutF32>(p, S, tiles_per_wg, blocks, s);
  } else if (planes == 1) {
    *err = launch_split<1, false, kOutF32>(p, S, tiles_per_wg, blocks, s);
  } else {
    *err = launch_split<2, false, kOutF32>(p, S, tiles_per_wg, blocks, s);
  }
  return true;
}

// The convolution on the same kernel (Xp, Wp as for launch_binary_conv2d).  Takes the problem when
// the filter rows are 16-byte aligned, and image and output fit 32-bit offsets.
bool launch_conv_fp4(const uint64_t* Xp, int Nimg, int C, int H, int W, const uint64_t* Wp, int O, int KH, int KW,
                     int stride, int pad, const float* alpha, int32_t* out_i32, float* out_f32, uint64_t* out_bits,
                     const float* thr, int out_pad, hipStream_t s, hipError_t* err) {
  if (gemm_engine == 1 || gemm_engine == 2 || gemm_engine == 4) return false;
  const int Ho = (H + 2 * pad - KH) / stride + 1;
  const int Wo = (W + 2 * pad - KW) / stride + 1;
  const int Cw = (int)words_for(C);
  const int kwords = KH * KW * Cw;
  const int64_t ld_words = conv_weight_row_words(kwords);
  const int64_t P = (int64_t)Nimg * Ho * Wo;
  const int Hp = H + 2 * pad, Wpp = W + 2 * pad;
  if ((ld_words & 1) || ((uintptr_t)Wp & 15)) return false;
  const bool odd = (KW * Cw) & 1;
  if ((int64_t)kwords * 64 >= ((int64_t)1 << 24)) return false;
  if ((int64_t)Nimg * Hp * Wpp * Cw * 8 >= ((int64_t)1 << 32) || (int64_t)O * ld_words * 8 >= ((int64_t)1 << 32))
    return false;
  if (P >= ((int64_t)1 << 31) || ((int64_t)Nimg * O + 64) * Ho * Wo >= ((int64_t)1 << 31)) return false;
  // (the halo's words are counted, and every word of the image addressed, in 32 bits)
  if (out_bits && (int64_t)Nimg * (Ho + 2 * out_pad) * (Wo + 2 * out_pad) * words_for(O) >= ((int64_t)1 << 30)) return false;
  // (a tile's results are addressed with 32 bits from its first image on: a tile of three images or more has less than 63 pixels
  // in each)
  if (O >= (1 << 23) && Ho * Wo < 63) return false;
  const int tiles_m = (int)ceil_div(O, 64), tiles_n = (int)ceil_div(P, 64);
  const int64_t tiles = (int64_t)tiles_m * tiles_n;
  if (tiles >= ((int64_t)1 << 28)) return false;
  Fp4Params p;
  p.A = Wp;
  p.B = Xp;
  p.lda_bytes = (uint32_t)(ld_words * 8);
  p.ldb_bytes = 0;
  p.Kd = 2 * kwords;
  p.M = O;
  p.N = (int)P;
  p.Kw = kwords;
  p.Kreal = C * KH * KW;
  const int ngroups = (int)ceil_div(kwords, 4);
  p.tiles_m = tiles_m;
  p.tiles_n = tiles_n;
  p.alpha = alpha;
  p.thr = thr;
  p.rowsum = nullptr;
  p.as_count = 0;
  p.C_i32 = out_i32;
  p.C_f32 = out_f32;
  p.C_bits = (uint32_t*)out_bits;
  p.Nimg = Nimg;
  p.Ho = Ho;
  p.opad = out_pad;
  p.oHp = Ho + 2 * out_pad;
  p.oWp = Wo + 2 * out_pad;
  p.oCw = (int)words_for(O);
  p.ldc = 0;
  p.nt = Ho * Wo % 32 == 0 && (((uintptr_t)out_i32 | (uintptr_t)out_f32) & 127) == 0;
  p.HoWo = Ho * Wo;
  p.Wo = Wo;
  p.Hp = Hp;
  p.Wpp = Wpp;
  p.Cw = Cw;
  p.stride = stride;
  p.run = (uint32_t)(KW * Cw);
  p.row_bytes = (uint32_t)((int64_t)Wpp * Cw * 8);
  p.div_howo = make_fast_div((uint32_t)(Ho * Wo));
  p.div_wo = make_fast_div((uint32_t)Wo);
  p.div_run = make_fast_div(p.run);
  p.div_two_runs = make_fast_div(2 * p.run);
  // (a wave may carry a single group of 256 bits)
  int S = gemm_fp4_split > 0 ? gemm_fp4_split : choose_k_split(tiles, kwords, Rows::patches);
  S = S > 8 ? 8 : S;
  if (S > ngroups) S = ngroups;
  if (S < 1) S = 1;
  set_tile_order(p, S);
  p.g_base = ngroups / S;
  p.g_rem = ngroups - p.g_base * S;
  const int tiles_per_wg = 4;
  const int64_t wgs = S > 1 ? tiles : ceil_div(tiles, tiles_per_wg);
  p.tiles_per_xcd = (int)ceil_div(wgs, 8);
  const int64_t blocks = 8 * (int64_t)p.tiles_per_xcd;
  if (out_bits) *err = odd ? launch_split<1, true, kOutBits, true, true>(p, S, tiles_per_wg, blocks, s)
                           : launch_split<1, true, kOutBits, true>(p, S, tiles_per_wg, blocks, s);
  else if (odd && out_i32) *err = launch_split<1, true, kOutI32, true, true>(p, S, tiles_per_wg, blocks, s);
  else if (odd) *err = launch_split<1, true, kOutF32, true, true>(p, S, tiles_per_wg, blocks, s);
  else if (out_i32) *err = launch_split<1, true, kOutI32, true>(p, S, tiles_per_wg, blocks, s);
  else *err = launch_split<1, true, kOutF32, true>(p, S, tiles_per_wg, blocks, s);
  return true;
}

}  // namespace bmx
