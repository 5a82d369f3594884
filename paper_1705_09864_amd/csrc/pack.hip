// Binarise / quantise + bit-pack kernels (HBM-bandwidth bound).
// Paper: Sec. 1 (sign binarisation, 64 values per word), Sec. 3.1 (the per-forward
// input binarisation step), Sec. 2.1 Eq. 1 (k-bit quantiser).
#include "bmx_internal.h"
#include "halo.h"

#include <algorithm>

namespace bmx {

static constexpr int kWave = 64;

// v_writelane_b32, which this compiler knows by no builtin: `old` with `value` (uniform) in lane `lane`.
extern "C" __device__ __attribute__((const)) uint32_t write_lane(uint32_t value, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");

// Row pack.  A wave packs segments of 16 consecutive words (1024 floats) of one row: lane
// <-> k, so every load instruction is a 256-byte coalesced read and the 64-lane compare
// mask is the packed word itself.  All 16 loads of a segment are issued before the first
// compare.  A workgroup owns one contiguous stretch of the segment list (its four waves
// interleave inside it).
constexpr int kSegWords = 16;

template <bool NT>
__device__ __forceinline__ void pack_row_segments(const float* __restrict__ x, uint32_t total,
                                                  int64_t cols, int64_t ldx,
                                                  uint64_t* __restrict__ out, int64_t out_ld,
                                                  int64_t Kw, FastDiv div_segs, uint32_t segs_per_row,
                                                  uint32_t first, uint32_t per) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), waves = blockDim.x / kWave;
  const uint32_t end = min(first + per, total);
  for (uint32_t seg = first + wave; seg < end; seg += waves) {
    const uint32_t r = fast_div(seg, div_segs);
    const int64_t b = seg - r * segs_per_row;
    const float* const xs = x + (int64_t)r * ldx + b * (64 * kSegWords);
    const int64_t left = cols - b * (64 * kSegWords);
    float v[kSegWords];
    if (left >= 64 * kSegWords) {  // whole segment inside the row (wave-uniform)
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) v[j] = NT ? __builtin_nontemporal_load(xs + 64 * j + lane) : xs[64 * j + lane];
    } else {  // (loads under no condition: all are in flight at once; out-of-row lanes contribute 0 bits)
      const int n = (int)max(left, (int64_t)0);  // (0: padding words only)
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) v[j] = n > 0 ? xs[(uint32_t)min(64 * j + lane, n - 1)] : 0.0f;
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) v[j] = 64 * j + lane < n ? v[j] : -1.0f;
    }
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < kSegWords; ++j) {
      const uint64_t m = __ballot(v[j] >= 0.0f);
      lo = write_lane((uint32_t)m, j, lo);
      hi = write_lane((uint32_t)(m >> 32), j, hi);
    }
    const int64_t w = b * kSegWords + lane;
    if (lane < kSegWords && w < Kw) out[(int64_t)r * out_ld + w] = ((uint64_t)hi << 32) | lo;
  }
}

template <bool NT>
__global__ void __launch_bounds__(256)
pack_rows_kernel(const float* __restrict__ x, uint32_t total, int64_t cols, int64_t ldx,
                 uint64_t* __restrict__ out, int64_t out_ld, int64_t Kw, FastDiv div_segs, uint32_t segs_per_row,
                 uint32_t segs_per_block) {
  pack_row_segments<NT>(x, total, cols, ldx, out, out_ld, Kw, div_segs, segs_per_row, blockIdx.x * segs_per_block,
                        segs_per_block);
}

// Matrices past this many bytes are read with the streaming hint: they would not stay in the L2s (4 MB on each of 8
// XCDs), and what they push out on the way costs more.  Row pack and alpha_mean_abs of 44 to 103 MB level or 10 %
// faster so, from HBM and on a second reading; 43 MB level, 37 MB 7.1 us instead of 5.8 on the second.  It depends on where the
// matrix is.  Both over 4096 x 9216 (151 MB, of the memory-side cache's 256), us without the hint / with it: several in turn 48.4 /
// 47.3, the same made one after the other in front of it 54.4 / 45.2, made long ago 52.1 / 52.1; but one matrix again and
// again 44.4 / 45.3, and weights made in the memory that the last ones left, read once, 47.8 / 49.7.
constexpr int64_t kStreamBytes = 48 << 20;

static void launch_pack_rows_grid(const float* x, int64_t rows, int64_t cols, int64_t ldx,
                                  uint64_t* out, int64_t out_ld, int64_t words_per_row,
                                  hipStream_t s) {
  // A wave per segment, in a grid of them all: waves that went on to their next segment (2048 workgroups) asked for it
  // only once they had the last (4096 x 9216 from HBM 29.9 us and now 24.1, 2 GiB 380 and 344: 6.2 TB/s).
  const uint32_t spr = (uint32_t)ceil_div(words_per_row, kSegWords);
  const int64_t most = std::max<int64_t>(((int64_t)1 << 30) / spr, 1);  // rows a launch: segments are counted in 32 bits
  if (rows > most) {
    launch_pack_rows_grid(x, most, cols, ldx, out, out_ld, words_per_row, s);
    launch_pack_rows_grid(x + most * ldx, rows - most, cols, ldx, out + most * out_ld, out_ld, words_per_row, s);
    return;
  }
  const uint32_t total = (uint32_t)rows * spr;
  const uint32_t blocks = (uint32_t)std::min<int64_t>(ceil_div(total, 4), 1 << 22);
  const bool nt = rows * cols * 4 > kStreamBytes;
  note_kernel("pack_rows_kernel<%s> grid %u x 256", nt ? "nontemporal" : "cached", blocks);
  const FastDiv div = make_fast_div(spr);
  auto go = [&](auto kern) {
    launch_kernel(kern, dim3(blocks), dim3(256), 0, s, x, total, cols, ldx, out, out_ld, words_per_row, div, spr,
                  (uint32_t)ceil_div(total, blocks));
  };
  if (nt) go(pack_rows_kernel<true>);
  else go(pack_rows_kernel<false>);
}

hipError_t launch_pack_rows(const float* x, int64_t rows, int64_t cols, int64_t ldx, uint64_t* out,
                            int64_t out_ld, hipStream_t s) {
  const int64_t Kw = words_for(cols);
  // A dense matrix whose rows are whole words is one long row.
  if (ldx == cols && out_ld == Kw && (cols % 64) == 0) {
    cols = rows * cols;
    ldx = cols;
    rows = 1;
    out_ld = cols / 64;
  }
  launch_pack_rows_grid(x, rows, cols, ldx, out, out_ld, words_for(cols), s);
  return launch_error();
}

// Row pack into rows of out_ld words, writing every word of a row (zeros past the last
// data word): the chunk-padded activation rows read by the scalar side of the GEMM kernel.
hipError_t launch_pack_rows_padded(const float* x, int64_t rows, int64_t cols, int64_t ldx,
                                   uint64_t* out, int64_t out_ld, hipStream_t s) {
  launch_pack_rows_grid(x, rows, cols, ldx, out, out_ld, out_ld, s);
  return launch_error();
}

// Inverse of the row pack: element k of row r -> +1.0f / -1.0f (a stored 1-bit model back
// to the float weights every pack routine starts from, Sec. 2.2.3).  A wave per word, lane =
// bit; grid-stride over the words.
__global__ void __launch_bounds__(256)
unpack_pm1_kernel(const uint64_t* __restrict__ bits, int64_t rows, int64_t K, int64_t ld_words,
                  float* __restrict__ out, int64_t ldo) {
  const int lane = threadIdx.x & 63;
  const int64_t Kw = words_for(K);
  const int64_t total = rows * Kw;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < total; i += (int64_t)gridDim.x * 4) {
    const int64_t r = i / Kw, w = i - r * Kw;
    const int64_t k = w * 64 + lane;
    const uint64_t word = bits[r * ld_words + w];
    if (k < K) out[r * ldo + k] = ((word >> lane) & 1) ? 1.0f : -1.0f;
  }
}

hipError_t launch_unpack_pm1(const uint64_t* bits, int64_t rows, int64_t K, int64_t ld_words, float* out,
                             int64_t ldo, hipStream_t s) {
  const int64_t blocks = ceil_div(rows * words_for(K), 4);
  launch_kernel(unpack_pm1_kernel, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, s, bits,
                     rows, K, ld_words, out, ldo);
  return launch_error();
}

// Rows of 32-bit words (the 32-bit BINARY_WORD flavour of Sec. 2.2.1) -> rows of 64-bit words:
// word w of a row is dwords 2w (low half) and 2w + 1 (high half, zero when the row has an odd
// number of dwords).  With bits LSB first and little-endian words this moves no bit: element k
// is bit k % 32 of dword k / 32 and bit k % 64 of word k / 64 alike.  One thread per word.
__global__ void __launch_bounds__(256)
widen_words32_kernel(const uint32_t* __restrict__ in, int64_t rows, int64_t Kd, int64_t ld_dw,
                     uint64_t* __restrict__ out, int64_t out_ld) {
  const int64_t Kw = (Kd + 1) / 2;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= rows * Kw) return;
  const int64_t r = i / Kw, w = i - r * Kw;
  const uint32_t* row = in + r * ld_dw;
  const uint32_t lo = row[2 * w];
  const uint32_t hi = 2 * w + 1 < Kd ? row[2 * w + 1] : 0u;
  out[r * out_ld + w] = ((uint64_t)hi << 32) | lo;
}

hipError_t launch_widen_words32(const uint32_t* in, int64_t rows, int64_t K, int64_t ld_dw, uint64_t* out,
                                int64_t out_ld, hipStream_t s) {
  const int64_t Kd = (K + 31) / 32;
  const int64_t total = rows * ((Kd + 1) / 2);
  launch_kernel(widen_words32_kernel, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, s, in, rows, Kd,
                     ld_dw, out, out_ld);
  return launch_error();
}

// Strided pack (the matrix is stored K x ncol, pack down the columns): a workgroup packs 64 columns of two words.  Each
// wave takes 16 rows (lanes span columns: a load is 256 bytes of a row, all 16 in flight) and leaves 16 bits per
// column in LDS; a column's two words are stored by neighbouring lanes.  Bound by the matrix's way in.  Where rows are no
// whole 128-byte lines the tiles beside each other share them: they are dealt to one XCD then, so that the second
// finds them in its L2, an eighth of the matrix each (ORDER kEighths) or, in a matrix that passes through, eight tiles at a
// time (kEights: XCDs at work an eighth of 9215 x 4095 apart meet in the same memory channels).
// With a wave per word, all 64 rows in its registers, and now, us a launch, from HBM: 9000 x 100 4.7 and 2.7, 300 x 4000
// 5.3 and 2.8, 3237 x 1338 7.5 and 4.9, 2944 x 3651 12.2 and 8.5 (5.1 TB/s), 8000 x 4001 29.0 and 23.7, 4096 x 9216
// 31.9 and 25.0 (6.0 TB/s).  Plain order, kEighths, kEights: 2944 x 3651 11.3, 8.5, 9.0; 8000 x 4001 32.3, 26.1, 23.7;
// 9215 x 4095 33.9, 31.9, 29.2; whole lines, 9216 x 4096, without the hint 28.4, 31.8, 27.6.  16 bytes a load on any
// dword, 256 columns a workgroup: 17.4 for 2944 x 3651.
enum { kPlain, kEighths, kEights };

template <int ORDER, bool NT>
__global__ void __launch_bounds__(512)
pack_strided_kernel(const float* __restrict__ x, int64_t K, int64_t ncol, int64_t ldx, uint64_t* __restrict__ out,
                    int64_t out_ld, int64_t Kw, uint32_t total, FastDiv div_groups, uint32_t groups) {
  constexpr int kWords = 2, kRows = 16;
  __shared__ __align__(8) uint16_t bits[64][4 * (kWords + 1)];  // (+1: other banks)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) {
    // workgroups b, b + 8, ... run on one XCD
    const uint32_t xcd = b & 7;
    uint32_t tile = b;
    if (ORDER == kEighths) tile = xcd * (total / 8) + min(xcd, total % 8) + b / 8;
    if (ORDER == kEights && b < total / 64 * 64) tile = b / 64 * 64 + xcd * 8 + b / 8 % 8;
    const uint32_t band = fast_div(tile, div_groups);
    const int64_t n0 = (int64_t)(tile - band * groups) * 64, w0 = (int64_t)band * kWords;
    const int64_t k0 = w0 * 64 + wave * kRows, left = K - k0;  // rows of this wave
    const float* const at = x + min(n0 + lane, ncol - 1);
    float v[kRows];
    if (left >= kRows) {
#pragma unroll
      for (int j = 0; j < kRows; ++j) v[j] = NT ? __builtin_nontemporal_load(at + (k0 + j) * ldx) : at[(k0 + j) * ldx];
    } else {
#pragma unroll
      for (int j = 0; j < kRows; ++j) v[j] = j < left ? at[(k0 + j) * ldx] : -1.0f;
    }
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kRows; ++j) mine |= (v[j] >= 0.0f ? 1u : 0u) << j;
    bits[lane][wave] = (uint16_t)mine;
    __syncthreads();
    if (threadIdx.x < 64 * kWords) {
      const int c = threadIdx.x / kWords, w = threadIdx.x % kWords;
      uint64_t word;
      __builtin_memcpy(&word, __builtin_assume_aligned(&bits[c][4 * w], 8), 8);
      if (n0 + c < ncol && w0 + w < Kw) out[(n0 + c) * out_ld + w0 + w] = word;
    }
    __syncthreads();
  }
}

hipError_t launch_pack_strided(const float* x, int64_t K, int64_t ncol, int64_t ldx, uint64_t* out, int64_t out_ld,
                               hipStream_t s) {
  const int64_t Kw = words_for(K);
  const uint32_t groups = (uint32_t)ceil_div(ncol, 64), total = groups * (uint32_t)ceil_div(Kw, 2);
  const uint32_t blocks = std::min<uint32_t>(total, 1u << 22);
  const bool lines = ldx % 32 == 0 && (uintptr_t)x % 128 == 0;
  const bool large = K * ncol * 4 > kStreamBytes;
  note_kernel("pack_strided_kernel<%s> grid %u x 512", lines ? "lines" : "per XCD", blocks);
  const FastDiv div = make_fast_div(groups);
  auto go = [&](auto kern) {
    launch_kernel(kern, dim3(blocks), dim3(512), 0, s, x, K, ncol, ldx, out, out_ld, Kw, total, div, groups);
  };
  if (lines && large) go(pack_strided_kernel<kPlain, true>);
  else if (lines) go(pack_strided_kernel<kPlain, false>);
  else if (large) go(pack_strided_kernel<kEights, false>);
  else go(pack_strided_kernel<kEighths, false>);
  return launch_error();
}

// NCHW channel pack.  A workgroup packs 64 consecutive pixels, counted through the images, for one
// 64-channel word: each of its four waves takes 16 of the channels (a load reads 256 bytes of a channel
// plane, all 16 in flight) and leaves 16 bits per pixel in LDS; the first wave stores the words.
// Bound by the fp32 image's way in: with a wave per 64 channels a small image left most of the chip
// without a load in flight, and counted per image 99 pixels are two waves of 64.
// The image is read exactly once, so where a plane is whole 128-byte lines the loads are non-temporal
// (they do not displace what the convolution that follows needs); elsewhere neighbouring loads share
// lines.  us a launch, against a wave per 64 channels, counted per image and in the order of the workgroups:
// 175 x 468 x 10 x 12 8.3 / 13.0, 17 x 505 x 49 x 49 14.6 / 21.3 (5.6 TB/s), 59 x 128 x 44 x 43 10.5 / 12.8, 16 x 64 x
// 56 x 56 4.0 / 4.5, 2 x 62 x 18 x 17 2.7 / 4.1.
// The halo (a constant per word) is spread over the workgroups of its word.
// THR: bit = (value >= thr[channel]) instead of (value >= 0): the packing behind a layer whose
// sign decision carries a folded per-channel threshold.
struct PackNchwParams {
  const float* x;
  const float* thr;
  uint64_t* xp;
  int images, C, HW, H, W, pad, Hp, Wp, Cw;
  uint32_t pixels, first;  // of all images; the launch's first
  FastDiv div_hw, div_w;
};

template <bool THR, bool NT>
__global__ void __launch_bounds__(256)
pack_nchw_kernel(const PackNchwParams p) {
  __shared__ uint16_t bits[64 * 4];
  asm volatile("" ::"s"(p.x), "s"(p.xp), "s"(p.C), "s"(p.HW), "s"(p.W), "s"(p.pad), "s"(p.Hp), "s"(p.Wp), "s"(p.Cw), "s"(p.pixels),
               "s"(p.first), "s"(p.div_hw.mul), "s"(p.div_hw.sh1), "s"(p.div_hw.sh2), "s"(p.div_w.mul), "s"(p.div_w.sh1), "s"(p.div_w.sh2));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cw = blockIdx.y, c0 = cw * 64 + wave * 16, real = min(16, p.C - c0);  // (real <= 0: channels past the last)
  // Workgroup b sits on XCD b % 8: every XCD gets a contiguous run of pixels, whose neighbours share lines
  // where planes are not whole ones (57 MB of 44 x 43 planes 14.1 us without).
  const uint32_t q = p.first + ((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * 64 + lane;
  const uint32_t qc = min(q, p.pixels - 1);  // lanes past the last pixel repeat it
  const uint32_t n = fast_div(qc, p.div_hw), px = qc - n * (uint32_t)p.HW;
  float v[16];
  if (real > 0) {
    const float* const xb = p.x + ((int64_t)n * p.C + c0) * p.HW + px;
    const int64_t plane = p.HW;
#pragma unroll
    for (int j = 0; j < 16; ++j) {  // (channels past the last repeat it and are masked)
      const float* const at = xb + plane * min(j, real - 1);
      v[j] = NT ? __builtin_nontemporal_load(at) : *at;
    }
  }
  const uint32_t h = fast_div(px, p.div_w), w = px - h * (uint32_t)p.W;
  if (p.pad > 0 && p.first == 0)
    write_halo(p.xp, p.images, p.H, p.W, p.pad, p.C, p.Cw, cw, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
  uint32_t b = 0;
  if (real > 0) {
#pragma unroll
    for (int j = 0; j < 16; ++j) b |= (v[j] >= (THR ? p.thr[min(c0 + j, p.C - 1)] : 0.0f) ? 1u : 0u) << j;
    if (real < 16) b &= (1u << real) - 1u;
  }
  bits[lane * 4 + wave] = (uint16_t)b;
  __syncthreads();
  if (wave == 0 && q < p.pixels) {
    typedef uint64_t __attribute__((may_alias)) word_alias;
    p.xp[(((int64_t)n * p.Hp + h + p.pad) * p.Wp + w + p.pad) * p.Cw + cw] = ((const word_alias*)bits)[lane];
  }
}

hipError_t launch_pack_nchw_thr(const float* x, int N, int C, int H, int W, int pad, const float* thr,
                                uint64_t* xp, hipStream_t s) {
  PackNchwParams p;
  p.thr = thr;
  p.C = C;
  p.HW = H * W;
  p.H = H;
  p.W = W;
  p.pad = pad;
  p.Hp = H + 2 * pad;
  p.Wp = W + 2 * pad;
  p.Cw = (int)words_for(C);
  p.div_hw = make_fast_div((uint32_t)p.HW);
  p.div_w = make_fast_div((uint32_t)W);
  const bool nt = p.HW % 32 == 0 && ((uintptr_t)x & 127) == 0;
  // images per launch: all of them unless they have 2^31 padded pixels or more
  const int most = (int)std::min<int64_t>(N, (((int64_t)1 << 31) - 1) / ((int64_t)p.Hp * p.Wp));
  for (int n0 = 0; n0 < N; n0 += most) {
    const int n = std::min(most, N - n0);
    p.x = x + (int64_t)n0 * C * p.HW;
    p.xp = xp + (int64_t)n0 * p.Hp * p.Wp * p.Cw;
    p.images = n;
    p.pixels = (uint32_t)n * (uint32_t)p.HW;
    auto kern = thr ? (nt ? pack_nchw_kernel<true, true> : pack_nchw_kernel<true, false>)
                    : (nt ? pack_nchw_kernel<false, true> : pack_nchw_kernel<false, false>);
    // four threads a pixel, and less than 2^32 threads a launch
    for (uint64_t first = 0; first < p.pixels; first += 1u << 29) {
      p.first = (uint32_t)first;
      const dim3 grid((unsigned)ceil_div(std::min(p.pixels - p.first, 1u << 29), 512) * 8, (unsigned)p.Cw);
      note_kernel("pack_nchw_kernel<%s> grid %u x %u x 256", thr ? "thr" : "sign", grid.x, grid.y);
      launch_kernel(kern, grid, dim3(256), 0, s, p);
    }
  }
  return launch_error();
}

hipError_t launch_pack_nchw(const float* x, int N, int C, int H, int W, int pad, uint64_t* xp,
                            hipStream_t s) {
  return launch_pack_nchw_thr(x, N, C, H, W, pad, nullptr, xp, s);
}

// Offline weight packing for the convolution: Wp[o][(kh*KW + kw)*Cw + cw] bit c = (w[o][64cw + c][kh][kw]
// >= 0); rows are ld words apart, the words between the data and ldb (the chunk-padded bit section)
// are zero, and with consts set the row's K - 2 * popcount follows as a float, with zeros behind it.
// A workgroup per filter, a wave per 64 channels: their 64 * T floats (T taps, contiguous) come in
// as T coalesced loads, all in flight, and pass through LDS, where lane c reads element c * T + t: the
// 64-lane mask of its sign is word t (T is odd, so the lanes' reads fall on different banks).
// One thread per word, reading 64 floats T apart, took 10 us for 137 x 64 x 3 x 3 with a launch before
// it to set up the sums; 272 x 256 x 3 x 3 now takes 3.5 us in one launch.
constexpr int kPackConvWaves = 4;

template <int T>
__global__ void __launch_bounds__(64 * kPackConvWaves)
pack_conv_weights_kernel(const float* __restrict__ w, int C, int Cw, int ld, int ldb, int consts,
                         uint64_t* __restrict__ Wp) {
  __shared__ float stage[kPackConvWaves][64 * T];
  __shared__ int ones[kPackConvWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int64_t o = blockIdx.x;
  const float* wo = w + o * C * T;
  uint64_t* row = Wp + o * ld;
  const int kwords = T * Cw;
  int pc = 0;
  for (int cw = wave; cw < Cw; cw += waves) {
    const int first = cw * 64 * T, last = C * T - 1;
    float v[T];
#pragma unroll
    for (int j = 0; j < T; ++j) v[j] = wo[min(first + 64 * j + lane, last)];
#pragma unroll
    for (int j = 0; j < T; ++j) stage[wave][64 * j + lane] = v[j];
    __builtin_amdgcn_wave_barrier();  // (LDS of one wave: its own accesses complete in order)
    const bool real = cw * 64 + lane < C;  // channels past the last are 0 bits
    uint64_t mine = 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const uint64_t word = __ballot(real && stage[wave][lane * T + t] >= 0.0f);
      if (lane == t) mine = word;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < T) row[lane * Cw + cw] = mine;
    pc += __popcll(mine);
  }
  for (int j = kwords + threadIdx.x; j < ldb; j += blockDim.x) row[j] = 0;
  if (!consts) return;  // (workgroup-uniform)
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) pc += __shfl_xor(pc, off);
  if (lane == 0) ones[wave] = pc;
  __syncthreads();
  if (threadIdx.x == 0) {
    int sum = 0;
    for (int i = 0; i < waves; ++i) sum += ones[i];
    row[ldb] = __float_as_uint((float)(C * T - 2 * sum));
    row[ldb + 1] = 0;
  }
}

// The same for 25 and 49 taps, where that is long for a wave: 49 loads, 49 ways through LDS and 49 ballots in a chain.  A
// workgroup per filter and 64 channels (per filter where a constant has to be added up over its words); the floats
// come 16 bytes at a time, on any dword since a filter starts anywhere, at most four a thread, and the four waves share the
// taps.  Bound by the launch to some 4 MB of weights, past that by the way in.  Before (a wave per 64 channels) and now, us
// a call, filters in turn from HBM: 432 x 10 x 7 x 7 6.6 and 3.9, 64 x 512 x 7 x 7 10.9 and 4.3, 294 x 461 x 7 x 7 (27 MB) 14.8
// and 9.3, 512 x 512 x 7 x 7 (51 MB) 17.0 and 14.3, 256 x 512 x 5 x 5 7.6 and 6.1, 400 x 400 x 5 x 5 8.3 and 6.6, 512 x 512 x 5 x 5 9.1 and
// 9.2; read again and again, from the caches, the last 6.7 and 7.1, 512 x 256 x 5 x 5 4.2 and 4.4, the others as above.  (Two words
// of channels a workgroup, the second requested while the first is packed: 512 x 512 x 5 x 5 9.9, 400 x 400 x 5 x 5 9.4.)
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float v4f_lds __attribute__((ext_vector_type(4), may_alias));

template <int T>
__global__ void __launch_bounds__(256)
pack_conv_taps_kernel(const float* __restrict__ w, uint32_t total, int C, int Cw, int ld, int ldb, int consts,
                      int parts, FastDiv div_parts, uint64_t* __restrict__ Wp) {
  constexpr int kVec = 16 * T, kLoads = (kVec + 255) / 256, kTaps = (T + 3) / 4;
  __shared__ v4f_lds stage[kVec];
  __shared__ int ones[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, last = C * T - 1;
  for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) {
    const uint32_t o = fast_div(b, div_parts);
    const int part = (int)(b - o * (uint32_t)parts);
    const float* const wo = w + (int64_t)o * C * T;
    uint64_t* const row = Wp + (int64_t)o * ld;
    int pc = 0;
    for (int cw = part; cw < Cw; cw += parts) {
      const int first = cw * 64 * T;
      v4f_any v[kLoads];
#pragma unroll
      for (int j = 0; j < kLoads; ++j) {
        const int i = first + 4 * min(256 * j + (int)threadIdx.x, kVec - 1);
        if (i + 3 <= last) {
          v[j] = *(const v4f_any*)(wo + i);
        } else {  // (behind the filter: its last value, masked below)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[j][e] = wo[min(i + e, last)];
        }
      }
#pragma unroll
      for (int j = 0; j < kLoads; ++j)
        if (256 * j + (int)threadIdx.x < kVec) stage[256 * j + threadIdx.x] = v[j];
      __syncthreads();
      const bool real = cw * 64 + lane < C;  // channels past the last are 0 bits
      const float* const at = (const float*)stage + lane * T + wave;
      uint64_t mine = 0;
#pragma unroll
      for (int u = 0; u < kTaps; ++u) {
        const bool tap = 4 * u + wave < T;
        const uint64_t word = __ballot(real && tap && at[tap ? 4 * u : 0] >= 0.0f);
        if (lane == u) mine = word;
      }
      if (lane < kTaps && 4 * lane + wave < T) row[(4 * lane + wave) * Cw + cw] = mine;
      pc += __popcll(mine);
      __syncthreads();
    }
    if (part == 0)
      for (int j = T * Cw + threadIdx.x; j < ldb; j += 256) row[j] = 0;
    if (!consts) continue;  // (workgroup-uniform)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) pc += __shfl_xor(pc, off);
    if (lane == 0) ones[wave] = pc;
    __syncthreads();
    if (threadIdx.x == 0) {
      row[ldb] = __float_as_uint((float)(C * T - 2 * (ones[0] + ones[1] + ones[2] + ones[3])));
      row[ldb + 1] = 0;
    }
    __syncthreads();
  }
}

hipError_t launch_pack_conv_weights(const float* w, int O, int C, int KH, int KW, uint64_t* Wp,
                                    hipStream_t s) {
  const int Cw = (int)words_for(C);
  const int kwords = KH * KW * Cw;
  const int ld = (int)conv_weight_row_words(kwords), ldb = (int)conv_weight_bits_words(kwords);
  const int consts = conv_weight_short_k(kwords) ? 1 : 0;
  if (KH * KW <= 9) {
    const dim3 grid((unsigned)O), block(64 * (Cw < kPackConvWaves ? Cw : kPackConvWaves));
    auto go = [&](auto kern) { launch_kernel(kern, grid, block, 0, s, w, C, Cw, ld, ldb, consts, Wp); };
    if (KH * KW == 1) go(pack_conv_weights_kernel<1>);
    else go(pack_conv_weights_kernel<9>);
    return launch_error();
  }
  const int parts = consts ? 1 : Cw;
  const uint32_t total = (uint32_t)O * (uint32_t)parts;  // (2^32 of them would be 800 GB of packed filters)
  const dim3 grid(std::min<uint32_t>(total, 1u << 20));
  const FastDiv div = make_fast_div((uint32_t)parts);
  auto go = [&](auto kern) { launch_kernel(kern, grid, dim3(256), 0, s, w, total, C, Cw, ld, ldb, consts, parts, div, Wp); };
  if (KH * KW == 25) go(pack_conv_taps_kernel<25>);
  else go(pack_conv_taps_kernel<49>);
  return launch_error();
}

// k-bit weights: T[m][n * bw + r] holds the 1-bit-weight form against weight plane r;
// S[m][n] = sum_r 2^r T[m][n * bw + r], out = float(S) / denom.
__global__ void __launch_bounds__(256)
quant_combine_kernel(const int32_t* __restrict__ T, int64_t M, int64_t N, int bw, float denom,
                     int32_t* __restrict__ S, float* __restrict__ out, int64_t ldo) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= M * N) return;
  const int64_t m = i / N, n = i - m * N;
  const int32_t* t = T + (m * N + n) * bw;
  int32_t acc = 0;
  for (int r = 0; r < bw; ++r) acc += t[r] << r;
  if (S) S[m * ldo + n] = acc;
  if (out) out[m * ldo + n] = (float)acc / denom;
}

hipError_t launch_quant_combine(const int32_t* T, int64_t M, int64_t N, int bw, float denom, int32_t* S,
                                float* out, int64_t ldo, hipStream_t s) {
  launch_kernel(quant_combine_kernel, dim3((unsigned)ceil_div(M * N, 256)), dim3(256), 0, s, T, M, N, bw,
                     denom, S, out, ldo);
  return launch_error();
}

// alpha[r] = mean |w[r][:]| in fp64: a wave or a workgroup of four per row, nine loads per lane in flight, 16 bytes
// each, on any dword: rows of 4n + 1 values start anywhere.  Bound by the way in of the weights.  Before and now, us a
// call: 4096 x 9215 48.9 (4-byte loads) and 22.8, 294 x 22589 17.3 (eleven trips to memory in a chain) and 4.6, 1000 x
// 9215 14.1 and 5.9; the kernel at 4096 x 9216 from HBM 27.2 (a wave per row, kept in the caches) and 23.7 (6.4 TB/s).
template <int WAVES, bool NT>
__global__ void __launch_bounds__(256)
alpha_mean_abs_kernel(const float* __restrict__ w, int64_t rows, int64_t cols, int64_t ldw,
                      float* __restrict__ alpha) {
  __shared__ double part[WAVES];
  constexpr int kAhead = 9, kLanes = 64 * WAVES, kRows = 4 / WAVES;  // rows a workgroup
  const int t = threadIdx.x & (kLanes - 1);
  const int64_t nvec = cols / 4;
  for (int64_t r0 = (int64_t)blockIdx.x * kRows; r0 < rows; r0 += (int64_t)gridDim.x * kRows) {
    const int64_t r = r0 + (int)(threadIdx.x / kLanes);
    double acc0 = 0.0, acc1 = 0.0;
    if (r < rows) {
      const float* x = w + r * ldw;
      const float rest = 4 * nvec + t < cols ? x[4 * nvec + t] : 0.f;  // (the last one to three values)
      for (int64_t i0 = 0; i0 < nvec; i0 += kAhead * kLanes) {
        v4f_any v[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
          const int64_t i = i0 + j * kLanes + t;
          if (i < nvec) v[j] = NT ? __builtin_nontemporal_load((const v4f_any*)x + i) : ((const v4f_any*)x)[i];
          else v[j] = v4f_any{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
          acc0 += fabs((double)v[j].x) + fabs((double)v[j].y);
          acc1 += fabs((double)v[j].z) + fabs((double)v[j].w);
        }
      }
      acc0 += fabs((double)rest);
    }
    double acc = acc0 + acc1;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (WAVES == 1) {
      if (t == 0 && r < rows) alpha[r] = (float)(acc / (double)cols);
    } else {
      if ((t & 63) == 0) part[t >> 6] = acc;
      __syncthreads();
      if (t == 0) {
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) sum += part[i];
        alpha[r] = (float)(sum / (double)cols);
      }
      __syncthreads();
    }
  }
}

hipError_t launch_alpha_mean_abs(const float* w, int64_t rows, int64_t cols, int64_t ldw,
                                 float* alpha, hipStream_t s) {
  // A wave per row where it takes the row in one trip, or two with rows enough to hide them (1338 x 3237 3.4 us with
  // one wave, 3.8 with four; 2048 x 4096 3.6 and 4.5, 512 x 4900 3.3 and 2.9, 1276 x 8576 8.8 and 7.9).
  const bool one = cols <= 2304 || (cols <= 4096 && rows >= 1024);
  const bool nt = rows * cols * 4 > kStreamBytes;
  const dim3 grid((unsigned)std::min<int64_t>(one ? ceil_div(rows, 4) : rows, 65535 * 16));
  auto go = [&](auto kern) { launch_kernel(kern, grid, dim3(256), 0, s, w, rows, cols, ldw, alpha); };
  if (one && nt) go(alpha_mean_abs_kernel<1, true>);
  else if (one) go(alpha_mean_abs_kernel<1, false>);
  else if (nt) go(alpha_mean_abs_kernel<4, true>);
  else go(alpha_mean_abs_kernel<4, false>);
  return launch_error();
}

// Eq. 1 quantiser + bit-plane pack.  A wave per segment of 16 words of a row, up to 16 of them (rows of one or two
// segments share a workgroup), lane <-> k, and all 16 loads of a segment are issued before
// the first of them is used.  q = round(L * clamp(x)), ties away from zero, from the single
// fp32 product L * x.  Plane p of word w is the 64-lane mask of bit p of q and goes to row
// m * bits + p of `planes` (words up to ld_words are written, zeros past the data).  The row
// sum of q, needed by the plane GEMM epilogue, is reduced through LDS.
// The weight operand of the same GEMM is sign-packed by the workgroups past the first ones of
// the same launch, so that the two inputs cost one kernel launch, not two.
// Bound by the two matrices' way in and, beside it, the vector ALU: 15 instructions a value at two bits with the quantiser
// itself.  The launch, from HBM, with it and four waves a row, and now: 1024 x 4096 and 1024 x 4096 weights 9.9 us and 7.6
// (4.4 TB/s), 2048 x 2048 twice 9.2 and 7.4, 300 x 5000 and 700 x 5000 (five segments) 8.8 and 6.8.
// One and two bits (BITS, else 0): the quantiser is monotone in x, so q >= i is x >= the smallest float that reaches i
// (tried on both sides below with the quantiser itself), and the compares' masks make the planes.
constexpr float kThird1 = 0x1.555556p-3f, kThird3 = 0x1.aaaaaap-1f;
static constexpr int quantised(float x, float L) {
#pragma clang fp contract(off)
  const float u = L * x;
  return (int)(u + 0x1.fffffep-2f);
}
static_assert(quantised(0.5f, 1.0f) == 1 && quantised(0x1.fffffep-2f, 1.0f) == 0);
static_assert(quantised(kThird1, 3.0f) == 1 && quantised(0x1.555554p-3f, 3.0f) == 0);
static_assert(quantised(0.5f, 3.0f) == 2 && quantised(0x1.fffffep-2f, 3.0f) == 1);
static_assert(quantised(kThird3, 3.0f) == 3 && quantised(0x1.aaaaa8p-1f, 3.0f) == 2);

template <int BITS>
__global__ void __launch_bounds__(1024)
quant_pack_kernel(const float* __restrict__ a, int64_t M, int64_t K, int64_t lda, int bits,
                  uint64_t* __restrict__ planes, int64_t ld_words, int32_t* __restrict__ rowsum,
                  const float* __restrict__ w, uint32_t wsegs, int64_t ldw, uint64_t* __restrict__ wbits, int64_t wb_ld,
                  FastDiv div_segs, uint32_t segs_per_row, uint32_t segs_per_block, uint32_t blocks_a, int per_row, int affine) {
  __shared__ int32_t part[16];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), waves = blockDim.x / kWave;
  if (blockIdx.x >= blocks_a) {
    pack_row_segments<false>(w, wsegs, K, ldw, wbits, wb_ld, words_for(K), div_segs, segs_per_row,
                          (blockIdx.x - blocks_a) * segs_per_block, segs_per_block);
    return;
  }
  const int sub = wave / per_row;  // row of the workgroup
  const int64_t m = (int64_t)blockIdx.x * (waves / per_row) + sub;
  const float L = (float)((1u << bits) - 1u);
  const float* ar = a + m * lda;
  uint64_t* prow = planes + m * bits * ld_words;
  int32_t sum = 0;
  for (int64_t w0 = (int64_t)(wave - sub * per_row) * kSegWords; m < M && w0 < ld_words; w0 += per_row * kSegWords) {
    const float* const as = ar + w0 * 64;
    const int64_t left = K - w0 * 64;  // (none where only padding words are left)
    float v[kSegWords];
    if (left >= 64 * kSegWords) {
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) v[j] = as[64 * j + lane];
      // (signed operand: [-1, 1] onto [0, 1] first, two fp32 operations)
      if (BITS == 0 && affine) {
#pragma unroll
        for (int j = 0; j < kSegWords; ++j) v[j] = __fmul_rn(__fadd_rn(v[j], 1.0f), 0.5f);
      }
    } else {
      const int n = (int)left;
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) v[j] = left > 0 ? as[(uint32_t)min(64 * j + lane, n - 1)] : 0.0f;
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) {
        if (BITS == 0 && affine) v[j] = __fmul_rn(__fadd_rn(v[j], 1.0f), 0.5f);
        v[j] = 64 * j + lane < n ? v[j] : 0.0f;
      }
    }
    if constexpr (BITS == 1 || BITS == 2) {
      uint64_t plane[BITS];
      uint32_t lo[BITS], hi[BITS];
#pragma unroll
      for (int p = 0; p < BITS; ++p) lo[p] = hi[p] = 0;
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) {
        plane[BITS - 1] = __ballot(v[j] >= 0.5f);
        if (BITS == 2) plane[0] = (__ballot(v[j] >= kThird1) & ~plane[BITS - 1]) | __ballot(v[j] >= kThird3);
#pragma unroll
        for (int p = 0; p < BITS; ++p) {
          lo[p] = write_lane((uint32_t)plane[p], j, lo[p]);
          hi[p] = write_lane((uint32_t)(plane[p] >> 32), j, hi[p]);
        }
      }
#pragma unroll
      for (int p = 0; p < BITS; ++p) {
        sum += (__popc(lo[p]) + __popc(hi[p])) << p;
        if (lane < kSegWords && w0 + lane < ld_words) prow[p * ld_words + w0 + lane] = ((uint64_t)hi[p] << 32) | lo[p];
      }
      continue;
    }
    // Half away from zero of u >= 0 is trunc(u + (0.5 - 2^-25)) in fp32 (with 0.5 itself the one value
    // 0.5 - 2^-25 would round up): one addition where roundf takes a truncation, a subtraction, a compare, a
    // selection, a sign and an addition.  us a call with roundf and now, 2 x 1 bits: 1024 x 1024 x 4096 14.0 / 13.9,
    // 2048 x 2048 x 2048 17.5 / 17.3, 4096 x 256 x 4096 20.4 / 19.5.
    // Product and sum are two roundings: fused, seven floats at 5 and 7 bits land on the level below.
    int q[kSegWords];
#pragma unroll
    for (int j = 0; j < kSegWords; ++j) {
#pragma clang fp contract(off)
      const float u = L * fminf(fmaxf(v[j], 0.0f), 1.0f);
      q[j] = (int)(u + 0x1.fffffep-2f);
      sum += q[j];
    }
    for (int p = 0; p < bits; ++p) {
      uint64_t mine = 0;
#pragma unroll
      for (int j = 0; j < kSegWords; ++j) {
        const uint64_t mask = __ballot((q[j] >> p) & 1);
        if (lane == j) mine = mask;
      }
      if (lane < kSegWords && w0 + lane < ld_words) prow[p * ld_words + w0 + lane] = mine;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, kWave);
  if (per_row == 1) {
    if (lane == 0 && m < M) rowsum[m] = sum;
    return;
  }
  if (lane == 0) part[wave] = sum;
  __syncthreads();
  if (lane == 0 && wave == sub * per_row && m < M) {
    for (int i = 1; i < per_row; ++i) sum += part[wave + i];
    rowsum[m] = sum;
  }
}

hipError_t launch_quant_pack(const float* a, int64_t M, int64_t K, int64_t lda, int bits,
                             uint64_t* planes, int64_t ld_words, int32_t* rowsum, const float* w,
                             int64_t wrows, int64_t ldw, uint64_t* wbits, int64_t wb_ld,
                             hipStream_t s, bool affine) {
  const int per_row = (int)std::min<int64_t>(ceil_div(ld_words, kSegWords), 16);
  const int rows = per_row <= 2 ? 4 / per_row : 1, waves = rows * per_row;
  const uint32_t spr = (uint32_t)ceil_div(words_for(K), kSegWords), wsegs = (uint32_t)wrows * spr;
  const uint32_t blocks_a = (uint32_t)ceil_div(M, rows), blocks_w = (uint32_t)std::min<int64_t>(ceil_div(wsegs, waves), 1 << 20);
  const uint32_t blocks = blocks_a + blocks_w, per_block = blocks_w ? (uint32_t)ceil_div(wsegs, blocks_w) : 0;
  note_kernel("quant_pack_kernel grid %u x %d", blocks, 64 * waves);
  const FastDiv div = make_fast_div(spr);
  auto go = [&](auto kern) {
    launch_kernel(kern, dim3(blocks), dim3(64 * waves), 0, s, a, M, K, lda, bits, planes, ld_words, rowsum, w, wsegs, ldw,
                  wbits, wb_ld, div, spr, per_block, blocks_a, per_row, affine ? 1 : 0);
  };
  if (affine || bits > 2) go(quant_pack_kernel<0>);
  else if (bits == 2) go(quant_pack_kernel<2>);
  else go(quant_pack_kernel<1>);
  return launch_error();
}

}  // namespace bmx
