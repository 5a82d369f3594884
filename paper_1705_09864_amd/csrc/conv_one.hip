// Binary convolution of an fp32 image in one launch.
// Paper: Sec. 2 (QConvolution: binarise the input, xnor GEMM, optional scale), Sec. 3.1 (M = filters,
// N = batch * output pixels, K = kh * kw * C).
//
// The general path is two launches, channel pack then convolution, each a launch on the host (2.7 us)
// and on the GPU a chain of trips to memory of 4 to 5 us however little there is to do.  Here a
// workgroup of up to 16 waves takes a band of output rows of one image and a share of the filters:
//   - its waves pack the band's input rows into LDS, 64 pixels x 16 channels per wave and step, all 16
//     loads in flight and the next step's behind them (the same bits as the packed image, halo
//     included, 16 of a word's bits at a time);
//   - after one barrier each wave takes units of 32 output pixels x 32 filters: the pixels' words come
//     from LDS, the filters' straight from the packed rows (16 bytes per lane, turned into the MFMA's
//     order by a half-wave swap), both are expanded to FP4 in registers and multiplied as in
//     conv_mfma.hip: out = alpha * ((K - 2 popcount(filter)) + 2 * sum f x).
// Where a workgroup has fewer units than waves, 2 to 8 waves share the K range of one and meet in LDS: what
// is left after packing is otherwise one wave's chain of K / 4 steps (7 x 7 x 64: 9.1 -> 6.1 us).
// Input rows are read once per band they belong to and per share of the filters, and a filter is
// expanded once per unit (8 vector instructions a word where the two-launch kernel shares them through
// LDS): that is what the form costs, and what the launcher weighs against the second launch.
//
// What bounds it is the chain of one workgroup (arguments, fp32 rows, bits in LDS, products, sums, results: 9 to 11 thousand
// clocks, of which the memory's part is 2 to 3) and the instructions on it: at one scalar and one vector instruction in four
// clocks a SIMD, what every wave repeats costs as much as what it shares.  Hence as few waves as do the work; sign bits
// gathered by carries; the halo, the places of a patch's words and the first filter operands made under the fp32 loads; scales
// requested with the filters; row constants read four at a time; results stored through a buffer that drops what is not part of them.
// Measured, us in a graph, with sixteen waves and none of that / now: 7 x 130 x 29 x 27 -> 70 3x3/2 6.85 / 5.14, 4 x 64 x 11 x 13 -> 60
// 3x3 5.0 / 3.8, 35 x 64 x 21 x 21 -> 40 1x1 4.85 / 3.55, 7 x 26 x 49 x 48 -> 68 3x3 7.8 / 6.0, 83 x 96 x 11 x 11 -> 115 1x1/2 5.1 / 3.9.
// One launch against two, a call: 1 x 64 x 8 x 8 -> 64 1x1 3.5 / 6.4, 7 x 130 x 29 x 27 -> 70 3x3/2 5.3 / 7.6 (in a graph 3.1 / 4.1
// and 5.1 / 5.6); 16 x 64 x 56 x 56 -> 64 3x3 would take 9.4 / 8.3 and stays with two.
#include <algorithm>
#include <type_traits>

#include "bmx_internal.h"
#include "conv_expand.h"

namespace bmx {

namespace {

constexpr int kWaves = 16;
constexpr int kLds = 64 * 1024;               // dynamic LDS without asking for more
constexpr int kRowBytes = kWaves * 64 * 4;     // row constants and scales, where a wave has units to itself
constexpr int kPartBytes = 64 * (16 + 1) * 4;  // a wave's sums, counts and scales in LDS

typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef uint16_t __attribute__((may_alias)) u16_alias;
typedef uint32_t __attribute__((may_alias)) u32_alias;
typedef float v4f_alias __attribute__((ext_vector_type(4), may_alias));

struct ConvOneParams {
  const float* x;
  const uint64_t* Wp;
  const float* alpha;
  void* out;  // int32 or fp32
  int C, H, W, O;
  int Ho, Wo;
  int K, Cw, KH, run;  // words of a patch; channel words; kernel rows; words per kernel row
  int stride, pad, rows, bands;  // output rows per band, bands per image
  int tiles;     // filter tiles of 32 per workgroup
  uint32_t ld_bytes;  // bytes per packed filter row
  int Kreal;
  int sums_at;  // byte offset in LDS of what stands behind the image
  FastDiv div_w, div_wp, div_wo, div_quarters, div_bands, div_run;
  FastDiv div_blocks, div_blocks_last;  // by the pixel blocks of a band, of the image's last one
  int items;  // bands of all images
  int quarters;  // sixteens of channels, the last maybe not whole
  int waves;     // per workgroup
};

// a uniform quotient, on the scalar unit
__device__ __forceinline__ int scalar_div(int n, FastDiv f) { return (int)__builtin_amdgcn_readfirstlane(fast_div((uint32_t)n, f)); }

// bits = 16 * bits + 8 * (d >= 0) + 4 * (c >= 0) + 2 * (b >= 0) + (a >= 0): a compare's mask is the carry of the sum that
// shifts, two instructions a value instead of three.  Four at a time: a mask is read two instructions after its compare
// or later, as the hardware wants it.
__device__ __forceinline__ void shift_in_signs(uint32_t& bits, float a, float b, float c, float d) {
  uint64_t ma, mb, mc, md;
  asm("v_cmp_le_f32 %4, 0, %8\n\tv_cmp_le_f32 %3, 0, %7\n\tv_cmp_le_f32 %2, 0, %6\n\tv_cmp_le_f32 %1, 0, %5\n\t"
      "v_addc_co_u32 %0, %4, %0, %0, %4\n\tv_addc_co_u32 %0, %3, %0, %0, %3\n\t"
      "v_addc_co_u32 %0, %2, %0, %0, %2\n\tv_addc_co_u32 %0, %1, %0, %0, %1"
      : "+v"(bits), "=&s"(ma), "=&s"(mb), "=&s"(mc), "=&s"(md)
      : "v"(a), "v"(b), "v"(c), "v"(d));
}

template <bool I32, int PARTS>
__global__ void __launch_bounds__(64 * kWaves)
conv_one_kernel(const ConvOneParams p) {
  extern __shared__ uint64_t img[];  // [band input rows][W + 2 pad][Cw]
  // (all arguments named at the top: fetched in one batch, one trip to memory instead of one per group)
  asm volatile("" ::"s"(p.x), "s"(p.Wp), "s"(p.alpha), "s"(p.C), "s"(p.H), "s"(p.W), "s"(p.O), "s"(p.Ho), "s"(p.Wo), "s"(p.K), "s"(p.Cw),
               "s"(p.KH), "s"(p.run), "s"(p.stride), "s"(p.pad), "s"(p.rows), "s"(p.bands), "s"(p.tiles), "s"(p.ld_bytes),
               "s"(p.div_quarters.mul), "s"(p.div_bands.mul), "s"(p.div_run.mul), "s"(p.div_blocks.mul), "s"(p.items), "s"(p.quarters));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;
  // Workgroup b sits on XCD b % 8: every XCD gets a contiguous run of bands, which share input rows (and this
  // batch of arguments: 12 x 390 x 24 x 26 -> 83 1x1 8.5 -> 7.3 us a call, 33 x 257 x 18 x 18 -> 240 1x1 10.7 -> 9.4)
  const int lin = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (lin >= p.items) return;  // (the whole workgroup)
  const int n = scalar_div(lin, p.div_bands), band = lin - n * p.bands;
  const int Wpp = p.W + 2 * p.pad, HW = p.H * p.W;
  const int ho0 = band * p.rows, nrows = min(p.rows, p.Ho - ho0);
  const int top = ho0 * p.stride - p.pad;             // input row of the band's first padded row
  const int rin = (nrows - 1) * p.stride + p.KH;      // padded rows of the band
  const int row0 = max(top, 0), row1 = min(top + rin, p.H);
  const int skip_top = row0 - top;
  const int npx = max(row1 - row0, 0) * p.W;          // real pixels of the band, contiguous in a plane

  // ---- this wave's units of 32 pixels x 32 filters; the first one's filter words are requested ahead of all
  const FastDiv div_blocks = nrows == p.rows ? p.div_blocks : p.div_blocks_last;
  const int px_blocks = (nrows * p.Wo + 31) >> 5;
  const int tile0 = blockIdx.y * p.tiles, ntiles = min(p.tiles, ((p.O + 31) >> 5) - tile0);
  const int units = px_blocks * ntiles;
  // PARTS waves share the K range of a unit (if more than one: units * PARTS <= kWaves in every workgroup)
  constexpr bool SPLIT = PARTS > 1;
  int part = 0;
  if (SPLIT) {
#pragma unroll
    for (int e = 1; e <= PARTS; ++e) part += wave >= e * units ? 1 : 0;  // (PARTS: none of the units is this wave's)
  }
  const int unit0 = SPLIT ? wave - part * units : wave, mine = SPLIT ? min(part, PARTS - 1) : 0;
  const int steps = (p.K + 3) >> 2;  // of four words (the packed rows are padded with zero words)
  const int first = SPLIT ? mine * steps / PARTS : 0;  // this wave's steps of every unit
  const int last = SPLIT ? (mine + 1) * steps / PARTS : steps;
  // What a unit needs beside its pixels: filter words (of four steps at a time), filter r's scale, where pixel r's patch
  // starts in the image (dword h of its words) and where filter 4 h and pixel r of the tile go in an image's results.
  struct Unit {
    v4u fw[4];
    uint32_t frow;
    float al;
    uint32_t patch, to;
  };
  const uint32_t pitch = (uint32_t)(p.Ho * p.Wo) * 4u, results = (uint32_t)p.O * pitch;
  auto open = [&](Unit& u, int k) {
    const int ft = scalar_div(k, div_blocks), m0 = (tile0 + ft) * 32;
    const uint32_t row = (uint32_t)min(m0 + r, p.O - 1);
    u.frow = row * p.ld_bytes + 16u * h;
#pragma unroll
    for (int i = 0; i < 4; ++i) u.fw[i] = *(const v4u*)((const char*)p.Wp + (u.frow + 32u * (uint32_t)min(first + i, last - 1)));
    u.al = (!I32 && p.alpha) ? p.alpha[row] : 1.0f;
    const int q = 32 * (k - ft * px_blocks) + r, qc = min(q, nrows * p.Wo - 1);
    const int ho = (int)fast_div((uint32_t)qc, p.div_wo), wo = qc - ho * p.Wo;
    u.patch = (uint32_t)((ho * Wpp + wo) * p.stride * p.Cw) * 8u + 4u * h;
    // (pixels past the band's last, like filters past O: behind the image's results, where nothing is stored)
    u.to = q == qc ? (uint32_t)(m0 + 4 * h) * pitch + (uint32_t)(ho0 * p.Wo + q) * 4u : results;
  };
  Unit u;
  open(u, min(unit0, units - 1));

  // ---- pack: item = (64 pixels, 16 channels)
  const int items = ((npx + 63) >> 6) * p.quarters;
  const uint32_t plane = (uint32_t)HW * 4u;
  struct Item {
    float v[16];
    bool last;
    int at, real;  // the 16 bits' place in the image (negative: none), channels
  };
  auto load = [&](Item& it, int t) {
    const int g = scalar_div(t, p.div_quarters), quarter = t - g * p.quarters, c0 = quarter * 16;
    const int px = g * 64 + lane;
    it.real = min(16, p.C - c0);
    it.last = quarter == p.quarters - 1;
    const char* const base = (const char*)(p.x + (((int64_t)n * p.C + c0) * HW + row0 * p.W));
    const __amdgpu_buffer_rsrc_t planes = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)0xffffffff, 0x00020000);
    const uint32_t off = 4u * (uint32_t)min(px, npx - 1);
    if (it.real == 16) {  // uniform
#pragma unroll
      for (int j = 0; j < 16; ++j) it.v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(planes, off, plane * (uint32_t)j, 0));
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j)  // (channels past the last repeat it and are masked)
        it.v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(planes, off, plane * (uint32_t)min(j, it.real - 1), 0));
    }
    const int hi = (int)fast_div((uint32_t)px, p.div_w), wi = px - hi * p.W;
    it.at = px < npx ? 4 * ((hi + skip_top) * Wpp + wi + p.pad) * p.Cw + quarter : -1;
  };
  auto pack = [&](const Item& it) {
    uint32_t b = 0;
#pragma unroll
    for (int j = 12; j >= 0; j -= 4) shift_in_signs(b, it.v[j], it.v[j + 1], it.v[j + 2], it.v[j + 3]);
    if (it.at >= 0) {
      ((u16_alias*)img)[it.at] = (uint16_t)(b & ((1u << it.real) - 1u));
      if (it.last) {  // uniform: the rest of the last word
        for (int i = p.quarters; i < 4 * p.Cw; ++i) ((u16_alias*)img)[it.at + 1 + i - p.quarters] = 0;
      }
    }
  };
  Item a, b;
  if (wave < items) load(a, wave);

  // ---- under those loads: the halo (the sign of the zero padding, +1 for every real channel), where the words of the
  // patch lie and the first step's filter operands
  if (p.pad > 0) {
    for (int i = threadIdx.x; i < rin * Wpp; i += 64 * p.waves) {
      const int hi = (int)fast_div((uint32_t)i, p.div_wp), wi = i - hi * Wpp;
      if (hi < skip_top || hi >= skip_top + (row1 - row0) || wi < p.pad || wi >= p.pad + p.W)
        for (int cw = 0; cw < p.Cw; ++cw)
          img[i * p.Cw + cw] = (cw == p.Cw - 1 && (p.C & 63)) ? ((uint64_t)1 << (p.C & 63)) - 1 : ~(uint64_t)0;
    }
  }
  // lane l: byte offset in a patch of word 4 first + l (words past K: the first); a wave's words are at most 64
  const uint32_t kw = 4u * (uint32_t)first + (uint32_t)lane;
  const uint32_t offs = kw < (uint32_t)p.K ? (fast_div(kw, p.div_run) * (uint32_t)(Wpp * p.Cw - p.run) + kw) * 8u : 0u;
  v4i ef[4];
  int pc = 0;
  // The filter words of a step as operands; those of four steps on are requested in their place.
  auto expand_step = [&](Unit& u, int i) {
    // lane (r, 0) holds words 4 i, 4 i + 1 of filter r, lane (r, 1) words 4 i + 2, 4 i + 3
    const v2u t = __builtin_amdgcn_permlane32_swap(u.fw[0][0], u.fw[0][1], false, false);
    const v2u s = __builtin_amdgcn_permlane32_swap(u.fw[0][2], u.fw[0][3], false, false);
    const uint32_t f[4] = {t[0], s[0], t[1], s[1]};
    u.fw[0] = u.fw[1], u.fw[1] = u.fw[2], u.fw[2] = u.fw[3];
    if (i + 4 < last) u.fw[3] = *(const v4u*)((const char*)p.Wp + (u.frow + 32u * (uint32_t)(i + 4)));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pc += __builtin_popcount(f[j]);
      ef[j] = expand_filter(f[j]);
    }
  };
  expand_step(u, first);

  for (int t = wave; t < items; t += 2 * p.waves) {
    if (t + p.waves < items) load(b, t + p.waves);
    pack(a);
    if (t + p.waves >= items) break;
    if (t + 2 * p.waves < items) load(a, t + 2 * p.waves);
    pack(b);
  }
  __syncthreads();

  // ---- multiply
  constexpr int kOwn = 16 / PARTS;
  v16f acc;  // (one chain: the SIMD's other three waves fill the matrix pipe)
  auto multiply = [&](Unit& u) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    uint32_t xw[4];
    auto read = [&](int i) {  // dword h of the words of step i
#pragma unroll
      for (int j = 0; j < 4; ++j)
        xw[j] = *(const u32_alias*)((const char*)img + (u.patch + (uint32_t)__builtin_amdgcn_readlane((int)offs, 4 * (i - first) + j)));
    };
    read(first);
    for (int i = first; i < last; ++i) {
      uint32_t x[4] = {xw[0], xw[1], xw[2], xw[3]};
      if (4 * i + 4 > p.K) {  // wave-uniform: the last step; words past K are zero pixels
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = 4 * i + j < p.K ? x[j] : 0u;
      }
      if (i + 1 < last) read(i + 1);
      // (without block scales, which cost the issue of an MFMA 6 clocks of 17: 0.98 of the time of 7 x 130 x 29 x 27 -> 70)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(ef[j]), widen(expand_pixel(x[j])), acc, 4, 4, 0, 0, 0, 0);
      if (i + 1 < last) expand_step(u, i + 1);
      __builtin_amdgcn_sched_barrier(0);  // (operands of later steps made early would spill: 128 registers)
    }
    pc += __shfl_xor(pc, 32);  // of filter r of the tile
  };
  // Results: register v of a wave's sixteen is filter 8 (v / 4) + 4 h + v % 4, pixel r.  Row constants c0 = K - 2 popcount and
  // scales pass through LDS, four rows a read.  (A buffer of one image's results: what lies past it is not stored.)
  const __amdgpu_buffer_rsrc_t image_out =
      __builtin_amdgcn_make_buffer_rsrc((char*)p.out + (int64_t)n * results, 0, (int)results, 0x00020000);
  auto store = [&](const Unit& u, int v, float sum, float c0, float al) {
    const float dot = fmaf(2.0f, sum, c0);
    const uint32_t bits = I32 ? (uint32_t)(int)dot : __float_as_uint(al * dot);
    __builtin_amdgcn_raw_buffer_store_b32(bits, image_out, u.to + (uint32_t)(8 * (v / 4) + v % 4) * pitch, 0, 0);
  };
  if (!SPLIT) {
    float* const rows = (float*)((char*)img + p.sums_at) + wave * 64;
    for (int k = wave; k < units; k += p.waves) {
      if (k != wave) {
        open(u, k);
        pc = 0;
        expand_step(u, 0);
      }
      multiply(u);
      if (h == 0) rows[r] = (float)(p.Kreal - 2 * pc);
      else rows[32 + r] = u.al;
      asm volatile("" ::: "memory");  // (the wave's own LDS accesses stay in this order)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v4f_alias c = *(const v4f_alias*)(rows + 8 * g + 4 * h), al = *(const v4f_alias*)(rows + 32 + 8 * g + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) store(u, 4 * g + e, acc[4 * g + e], c[e], al[e]);
      }
      asm volatile("" ::: "memory");
    }
    return;
  }
  // SPLIT: the parts of a unit meet in LDS behind the image, [unit]([part][four rows][lane][4], [part][32 counts], [32 scales]),
  // and each finishes its share of the sixteen
  const bool busy = part < PARTS;
  char* const sums = (char*)img + p.sums_at + unit0 * (PARTS * kPartBytes);
  float* const counts = (float*)(sums + PARTS * 4096);
  if (busy) {
    multiply(u);
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(v4f_alias*)(sums + part * 4096 + g * 1024 + lane * 16) = v4f_alias{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    if (h == 0) counts[part * 32 + r] = (float)((part == 0 ? p.Kreal : 0) - 2 * pc);
    else if (part == 0) counts[PARTS * 32 + r] = u.al;
  }
  __syncthreads();
  if (!busy) return;
  constexpr int kRun = kOwn < 4 ? kOwn : 4;  // consecutive registers of a share
  typedef float run_t __attribute__((ext_vector_type(kRun), may_alias));
#pragma unroll
  for (int o = 0; o < kOwn; o += kRun) {
    const int v = part * kOwn + o, row = 8 * (v >> 2) + (v & 3) + 4 * h;
    run_t t[PARTS], c[PARTS];
#pragma unroll
    for (int e = 0; e < PARTS; ++e) {
      t[e] = *(const run_t*)(sums + e * 4096 + (v >> 2) * 1024 + lane * 16 + (v & 3) * 4);
      c[e] = *(const run_t*)(counts + e * 32 + row);
    }
    const run_t al = *(const run_t*)(counts + PARTS * 32 + row);
#pragma unroll
    for (int e = 1; e < PARTS; ++e) t[0] += t[e], c[0] += c[e];
#pragma unroll
    for (int e = 0; e < kRun; ++e) store(u, v + e, t[0][e], c[0][e], al[e]);
  }
}

}  // namespace

// (Not asked of the default stream, which cannot: the question would be an error while another stream's are.)
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (!s) return false;
  if (hipStreamIsCapturing(s, &status) == hipSuccess) return status == hipStreamCaptureStatusActive;
  (void)hipGetLastError();
  return false;
}

int conv_one = 0;  // 1 = never, 2 = wherever a workgroup holds a band (measurements and tests of either path)

bool launch_conv_one(const float* x, int N, int C, int H, int W, const uint64_t* Wp, int O, int KH, int KW, int stride,
                     int pad, const float* alpha, int32_t* out_i32, float* out_f32, hipStream_t s, hipError_t* err) {
  if (conv_one == 1 || conv_path != 0 || gemm_engine != 0 || ((uintptr_t)Wp & 15)) return false;
  const int Ho = (H + 2 * pad - KH) / stride + 1, Wo = (W + 2 * pad - KW) / stride + 1;
  const int Cw = (int)words_for(C), K = KH * KW * Cw, Wpp = W + 2 * pad;
  if (N > 65535 || O > 65535 * 32 || (int64_t)H * W * 4 >= ((int64_t)1 << 31) || (int64_t)C * KH * KW >= ((int64_t)1 << 24)) return false;
  // (32-bit offsets in an image's results, in sixteen planes of the image and in the filters)
  if (((int64_t)N * O + 32) * Ho * Wo * 4 >= ((int64_t)1 << 32) || (int64_t)H * W >= (1 << 26) ||
      O * conv_weight_row_words(K) * 8 >= ((int64_t)1 << 32))
    return false;
  const int tiles = (int)ceil_div(O, 32);
  // The two launches' time on the GPU in us, fitted to 5225 shapes (6 % rms): KB of input and of results, words of 32 x 32 results,
  // the chain of a patch's words.  As calls they take never less than the host does for two launches and a workspace, 6.9 to 8.2 us by
  // the process.
  const double in_kb_all = (double)N * C * H * W / 256, out_kb_all = (double)N * O * Ho * Wo / 256;
  const double unit_words = (double)N * Ho * Wo * tiles * K;
  const double two = 5.03 + in_kb_all * 1.11e-4 + out_kb_all * 1.81e-4 + unit_words * 9.27e-7 + K * 0.0114;
  const double limit = conv_one == 2 ? 1e30 : 0.98 * std::max(7.6, two);
  // Output rows per band, filter tiles per workgroup and waves per unit: those of the shortest modelled
  // time, fitted to the same shapes (5 % rms).  Beside what all launches pay, a round of workgroups
  // costs its fp32 rows (KB), the loads of them (64 pixels x 16 channels each, whole or not), its words per SIMD (one unit in four
  // waves: 1) and its results (KB).  One launch or two by it, over these shapes: 0.33 % behind the better as calls, 0.32 % in a graph (0.5
  // and 1.35 % while rounds were counted by the chip and rows in KB alone).
  auto cost_of = [](double rounds, double in_kb, double loads, double words, double out_kb) {
    return 3.375 + rounds * 0.05 + in_kb * 0.0051 + loads * 0.067 + words * 0.0565 + out_kb * 0.0373;
  };
  // (no plan is below an even share of everything: most layers that stay with two launches end here)
  const double in_share = in_kb_all * std::min(1.0, (double)KH / stride) / 256;
  if (cost_of(1, in_share, in_share / 4, unit_words / (32 * 4 * 256), out_kb_all / 256) > limit) return false;
  double best = 1e30;
  int rows = 0, share = 0, parts = 1, units_max = 0;
  const int steps = (K + 3) / 4, quarters = (C + 15) / 16;
  for (int rr = 1; rr <= Ho; rr = rr < 4 ? rr + 1 : rr + (rr + 1) / 2) {
    const int rin = (rr - 1) * stride + KH;
    if ((int64_t)rin * Wpp * Cw * 8 > kLds - kRowBytes) break;
    const int image = (rin * Wpp * Cw * 8 + 15) & ~15;
    const int bands = (Ho + rr - 1) / rr, px_blocks = (rr * Wo + 31) / 32;  // (32-bit: this runs on every call)
    const int px = std::min(rin, H) * W;
    const double in_kb = (double)px * C / 256, loads = (double)((px + 63) / 64) * quarters;
    double rounds = 0;
    for (int g = 1; g <= tiles; g *= 2) {
      const int per = (tiles + g - 1) / g, units = px_blocks * per;
      // K is split over idle waves: down to a step of four words each while that leaves every SIMD two
      // waves at most, to two steps each beyond (parts of one step lose more in the sums than they gain)
      int ks = 1;
      while (ks < 8 && ks * 2 * units <= kWaves && ks * 2 <= (ks * 2 * units <= kWaves / 2 ? steps : steps / 2) &&
             image + ks * 2 * units * kPartBytes <= kLds) ks *= 2;
      if ((steps + ks - 1) / ks > 16) continue;  // (a lane of the wave holds the place of each of its words)
      const double words = ks > 1 ? std::max(1.0, units * ks / 4.0) * ((K + ks - 1) / ks) : (double)((units + 3) / 4) * K;
      // (An XCD has 32 CUs, and the first of them a whole eighth of the bands, rounded up: 25 x 40 x 21 x 21 -> 320 5x5/2 in 50 bands of 5
      // workgroups is 35 of them on one, two rounds: 11.7 us where two launches take 7.1)
      rounds = (double)(((((int64_t)bands * N + 7) >> 3) * ((tiles + per - 1) / per) + 31) >> 5);
      const double cost = cost_of(rounds, rounds * in_kb, rounds * loads, rounds * words, rounds * rr * Wo * std::min(O, 32 * per) / 256);
      if (cost < best) best = cost, rows = rr, share = per, parts = ks, units_max = units;
    }
    if (rounds == 1) break;  // one round however the filters are shared: longer bands cost more
  }
  if (rows == 0 || best > limit) return false;
  // A replayed graph pays the GPU's part of two launches alone: 3 x 256 x 25 x 25 -> 128 3x3 takes 7.6 us in one launch; two are 8.5 in a
  // call, 5.7 in a graph.  (Of 1770 layers in a graph the line at 0.98 left 1.4 % on one launch and 2.9 % on two that are more than 3 %
  // behind the other form there, at 1.02 2.6 and 0.7 %; behind the better form by 0.39 and 0.26 % on average.)
  if (conv_one != 2 && best > 1.02 * two && capturing(s)) return false;
  ConvOneParams p;
  p.x = x;
  p.Wp = Wp;
  p.alpha = alpha;
  p.out = out_i32 ? (void*)out_i32 : (void*)out_f32;
  p.C = C;
  p.H = H;
  p.W = W;
  p.O = O;
  p.Ho = Ho;
  p.Wo = Wo;
  p.K = K;
  p.Cw = Cw;
  p.KH = KH;
  p.run = KW * Cw;
  p.stride = stride;
  p.pad = pad;
  p.rows = rows;
  p.bands = (int)ceil_div(Ho, rows);
  p.tiles = share;
  p.ld_bytes = (uint32_t)(conv_weight_row_words(K) * 8);
  p.Kreal = C * KH * KW;
  p.div_w = make_fast_div((uint32_t)W);
  p.div_wp = make_fast_div((uint32_t)Wpp);
  p.div_wo = make_fast_div((uint32_t)Wo);
  p.quarters = quarters;
  p.div_quarters = make_fast_div((uint32_t)p.quarters);
  p.div_bands = make_fast_div((uint32_t)p.bands);
  p.div_run = make_fast_div((uint32_t)p.run);
  p.div_blocks = make_fast_div((uint32_t)ceil_div(rows * Wo, 32));
  p.div_blocks_last = make_fast_div((uint32_t)ceil_div((Ho - (p.bands - 1) * rows) * Wo, 32));
  p.items = p.bands * N;
  // As few waves as do it: one for every four items of the pack and one for every unit or part of one.  A wave costs its CU the
  // instructions ahead of its loads, and a SIMD issues one scalar instruction in four clocks: of sixteen waves the last has
  // its loads out 3000 clocks after the first has (6 x 64 x 11 x 11 -> 398 1x1 in four waves 0.69 of the time in sixteen; 7 x 130 x 29
  // x 27 -> 70 3x3/2 in eight 0.94).
  const int items_max = (int)(ceil_div((int64_t)std::min((rows - 1) * stride + KH, H) * W, 64) * p.quarters);
  p.waves = std::min(kWaves, (std::max((items_max + 3) / 4, units_max * parts) + 3) / 4 * 4);
  const dim3 grid((unsigned)ceil_div(p.items, 8) * 8, (unsigned)ceil_div(tiles, share));
  const int image = (((rows - 1) * stride + KH) * Wpp * Cw * 8 + 15) & ~15;
  p.sums_at = image;
  const size_t lds = (size_t)image + (parts > 1 ? (size_t)parts * units_max * kPartBytes : kRowBytes);
  note_kernel("conv_one_kernel grid %u x %u x %d, %d rows, %d filter tiles, %d parts of K", grid.x, grid.y, 64 * p.waves, rows, share, parts);
  auto pick = [&](auto i32) {
    constexpr bool I = decltype(i32)::value;
    return parts == 1 ? conv_one_kernel<I, 1> : parts == 2 ? conv_one_kernel<I, 2> : parts == 4 ? conv_one_kernel<I, 4> : conv_one_kernel<I, 8>;
  };
  auto kernel = out_i32 ? pick(std::true_type{}) : pick(std::false_type{});
  launch_kernel(kernel, grid, dim3(64 * p.waves), lds, s, p);
  *err = launch_error();
  return true;
}

}  // namespace bmx
