// Binary convolution of an fp32 image in one launch.
// Paper: Sec. 2 (QConvolution: binarise the input, xnor GEMM, optional scale), Sec. 3.1 (M = filters,
// N = batch * output pixels, K = kh * kw * C).
//
// The general path is two launches, channel pack then convolution, each a launch on the host (2.7 us)
// and on the GPU a chain of trips to memory of 4 to 5 us however little there is to do.  Here a
// workgroup of 16 waves takes a band of output rows of one image and a share of the filters:
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
// Measured, one launch against two (us per call): 1 x 64 x 8 x 8 -> 64 1x1 4.8 / 7.9, 1 x 60 x 20 x 19 -> 64
// 3x3 5.1 / 8.6, 38 x 49 x 25 x 25 -> 64 1x1/2 5.2 / 8.5, 22 x 64 x 13 x 13 -> 167 3x3 6.9 / 8.7, 7 x 130 x 29 x
// 27 -> 70 3x3/2 7.1 / 8.1; 16 x 64 x 56 x 56 -> 64 3x3 would take 12.1 / 9.4 and stays with two.
#include <algorithm>
#include <type_traits>

#include "bmx_internal.h"
#include "conv_expand.h"

namespace bmx {

namespace {

constexpr int kWaves = 16;
constexpr int kLds = 64 * 1024;               // dynamic LDS without asking for more
constexpr int kPartBytes = 64 * (16 + 1) * 4;  // a wave's sums and counts

typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef uint16_t __attribute__((may_alias)) u16_alias;
typedef uint32_t __attribute__((may_alias)) u32_alias;

struct ConvOneParams {
  const float* x;
  const uint64_t* Wp;
  const float* alpha;
  int32_t* out_i32;
  float* out_f32;
  int C, H, W, O;
  int Ho, Wo;
  int K, Cw, KH, run;  // words of a patch; channel words; kernel rows; words per kernel row
  int stride, pad, rows, bands;  // output rows per band, bands per image
  int tiles;     // filter tiles of 32 per workgroup
  int ld_words;  // words per packed filter row
  int Kreal;
  int sums_at;  // byte offset in LDS of the sums of units split over K
  FastDiv div_w, div_wp, div_wo, div_cw, div_bands;
  int items;  // bands of all images
};

template <bool I32, int PARTS>
__global__ void __launch_bounds__(64 * kWaves)
conv_one_kernel(const ConvOneParams p) {
  extern __shared__ uint64_t img[];  // [band input rows][W + 2 pad][Cw]
  // (all arguments named at the top: fetched in one batch, one trip to memory instead of one per group)
  asm volatile("" ::"s"(p.x), "s"(p.Wp), "s"(p.C), "s"(p.H), "s"(p.W), "s"(p.O), "s"(p.Ho), "s"(p.Wo), "s"(p.K), "s"(p.Cw), "s"(p.KH),
               "s"(p.stride), "s"(p.pad), "s"(p.rows), "s"(p.bands), "s"(p.tiles), "s"(p.ld_words), "s"(p.div_cw.mul),
               "s"(p.div_cw.sh1), "s"(p.div_cw.sh2), "s"(p.div_bands.mul), "s"(p.div_bands.sh1), "s"(p.div_bands.sh2), "s"(p.items));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;
  // Workgroup b sits on XCD b % 8: every XCD gets a contiguous run of bands, which share input rows (and this
  // batch of arguments: 12 x 390 x 24 x 26 -> 83 1x1 8.5 -> 7.3 us a call, 33 x 257 x 18 x 18 -> 240 1x1 10.7 -> 9.4)
  const int lin = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (lin >= p.items) return;  // (the whole workgroup)
  const int n = (int)__builtin_amdgcn_readfirstlane(fast_div((uint32_t)lin, p.div_bands)), band = lin - n * p.bands;
  const int group = blockIdx.y;
  const int Wpp = p.W + 2 * p.pad, HW = p.H * p.W;
  const int ho0 = band * p.rows, nrows = min(p.rows, p.Ho - ho0);
  const int top = ho0 * p.stride - p.pad;             // input row of the band's first padded row
  const int rin = (nrows - 1) * p.stride + p.KH;      // padded rows of the band
  const int row0 = max(top, 0), row1 = min(top + rin, p.H);
  const int skip_top = row0 - top;
  const int npx = max(row1 - row0, 0) * p.W;          // real pixels of the band, contiguous in a plane

  // ---- this wave's units of 32 pixels x 32 filters; the first one's filter words are requested ahead of all
  const int px_blocks = (nrows * p.Wo + 31) >> 5;
  const int tile0 = group * p.tiles, ntiles = min(p.tiles, (p.O + 31) / 32 - tile0);
  const int units = px_blocks * ntiles;
  // PARTS waves share the K range of a unit (if more than one: units * PARTS <= kWaves in every workgroup)
  constexpr bool SPLIT = PARTS > 1;
  const int part = SPLIT ? wave / units : 0, unit0 = SPLIT ? wave - part * units : wave;
  const int steps = (p.K + 3) >> 2;  // of four words (the packed rows are padded with zero words)
  v4u fw[4];
  auto filter_row = [&](int u) {
    const int tile = tile0 + u / px_blocks;
    return (const char*)(p.Wp + (int64_t)min(tile * 32 + r, p.O - 1) * p.ld_words) + 16 * h;
  };
  const int first = SPLIT ? min(part, PARTS - 1) * steps / PARTS : 0;  // this wave's steps of every unit
  const int last = SPLIT ? (min(part, PARTS - 1) + 1) * steps / PARTS : steps;
  const char* frow = filter_row(min(unit0, units - 1));
#pragma unroll
  for (int i = 0; i < 4; ++i) fw[i] = *(const v4u*)(frow + 32 * min(first + i, last - 1));

  // ---- pack: item = (64 pixels, channel word, 16 of its channels)
  const int items = ((npx + 63) >> 6) * p.Cw * 4;
  struct Item {
    float v[16];
    int px, word, quarter, real;
  };
  auto load = [&](Item& it, int t) {
    t = min(t, items - 1);
    it.quarter = t & 3;
    const int rest = t >> 2, g = __builtin_amdgcn_readfirstlane((int)fast_div((uint32_t)rest, p.div_cw));
    it.word = rest - g * p.Cw;
    it.px = g * 64 + lane;
    const int c0 = it.word * 64 + it.quarter * 16;
    it.real = min(16, p.C - c0);  // (may be negative: a quarter without channels)
    const float* base = p.x + ((int64_t)n * p.C + min(c0, p.C - 1)) * HW + row0 * p.W;
    const uint32_t off = 4u * (uint32_t)min(it.px, npx - 1);
    const int64_t plane = (int64_t)HW * 4;
#pragma unroll
    for (int j = 0; j < 16; ++j)  // (channels past the last repeat it and are masked)
      it.v[j] = *(const float*)((const char*)base + plane * min(j, max(it.real - 1, 0)) + off);
  };
  auto pack = [&](const Item& it) {
    uint32_t b = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) b |= (it.v[j] >= 0.0f ? 1u : 0u) << j;
    b &= it.real >= 16 ? 0xffffu : (it.real <= 0 ? 0u : (1u << it.real) - 1u);
    if (it.px < npx) {
      const int hi = (int)fast_div((uint32_t)it.px, p.div_w), wi = it.px - hi * p.W;
      const int at = ((hi + skip_top) * Wpp + wi + p.pad) * p.Cw + it.word;
      ((u16_alias*)img)[4 * at + it.quarter] = (uint16_t)b;
    }
  };
  if (npx > 0) {
    Item a, b;
    load(a, wave);
    for (int t = wave; t < items; t += 2 * kWaves) {
      load(b, t + kWaves);
      pack(a);
      if (t + kWaves >= items) break;
      load(a, t + 2 * kWaves);
      pack(b);
    }
  }
  // halo: the sign of the zero padding, +1 for every real channel
  if (p.pad > 0) {
    for (int i = threadIdx.x; i < rin * Wpp; i += 64 * kWaves) {
      const int hi = (int)fast_div((uint32_t)i, p.div_wp), wi = i - hi * Wpp;
      if (hi < skip_top || hi >= skip_top + (row1 - row0) || wi < p.pad || wi >= p.pad + p.W)
        for (int cw = 0; cw < p.Cw; ++cw)
          img[i * p.Cw + cw] = (cw == p.Cw - 1 && (p.C & 63)) ? ((uint64_t)1 << (p.C & 63)) - 1 : ~(uint64_t)0;
    }
  }
  __syncthreads();

  // ---- multiply
  const int skip = (Wpp * p.Cw - p.run) * 8;  // bytes from the end of a kernel row's run to the next
  const int kh0 = SPLIT ? (4 * first) / p.run : 0;
  const int off0 = SPLIT ? kh0 * Wpp * p.Cw * 8 + (4 * first - kh0 * p.run) * 8 : 0;
  const int left0 = SPLIT ? (kh0 + 1) * p.run - 4 * first : p.run;
  constexpr int kOwn = 16 / PARTS;
  v16f acc;  // (one chain: the SIMD's other three waves fill the matrix pipe)
  float c0;
  auto multiply = [&](int u) {
    const int pb = u - u / px_blocks * px_blocks;
    const int qc = min(pb * 32 + r, nrows * p.Wo - 1);
    const int ho = (int)fast_div((uint32_t)qc, p.div_wo), wo = qc - ho * p.Wo;
    const char* patch = (const char*)img + (((ho * p.stride) * Wpp + wo * p.stride) * p.Cw) * 8 + 4 * h;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    int pc = 0;
    int off = off0, left = left0;  // byte offset of the next word in the patch, words left in its run (wave-uniform)
    uint32_t xw[4];
    auto read = [&](int k) {  // dword h of words k .. k + 3 of the patch; words past K repeat its last
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        xw[j] = *(const u32_alias*)(patch + off);
        const bool more = k + j + 1 < p.K;
        left -= more ? 1 : 0;
        const bool wrap = left == 0;
        off += more ? (wrap ? 8 + skip : 8) : 0;
        left = wrap ? p.run : left;
      }
    };
    read(4 * first);
    for (int i0 = first; i0 < last; i0 += 4) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i0 + i >= last) break;  // wave-uniform
        // lane (r, 0) holds words 4 i, 4 i + 1 of filter r, lane (r, 1) words 4 i + 2, 4 i + 3
        const v2u t = __builtin_amdgcn_permlane32_swap(fw[i][0], fw[i][1], false, false);
        const v2u s = __builtin_amdgcn_permlane32_swap(fw[i][2], fw[i][3], false, false);
        const uint32_t f[4] = {t[0], s[0], t[1], s[1]};
        fw[i] = *(const v4u*)(frow + 32 * min(i0 + i + 4, last - 1));
        uint32_t x[4] = {xw[0], xw[1], xw[2], xw[3]};
        if (4 * (i0 + i) + 4 > p.K) {  // wave-uniform: the last step; words past K are zero pixels
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = 4 * (i0 + i) + j < p.K ? x[j] : 0u;
        }
        if (i0 + i + 1 < last) read(4 * (i0 + i + 1));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          pc += __builtin_popcount(f[j]);
          acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(expand_filter(f[j])), widen(expand_pixel(x[j])), acc, 4, 4,
                                                               0, 127, 0, 127);
        }
        __builtin_amdgcn_sched_barrier(0);  // (operands of later steps made early would spill: 128 registers)
      }
    }
    pc += __shfl_xor(pc, 32);
    c0 = (float)((part == 0 ? p.Kreal : 0) - 2 * pc);  // of filter r of the tile
  };
  auto store = [&](int u) {
    const int ft = u / px_blocks, pb = u - ft * px_blocks;
    const int m0 = (tile0 + ft) * 32;
    const int q = pb * 32 + r;
    const float al = p.alpha ? p.alpha[min(m0 + r, p.O - 1)] : 1.0f;
    const bool valid = q < nrows * p.Wo;
    // register v of a wave's sixteen: filter m0 + 8 (v / 4) + 4 h + v % 4, pixel r of the block
    const uint32_t pitch = (uint32_t)(p.Ho * p.Wo) * 4u;
    const uint32_t at = (uint32_t)(n * p.O + m0 + 4 * h) * pitch + (uint32_t)(ho0 * p.Wo + q) * 4u;
    char* const out = I32 ? (char*)p.out_i32 : (char*)p.out_f32;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      const int v = SPLIT ? part * kOwn + i : i, mi = 8 * (v / 4) + (v % 4);
      const float t = fmaf(2.0f, acc[i], __shfl(c0, mi + 4 * h));
      const float a = I32 ? 1.0f : __shfl(al, mi + 4 * h);
      if (!valid || m0 + mi + 4 * h >= p.O) continue;
      if (I32) *(int32_t*)(out + (size_t)(at + (uint32_t)mi * pitch)) = (int)t;
      else *(float*)(out + (size_t)(at + (uint32_t)mi * pitch)) = a * t;
    }
  };
  if (!SPLIT) {
    for (int u = wave; u < units; u += kWaves) {
      if (u != wave) {
        frow = filter_row(u);
#pragma unroll
        for (int i = 0; i < 4; ++i) fw[i] = *(const v4u*)(frow + 32 * min(i, steps - 1));
      }
      multiply(u);
      store(u);
    }
    return;
  }
  // SPLIT: the parts of a unit meet in LDS behind the image, [unit][part][16 sums and the count][lane],
  // and each finishes its share of the sixteen
  const bool busy = part < PARTS;
  float* const sums = (float*)((char*)img + p.sums_at) + unit0 * (PARTS * kPartBytes / 4) + lane;
  if (busy) {
    multiply(unit0);
    float* const mine = sums + part * (kPartBytes / 4);
#pragma unroll
    for (int v = 0; v < 16; ++v) mine[v * 64] = acc[v];
    mine[16 * 64] = c0;
  }
  __syncthreads();
  if (!busy) return;
  c0 = 0.0f;
#pragma unroll
  for (int e = 0; e < PARTS; ++e) c0 += sums[(e * 17 + 16) * 64];
#pragma unroll
  for (int v = 0; v < kOwn; ++v) {
    acc[v] = 0.0f;
#pragma unroll
    for (int e = 0; e < PARTS; ++e) acc[v] += sums[(e * 17 + part * kOwn + v) * 64];
  }
  store(unit0);
}

}  // namespace

int conv_one = 0;  // 1 = never (measurements and tests of the two-launch path)

bool launch_conv_one(const float* x, int N, int C, int H, int W, const uint64_t* Wp, int O, int KH, int KW, int stride,
                     int pad, const float* alpha, int32_t* out_i32, float* out_f32, hipStream_t s, hipError_t* err) {
  if (conv_one == 1 || conv_path != 0 || gemm_engine != 0 || ((uintptr_t)Wp & 15)) return false;
  const int Ho = (H + 2 * pad - KH) / stride + 1, Wo = (W + 2 * pad - KW) / stride + 1;
  const int Cw = (int)words_for(C), K = KH * KW * Cw, Wpp = W + 2 * pad;
  if (N > 65535 || O > 65535 * 32 || (int64_t)H * W * 4 >= ((int64_t)1 << 31) || (int64_t)C * KH * KW >= ((int64_t)1 << 24)) return false;
  if (((int64_t)N * O + 32) * Ho * Wo * 4 >= ((int64_t)1 << 32)) return false;  // 32-bit output offsets
  const int tiles = (int)ceil_div(O, 32);
  // The two launches' time in us, fitted to 850 shapes (9 % rms; 7.1 to 8.4 of it is the host's part): MB of input and of results, 1e9
  // products, the chain of a patch's words.  This form is taken where its own estimate is 5 % below.
  const double in_kb_all = (double)N * C * H * W / 256, out_kb_all = (double)N * O * Ho * Wo / 256;
  const double unit_words = (double)N * Ho * Wo * tiles * K;
  const double limit = 0.95 * (7.6 + in_kb_all * (0.16 / 977) + out_kb_all * (0.1 / 977) + unit_words * (32 * 64 * 0.4e-9) + K * 0.012);
  // Output rows per band, filter tiles per workgroup and waves per unit: those of the shortest modelled
  // time, fitted to the same shapes (6.5 % rms).  A round of workgroups pays its trips to memory, its fp32
  // rows (KB), its words per SIMD (one unit in four waves: 1) and its results (KB).
  auto cost_of = [](double rounds, double in_kb, double words, double out_kb) {
    return 2.3 + rounds * 2.4 + in_kb * (1 / 37.0) + words * (1 / 15.0) + out_kb * (1 / 21.0);
  };
  // (no plan is below an even share of everything: most layers that stay with two launches end here)
  if (cost_of(1, in_kb_all * std::min(1.0, (double)KH / stride) / 256, unit_words / (32 * 4 * 256), out_kb_all / 256) > limit) return false;
  double best = 1e30;
  int rows = 0, share = 0, parts = 1, units_max = 0;
  const int steps = (K + 3) / 4;
  for (int rr = 1; rr <= Ho; rr = rr < 4 ? rr + 1 : rr + (rr + 1) / 2) {
    const int rin = (rr - 1) * stride + KH;
    if ((int64_t)rin * Wpp * Cw * 8 > kLds) break;
    const int image = (rin * Wpp * Cw * 8 + 15) & ~15;
    const int bands = (Ho + rr - 1) / rr, px_blocks = (rr * Wo + 31) / 32;  // (32-bit: this runs on every call)
    const double in_kb = (double)std::min(rin, H) * W * C / 256;
    double rounds = 0;
    for (int g = 1; g <= tiles; g *= 2) {
      const int per = (tiles + g - 1) / g, units = px_blocks * per;
      // K is split over idle waves: down to a step of four words each while that leaves every SIMD two
      // waves at most, to two steps each beyond (parts of one step lose more in the sums than they gain)
      int ks = 1;
      while (ks < 8 && ks * 2 * units <= kWaves && ks * 2 <= (ks * 2 * units <= kWaves / 2 ? steps : steps / 2) &&
             image + ks * 2 * units * kPartBytes <= kLds) ks *= 2;
      const double words = ks > 1 ? std::max(1.0, units * ks / 4.0) * ((K + ks - 1) / ks) : (double)((units + 3) / 4) * K;
      rounds = (double)(((int64_t)bands * ((tiles + per - 1) / per) * N + 255) >> 8);
      const double cost = cost_of(rounds, rounds * in_kb, rounds * words, rounds * rr * Wo * std::min(O, 32 * per) / 256);
      if (cost < best) best = cost, rows = rr, share = per, parts = ks, units_max = units;
    }
    if (rounds == 1) break;  // one round however the filters are shared: longer bands cost more
  }
  if (rows == 0 || best > limit) return false;
  ConvOneParams p;
  p.x = x;
  p.Wp = Wp;
  p.alpha = alpha;
  p.out_i32 = out_i32;
  p.out_f32 = out_f32;
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
  p.ld_words = (int)conv_weight_row_words(K);
  p.Kreal = C * KH * KW;
  p.div_w = make_fast_div((uint32_t)W);
  p.div_wp = make_fast_div((uint32_t)Wpp);
  p.div_wo = make_fast_div((uint32_t)Wo);
  p.div_cw = make_fast_div((uint32_t)Cw);
  p.div_bands = make_fast_div((uint32_t)p.bands);
  p.items = p.bands * N;
  const dim3 grid((unsigned)ceil_div(p.items, 8) * 8, (unsigned)ceil_div(tiles, share));
  const int image = (((rows - 1) * stride + KH) * Wpp * Cw * 8 + 15) & ~15;
  p.sums_at = image;
  const size_t lds = (size_t)image + (parts > 1 ? (size_t)parts * units_max * kPartBytes : 0);
  note_kernel("conv_one_kernel grid %u x %u x %d, %d rows, %d filter tiles, %d parts of K", grid.x, grid.y, 64 * kWaves, rows, share, parts);
  auto pick = [&](auto i32) {
    constexpr bool I = decltype(i32)::value;
    return parts == 1 ? conv_one_kernel<I, 1> : parts == 2 ? conv_one_kernel<I, 2> : parts == 4 ? conv_one_kernel<I, 4> : conv_one_kernel<I, 8>;
  };
  auto kernel = out_i32 ? pick(std::true_type{}) : pick(std::false_type{});
  launch_kernel(kernel, grid, dim3(64 * kWaves), lds, s, p);
  *err = launch_error();
  return true;
}

}  // namespace bmx
