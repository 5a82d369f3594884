// Binary convolution of a packed image for small problems: 32 filters x 32 output pixels per workgroup, K
// split over its 1 to 16 waves.
// Paper: Sec. 3.1 (M = filters, N = batch * output pixels, K = kh * kw * C), Sec. 2.2.2 (Eq. 2).
//
// gemm_small.hip with im2col columns, and for its reasons: at this size a launch is a chain of trips to
// memory and barriers, and of code that no cache holds.  A wave requests the filter words (16 bytes per
// lane, lane (r, h) of row r) and the pixel words (two 8-byte loads per lane: the words of a kernel row are
// consecutive in the image, from row to row there is a jump) of up to four steps of 256 bits before it
// uses the first; the waves' sums meet in LDS behind one barrier.  Any K: where the kernels for long K
// have no form that writes packed bits, this one does.
//
// Arithmetic as in gemm_small.hip: dot = K - 2 pc(filter) - 2 pc(patch) + 4 * sum of products.
//
// Measured, us per launch in a graph, against the other kernels: 3 x 192 x 22 x 21 -> 132 3x3/2 3.3 / 4.8, 3 x 64 x 37 x
// 36 -> 64 7x7 3.8 / 5.7, 20 x 258 x 9 x 11 -> 82 3x3 3.7 / 6.3 and as packed bits 4.1 / 11.3, 3 x 384 x 27 x 26 -> 64
// 7x7 6.7 / 9.0 and 7.2 / 14.2.

#include <type_traits>

#include "bmx_internal.h"
#include "halo.h"

namespace bmx {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(8)));

constexpr int kF32 = 0, kI32 = 1, kBits = 2;

struct SmallConvParams {
  const char* X;  // halo-padded packed image
  const char* W;  // packed filters, rows padded with zero words to a multiple of four
  uint32_t ldw;   // bytes
  int O, P, K, Kreal;  // filters, output pixels, words and bits of a patch
  int s_base, s_rem;   // steps of four words per wave: s_base, the first s_rem waves one more
  int run;             // words of a patch per kernel row
  uint32_t row_bytes;  // from kernel row to kernel row in the image
  int HoWo, Wo, Hp, Wpp, Cw, stride;
  FastDiv div_howo, div_wo, div_run;
  const float* alpha;  // per filter, or null
  const float* thr;    // packed bits: per filter threshold, or null (0)
  void* out;           // fp32 or int32 NCHW, or the next convolution's packed image in dwords
  int Nimg, Ho, oHp, oWp, oCw, opad;  // packed image: its size, words per pixel, halo
  int blocks, per_xcd;  // blocks of 32 pixels, and how many of them in a row every XCD takes (RUNS)
};

__device__ __forceinline__ v8i plane(const v4u& w, int n) {
  v8i e;
#pragma unroll
  for (int d = 0; d < 4; ++d) e[d] = (int)(n == 3 ? (w[d] >> 3) & 0x11111111u : w[d] & (0x11111111u << n));
#pragma unroll
  for (int d = 4; d < 8; ++d) e[d] = 0;
  return e;
}

// RUNS: a run of blocks of pixels per XCD, else in the grid's order.  (A kernel of its own: as a choice in one kernel the others, whose first
// addresses wait for it, lost 0.6 % in the mean.)
template <int OUT, int S, bool RUNS>
__global__ void __launch_bounds__(64 * S)
conv_small_kernel(const SmallConvParams p) {
  __shared__ float sums[S > 1 ? S : 1][17][64];  // a wave's sixteen sums per lane and its popcounts
  __shared__ uint32_t masks[S > 1 && OUT == kBits ? S : 1][32];
  asm volatile("" ::"s"(p.X), "s"(p.W), "s"(p.ldw), "s"(p.O), "s"(p.P), "s"(p.K), "s"(p.s_base), "s"(p.s_rem), "s"(p.run),
               "s"(p.row_bytes), "s"(p.HoWo), "s"(p.Wo), "s"(p.Hp), "s"(p.Wpp), "s"(p.Cw), "s"(p.stride), "s"(p.div_howo.mul),
               "s"(p.div_howo.sh1), "s"(p.div_howo.sh2), "s"(p.div_wo.mul), "s"(p.div_wo.sh1), "s"(p.div_wo.sh2));
  if (RUNS) asm volatile("" ::"s"(p.per_xcd));
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int wave = S > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const int block = RUNS ? (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  if (RUNS && block * 32 >= p.P) return;  // (the whole workgroup)
  const int m0 = blockIdx.y * 32, q = block * 32 + r;
  const int s0 = wave * p.s_base + min(wave, p.s_rem), s1 = s0 + p.s_base + (wave < p.s_rem ? 1 : 0);
  // (filters and pixels past the last repeat it; their results are not stored)
  const int qc = min(q, p.P - 1);
  const uint32_t img = fast_div((uint32_t)qc, p.div_howo), rem = (uint32_t)qc - img * (uint32_t)p.HoWo;
  const uint32_t ho = fast_div(rem, p.div_wo), wo = rem - ho * (uint32_t)p.Wo;
  const uint32_t patch = (((img * (uint32_t)p.Hp + ho * (uint32_t)p.stride) * (uint32_t)p.Wpp + wo * (uint32_t)p.stride) * (uint32_t)p.Cw) * 8u;
  const int mrow = min(m0 + r, p.O - 1);
  const uint32_t frow = (uint32_t)mrow * p.ldw + 16u * (uint32_t)h;

  // byte offset of the wave's next word in the patch and the words left of its kernel row (wave-uniform)
  const int kh0 = S > 1 ? (int)fast_div((uint32_t)(4 * s0), p.div_run) : 0;
  int left = (kh0 + 1) * p.run - 4 * s0;
  uint32_t off = (uint32_t)kh0 * p.row_bytes + (uint32_t)(p.run - left) * 8u;
  const uint32_t jump = p.row_bytes - (uint32_t)p.run * 8u;
  v4u a[4];
  uint64_t b[4][2];
  auto fetch = [&](int i, int s) {
    a[i] = *(const v4u_any*)(p.W + (frow + 32u * (uint32_t)s));
    uint32_t o[4];  // of words 4 s .. 4 s + 3; those past the patch repeat its last
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      o[j] = off;
      const bool more = 4 * s + j + 1 < p.K;
      left -= more ? 1 : 0;
      off += more ? 8u : 0u;
      if (left == 0) left = p.run, off += jump;
    }
    b[i][0] = *(const uint64_t*)(p.X + (patch + (h ? o[2] : o[0])));
    b[i][1] = *(const uint64_t*)(p.X + (patch + (h ? o[3] : o[1])));
  };
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (s0 + i < s1) fetch(i, s0 + i);
  const float al_l = (OUT != kI32 && p.alpha) ? p.alpha[mrow] : 1.0f;  // of filter r
  const float th_l = (OUT == kBits && p.thr) ? p.thr[mrow] : 0.0f;

  if (OUT == kBits && p.opad > 0 && (m0 & 63) == 0) {
    // word m0 / 64 of the output image's halo, spread over the workgroups of this filter tile
    write_halo((uint64_t*)p.out, p.Nimg, p.Ho, p.Wo, p.opad, p.O, p.oCw, m0 >> 6, block * (64 * S) + threadIdx.x,
               p.blocks * (64 * S));
  }

  v16f acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
  int pa = 0, pb = 0;
  for (int s = s0; s < s1; s += 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (s + i >= s1) break;  // wave-uniform
      const v4u x = a[i];
      v4u y = {(uint32_t)b[i][0], (uint32_t)(b[i][0] >> 32), (uint32_t)b[i][1], (uint32_t)(b[i][1] >> 32)};
      if (s + i + 4 < s1) fetch(i, s + i + 4);
      if (4 * (s + i) + 4 > p.K) {  // wave-uniform: words past the patch are zero
        const int k = 4 * (s + i) + 2 * h;
        if (k >= p.K) y[0] = y[1] = 0u;
        if (k + 1 >= p.K) y[2] = y[3] = 0u;
      }
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
  // filter r's count in lane (r, 0), pixel r's in lane (r, 1): a lane counted its half of K
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
  uint32_t mask = 0;
  const uint32_t at = (img * (uint32_t)p.O + (uint32_t)(m0 + 4 * h)) * (uint32_t)p.HoWo + rem;
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    const int v = S > 1 ? wave * kOwn + i : i;
    const int mu = 8 * (v >> 2) + (v & 3), mi = mu + 4 * h;  // register v: filter m0 + mi, pixel r
    const float dot = fmaf(4.0f, acc[i], base - 2.0f * __shfl(cnt, mi));  // exact: whole numbers below 2^24
    const float al = OUT == kI32 ? 1.0f : __shfl(al_l, mi);
    if (OUT == kBits) {
      if (al * dot >= __shfl(th_l, mi) && m0 + mi < p.O) mask |= 1u << mi;
    } else if (q < p.P && m0 + mi < p.O) {
      const uint32_t to = at + (uint32_t)mu * (uint32_t)p.HoWo;
      if (OUT == kI32) ((int32_t*)p.out)[to] = (int)dot;
      else ((float*)p.out)[to] = al * dot;
    }
  }
  if (OUT != kBits) return;
  mask |= (uint32_t)__shfl_xor((int)mask, 32);
  if (S > 1) {
    if (h == 0) masks[wave][r] = mask;
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 1; w < S; ++w) mask |= masks[w][r];
  }
  if (h == 0 && q < p.P) {
    const uint32_t word = ((img * (uint32_t)p.oHp + ho + (uint32_t)p.opad) * (uint32_t)p.oWp + wo + (uint32_t)p.opad) * (uint32_t)p.oCw + (uint32_t)(m0 >> 6);
    uint32_t* const dst = (uint32_t*)p.out + 2 * (size_t)word + ((m0 >> 5) & 1);
    dst[0] = mask;
    if ((m0 & 32) == 0 && m0 + 32 >= p.O) dst[1] = 0;  // nobody else owns the upper half
  }
}

template <int OUT>
void launch_kind(const SmallConvParams& p, int S, dim3 grid, hipStream_t s) {
  auto of = [&](auto runs) {
    constexpr bool R = decltype(runs)::value;
    return S == 1 ? conv_small_kernel<OUT, 1, R> : S == 2 ? conv_small_kernel<OUT, 2, R> : S == 4 ? conv_small_kernel<OUT, 4, R>
         : S == 8 ? conv_small_kernel<OUT, 8, R> : conv_small_kernel<OUT, 16, R>;
  };
  auto kern = p.per_xcd ? of(std::true_type{}) : of(std::false_type{});
  launch_kernel(kern, grid, dim3(64 * S), 0, s, p);
}

}  // namespace

int conv_small = 0;  // 1 = never (measurements and tests of the other kernels)

bool launch_conv_small(const uint64_t* Xp, int Nimg, int C, int H, int W, const uint64_t* Wp, int O, int KH, int KW, int stride,
                       int pad, const float* alpha, int32_t* out_i32, float* out_f32, uint64_t* out_bits, const float* thr,
                       int out_pad, hipStream_t s, hipError_t* err) {
  if (conv_small == 1 || conv_path || gemm_engine || conv_filters_per_wave || conv_ws_x4) return false;
  const int Ho = (H + 2 * pad - KH) / stride + 1, Wo = (W + 2 * pad - KW) / stride + 1;
  const int Cw = (int)words_for(C), K = KH * KW * Cw, Hp = H + 2 * pad, Wpp = W + 2 * pad;
  const int64_t P = (int64_t)Nimg * Ho * Wo, row_words = conv_weight_row_words(K);
  const int64_t lim = (int64_t)1 << 32;
  if ((int64_t)Nimg * Hp * Wpp * Cw * 8 >= lim || O * row_words * 8 >= lim || ((int64_t)Nimg * O + 32) * Ho * Wo >= lim / 4) return false;
  const int64_t oq = (int64_t)(Ho + 2 * out_pad) * (Wo + 2 * out_pad), oCw = words_for(O);
  if (out_bits && Nimg * oq * oCw >= lim / 2) return false;
  if ((int64_t)C * KH * KW >= (1 << 24) || O > 65535 * 32) return false;
  const int64_t tiles_p = ceil_div(P, 32), tiles_o = ceil_div(O, 32), tiles = tiles_p * tiles_o;
  const int steps = (K + 3) / 4;
  const int64_t work = tiles * steps, tiles64 = ceil_div(P, 64) * ceil_div(O, 64);
  // Against the kernels with an eye to K (us in a graph): the short-K kernel shares its filters, which pays
  // from a few hundred tiles on, and at 9 words from the first (18 words: 400 tiles 3.9 against 4.3, 700
  // tiles 4.3 / 4.0; 27 words: 95 tiles 3.3 / 4.8; 49 words: 530 tiles 5.3 / 6.0, 1170 tiles 8.4 / 8.0); the
  // stationary kernel has nothing to share at 1 to 4 words.  A long K is gemm_fp4_kernel's from
  // 12288 tile steps on (its time over this kernel's: at 8000 to 12000 steps 1.0 to 1.2, at 12540 to 16000 0.81 to 1.07, mean 0.93),
  // where it has 64 tiles of its own that are not half empty (at most three of these in one of those: at 12288 to 16384 steps 0.9 to
  // 1.7, mean 1.15; 9 x 545 x 48 x 48 -> 30, 3 x 3, 8.7 / 6.9) and it takes the filters, 16-byte aligned; from 16384 on in any case.
  // As packed bits the line is where 3.4 us and 0.25 ns a tile
  // step, this kernel's time, meet the estimate of the kernels for long K (211 filters, 3780 pixels, 196 words: 13.4 / 9.5; 32, 22707, 100,
  // half of their tiles empty: 7.5 / 10.9; 64, 20064, 63: 7.8 / 9.7), 12000 steps at least; and gemm_block.hip's for few words.
  if (conv_weight_short_k(K)) {
    if (steps < 5 || tiles > (steps == 5 ? 400 : 700)) return false;
  } else if (out_bits) {
    int form;
    if (work > 72000) return false;
    if (((uintptr_t)Wp & 15) == 0 && !conv_block && !gemm_fp4_split && !gemm_fp4_half && !gemm_fp4_band) {
      if (K < 8 ? tiles >= 7000 : work > 12000 && 3.4 + 2.5e-4 * work > conv_long_us(P, O, K, (KW * Cw) & 1, &form)) return false;
    }
  } else if (K == 1 || K == 2 || K == 4 || work > (tiles64 >= 64 && tiles > 3 * tiles64 && ((uintptr_t)Wp & 15) == 0 ? 12288 : 16384) || tiles > 4096) {
    return false;
  }
  int S = 1;
  while (S < 16 && 2 * S <= steps && 2 * S * tiles <= (work > 12288 ? 8192 : 4096)) S *= 2;
  SmallConvParams p;
  p.X = (const char*)Xp;
  p.W = (const char*)Wp;
  p.ldw = (uint32_t)(row_words * 8);
  p.O = O;
  p.P = (int)P;
  p.K = K;
  p.Kreal = C * KH * KW;
  p.s_base = steps / S;
  p.s_rem = steps % S;
  p.run = KW * Cw;
  p.row_bytes = (uint32_t)Wpp * (uint32_t)Cw * 8u;
  p.HoWo = Ho * Wo;
  p.Wo = Wo;
  p.Hp = Hp;
  p.Wpp = Wpp;
  p.Cw = Cw;
  p.stride = stride;
  p.div_howo = make_fast_div((uint32_t)(Ho * Wo));
  p.div_wo = make_fast_div((uint32_t)Wo);
  p.div_run = make_fast_div((uint32_t)p.run);
  p.alpha = alpha;
  p.thr = thr;
  p.out = out_bits ? (void*)out_bits : out_i32 ? (void*)out_i32 : (void*)out_f32;
  p.Nimg = Nimg;
  p.Ho = Ho;
  p.opad = out_pad;
  p.oHp = Ho + 2 * out_pad;
  p.oWp = Wo + 2 * out_pad;
  p.oCw = (int)oCw;
  p.blocks = (int)tiles_p;
  // Workgroup b sits on XCD b % 8: with a run of pixels and all filters to itself an XCD fetches few rows of the image, and one that
  // several blocks' patches share once (us in a graph, in the grid's order / so: 47 x 243 x 26 x 28 -> 64, 3 x 3 / 2, 4.65 / 4.46, 100 x 320 x
  // 14 x 14 -> 64, 1 x 1, 4.75 / 4.38; 211 drawn ones of 32 blocks of pixels and more 1.014 in the mean).
  // Not of few blocks, which leave XCDs without any (170 drawn ones of up to 80 0.999, some of two to twenty 0.98: 3 x 238 x 10 x 10 -> 64, 7 x 7,
  // 7.66 / 7.86); and not where the runs do not come out even and a CU would have a workgroup more (51 x 53 pixels, 3 tiles of filters, 7 x 7,
  // 7.1 / 9.2).
  p.per_xcd = (int)ceil_div(tiles_p, 8);
  if (tiles_p < 48 || ceil_div(p.per_xcd * tiles_o, 32) > ceil_div(tiles, 256)) p.per_xcd = 0;
  const dim3 grid((unsigned)(p.per_xcd ? 8 * p.per_xcd : tiles_p), (unsigned)tiles_o);
  note_kernel("conv_small_kernel<%s> grid %u x %u x %d", out_bits ? "bits" : out_i32 ? "i32" : "f32", grid.x, grid.y, 64 * S);
  if (out_bits) launch_kind<kBits>(p, S, grid, s);
  else if (out_i32) launch_kind<kI32>(p, S, grid, s);
  else launch_kind<kF32>(p, S, grid, s);
  *err = launch_error();
  return true;
}

}  // namespace bmx
