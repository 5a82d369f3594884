// Binary fully connected layer in one launch, for problems of a few microseconds of work or less.
// Paper: Sec. 2 (QFullyConnected: binarise the input, xnor GEMM against the packed weights,
// optional scale), Sec. 2.2.1 / 2.2.2 (Eq. 2): out[m][n] = K - 2 * popcount(x_bits[m] xor W[n]).
//
// The general path is two launches, pack then GEMM, each a launch on the host (2.7 us) and on the
// GPU a chain of trips to memory of about 4 us however little there is to do.  Here a workgroup
// takes RM batch rows and a run of output features: it requests its first weight words, turns its
// rows' fp32 values into sign bits in LDS (one coalesced load and one ballot per 64 values), and
// then counts xor + popcount over lanes: L lanes share a feature, lane l taking words l, l + L, ...
// of its row (whole runs of the weights per load, any alignment), the next words in flight while one
// set is counted, and the lanes' counts are added by DPP and half-wave swaps.
//
// Every workgroup packs its rows for itself, so a row of x is read once per run of features, and
// that is what decides where this form ends: the L1 path of a CU takes in 64 bytes per clock.  The
// launcher weighs the bytes a CU has to move against the second launch.
#include "bmx_internal.h"

#include <algorithm>

namespace bmx {

namespace {

// (up to sixteen waves, so that a row's runs are requested at once: 8 x 9216 -> 4096 6.0 us a call, with eight
// waves 7.2, with eight that request a run ahead 7.5)
constexpr int kWaves = 16;

struct FcSmallParams {
  const float* x;
  int64_t ldx;
  const uint64_t* W;
  int64_t ldw;
  const float* alpha;
  int M, N, K, Kw, Kpad;  // Kpad: words of an LDS row, a multiple of W * L
  int cols;               // output features per workgroup
  int waves;              // per workgroup
  int32_t* out_i32;
  float* out_f32;
  int64_t ldo;
};

template <int CTRL>
__device__ __forceinline__ int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}

// Sums over the wave, two values at a time: after the swap one register holds the two halves of a,
// the other those of b, so the sum is a's in the lower lanes and b's in the upper.
__device__ __forceinline__ int swap_add32(int a, int b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  return (int)r[0] + (int)r[1];
}
__device__ __forceinline__ int swap_add16(int a, int b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  return (int)r[0] + (int)r[1];
}

// L lanes per feature, U features per lane group and step, W words per lane and step.
template <int RM, int L, int U, int W>
__global__ void __launch_bounds__(64 * kWaves)
fc_small_kernel(const FcSmallParams p) {
  extern __shared__ uint64_t bits[];  // [RM][Kpad] sign bits
  asm volatile("" ::"s"(p.x), "s"(p.ldx), "s"(p.W), "s"(p.ldw), "s"(p.alpha), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.Kw),
               "s"(p.Kpad), "s"(p.cols), "s"(p.waves), "s"(p.out_i32), "s"(p.out_f32), "s"(p.ldo));
  constexpr int NV = RM * U;         // counts per lane group
  constexpr int kGroupsPerWave = 64 / L;
  constexpr int kPass = kGroupsPerWave * U;  // features per wave and pass
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.y * RM, n0 = blockIdx.x * p.cols;
  const int l = lane & (L - 1), grp = lane / L;
  const int nchunks = p.Kpad / (W * L);
  const int n_end = min(n0 + p.cols, p.N);
  // passes of this wave: features n0 + (wave + waves * i) * kPass ...
  int npass = 0;
  for (int n = n0 + wave * kPass; n < n_end; n += p.waves * kPass) ++npass;
  // which of the group's counts this lane stores: value v = m * U + u
  int v_mine;
  bool stores;
  if constexpr (L == 64) {
    const int q = lane >> 4, i = lane & 15;
    v_mine = 4 * i + 2 * (q & 1) + (q >> 1);
    stores = v_mine < NV;
  } else {
    v_mine = l;
    stores = l < NV;
  }
  const int u_mine = v_mine % U;

  uint64_t w[U][W], nxt[U][W];
  float al = 1.0f, al_nxt = 1.0f;
  auto request = [&](int it) {
    const int pass = it / nchunks, chunk = it - pass * nchunks;
    const int nb = n0 + (wave + p.waves * pass) * kPass + grp * U;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t* row = p.W + (int64_t)min(nb + u, p.N - 1) * p.ldw;
#pragma unroll
      for (int j = 0; j < W; ++j) nxt[u][j] = row[min((chunk * W + j) * L + l, p.Kw - 1)];
    }
    if (p.alpha) al_nxt = p.alpha[min(nb + u_mine, p.N - 1)];
  };
  const int total = npass * nchunks;
  if (total > 0) request(0);

  // ---- sign bits of the rows; values past K count as negative (bit 0, like the weights' tail).  A
  // row is read as a buffer of K floats: what lies beyond reads as zero (and is masked), so a run of
  // 16 words that ends past the row needs no addresses of its own.
  const int cpr = (p.Kpad + 15) >> 4;  // runs per row
  int m = 0, c = wave;
  while (c >= cpr) c -= cpr, ++m;
  while (m < RM) {
    const float* xr = p.x + (int64_t)min(m0 + m, p.M - 1) * p.ldx;
    const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc((void*)xr, 0, 4 * p.K, 0x00020000);
    const uint32_t off = (uint32_t)c * 4096u + 4u * (uint32_t)lane;
    uint32_t v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = __builtin_amdgcn_raw_buffer_load_b32(row, off + 256u * j, 0, 0);
    uint32_t lo = 0, hi = 0;  // lane j: word j of the run
#pragma unroll
    for (int j = 0; j < 16; j += 4) {
      uint64_t b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = __ballot(__uint_as_float(v[j + i]) >= 0.0f);
      // (the wait states between the compares that write b and their readers are part of the statement: the
      // compiler, which puts them between its own instructions, does not look into one)
      asm("s_nop 1\n\t"
          "v_writelane_b32 %0, %2, %10\n\tv_writelane_b32 %1, %3, %10\n\t"
          "v_writelane_b32 %0, %4, %10 + 1\n\tv_writelane_b32 %1, %5, %10 + 1\n\t"
          "v_writelane_b32 %0, %6, %10 + 2\n\tv_writelane_b32 %1, %7, %10 + 2\n\t"
          "v_writelane_b32 %0, %8, %10 + 3\n\tv_writelane_b32 %1, %9, %10 + 3"
          : "+v"(lo), "+v"(hi)
          : "s"((uint32_t)b[0]), "s"((uint32_t)(b[0] >> 32)), "s"((uint32_t)b[1]), "s"((uint32_t)(b[1] >> 32)),
            "s"((uint32_t)b[2]), "s"((uint32_t)(b[2] >> 32)), "s"((uint32_t)b[3]), "s"((uint32_t)(b[3] >> 32)), "i"(j));
    }
    // Values past K, a word on its lane: 100 x 2100 -> 1000 takes 4.76 us a call so; with a branch per word around a
    // scalar mask, and so the wait once per word, 5.07.
    const int real = min(max(p.K - c * 1024 - 64 * lane, 0), 64);
    const uint64_t word = ((uint64_t)hi << 32 | lo) & (real < 64 ? (1ull << real) - 1 : ~0ull);
    if (lane < 16 && 16 * c + lane < p.Kpad) bits[m * p.Kpad + 16 * c + lane] = word;
    c += p.waves;
    while (c >= cpr) c -= cpr, ++m;
  }
  __syncthreads();

  int pc[NV];
  int pass = 0, chunk = 0;
  for (int it = 0; it < total; ++it) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < W; ++j) w[u][j] = nxt[u][j];
    al = al_nxt;
    if (it + 1 < total) request(it + 1);
    if (chunk == 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) pc[i] = 0;
    }
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const int wi = (chunk * W + j) * L + l;
      if (wi >= p.Kw) {  // (the rows' bits are zero there too)
#pragma unroll
        for (int u = 0; u < U; ++u) w[u][j] = 0;
      }
#pragma unroll
      for (int m = 0; m < RM; ++m) {
        const uint64_t xb = bits[m * p.Kpad + wi];
#pragma unroll
        for (int u = 0; u < U; ++u) pc[m * U + u] += __popcll(xb ^ w[u][j]);
      }
    }
    if (++chunk < nchunks) continue;
    chunk = 0;
    // ---- the pass's features are counted: add the lanes up, one count per storing lane
    int mine = 0;
    if constexpr (L == 64) {
      constexpr int N4 = (NV + 3) / 4;
#pragma unroll
      for (int i = 0; i < N4; ++i) {
        int a[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] = 4 * i + k < NV ? pc[4 * i + k] : 0;
        int s = swap_add16(swap_add32(a[0], a[1]), swap_add32(a[2], a[3]));
        s = dpp_add<0x121>(dpp_add<0x122>(dpp_add<0x124>(dpp_add<0x128>(s))));  // row_ror 8, 4, 2, 1
        if ((lane & 15) == i) mine = s;
      }
    } else if constexpr (L == 16) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int s = dpp_add<0x121>(dpp_add<0x122>(dpp_add<0x124>(dpp_add<0x128>(pc[i]))));
        if (l == i) mine = s;
      }
    }
    const int nb = n0 + (wave + p.waves * pass) * kPass + grp * U;
    ++pass;
    auto store = [&](int v, int count) {
      const int m = m0 + v / U, n = nb + v % U;
      if (m >= p.M || n >= n_end) return;
      const int dot = p.K - 2 * count;
      if (p.out_i32) p.out_i32[(int64_t)m * p.ldo + n] = dot;
      else p.out_f32[(int64_t)m * p.ldo + n] = al * (float)dot;
    };
    if constexpr (L == 4) {  // U = 1: lane l of a group stores rows l, l + 4
      static_assert(L != 4 || U == 1, "");
#pragma unroll
      for (int i = 0; i < NV; i += 4) {
        int t = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (i + k >= NV) break;
          const int s = dpp_add<0x4e>(dpp_add<0xb1>(pc[i + k]));  // quad_perm [1,0,3,2], [2,3,0,1]
          if (l == k) t = s;
        }
        if (i + l < NV) store(i + l, t);
      }
    } else if (stores) {
      store(v_mine, mine);
    }
  }
}

// Lanes per feature and words per lane and step.  Few lanes, since what their sums cost is then shared by more words, as long as
// a row is at most three steps (four lanes, up to 48 words; sixteen, up to 192) and the features make work for eight waves
// (four waves: 599 x 2940 -> 64 3.84 -> 4.30 us; twelve: 153 x 4544 -> 108 3.9 -> 4.7); but not so many that a row does not fill
// them once.  Then the least padding.  In a graph, before (sixteen lanes from 17 words on, sixty-four from 65) and now: 100 x 2100 -> 1000 4.76
// and 4.14 us, 23 x 4206 -> 1920 6.3 and 5.0, 111 x 2176 -> 632 4.8 and 4.1.
struct Lanes {
  int L, W, padded;  // padded: words of a row, in whole steps
};
constexpr int features_per_pass(int L) { return L == 4 ? 16 : L == 16 ? 8 : 2; }
Lanes lanes_of(int L, int Kw) {
  // (in columns of L words and by constants only: six divisions were a percent of a small call)
  const unsigned cols = (unsigned)(Kw + L - 1) >> (L == 4 ? 2 : L == 16 ? 4 : 6);
  const unsigned four = (cols + 3) / 4 * 4, three = (cols + 2) / 3 * 3, two = (cols + 1) / 2 * 2;
  Lanes best = {L, 4, (int)four};
  if (three < four) best.W = 3, best.padded = (int)three;
  if ((int)two < best.padded) best.W = 2, best.padded = (int)two;
  best.padded *= L;
  return best;
}

inline int64_t shift_up(int64_t n, int log) { return (n + ((int64_t)1 << log) - 1) >> log; }

template <int RM>
void launch_rm(const FcSmallParams& p, Lanes l, dim3 grid, hipStream_t s) {
  const size_t lds = (size_t)RM * p.Kpad * 8;
  note_kernel("fc_small_kernel<%d,%d,%d> grid %u x %u x %d, %d features", RM, l.L, l.W, grid.x, grid.y, 64 * p.waves, p.cols);
  auto go = [&](auto kern) { launch_kernel(kern, grid, dim3(64 * p.waves), lds, s, p); };
  if (l.L == 64) {
    if (l.W == 2) go(fc_small_kernel<RM, 64, 2, 2>);
    else if (l.W == 3) go(fc_small_kernel<RM, 64, 2, 3>);
    else go(fc_small_kernel<RM, 64, 2, 4>);
  } else if (l.L == 16) {
    if (l.W == 2) go(fc_small_kernel<RM, 16, 2, 2>);
    else if (l.W == 3) go(fc_small_kernel<RM, 16, 2, 3>);
    else go(fc_small_kernel<RM, 16, 2, 4>);
  } else {
    if (l.W == 2) go(fc_small_kernel<RM, 4, 1, 2>);
    else if (l.W == 3) go(fc_small_kernel<RM, 4, 1, 3>);
    else go(fc_small_kernel<RM, 4, 1, 4>);
  }
}

}  // namespace

int fc_small = 0;  // 1 = never (measurements and tests of the general path on small layers)

// Takes the layer where what the busiest CU has to move in this form costs less than a second
// launch; false otherwise (nothing launched then).
bool launch_fc_small(const float* x, int64_t ldx, const uint64_t* Wp, int64_t ldw_w, const float* alpha, int batch,
                     int in_features, int out_features, int32_t* out_i32, float* out_f32, int64_t ldo, bool shared,
                     hipStream_t s, hipError_t* err) {
  // (a GEMM engine pinned through the tuning hook is what the caller wants to run)
  if (fc_small == 1 || gemm_engine != 0) return false;
  const int64_t Kw = words_for(in_features);
  if (Kw > 4096 || batch > 65535) return false;
  // (32-bit and few divisions: the calls that come here are bound by the host)
  const int few = Kw <= 48 ? 4 : Kw <= 192 ? 16 : 64, many = Kw <= 16 ? 4 : Kw <= 64 ? 16 : 64;  // lanes: fewest and most
  const Lanes least_lanes = lanes_of(few, (int)Kw), most_lanes = many == few ? least_lanes : lanes_of(many, (int)Kw);
  auto lanes_for = [&](int cols) -> const Lanes& { return cols < 8 * features_per_pass(few) ? most_lanes : least_lanes; };
  // Rows and features per workgroup: the pair that leaves the busiest CU the least to move (fp32 rows
  // and packed weights of its workgroups, and a fixed share per workgroup for its latencies).
  const bool long_and_many = Kw > 28 && (int64_t)batch * 12 > out_features;
  int64_t best = INT64_MAX;
  int rm_log = 0, cols_log = 4;
  for (int c = 4; c <= 9; ++c) {
    if (c > 4 && (1 << c) / 2 >= out_features) break;
    const int64_t Kpad = lanes_for(std::min(1 << c, out_features)).padded, groups = shift_up(out_features, c);
    for (int r = 0; r <= 3; ++r) {
      if (r > 0 && ((1 << r) / 2 >= batch || (Kpad * 8 << r) > 48 * 1024)) break;
      const int64_t wgs = shift_up(batch, r) * groups;
      const int64_t cost = shift_up(wgs, 8) * (((int64_t)in_features * 4 << r) + (Kw * 8 << c) + (4 * Kpad << (r + c)) + (16 << 10));
      // (Twice the rows and half the features is level where K is whole words.  Then four rows and not eight (0.96 of the time over 95
      // layers, 320 x 1536 -> 716 5.8 / 4.6 us); two and not four from 17 to 47 words (0.96); and fewer where rows are long and many, as each
      // of the fewer groups of features reads them again: from 29 words and a row for twelve features on 0.72 to 1.06 of the
      // time, mean 0.92, 343 x 7424 -> 95 5.5 us in pairs of rows, 7.6 in fours; else 0.95 to 1.14, mean 1.01.)
      const bool fewer = rm_log == 3 || (rm_log == 2 && Kw > 16 && Kw < 48) || long_and_many;
      if (cost < best || (cost == best && r < rm_log && fewer)) best = cost, rm_log = r, cols_log = c;
    }
  }
  // Level with two launches at about 320 KB (8 x 9216 -> 4096, 256 KB: 6.0 against 7.4 us; 767 x 3740 -> 124,
  // 261 KB: 6.0 / 7.8; 719 x 832 -> 739, 7.3 / 7.3 to 8.6; 287 x 1598 -> 1213, 371 KB: 8.4 / 7.5).  A few workgroups have the memory system
  // to themselves, and the general path's one or two tiles take a chain as long (2 x 65536 -> 16: 7.0
  // against 13.3 us).  Eight rows a workgroup, of 489 layers: 256 to 320 KB in more than a round of workgroups the two launches take 0.86 to
  // 0.96 of this form's time as calls, 0.77 to 0.88 in a graph; in one round 0.88 to 1.17 as calls, 0.84 to 0.97 in a graph, where the host's
  // part is not paid on replay: the line is at 256 KB for both.  Four rows in a graph likewise where four lanes share a feature (168 x 2432 ->
  // 1064 6.3 / 5.7), else level or this form ahead (568 x 7217 -> 64 7.2 / 9.1).
  const int rm = 1 << rm_log, cols = 1 << cols_log;
  const int64_t wgs = shift_up(batch, rm_log) * shift_up(out_features, cols_log);
  if (best > (wgs <= 32 ? 768 << 10 : 320 << 10)) return false;
  const Lanes lanes = lanes_for(std::min(cols, out_features));
  if (best > 256 << 10 && wgs > 32 && !shared && ((rm == 8 && wgs > 256) || ((rm == 8 || lanes.L == 4) && capturing(s)))) return false;
  const int64_t Kpad = lanes.padded;
  FcSmallParams p;
  p.x = x;
  p.ldx = ldx;
  p.W = Wp;
  p.ldw = ldw_w;
  p.alpha = alpha;
  p.M = batch;
  p.N = out_features;
  p.K = in_features;
  p.Kw = (int)Kw;
  p.Kpad = (int)Kpad;
  p.cols = cols;
  const int nitems = rm * ((lanes.padded + 15) / 16), pass = features_per_pass(lanes.L), npass = (std::min(cols, out_features) + pass - 1) / pass;
  // As many waves as runs of sixteen words to pack or passes over the features, whichever is more: a wave costs its CU the
  // instructions ahead of its loads (64 x 512 -> 256 2.61 -> 2.29 us in a graph, 112 x 73 -> 216 2.76 -> 2.38).
  p.waves = std::min(kWaves, (std::max(nitems, npass) + 3) / 4 * 4);
  p.out_i32 = out_i32;
  p.out_f32 = out_f32;
  p.ldo = ldo;
  const dim3 grid((unsigned)shift_up(out_features, cols_log), (unsigned)shift_up(batch, rm_log));
  if (rm == 1) launch_rm<1>(p, lanes, grid, s);
  else if (rm == 2) launch_rm<2>(p, lanes, grid, s);
  else if (rm == 4) launch_rm<4>(p, lanes, grid, s);
  else launch_rm<8>(p, lanes, grid, s);
  *err = launch_error();
  return true;
}

}  // namespace bmx
