// Bound-pruned library argmax (gfx950): the best template of every pattern under the FP32 FFT search (or
// the windowed forms of k_xcf_even.hip), without the full correlation of the pairs that cannot win.
//
// For band-limited spectra the correlation splits into rho = low + high, low the part of the
// coefficients with |u|, |v| <= 15:
//   |high(s)| <= sum_high |E||T| <= sqrt(eh_E eh_T)      (Cauchy-Schwarz; eh = energy of the high part),
//   low(s)    <= max of low over the corners of s's cell of a 32 x 32 shift grid, h = N / 32 px apart,
//                + h^2 / 8 (|low_xx| + |low_yy|)          (a bilinear interpolant's error),
//   |low_xx| + |low_yy| <= (2 pi / N)^2 sum_low |E||T| (u^2 + v^2) <= sqrt(k_E k_T),
//                k = (2 pi / N)^2 sum_low |X|^2 (u^2 + v^2).
// So   score(p, l) <= coarse(p, l) + h^2 / 8 sqrt(k_p k_l) + sqrt(eh_p eh_l) + rounding,
// where coarse is the largest low value of the grid and the other terms are products of two numbers
// per spectrum.  With h0, the full-size score of the template with the largest coarse value, every
// template whose bound lies below h0 is out (99 % of a 4,000-template library for patterns that match it,
// SNR 5), and of the rest those whose bound from a grid of half the step does.  What remains gets its
// full score from the search kernel itself, so the pick is that of the whole score matrix, bit for bit,
// ties included.  What patterns that match less well keep depends on their size.  Whole calls of 200 patterns
// against 4,000 templates of 15 bands, every pair / matching / another crystal's / noise, in ms: 64 2.06 / 0.26 /
// 0.29 / 0.62, 96 5.48 / 0.25 / 0.32 / 2.38, 128 8.81 / 0.28 / 0.38 / 8.91, 160 18.9 / 0.30 / 0.54 / 19.8; windows
// of +-15 px, split: 128 2.50 / 0.29 / 0.56 / 2.66, 256 7.78 / 0.59 / 2.97 / 8.22.  Against fewer templates or
// patterns noise costs up to a quarter more than every pair (11 x 6,000 at 160, split, 465 -> 589 us; prune_pays).
#include "ebsd_common.hpp"
#include "ebsd_internal.hpp"

#include <math.h>

#include <algorithm>

namespace ebsd {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr int BL = 15, G = 32;       // low band, grid points per axis
constexpr int FRAG = 2 * 64;         // h8 values of one spectrum's low part
constexpr int PT = 32, TC = 16;      // patterns per block, most templates per wave of the coarse kernel
constexpr float kScale = 64.0f;      // of the FP16 low parts: products to 4096, sums to 11586, nothing subnormal that counts

// The coarse values are a filter, not a result, and their error is part of the bound: with u = 2^-11
// each product of the low parts carries 2 u of its operands' and 5 u of its own rounding, u of the
// first constant, u of the conversion between the stages and u of the second constant, all against
// |E||T| (|c1| + |s1|) (|c2| + |s2|) <= 2 |E||T|, and sum |E||T| <= 1: 20 u = 0.0098.  The FP32 sums and the
// exact score add a few ulp.  (On the bounds' own slack of 0.11 to 0.14 this keeps 1.1x the templates.)
constexpr float kRound = 0.0102f;

// The low part of each spectrum in the coarse kernel's order, FP16 times kScale: X(u), X(-u) of
// u = 4 (lane / 16) + j, v = lane % 16 (X(-0) = 0), j < 4, as re, im of u at [0][lane] and of -u at
// [1][lane]; and stat = (sqrt(eh), sqrt(k)); one block per spectrum
__global__ __launch_bounds__(256) void k_low_spectra(const cf* __restrict__ spec, int n, int bnd,
                                                     h8* __restrict__ low, float2* __restrict__ stat) {
  const int nv = bnd + 1, nk = 2 * bnd + 1, spec_n = nv * nk;
  const int64_t k = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const cf* S = spec + k * spec_n;
  if (tid < 128) {
    h8 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int u = 4 * (lane >> 4) + j, v = lane & 15;
      const cf x = tid < 64 ? S[u * nv + v] : (u ? S[(nk - u) * nv + v] : cf{0.f, 0.f});
      o[j] = (_Float16)(kScale * x.x);
      o[4 + j] = (_Float16)(kScale * x.y);
    }
    low[k * FRAG + tid] = o;
  }
  float eh = 0.0f, kl = 0.0f;
  for (int t = tid; t < spec_n; t += 256) {
    const int kk = t / nv, v = t - kk * nv;
    const int u = kk <= bnd ? kk : kk - nk;
    const cf z = S[t];
    const float e = (v == 0 ? 1.0f : 2.0f) * (z.x * z.x + z.y * z.y);
    if (abs(u) <= BL && v <= BL) kl += e * (float)(u * u + v * v);
    else eh += e;
  }
  eh = wave_sum(eh);
  kl = wave_sum(kl);
  __shared__ float red[2][4];
  if (lane == 0) {
    red[0][tid >> 6] = eh;
    red[1][tid >> 6] = kl;
  }
  __syncthreads();
  if (tid == 0) {
    const float tpn = 6.2831855f / (float)n;
    stat[k] = make_float2(sqrtf(red[0][0] + red[0][1] + red[0][2] + red[0][3]),
                          tpn * sqrtf(red[1][0] + red[1][1] + red[1][2] + red[1][3]));
  }
}

// The larger of a lane's and another lane's value (NaN is passed over)
template <int CTRL>
__device__ __forceinline__ float dpp_max(float v) {
  return fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true)));
}

// A = Z(u) + Z(-u), D = Z(u) - Z(-u) of Z = E conj(T) for a lane's four u: (Re A, Im D) and (Im A, Re D)
__device__ __forceinline__ void form_sums(h8 ea, h8 eb, h8 xp, h8 xm, h8* ad, h8* bd) {
  const h4 er = ea.lo, ei = ea.hi, fr = eb.lo, fi = eb.hi;
  const h4 xpr = xp.lo, xpi = xp.hi, xmr = xm.lo, xmi = xm.hi;
  const h4 mr = __builtin_elementwise_fma(fr, xmr, fi * xmi), mi = __builtin_elementwise_fma(fi, xmr, -(fr * xmi));
  const h4 ar = __builtin_elementwise_fma(er, xpr, __builtin_elementwise_fma(ei, xpi, mr));
  const h4 ai = __builtin_elementwise_fma(ei, xpr, __builtin_elementwise_fma(-er, xpi, mi));
  const h4 two = {(_Float16)-2.0f, (_Float16)-2.0f, (_Float16)-2.0f, (_Float16)-2.0f};
  const h4 dr = __builtin_elementwise_fma(two, mr, ar), di = __builtin_elementwise_fma(two, mi, ai);
  *ad = __builtin_shufflevector(ar, di, 0, 1, 2, 3, 4, 5, 6, 7);
  *bd = __builtin_shufflevector(ai, dr, 0, 1, 2, 3, 4, 5, 6, 7);
}

// coarse[p][l] = the largest low value over the grid points t h, t = +-(j + 1/2), j <= last (both axes), by
// the +-u, +-s symmetric products of k_xcf_even.hip.  One 16 x 16 tile per stage (u and j below 16, v
// and j below 16): with A = Z(u) + Z(-u), D = Z(u) - Z(-u) the first stage's four sums
//   F1, F2 = sum_u Re A cos -+ Im D sin,   F3, F4 = sum_u Im A cos +- Re D sin
// are one product of depth 32 each, the second stage's four of depth 16 give
//   max(cos F1 + |sin F3|, cos F2 + |sin F4|)
// over the four sign pairs.  A block holds PT patterns in LDS; each of its 8 waves takes tc templates in turn,
// a template's 16 values per lane serving all the patterns; every phase constant stays in registers.
// Bound by issue: 8 matrix products and 60 vector instructions a pair, 43 and 83 % of the SIMD cycles.  200 x 3,000 pairs
// take 119 us, 5,000 x 4,000 2.84 ms (7.0e9 pairs/s); with FP32 products (32 of 16x16x4) 424 us and 12.0 ms; a
// 64 x 64 FFT search of wider low parts (|u|, |v| <= 24) ran at 4.2e8 pairs/s.  2 KB a spectrum are read once
// per block of 32 patterns and 128 templates.  Fewer templates per wave (tc) fill the chip for few pairs:
// whole calls at 128 of 11 x 3,000 pairs 176 -> 124 us, 33 x 1,000 276 -> 134, 500 x 1,000 355 -> 268.
// ALL: every grid point counts (last = 15), no masks between the two patterns of a step.
template <bool ALL>
__global__ __launch_bounds__(512, 4) void k_coarse(const h8* __restrict__ low_p, int64_t np,
                                                   const h8* __restrict__ low_l, int64_t nl, int64_t npt,
                                                   int64_t nblk, int tc, int last, float* __restrict__ coarse,
                                                   int* __restrict__ queue, unsigned long long* __restrict__ fill) {
  __shared__ h8 ep[PT * FRAG];
  __shared__ float out[8 * TC * PT];
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, q4 = lane >> 4;
  if (blockIdx.x == 0 && tid < 8) queue[tid] = 0;  // for the lists of the templates that are kept
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t per = (nblk + 7) / 8;
  const int64_t g = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (g >= nblk) return;
  const int64_t chunk = g / npt, p0 = (g - chunk * npt) * PT, l0 = chunk * (8 * tc);
  const int pc = (int)(np - p0 < PT ? np - p0 : PT);
  if (chunk == 0 && tid < pc) fill[p0 + tid] = 0;
  for (int i = tid; i < pc * FRAG; i += 512) ep[i] = low_p[p0 * FRAG + i];
  // stage 1: cos, +-sin of 2 pi u (j + 1/2) / G for this lane's column j = r16 and rows u = 4 q4 + i; stage 2: the
  // same with v in the place of u and the Hermitian weight
  h8 cp, cm;
  h4 c2, s2;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int f = 4 * q4 + i;
    float s, c;
    sincospif((float)(f * (2 * r16 + 1)) / (float)G, &s, &c);
    cp[i] = cm[i] = (_Float16)c;
    cp[4 + i] = (_Float16)s;
    cm[4 + i] = (_Float16)(-s);
    c2[i] = (_Float16)(f ? 2.0f * c : c);
    s2[i] = (_Float16)(f ? 2.0f * s : s);
  }
  const bool col = r16 <= last;
  __syncthreads();
#pragma unroll 1
  for (int t = 0; t < tc; ++t) {
    const int64_t l = l0 + wave * tc + t;
    if (l >= nl) break;
    const h8 xp = low_l[l * FRAG + lane], xm = low_l[l * FRAG + 64 + lane];
    float* const o = out + (wave * tc + t) * PT;
    const auto best_of = [&](int pb) -> float {
      const h8 ea = ep[pb * FRAG + lane], eb = ep[pb * FRAG + 64 + lane];
      h8 ad, bd;
      form_sums(ea, eb, xp, xm, &ad, &bd);
      const f4 z = {0.f, 0.f, 0.f, 0.f};
      const f4 f1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ad, cm, z, 0, 0, 0);
      const f4 f2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(ad, cp, z, 0, 0, 0);
      const f4 f3 = __builtin_amdgcn_mfma_f32_16x16x32_f16(bd, cp, z, 0, 0, 0);
      const f4 f4_ = __builtin_amdgcn_mfma_f32_16x16x32_f16(bd, cm, z, 0, 0, 0);
      const f4 u1 = __builtin_amdgcn_mfma_f32_16x16x16f16(c2, __builtin_convertvector(f1, h4), z, 0, 0, 0);
      const f4 u2 = __builtin_amdgcn_mfma_f32_16x16x16f16(c2, __builtin_convertvector(f2, h4), z, 0, 0, 0);
      const f4 w1 = __builtin_amdgcn_mfma_f32_16x16x16f16(s2, __builtin_convertvector(f3, h4), z, 0, 0, 0);
      const f4 w2 = __builtin_amdgcn_mfma_f32_16x16x16f16(s2, __builtin_convertvector(f4_, h4), z, 0, 0, 0);
      float m = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = fmaxf(u1[i] + fabsf(w1[i]), u2[i] + fabsf(w2[i]));
        m = fmaxf(m, ALL || (col && 4 * q4 + i <= last) ? v : -INFINITY);
      }
      return m;
    };
    // two patterns at a time, independent of each other (an odd count's last one pairs with unused LDS)
#pragma unroll 1
    for (int pb = 0; pb < pc; pb += 2) {
      const unsigned m0 = __builtin_bit_cast(unsigned, best_of(pb)), m1 = __builtin_bit_cast(unsigned, best_of(pb + 1));
      // the halves exchanged: the first pattern's values in lanes 0 to 31, the second's in 32 to 63
      const auto sw = __builtin_amdgcn_permlane32_swap(m0, m1, false, false);
      float m = fmaxf(__builtin_bit_cast(float, (unsigned)sw[0]), __builtin_bit_cast(float, (unsigned)sw[1]));
      m = dpp_max<0x128>(m);  // row_ror 8, 4, 2, 1
      m = dpp_max<0x124>(m);
      m = dpp_max<0x122>(m);
      m = dpp_max<0x121>(m);
      m = dpp_max<0x142>(m);  // row_bcast 15: of the half, in its last lane
      if ((lane & 31) == 31) o[pb + (lane >> 5)] = m;
    }
  }
  __syncthreads();
  for (int i = tid; i < pc * 8 * tc; i += 512) {
    const int pb = i / (8 * tc), c = i - pb * (8 * tc);
    if (l0 + c < nl) coarse[(p0 + pb) * nl + l0 + c] = out[c * PT + pb] * (1.0f / (kScale * kScale));
  }
}

// Lists of one template per pattern (its list is the argmax itself, rows of 1), queue[2 ..]
__global__ __launch_bounds__(256) void k_one_each(int64_t p, int32_t* __restrict__ count, int2* __restrict__ items,
                                                  int* __restrict__ queue) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0) queue[3] = (int)p;
  if (i >= p) return;
  count[i] = 1;
  items[i] = make_int2((int)i, 0);
}

// cos, sin of pi k / (2 G) in FP16, k in [0, 4 G): the half-step grid's phases from a table, worked out per block
// (eight sincospif a lane) they took longer than the few templates that a block bounds
struct Phases {
  _Float16 cs[4 * G][2];
  constexpr Phases() : cs() {
    for (int k = 0; k < 4 * G; ++k) {
      cs[k][0] = (_Float16)(float)cx::cos2pi(k, 4 * G);
      cs[k][1] = (_Float16)(float)cx::sin2pi(k, 4 * G);
    }
  }
};
__constant__ Phases c_phases = Phases();

// The largest low value over the 64 x 64 grid of half the step (products as in k_coarse, two tiles per axis), in
// the wave's last lane; e, x: the low parts of pattern and template
struct FineConsts {
  h8 cp[2], cm[2];
  h4 c2[2], s2[2];
  __device__ __forceinline__ void init(int r16, int q4) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int f = 4 * q4 + i, k = (f * (2 * (16 * a + r16) + 1)) & (4 * G - 1);
        const _Float16 c = c_phases.cs[k][0], s = c_phases.cs[k][1], w = f ? (_Float16)2.0f : (_Float16)1.0f;
        cp[a][i] = cm[a][i] = c;
        cp[a][4 + i] = s;
        cm[a][4 + i] = -s;
        c2[a][i] = w * c;
        s2[a][i] = w * s;
      }
  }
};
__device__ __forceinline__ float fine_max(const FineConsts& k, h8 ea, h8 eb, h8 xp, h8 xm, int r16, int q4, int last) {
  h8 ad, bd;
  form_sums(ea, eb, xp, xm, &ad, &bd);
  const f4 z = {0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const h4 f1 = __builtin_convertvector(__builtin_amdgcn_mfma_f32_16x16x32_f16(ad, k.cm[a], z, 0, 0, 0), h4);
    const h4 f2 = __builtin_convertvector(__builtin_amdgcn_mfma_f32_16x16x32_f16(ad, k.cp[a], z, 0, 0, 0), h4);
    const h4 f3 = __builtin_convertvector(__builtin_amdgcn_mfma_f32_16x16x32_f16(bd, k.cp[a], z, 0, 0, 0), h4);
    const h4 f4_ = __builtin_convertvector(__builtin_amdgcn_mfma_f32_16x16x32_f16(bd, k.cm[a], z, 0, 0, 0), h4);
    const bool col = 16 * a + r16 <= last;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const f4 u1 = __builtin_amdgcn_mfma_f32_16x16x16f16(k.c2[b], f1, z, 0, 0, 0);
      const f4 u2 = __builtin_amdgcn_mfma_f32_16x16x16f16(k.c2[b], f2, z, 0, 0, 0);
      const f4 w1 = __builtin_amdgcn_mfma_f32_16x16x16f16(k.s2[b], f3, z, 0, 0, 0);
      const f4 w2 = __builtin_amdgcn_mfma_f32_16x16x16f16(k.s2[b], f4_, z, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = fmaxf(u1[i] + fabsf(w1[i]), u2[i] + fabsf(w2[i]));
        m = fmaxf(m, col && 16 * b + 4 * q4 + i <= last ? v : -INFINITY);
      }
    }
  }
  m = dpp_max<0x128>(m);
  m = dpp_max<0x124>(m);
  m = dpp_max<0x122>(m);
  m = dpp_max<0x121>(m);
  m = dpp_max<0x142>(m);
  return dpp_max<0x143>(m);
}

// The templates of each pattern that its bound keeps: cand[p l ..] (any order) and count[p], and their chunks
// in the queue, of list_chunk(count) entries or, with rows, of kListChunk.  What the first bound keeps is bounded
// once more from the grid of half the step, with a quarter of the curvature term (0.11 to 0.14 -> 0.03), one
// wave a template: 5,000 x 4,000 pairs at 128 keep so few that their full scores take 0.76 ms instead of 2.53,
// 1,500 x 1,859 at 160 0.30 instead of 0.91.  Of 4,000 templates patterns of another crystal (15 bands, SNR 5)
// keep 2.8 / 7.7 / 12 / 17 % after the first bound and 0.2 / 0.3 / 0.4 / 0.5 % after the second at 64 / 96 / 128 /
// 160, and patterns of noise 88 / 100 / 100 / 100 % and 2.7 / 27 / 92 / 100 %, so a block that finds most of its
// first SAMPLE templates still kept (with rows: too many for a list) leaves the others with the first bound.
// A block takes `slice` templates of a pattern, so that few patterns fill the chip as well; the last block of a
// pattern (fill[p]: entries so far, and blocks in the upper half) puts its list in the queue.
// With rows, a pattern that keeps more than 1 / part of the library goes there instead (queue[5] counts them)
// and its count is -1: a pair of a list costs 2 to 4 times one of a row in the even forms, whose rows share
// patterns (200 patterns of noise against 4,000 templates at 96, split, part 4 and 8: 0.89 and 1.40 ms; at 256,
// part 3, 4, 8: 8.80, 8.56, 8.49, where the second bound gains noise nothing and is left out: 8.05), and 1.4 times
// at 64, whose rows share a template load; at 96 to 160 it is 1.05 and a row launch would not pay.
constexpr int SLICE = 4096, SAMPLE = 32;
__global__ __launch_bounds__(512, 4) void k_prune_select(const float* __restrict__ coarse, int64_t l, int slice, int ns,
                                                         float h28, const h8* __restrict__ low_p,
                                                         const h8* __restrict__ low_l,
                                                         const float2* __restrict__ stat_p,
                                                         const float2* __restrict__ stat_l,
                                                         const float* __restrict__ h0, int last,
                                                         int32_t* __restrict__ cand, int32_t* __restrict__ count,
                                                         unsigned long long* __restrict__ fill, int2* __restrict__ items,
                                                         int* __restrict__ queue, int32_t* __restrict__ rows,
                                                         int part) {
  const int64_t p = blockIdx.x / ns, i0 = (int64_t)(blockIdx.x - p * ns) * slice;
  const int len = (int)(l - i0 < slice ? l - i0 : slice);
  const int tid = threadIdx.x, lane = tid & 63;
  __shared__ int kept, fine, at0, total;
  __shared__ unsigned short list[SLICE], best[SLICE];
  if (tid == 0) kept = fine = 0;
  __syncthreads();
  const float2 sp = stat_p[p];
  const float eh = 1.0002f * sp.x, kl = 1.0002f * h28 * sp.y, least = h0[p] - kRound;
  for (int j0 = 0; j0 < len; j0 += 512) {
    const int j = j0 + tid;
    bool keep = false;
    if (j < len) {
      const float2 sl = stat_l[i0 + j];
      keep = coarse[p * l + i0 + j] + __fmaf_rn(kl, sl.y, eh * sl.x) >= least;
    }
    const unsigned long long mask = __ballot(keep);
    if (mask == 0) continue;
    int at = 0;
    if (lane == 0) at = atomicAdd(&kept, __popcll(mask));
    at = __shfl(at, 0, 64) + __popcll(mask & ((1ull << lane) - 1));
    if (keep) list[at] = (unsigned short)j;
  }
  __syncthreads();
  int n = kept;
  const unsigned short* out = list;
  if ((n > 1 || (n == 1 && ns > 1)) && !(rows && part > 4 && 3 * n > len)) {
    const int r16 = lane & 15, q4 = lane >> 4;
    FineConsts k;
    k.init(r16, q4);
    const h8 ea = low_p[p * FRAG + lane], eb = low_p[p * FRAG + 64 + lane];
    const auto bound = [&](int from, int to) {
      for (int j = from + __builtin_amdgcn_readfirstlane(tid >> 6); j < to; j += 8) {
        const int64_t i = i0 + list[j];
        const h8 xp = low_l[i * FRAG + lane], xm = low_l[i * FRAG + 64 + lane];
        const float2 sl = stat_l[i];
        const float m = fine_max(k, ea, eb, xp, xm, r16, q4, last) * (1.0f / (kScale * kScale));
        if (lane == 63 && m + __fmaf_rn(0.25f * kl, sl.y, eh * sl.x) >= least) best[atomicAdd(&fine, 1)] = list[j];
      }
      __syncthreads();
    };
    bound(0, min(n, SAMPLE));
    if (n <= SAMPLE) {
      n = fine;
      out = best;
    } else if (rows ? part * fine * n <= SAMPLE * len : 4 * fine <= 3 * SAMPLE) {
      __syncthreads();
      bound(SAMPLE, n);
      n = fine;
      out = best;
    }
  }
  if (tid == 0) {
    const unsigned long long old = ns > 1 ? atomicAdd(fill + p, (1ull << 32) | (unsigned)n) : 0;
    at0 = (int)(unsigned)old;
    total = (int)(old >> 32) == ns - 1 ? at0 + n : -1;
  }
  __syncthreads();
  for (int t = tid; t < n; t += 512) cand[p * l + at0 + t] = (int32_t)(i0 + out[t]);
  n = total;
  if (n < 0) return;
  if (rows && part * n > l) {
    if (tid == 0) {
      count[p] = -1;
      rows[atomicAdd(queue + 5, 1)] = (int)p;
    }
    return;
  }
  const int ch = rows ? kListChunk : list_chunk(n), nc = (n + ch - 1) / ch;
  __shared__ int first;
  if (tid == 0) {
    count[p] = n;
    first = nc ? atomicAdd(queue + 1, nc) : 0;
  }
  __syncthreads();
  for (int i = tid; i < nc; i += 512) items[first + i] = make_int2((int)p, i * ch);
}

// bound[p k + j] = the half-step bound of candidate cand[p k + j]; first[p] = the candidate with the largest low
// value; one wave a candidate
__global__ __launch_bounds__(256) void k_cand_bounds(const h8* __restrict__ low_p, const float2* __restrict__ stat_p,
                                                     const h8* __restrict__ low_l, const float2* __restrict__ stat_l,
                                                     int64_t l, const int32_t* __restrict__ cand, int k, float h28,
                                                     int last, float* __restrict__ bound, int32_t* __restrict__ first,
                                                     int* __restrict__ queue) {
  const int64_t p = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (p == 0 && tid < 2) queue[tid] = 0;
  FineConsts c;
  c.init(r16, q4);
  const h8 ea = low_p[p * FRAG + lane], eb = low_p[p * FRAG + 64 + lane];
  const float2 sp = stat_p[p];
  const float eh = 1.0002f * sp.x, kl = 1.0002f * h28 * sp.y;
  float bv = -INFINITY;
  int bi = cand[p * k];
  for (int j = wave; j < k; j += 4) {
    int64_t i = cand[p * k + j];
    i = i < 0 ? 0 : (i >= l ? l - 1 : i);
    const h8 xp = low_l[i * FRAG + lane], xm = low_l[i * FRAG + 64 + lane];
    const float2 sl = stat_l[i];
    const float m = fine_max(c, ea, eb, xp, xm, r16, q4, last) * (1.0f / (kScale * kScale));
    if (lane == 63) {
      bound[p * k + j] = m + __fmaf_rn(kl, sl.y, eh * sl.x);
      if (m > bv) {
        bv = m;
        bi = (int)i;
      }
    }
  }
  __shared__ float rv[4];
  __shared__ int ri[4];
  if (lane == 63) {
    rv[wave] = bv;
    ri[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w)
      if (rv[w] > rv[0]) {
        rv[0] = rv[w];
        ri[0] = ri[w];
      }
    first[p] = ri[0];
  }
}

// The candidates that reach the score of `first`, and where they stand; scores are -infinity until they have one
__global__ __launch_bounds__(64) void k_cand_select(const float* __restrict__ bound, const int32_t* __restrict__ cand,
                                                    int k, const float* __restrict__ h0, int32_t* __restrict__ list,
                                                    int32_t* __restrict__ pos, int32_t* __restrict__ count,
                                                    int2* __restrict__ items, int* __restrict__ queue,
                                                    float* __restrict__ scores) {
  const int64_t p = blockIdx.x;
  const int lane = threadIdx.x;
  const float least = h0[p] - kRound;
  int n = 0;
  for (int j0 = 0; j0 < k; j0 += 64) {
    const int j = j0 + lane;
    const bool keep = j < k && bound[p * k + j] >= least;
    if (j < k) scores[p * k + j] = -INFINITY;
    const unsigned long long mask = __ballot(keep);
    if (keep) {
      const int at = n + __popcll(mask & ((1ull << lane) - 1));
      list[p * k + at] = cand[p * k + j];
      pos[p * k + at] = j;
    }
    n += __popcll(mask);
  }
  const int ch = list_chunk(n), nc = (n + ch - 1) / ch;
  int base = 0;
  if (lane == 0) {
    count[p] = n;
    base = nc ? atomicAdd(queue + 1, nc) : 0;
  }
  base = __shfl(base, 0, 64);
  for (int i = lane; i < nc; i += 64) items[base + i] = make_int2((int)p, i * ch);
}

__global__ __launch_bounds__(64) void k_cand_scatter(const float* __restrict__ listed, const int32_t* __restrict__ pos,
                                                     const int32_t* __restrict__ count, int k,
                                                     float* __restrict__ scores) {
  const int64_t p = blockIdx.x;
  for (int i = threadIdx.x; i < count[p]; i += 64) scores[p * k + pos[p * k + i]] = listed[p * k + i];
}

// Best of the kept templates, or of the whole row where count is -1 (ties: smallest index; none kept, every
// score NaN: 0)
__global__ __launch_bounds__(256) void k_prune_argmax(const float* __restrict__ scores,
                                                      const int32_t* __restrict__ cand,
                                                      const int32_t* __restrict__ count, int64_t l,
                                                      int32_t* __restrict__ best) {
  const int64_t p = blockIdx.x;
  float bv = -INFINITY;
  int bi = 0x7fffffff;
  const int c = count[p];
  const int64_t m = c < 0 ? l : c;
  for (int64_t i = threadIdx.x; i < m; i += 256)
    argmax_merge(bv, bi, scores[p * l + i], c < 0 ? (int)i : cand[p * l + i]);
  wave_argmax(bv, bi);
  __shared__ float rv[4];
  __shared__ int ri[4];
  if ((threadIdx.x & 63) == 0) {
    rv[threadIdx.x >> 6] = bv;
    ri[threadIdx.x >> 6] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) argmax_merge(bv, bi, rv[w], ri[w]);
    best[p] = bi < 0 || bi >= l ? 0 : bi;
  }
}

}  // namespace

bool prune_supported(int n, PruneBy by, int max_shift) {
  if (by == PruneBy::Fft) return fft_supported(n);
  return by != PruneBy::None && even_supported(n, max_shift);
}

// Below some number of pairs the pruned search's launches and its lists cost more than they save, and patterns that
// match nothing pay for them on top of what they keep.  The lines lie where matching patterns gain what patterns of
// noise lose or more.  Whole calls of a plan, every pair / matching / noise, in us:
//   FFT    64: 33,000 pairs 144 / 111 / 154, 66,000 240 / 126 / 171
//          96: 17,000 210 / 102 / 162;  128: 8,400 180 / 118 / 193, 17,000 280 / 121 / 198
//          160: 8,400 383 / 137 / 269
//   split  64: 33,000 104 / 98 / 126, 66,000 152 / 113 / 144;  96: 17,000 133 / 115 / 180, 33,000 170 / 129 / 200
//          128: 33,000 189 / 142 / 260, 66,000 283 / 153 / 353;  160: 33,000 267 / 176 / 361, 66,000 399 / 189 / 524
//          256: 8,400 491 / 364 / 617, 17,000 530 / 413 / 625
//   FP32   64: 33,000 137 / 101 / 127;  128: 17,000 181 / 132 / 243, 33,000 256 / 146 / 305
//          160: 17,000 262 / 162 / 349, 33,000 384 / 183 / 472;  256: 8,400 548 / 390 / 670
// (windows of +-15 px; the split form's own products are the cheapest, its lists the dearest).
bool prune_pays(int n, PruneBy by, int max_shift, int64_t pairs) {
  if (!prune_supported(n, by, max_shift)) return false;
  int at;
  if (by == PruneBy::Fft) at = n == 64 ? 15 : n == 96 ? 14 : 13;
  else at = (n == 256 ? 13 : n == 96 ? 14 : 15) + (by == PruneBy::EvenSplit);
  return pairs >= int64_t(1) << at;
}

int64_t prune_slab(int64_t p, int64_t l) {
  return std::max<int64_t>(1, std::min({p, (int64_t(1) << 26) / l, int64_t(1) << 21}));
}

int64_t low_spec_complex() { return FRAG * (int)sizeof(h8) / (int)sizeof(float2); }

hipError_t launch_low_spectra(int n, const float2* spec, int64_t k, float2* low, float2* stat, hipStream_t stream) {
  if (k <= 0) return hipSuccess;
  const int bnd = band_of(n);
  if (bnd < BL + 1) return hipErrorInvalidValue;
  const int64_t sc = (int64_t)(bnd + 1) * (2 * bnd + 1), kmax = (int64_t(1) << 31) / 256;
  for (int64_t s = 0; s < k; s += kmax) {
    hipLaunchKernelGGL(k_low_spectra, dim3((unsigned)(k - s < kmax ? k - s : kmax)), dim3(256), 0, stream,
                       (const cf*)spec + s * sc, n, bnd, (h8*)low + s * FRAG, stat + s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_pruned_best(int n, PruneBy by, const float2* spec_p, const float2* low_p, const float2* stat_p,
                              int64_t p, const float2* spec_l, const float2* low_l, const float2* stat_l, int64_t l,
                              int max_shift, const PruneScratch& ws, int32_t* best, hipStream_t stream) {
  if (p <= 0) return hipSuccess;
  if (p > (int64_t(1) << 31) / 256) return hipErrorInvalidValue;
  hipError_t e;
  const float h = (float)n / (float)G;
  // the cells of a grid of step s that cover a shift window
  const auto last_of = [&](float s, int all) {
    return max_shift < 0 ? all : std::min(all, std::max(0, (int)ceilf((float)max_shift / s - 0.5f)));
  };
  const int last = last_of(h, 15);
  // templates per wave: TC, fewer where that leaves less than four rounds of the 512 blocks that run at once
  int tc = TC;
  while (tc > 1 && ((p + PT - 1) / PT) * ((l + 8 * tc - 1) / (8 * tc)) < 2048) tc >>= 1;
  const int64_t nch = (l + 8 * tc - 1) / (8 * tc), pmax = std::max<int64_t>(1, ((int64_t(1) << 31) / 512 - 8) / nch) * PT;
  for (int64_t s = 0; s < p; s += pmax) {
    const int64_t pc = p - s < pmax ? p - s : pmax, npt = (pc + PT - 1) / PT, nblk = npt * nch;
    hipLaunchKernelGGL(last == 15 ? k_coarse<true> : k_coarse<false>, dim3((unsigned)((nblk + 7) / 8 * 8)), dim3(512), 0,
                       stream, (const h8*)low_p + s * FRAG, pc, (const h8*)low_l, l, npt, nblk, tc, last,
                       ws.scores + s * l, ws.queue, ws.fill + s);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = launch_library_argmax(ws.scores, p, l, best, ws.h0, stream)) != hipSuccess) return e;
  const bool split = by == PruneBy::EvenSplit;
  if (by == PruneBy::Fft) {
    e = launch_xcf_scores_cand(n, spec_p, p, spec_l, l, best, 1, max_shift, ws.h0, stream);
  } else {
    hipLaunchKernelGGL(k_one_each, dim3((unsigned)((p + 255) / 256)), dim3(256), 0, stream, p, ws.count, ws.items,
                       ws.queue);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    e = launch_xcf_even_lists(n, split, spec_p, p, spec_l, l, 1, best, ws.count, ws.items, ws.queue + 2, max_shift,
                              ws.frag, true, ws.h0, stream);
  }
  if (e != hipSuccess) return e;
  // slices down to 256 templates while they leave CUs without two blocks: 11 patterns of noise against 3,000
  // templates at 64 in whole rows 0.31 ms, in slices 0.14; 500 against 1,000 in four slices each lose 2 %
  int slice = SLICE;
  while (slice > 256 && p * ((l + slice - 1) / slice) < 512) slice >>= 1;
  const int64_t ns = (l + slice - 1) / slice;
  hipLaunchKernelGGL(k_prune_select, dim3((unsigned)(p * ns)), dim3(512), 0, stream, ws.scores, l, slice, (int)ns,
                     0.125f * h * h, (const h8*)low_p, (const h8*)low_l, stat_p, stat_l, ws.h0, last_of(0.5f * h, 31),
                     ws.cand, ws.count, ws.fill, ws.items, ws.queue,
                     by == PruneBy::Fft && n != 64 ? nullptr : ws.rows, n < 160 ? 4 : 8);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t most = p * list_chunks(l);
  e = by == PruneBy::Fft
          ? launch_xcf_scores_lists(n, spec_p, most, spec_l, l, l, ws.cand, ws.count, ws.items, ws.queue, max_shift,
                                    ws.scores, stream)
          : launch_xcf_even_lists(n, split, spec_p, most, spec_l, l, l, ws.cand, ws.count, ws.items, ws.queue,
                                  max_shift, ws.frag, false, ws.scores, stream);
  if (e != hipSuccess) return e;
  if (by != PruneBy::Fft)
    e = launch_xcf_even_rows(n, split, spec_p, p, ws.rows, spec_l, l, ws.queue + 4, max_shift, ws.frag, ws.scores, stream);
  else if (n == 64)
    e = launch_xcf_scores_rows64(spec_p, p, ws.rows, spec_l, l, ws.queue + 4, max_shift, ws.scores, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_prune_argmax, dim3((unsigned)p), dim3(256), 0, stream, ws.scores, ws.cand, ws.count, l, best);
  return hipGetLastError();
}

// Candidates are read at random, 38 KB of spectrum each, so 32 for each of 4,096 patterns out of 8,000 templates
// take 1.62 ms in full (the whole call 5.99 ms, pruned 4.99).  The bounds need the library's low parts (8 ns a
// template) and one full score a pattern, which is too much of what 8 candidates a pattern cost (4.81 -> 4.95 ms)
// and where the library is half as many templates as there are pairs (32 x 1,024 of 16,000: 3.69 -> 3.65).
bool prune_cand_pays(int n, int64_t p, int k, int64_t l) {
  return n == 128 && k >= 16 && p * k >= (int64_t(1) << 15) && p * k >= 2 * l && p <= (int64_t(1) << 31) / 256;
}

hipError_t launch_pruned_cand(int n, const float2* spec_p, const float2* low_p, const float2* stat_p, int64_t p,
                              const float2* spec_l, const float2* low_l, const float2* stat_l, int64_t l,
                              const int32_t* cand, int k, int max_shift, const CandScratch& ws, float* scores,
                              hipStream_t stream) {
  if (p <= 0 || k <= 0) return hipSuccess;
  if (p > (int64_t(1) << 31) / 256) return hipErrorInvalidValue;
  hipError_t e;
  const float h = (float)n / (float)(2 * G);
  const int last = max_shift < 0 ? 31 : std::min(31, std::max(0, (int)ceilf((float)max_shift / h - 0.5f)));
  hipLaunchKernelGGL(k_cand_bounds, dim3((unsigned)p), dim3(256), 0, stream, (const h8*)low_p, stat_p,
                     (const h8*)low_l, stat_l, l, cand, k, 0.125f * h * h, last, ws.bound, ws.first, ws.queue);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_xcf_scores_cand(n, spec_p, p, spec_l, l, ws.first, 1, max_shift, ws.h0, stream)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(k_cand_select, dim3((unsigned)p), dim3(64), 0, stream, ws.bound, cand, k, ws.h0, ws.list, ws.pos,
                     ws.count, ws.items, ws.queue, scores);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // the bounds have served: the listed scores take their place
  if ((e = launch_xcf_scores_lists(n, spec_p, p * list_chunks(k), spec_l, l, k, ws.list, ws.count, ws.items, ws.queue,
                                   max_shift, ws.bound, stream)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(k_cand_scatter, dim3((unsigned)p), dim3(64), 0, stream, ws.bound, ws.pos, ws.count, k, scores);
  return hipGetLastError();
}

}  // namespace ebsd
