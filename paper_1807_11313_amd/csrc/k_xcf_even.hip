// Correlation search over a shift window as DFT products on the matrix cores (gfx950), in FP32 or in
// split FP16, with the +-u and +-s symmetries of the phase factors used in both stages.
//
// For one pattern-template pair with Z = E conj(T) over the stored band
// (u in [-B, B], v in [0, B]; w_0 = 1, w_v = 2 for the Hermitian half)
//   rho(s_y, s_x) = Re sum_v w_v exp(2 pi i v s_x / N) sum_u Z(u, v) exp(2 pi i u s_y / N).
// With A(u) = Z(u) + Z(-u), D(u) = Z(u) - Z(-u) for u >= 0 (Z(-0) = 0) and, for s_y >= 0,
//   C(s_y, v) = sum_u A(u, v) cos(2 pi u s_y / N),   S(s_y, v) = sum_u D(u, v) sin(2 pi u s_y / N)
// the inner sum at +-s_y is C +- i S; with, for s_x >= 0,
//   P1 = sum_v w Re C cos,  P2 = sum_v w Im S cos,  Q1 = sum_v w Im C sin,  Q2 = sum_v w Re S sin
// (cos, sin of 2 pi v s_x / N) the four correlation values are
//   rho(y s_y, x s_x) = (P1 - y P2) - x (Q1 + y Q2),   x, y = +-1.
// Every product is real: stage 1 costs a quarter and stage 2 half of the
// complex products over the full range of u and s.
//
// Z, A and D are formed in FP32 on the vector ALU.  The products take one of two forms (SPLIT):
//  - FP32 operands on v_mfma_f32_16x16x4_f32 (exact products, FP32 sums);
//  - every operand split into two FP16 halves x = hi + lo, both rounded to nearest even, the
//    product formed as hi*hi + hi*lo + lo*hi with FP32 sums.  E is scaled by 2^10 first (exact),
//    so that the lo halves of typical band values are normal FP16 numbers; |A|, |C|, |S| are at most
//    2^10 |E| |T|, below the FP16 maximum up to a product of 63 of the spectra's norms (2^12: 15).
//    The largest error of unit-energy spectra is the same with either factor.
//
// One wave owns one pair at a time.  Stage 1 runs transposed: A operand = the formed values (row
// v = lane % 16, this lane's eight rows u = 32 kc + 8 (lane / 16) + j), B operand = the phase
// constants (column s_y = lane % 16).  Its accumulator tile (lane: v = 4 (lane / 16) + i, s_y = lane % 16)
// is the B operand of stage 2, value i in its i-th product (FP32) or all four in one 16-deep
// product (FP16 halves).
#include "ebsd_common.hpp"
#include "ebsd_internal.hpp"

#include <math.h>

#include <type_traits>

namespace ebsd {

namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr float kScale = 1024.0f;
constexpr float kUnscale = 1.0f / 1024.0f;

constexpr int kRing = 4 * 8 * 64 * 16;  // bytes of LDS per pattern of a block

// ST: tiles of 16 shifts s >= 0 (max_shift < 16 ST).  DISC: the spectra are zero outside the filter's
// disc, as every spectrum this library writes is
template <int N, int ST, bool DISC>
struct EvenLay {
  static constexpr int B = Plan<N>::B, NV = B + 1, NK = 2 * B + 1, SPEC = NV * NK;
  // rows u in [0, 32 KC + 16 HALF) and columns v in [0, 16 VT) run through the products.  Where B is a
  // multiple of 16 the row u = B and the column v = B, which in the disc are non-zero at v = 0 and u = 0
  // only, are added to the result in FP32 instead of opening another chunk
  static constexpr bool UTOP = DISC && B % 16 == 0, VTOP = UTOP;
  static constexpr int ROWS16 = UTOP ? B / 16 : B / 16 + 1;
  static constexpr int KC = ROWS16 / 2, HALF = ROWS16 % 2, NS = KC + HALF;  // chunks of 32 rows, of 16; both
  static constexpr int VT = VTOP ? B / 16 : B / 16 + 1;
  // constants, the same bytes in both forms: stage 1 [KC][ST][cos, sin] x 2 x 64 lanes x 16 B
  // (FP16: hi, lo halves of 8 rows; FP32: rows 0-3, 4-7), its half chunk [ST][cos, sin] x 1024 B, stage 2
  // [VT][ST][w cos, w sin] x 1024 B (FP16: [hi, lo][lane] x 4 halves; FP32: [lane] x 4)
  static constexpr int H_AT = KC * ST * 4096, W_BYTES = H_AT + HALF * ST * 2048, C_BYTES = VT * ST * 2048;
  static constexpr int FRAG_BYTES = W_BYTES + C_BYTES;
};

template <int N, int ST, bool SPLIT, bool DISC>
__global__ void k_even_consts(unsigned char* __restrict__ frag) {
  using L = EvenLay<N, ST, DISC>;
  constexpr int nf = L::H_AT / 4, nw = L::W_BYTES / 4;
  const int i = blockIdx.x * 256 + threadIdx.x;  // one constant per thread
  if (i >= nw + L::C_BYTES / 4) return;
  const bool full = i < nf, first = i < nw;
  const int per = full ? 8 : 4, at = full ? 0 : (first ? nf : nw), c = i - at;
  const int j = c % per, lane = (c / per) & 63, rest = c / (per * 64);
  const int part = rest & 1, st = (rest >> 1) % ST, chunk = full || !first ? (rest >> 1) / ST : L::KC;
  const int s = st * 16 + (lane & 15);
  const int f = chunk * (first ? 32 : 16) + per * (lane >> 4) + j;
  double val = 0.0;
  if (f < (first ? (L::UTOP ? L::B : L::B + 1) : (L::VTOP ? L::B : L::NV))) {
    double sn, cs;
    sincospi(2.0 * (double)((f * s) % N) / (double)N, &sn, &cs);
    val = part ? sn : cs;
    if (!first && f > 0) val *= 2.0;
  }
  const float x = (float)val;
  unsigned char* base = frag + at * 4 + rest * per * 256;
  if constexpr (SPLIT) {
    const _Float16 h = (_Float16)x, l = (_Float16)(x - (float)h);
    _Float16* o = reinterpret_cast<_Float16*>(base) + lane * per + j;
    o[0] = h;
    o[64 * per] = l;
  } else {
    reinterpret_cast<float*>(base)[((j >> 2) * 64 + lane) * 4 + (j & 3)] = x;
  }
}

// Four pairs of floats split into packed FP16 halves: hi[i] = (x[2i], x[2i + 1]) rounded, lo[i] =
// the exact remainders (one mixed-precision FMA each) rounded: four full-rate instructions a pair.
// The empty asm keeps the compiler from folding the conversion into the FMA that made x, as a
// mixed FMA that writes one FP16 half: those run at half rate.  The waits between a matrix instruction
// and others are the compiler's, who does not look into an asm: each FMA works in place, on a register
// that the conversion before it has read and that no matrix instruction in flight reads or writes, and the
// conversions are left to the compiler.
__device__ __forceinline__ unsigned pack_f16(float a, float b) {
  return __builtin_bit_cast(unsigned, h2{(_Float16)a, (_Float16)b});
}
__device__ __forceinline__ void split4(const float* x, unsigned* hi, unsigned* lo) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
    asm("" : "+v"(a), "+v"(b));
    hi[i] = pack_f16(a, b);
    asm("v_fma_mix_f32 %0, -%1, 1.0, %0 op_sel_hi:[1,0,0]" : "+v"(a) : "v"(hi[i]));
    asm("v_fma_mix_f32 %0, -%1, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(b) : "v"(hi[i]));
    lo[i] = pack_f16(a, b);
  }
}

__device__ __forceinline__ f4 mfma32(const u4v& a, const u4v& b, const f4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f4 mfma16(const u2v& a, const u2v& b, const f4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(h4, a), __builtin_bit_cast(h4, b), c, 0, 0, 0);
}

__device__ __forceinline__ f4 mfma4(float a, float b, const f4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// exp(i pi k / 4), k in [0, 8): B / N = 3 / 8, so the top row's and column's phases are eighths of a turn
__device__ __forceinline__ cf oct_root(int k) {
  constexpr float r = 0.70710678118654752440f;
  const float c[8] = {1.0f, r, 0.0f, -r, -1.0f, -r, 0.0f, r};
  return cf{c[k], c[(k + 6) & 7]};
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const cf* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<cf*>(p), (short)0, bytes, 0x00020000);
}
__device__ __forceinline__ cf load_cf(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(cf, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}

// Byte offsets of a lane's values of chunk (vt, kc): rows u0 + j, u0 = 32 kc + 8 q (32 KC + 4 q of the half
// chunk, whose j >= 4 are not used), at pos + j * row, rows -(u0 + j) at neg + (7 - j) * row.  The row of u = -0 lies past the end of the spectrum (a buffer load
// there returns zero); rows above B hold other values of the spectrum and meet zero constants, as do
// the columns past the last one, which read the last.
// rows8: 8 q rows in bytes; everything else of the rows is uniform.
template <class L>
__device__ __forceinline__ void chunk_offsets(int step, int r16, int rows8, int* pos, int* neg) {
  constexpr int ROW = L::NV * (int)sizeof(cf);
  const int vt = step / L::NS, kc = step - vt * L::NS;
  const int v = min(vt * 16 + r16, L::NV - 1) * (int)sizeof(cf);
  const int u0 = kc * 32 * ROW + (L::HALF && kc == L::KC ? rows8 / 2 : rows8);
  *pos = u0 + v;
  *neg = (L::NK - 7) * ROW - u0 + v;
}

// A block of 8 waves correlates PB patterns with 8 templates, one per wave.  The patterns' values of each
// step (vt, kc) are staged once per block in a four-slot ring in LDS, two steps ahead (so one barrier
// closes two steps); wave w stages value j = w of every pattern.  A template value a wave loads serves PB patterns, and is replaced by the next step's as soon as
// the last pattern has used it.
// Bound by issue: vector and matrix instructions of the waves on one SIMD hardly overlap here (128 FMAs
// and 32 of the 16-cycle products take 1,886 cycles a pair of waves, 2,155 one after the other), so the cost of a
// step is their sum: 80 VALU instructions to form A and D, 64 to split them, 12 products (split), or 80 and 32
// products of 32 cycles (FP32); 61 and 24 % of the cycles issue vector and matrix work at 128 split, 70 and 22 at 256,
// 30 and 63 in FP32.  The half chunk of 16 rows takes half of the vector instructions: 1,200 x 1,500 split
// pairs (whole calls) at 96 6.07 -> 5.27 ms, at 128 6.11 -> 5.37, at max_shift 31 12.7 -> 11.0 and 12.9 -> 10.9.
// Measured, max_shift 15, 1,200 x 1,500 pairs at 128 and 500 x 1,500 at 256: split 3.4e8 / 1.16e8 pairs/s (complex
// products over every u and s: 2.5e8 / 0.84e8).
// Super-tiles of TS template blocks: consecutive blocks (running at one time on an XCD) cycle through
// the TS template blocks of one pattern block, so both stay in that XCD's L2
template <int N>
__device__ __forceinline__ void tile_of(int64_t g, int64_t npb, int64_t nl, int64_t* tb, int64_t* pbk) {
  constexpr int TS = N >= 256 ? 2 : 4;
  const int64_t ntb = (nl + 7) / 8;
  const int64_t tb0 = g / (TS * npb) * TS;
  const int64_t ts = ntb - tb0 < TS ? ntb - tb0 : TS;
  const int64_t r = g - tb0 * npb;
  *pbk = r / ts;
  *tb = tb0 + (r - *pbk * ts);
}

// One wave's part: the PB patterns pat(0 .. cnt - 1) (cnt >= 1) against template T (any valid one where !lok),
// scores to out[pattern * row].  smem: the constants, loaded before or by the same block without a
// barrier since, then the ring.
template <int N, int ST, int PB, bool SPLIT, bool DISC, class Pat>
__device__ __forceinline__ void even_tile(unsigned char* smem, const cf* __restrict__ spec_p, Pat pat, int64_t cnt,
                                          const cf* __restrict__ T, bool lok, int max_shift, float* __restrict__ out,
                                          int64_t row) {
  using L = EvenLay<N, ST, DISC>;
  constexpr int VT = L::VT, KC = L::KC, NV = L::NV, NSTEP = VT * L::NS, ROW = NV * (int)sizeof(cf);
  constexpr int NSLOT = 4, AHEAD = 2;
  constexpr float SCALE = SPLIT ? kScale : 1.0f, UNSCALE = SPLIT ? kUnscale : 1.0f;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, q4 = lane >> 4, rows8 = 8 * ROW * q4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const u4v* wf = reinterpret_cast<const u4v*>(smem);
  const unsigned char* cfr = smem + L::W_BYTES;
  f4* ring = reinterpret_cast<f4*>(smem + L::FRAG_BYTES);  // [slot][pb][j][lane] (E(u), E(-u))
  const __amdgpu_buffer_rsrc_t tr = rsrc_of(T, L::SPEC * (int)sizeof(cf));
  __amdgpu_buffer_rsrc_t er[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
    er[pb] = rsrc_of(spec_p + pat(pb < cnt ? pb : 0) * L::SPEC, L::SPEC * (int)sizeof(cf));

  cf es[PB][2];
  auto stage_load = [&](int pos, int neg) {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      es[pb][0] = load_cf(er[pb], pos, wave * ROW);
      es[pb][1] = load_cf(er[pb], neg, (7 - wave) * ROW);
    }
  };
  auto stage_store = [&](int slot) {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
      ring[((slot * PB + pb) * 8 + wave) * 64 + lane] =
          f4{es[pb][0].x * SCALE, es[pb][0].y * SCALE, es[pb][1].x * SCALE, es[pb][1].y * SCALE};
  };
  cf tp[8], tn[8];
#pragma unroll
  for (int step = 0; step < AHEAD; ++step) {
    int pos, neg;
    chunk_offsets<L>(step, r16, rows8, &pos, &neg);
    stage_load(pos, neg);
    if (step == 0) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        tp[j] = load_cf(tr, pos, j * ROW);
        tn[j] = load_cf(tr, neg, (7 - j) * ROW);
      }
    }
    stage_store(step);
  }
  __syncthreads();

  f4 rho[PB][ST][ST][4];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int a = 0; a < ST; ++a)
#pragma unroll
      for (int b = 0; b < ST; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) rho[pb][a][b][c] = f4{0.f, 0.f, 0.f, 0.f};

#pragma unroll 1
  for (int vt = 0; vt < VT; ++vt) {
    f4 acc[PB][ST][4];  // C re, C im, S re, S im
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[pb][s][c] = f4{0.f, 0.f, 0.f, 0.f};
    const auto chunk = [&](auto half, int kc) {
      constexpr bool HF = decltype(half)::value;
      constexpr int J = HF ? 4 : 8;
      const int step = vt * L::NS + kc, slot = step & (NSLOT - 1);
      int pos, neg;
      {
        chunk_offsets<L>(min(step + AHEAD, NSTEP - 1), r16, rows8, &pos, &neg);
        stage_load(pos, neg);
        chunk_offsets<L>(min(step + 1, NSTEP - 1), r16, rows8, &pos, &neg);
      }
      if constexpr (HF) {  // the full chunk that follows
#pragma unroll
        for (int j = J; j < 8; ++j) {
          tp[j] = load_cf(tr, pos, j * ROW);
          tn[j] = load_cf(tr, neg, (7 - j) * ROW);
        }
      }
      f4 e[J];
#pragma unroll
      for (int j = 0; j < J; ++j) e[j] = ring[((slot * PB) * 8 + j) * 64 + lane];
      u4v w[ST][4];  // [cos, cos, sin, sin]: hi, lo halves or rows 0-3, 4-7
      u2v w2[ST][4];  // the half chunk's halves
#pragma unroll
      for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if constexpr (!HF) w[s][c] = wf[((kc * ST + s) * 4 + c) * 64 + lane];
          else if constexpr (SPLIT) w2[s][c] = reinterpret_cast<const u2v*>(smem + L::H_AT)[(s * 4 + c) * 64 + lane];
          else if (!(c & 1)) w[s][c] = reinterpret_cast<const u4v*>(smem + L::H_AT)[(s * 2 + c / 2) * 64 + lane];
        }
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        u4v zh[4], zl[4];  // A re, A im, D re, D im
#pragma unroll
        for (int j = 0; j < J; j += 2) {
          float x[8];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const f4 ej = e[j + h];
            const cf t0 = tp[j + h], t1 = tn[j + h];
            const float mr = __fmaf_rn(ej[2], t1.x, ej[3] * t1.y), mi = __fmaf_rn(ej[3], t1.x, -(ej[2] * t1.y));
            const float ar = __fmaf_rn(ej[0], t0.x, __fmaf_rn(ej[1], t0.y, mr));
            const float ai = __fmaf_rn(ej[1], t0.x, __fmaf_rn(-ej[0], t0.y, mi));
            x[h] = ar;
            x[2 + h] = ai;
            x[4 + h] = __fmaf_rn(-2.0f, mr, ar);
            x[6 + h] = __fmaf_rn(-2.0f, mi, ai);
            if (pb + 1 < PB) {
              e[j + h] = ring[((slot * PB + pb + 1) * 8 + j + h) * 64 + lane];
            } else if (HF || KC > 1 || !L::HALF || j < 4) {  // a half chunk follows the only full one
              tp[j + h] = load_cf(tr, pos, (j + h) * ROW);
              tn[j + h] = load_cf(tr, neg, (7 - j - h) * ROW);
            }
          }
          if constexpr (SPLIT) {
            unsigned hi[4], lo[4];
            split4(x, hi, lo);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              zh[c][j / 2] = hi[c];
              zl[c][j / 2] = lo[c];
            }
          } else {
#pragma unroll
            for (int s = 0; s < ST; ++s)
#pragma unroll
              for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                  acc[pb][s][c] = mfma4(x[2 * c + h],
                                        __builtin_bit_cast(f4, w[s][(c & 2) + (j + h) / 4])[(j + h) & 3],
                                        acc[pb][s][c]);
          }
        }
        if constexpr (SPLIT) {
          // (16-deep products one or two instructions after 32-deep ones into the same accumulators gave wrong
          // sums in a trial; between those of two chunks lie the vector instructions of a chunk)
          const auto product = [&](const u4v& z, int s, int k, const f4& a) {
            if constexpr (HF) return mfma16(u2v{z[0], z[1]}, w2[s][k], a);
            else return mfma32(z, w[s][k], a);
          };
#pragma unroll
          for (int s = 0; s < ST; ++s) {
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[pb][s][c] = product(zh[c], s, c & 2, acc[pb][s][c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[pb][s][c] = product(zh[c], s, (c & 2) + 1, acc[pb][s][c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[pb][s][c] = product(zl[c], s, c & 2, acc[pb][s][c]);
          }
        }
      }
      stage_store((step + AHEAD) & (NSLOT - 1));
      if (step & 1) __syncthreads();
    };
#pragma unroll 1
    for (int kc = 0; kc < KC; ++kc) chunk(std::false_type{}, kc);
    if constexpr (L::HALF) chunk(std::true_type{}, KC);
    // stage 2: P1 += cos C re, P2 += cos S im, Q1 += sin C im, Q2 += sin S re
    constexpr int src[4] = {0, 3, 1, 2};  // C re, S im, C im, S re
    if constexpr (SPLIT) {
      u2v cw[ST][4];
#pragma unroll
      for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          cw[s][c] = reinterpret_cast<const u2v*>(cfr)[((vt * ST + s) * 4 + c) * 64 + lane];
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int sy = 0; sy < ST; ++sy) {
          u2v bh[4], bl[4];
#pragma unroll
          for (int i = 0; i < 4; i += 2) {
            float x[8];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              x[2 * c] = acc[pb][sy][c][i];
              x[2 * c + 1] = acc[pb][sy][c][i + 1];
            }
            unsigned hi[4], lo[4];
            split4(x, hi, lo);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              bh[c][i / 2] = hi[c];
              bl[c][i / 2] = lo[c];
            }
          }
#pragma unroll
          for (int sx = 0; sx < ST; ++sx) {
            f4* r = rho[pb][sx][sy];
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = mfma16(cw[sx][c & 2], bh[src[c]], r[c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = mfma16(cw[sx][(c & 2) + 1], bh[src[c]], r[c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = mfma16(cw[sx][c & 2], bl[src[c]], r[c]);
          }
        }
    } else {
#pragma unroll
      for (int sx = 0; sx < ST; ++sx) {
        const f4 cc = reinterpret_cast<const f4*>(cfr)[((vt * ST + sx) * 2) * 64 + lane];
        const f4 cs = reinterpret_cast<const f4*>(cfr)[((vt * ST + sx) * 2 + 1) * 64 + lane];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
          for (int sy = 0; sy < ST; ++sy)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
              for (int c = 0; c < 4; ++c)
                rho[pb][sx][sy][c] = mfma4(c < 2 ? cc[i] : cs[i], acc[pb][sy][src[c]][i], rho[pb][sx][sy][c]);
      }
    }
  }
  if (!lok) return;
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    if (pb >= cnt) break;
    const cf* E = spec_p + pat(pb) * L::SPEC;
    cf za{0.f, 0.f}, zd{0.f, 0.f}, zc{0.f, 0.f};
    if constexpr (L::UTOP) {
      const cf zp = cmulc(E[L::B * NV], T[L::B * NV]), zm = cmulc(E[(L::B + 1) * NV], T[(L::B + 1) * NV]);
      za = cscale(cadd(zp, zm), SCALE);
      zd = cscale(csub(zp, zm), SCALE);
    }
    if constexpr (L::VTOP) zc = cscale(cmulc(E[L::B], T[L::B]), 2.0f * SCALE);
    float m = -INFINITY;
#pragma unroll
    for (int sx = 0; sx < ST; ++sx)
#pragma unroll
      for (int sy = 0; sy < ST; ++sy) {
        const int y = sy * 16 + r16;
        const cf wy = oct_root((3 * y) & 7);
        const f4* r = rho[pb][sx][sy];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int x = sx * 16 + 4 * q4 + i;
          const cf wx = oct_root((3 * x) & 7);
          const float p1 = __fmaf_rn(zc.x, wx.x, __fmaf_rn(za.x, wy.x, r[0][i]));
          const float p2 = __fmaf_rn(zd.y, wy.y, r[1][i]);
          const float q1 = __fmaf_rn(zc.y, wx.y, r[2][i]), q2 = r[3][i];
          const float v = fmaxf((p1 - p2) + fabsf(q1 + q2), (p1 + p2) + fabsf(q1 - q2));
          if (x <= max_shift && y <= max_shift) m = fmaxf(m, v);
        }
      }
    m = wave_max(m);
    if (lane == 0) out[pat(pb) * row] = m * UNSCALE;
  }
}

template <int N, int ST, int PB, bool SPLIT, bool DISC>
__global__ __launch_bounds__(512) void k_xcf_even(const cf* __restrict__ spec_p, int64_t np,
                                                  const cf* __restrict__ spec_l, int64_t nl, int64_t npb,
                                                  int64_t nblk, int max_shift,
                                                  const unsigned char* __restrict__ frag_g,
                                                  float* __restrict__ scores) {
  using L = EvenLay<N, ST, DISC>;
  __shared__ __align__(16) unsigned char smem[L::FRAG_BYTES + kRing * PB];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t per = (nblk + 7) / 8;
  const int64_t g = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (g >= nblk) return;
  int64_t tb, pbk;
  tile_of<N>(g, npb, nl, &tb, &pbk);
  const int64_t p0 = pbk * PB, l = tb * 8 + wave;
  const bool lok = l < nl;
  for (int i = tid; i < L::FRAG_BYTES / 16; i += 512)
    reinterpret_cast<uint4*>(smem)[i] = reinterpret_cast<const uint4*>(frag_g)[i];
  even_tile<N, ST, PB, SPLIT, DISC>(smem, spec_p, [p0](int pb) { return p0 + pb; }, np - p0,
                                    spec_l + (lok ? l : 0) * L::SPEC, lok, max_shift, scores + l, nl);
}

// The same for lists: scores[p nl + j] for template cand[p nl + j], j < count[p], in chunks of 8 templates
// items[g] = (pattern, first entry), g < queue[1], which a resident grid takes from queue[0].  A chunk's
// templates share one pattern only, so a pair costs up to three times k_xcf_even's.
template <int N, int ST, bool SPLIT>
__global__ __launch_bounds__(512) void k_xcf_even_lists(const cf* __restrict__ spec_p, const cf* __restrict__ spec_l,
                                                        int64_t lib_n, int64_t nl, const int32_t* __restrict__ cand,
                                                        const int32_t* __restrict__ count,
                                                        const int2* __restrict__ items, int* __restrict__ queue,
                                                        int max_shift, const unsigned char* __restrict__ frag_g,
                                                        float* __restrict__ scores) {
  using L = EvenLay<N, ST, true>;
  __shared__ __align__(16) unsigned char smem[L::FRAG_BYTES + kRing];
  __shared__ int item;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int total = queue[1];
  for (int i = tid; i < L::FRAG_BYTES / 16; i += 512)
    reinterpret_cast<uint4*>(smem)[i] = reinterpret_cast<const uint4*>(frag_g)[i];
  for (;;) {
    __syncthreads();
    if (tid == 0) item = atomicAdd(queue, 1);
    __syncthreads();
    const int g = __builtin_amdgcn_readfirstlane(item);
    if (g >= total) return;
    const int64_t p = items[g].x, j = items[g].y + wave;
    const bool lok = j < count[p];
    int64_t tl = lok ? cand[p * nl + j] : 0;
    tl = tl < 0 ? 0 : (tl >= lib_n ? lib_n - 1 : tl);
    even_tile<N, ST, 1, SPLIT, true>(smem, spec_p, [p](int) { return p; }, 1, spec_l + tl * L::SPEC, lok, max_shift,
                                     scores + j, nl);
  }
}

// And for patterns that keep most of the library: rows[0 .. queue[1]) against all of it, PB patterns a block
// as in k_xcf_even, tiles taken from queue[0] by a resident grid
template <int N, int ST, int PB, bool SPLIT>
__global__ __launch_bounds__(512) void k_xcf_even_rows(const cf* __restrict__ spec_p, const int32_t* __restrict__ rows,
                                                       const cf* __restrict__ spec_l, int64_t nl,
                                                       int* __restrict__ queue, int max_shift,
                                                       const unsigned char* __restrict__ frag_g,
                                                       float* __restrict__ scores) {
  using L = EvenLay<N, ST, true>;
  __shared__ __align__(16) unsigned char smem[L::FRAG_BYTES + kRing * PB];
  __shared__ int item;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nr = queue[1];
  const int64_t npb = (nr + PB - 1) / PB, nblk = npb * ((nl + 7) / 8);
  if (nblk == 0) return;
  for (int i = tid; i < L::FRAG_BYTES / 16; i += 512)
    reinterpret_cast<uint4*>(smem)[i] = reinterpret_cast<const uint4*>(frag_g)[i];
  for (;;) {
    __syncthreads();
    if (tid == 0) item = atomicAdd(queue, 1);
    __syncthreads();
    const int g = __builtin_amdgcn_readfirstlane(item);
    if (g >= nblk) return;
    int64_t tb, pbk;
    tile_of<N>(g, npb, nl, &tb, &pbk);
    const int64_t l = tb * 8 + wave;
    const bool lok = l < nl;
    const int32_t* r = rows + pbk * PB;
    even_tile<N, ST, PB, SPLIT, true>(smem, spec_p, [r](int pb) { return (int64_t)r[pb]; }, nr - pbk * PB,
                                      spec_l + (lok ? l : 0) * L::SPEC, lok, max_shift, scores + l, nl);
  }
}

template <int N, int ST, int PB, bool SPLIT, bool DISC>
hipError_t run_even(const float2* spec_p, int64_t p, const float2* spec_l, int64_t l, int max_shift,
                    unsigned char* frag, float* scores, hipStream_t stream) {
  using L = EvenLay<N, ST, DISC>;
  hipLaunchKernelGGL((k_even_consts<N, ST, SPLIT, DISC>), dim3((L::FRAG_BYTES / 4 + 255) / 256), dim3(256), 0, stream,
                     frag);
  const int64_t ntb = (l + 7) / 8;
  // patterns per dispatch so that blocks x threads stays below 2^31
  const int64_t pmax = (((int64_t(1) << 31) / 512 - 8) / ntb) * PB;
  if (pmax < PB) return hipErrorInvalidValue;
  for (int64_t s = 0; s < p; s += pmax) {
    const int64_t pc = p - s < pmax ? p - s : pmax;
    const int64_t npb = (pc + PB - 1) / PB, nblk = npb * ntb;
    hipLaunchKernelGGL((k_xcf_even<N, ST, PB, SPLIT, DISC>), dim3((unsigned)((nblk + 7) / 8 * 8)), dim3(512), 0,
                       stream, (const cf*)spec_p + s * L::SPEC, pc, (const cf*)spec_l, l, npb, nblk, max_shift, frag,
                       scores + s * l);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Patterns per block: as many as the registers of two waves per SIMD hold.  Split 2 / 3 / 4 patterns: 2.72 /
// 3.00 / 2.56e8 pairs/s at 128 (before its half chunk; with it 3 take 3.35), 0.98 / 1.07 / 0.92e8 at 256 (four
// spill); FP32 2 / 4 / 5: 1.85 / 1.99 / 1.93e8 and 0.66 / 0.72 / 0.68e8.  Two tiles of shifts (16 <= max_shift) take a quarter as many accumulators' patterns: one.
// Few blocks: a CU runs one at a time, so a search takes ceil(blocks / CUs) rounds, and what counts is rounds times
// the time of a block.  Split blocks of 1 / 2 / 3 patterns take about 1 / 1.75 / 2.5 (64 to 160) or 1 / 1.35 / 1.75
// (256): 16 patterns x 500 templates (1,008 / 504 / 378 blocks) 40 / 36 / 45 us at 128, 59 / 49 / 61 at 160, 128 / 91 /
// 113 at 256; 4 x 1,000 (500 / 250 / 250) 40 / 31 / 38 at 160, 75 / 58 / 69 at 256; 40 x 500 (2,520 / 1,260 / 882) 82 /
// 76 / 82, 125 / 106 / 117, 302 / 210 / 219; 100 x 1,000 354 / 341 / 320, 555 / 485 / 466, 1,438 / 1,010 / 900.
// FP32 in blocks of four: one where these would leave CUs without one, as a block works out all of its patterns'
// places: 4 patterns x 200 templates 63 -> 29 us at 128, 63 -> 30 at 160, 176 -> 66 at 256, x 1,000 (125 blocks of
// four) 64 -> 42, 64 -> 44, 177 -> 113; 16 x 500 (252) 64 -> 68, 64 -> 71, 177 -> 197.
template <bool SPLIT, int ST>
constexpr int even_pb() { return ST == 2 ? 1 : SPLIT ? 3 : 4; }
template <int N, bool SPLIT, bool DISC>
hipError_t pick_even(const float2* spec_p, int64_t p, const float2* spec_l, int64_t l, int max_shift,
                     unsigned char* frag, float* scores, hipStream_t stream) {
  if (max_shift >= 16)
    return run_even<N, 2, even_pb<SPLIT, 2>(), SPLIT, DISC>(spec_p, p, spec_l, l, max_shift, frag, scores, stream);
  constexpr int PB = even_pb<SPLIT, 1>();
  const int64_t ntb = (l + 7) / 8;
  if constexpr (SPLIT) {
    const auto rounds = [p, ntb](int pb) { return ((p + pb - 1) / pb * ntb + 255) / 256; };
    const int64_t one = 20 * rounds(1), two = (N == 256 ? 27 : 35) * rounds(2), three = (N == 256 ? 35 : 50) * rounds(3);
    if (p > 1 && two < three && two < one)
      return run_even<N, 1, 2, SPLIT, DISC>(spec_p, p, spec_l, l, max_shift, frag, scores, stream);
    if (p > 1 && three <= one)
      return run_even<N, 1, PB, SPLIT, DISC>(spec_p, p, spec_l, l, max_shift, frag, scores, stream);
    return run_even<N, 1, 1, SPLIT, DISC>(spec_p, p, spec_l, l, max_shift, frag, scores, stream);
  } else {
    if ((p + PB - 1) / PB * ntb <= 192 || p == 1)
      return run_even<N, 1, 1, SPLIT, DISC>(spec_p, p, spec_l, l, max_shift, frag, scores, stream);
    return run_even<N, 1, PB, SPLIT, DISC>(spec_p, p, spec_l, l, max_shift, frag, scores, stream);
  }
}

template <int N, int ST, bool SPLIT>
hipError_t run_lists(const float2* spec_p, int64_t max_items, const float2* spec_l, int64_t lib_n, int64_t row,
                     const int32_t* cand, const int32_t* count, const int2* items, int* queue, int max_shift,
                     unsigned char* frag, bool consts, float* scores, hipStream_t stream) {
  using L = EvenLay<N, ST, true>;
  if (consts)
    hipLaunchKernelGGL((k_even_consts<N, ST, SPLIT, true>), dim3((L::FRAG_BYTES / 4 + 255) / 256), dim3(256), 0,
                       stream, frag);
  hipLaunchKernelGGL((k_xcf_even_lists<N, ST, SPLIT>),
                     dim3((unsigned)(max_items < kListBlocks ? max_items : kListBlocks)), dim3(512), 0, stream,
                     (const cf*)spec_p, (const cf*)spec_l, lib_n, row, cand, count, items, queue, max_shift, frag,
                     scores);
  return hipGetLastError();
}

template <int N, int ST, int PB, bool SPLIT>
hipError_t run_rows(const float2* spec_p, int64_t most, const int32_t* rows, const float2* spec_l, int64_t l,
                    int* queue, int max_shift, const unsigned char* frag, float* scores, hipStream_t stream) {
  const int64_t tiles = (most + PB - 1) / PB * ((l + 7) / 8);
  if (tiles > 0x7ffffff0LL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_xcf_even_rows<N, ST, PB, SPLIT>), dim3((unsigned)(tiles < kListBlocks ? tiles : kListBlocks)),
                     dim3(512), 0, stream, (const cf*)spec_p, rows, (const cf*)spec_l, l, queue, max_shift, frag,
                     scores);
  return hipGetLastError();
}

}  // namespace

#define EBSD_EVEN_SIZES(X) X(64) X(96) X(128) X(160) X(256)

bool even_supported(int n, int max_shift) {
  return band_of(n) > 0 && max_shift >= 0 && max_shift <= 31 && 2 * max_shift < n;
}

size_t even_frag_bytes(int n, int max_shift) {
#define EBSD_EB(NN) \
  if (n == NN) return max_shift < 16 ? EvenLay<NN, 1, false>::FRAG_BYTES : EvenLay<NN, 2, false>::FRAG_BYTES;
  EBSD_EVEN_SIZES(EBSD_EB)
#undef EBSD_EB
  return 0;
}

hipError_t launch_xcf_even(int n, bool split, bool disc, const float2* spec_p, int64_t p, const float2* spec_l,
                           int64_t l, int max_shift, void* frag_v, float* scores, hipStream_t stream) {
  if (p <= 0 || l <= 0) return hipSuccess;
  if (!even_supported(n, max_shift)) return hipErrorInvalidValue;
  unsigned char* frag = static_cast<unsigned char*>(frag_v);
  // the shortcuts for the disc exist at 128 and 256 only (B = 48, 96)
#define EBSD_EL(NN)                                                                                      \
  if (n == NN) {                                                                                         \
    if (split) return pick_even<NN, true, true>(spec_p, p, spec_l, l, max_shift, frag, scores, stream);  \
    return disc || Plan<NN>::B % 16 != 0                                                                 \
               ? pick_even<NN, false, true>(spec_p, p, spec_l, l, max_shift, frag, scores, stream)       \
               : pick_even<NN, false, Plan<NN>::B % 16 != 0>(spec_p, p, spec_l, l, max_shift, frag,      \
                                                             scores, stream);                            \
  }
  EBSD_EVEN_SIZES(EBSD_EL)
#undef EBSD_EL
  return hipErrorInvalidValue;
}

hipError_t launch_xcf_even_lists(int n, bool split, const float2* spec_p, int64_t max_items, const float2* spec_l,
                                 int64_t lib_n, int64_t row, const int32_t* cand, const int32_t* count,
                                 const int2* items, int* queue, int max_shift, void* frag_v, bool consts,
                                 float* scores, hipStream_t stream) {
  if (max_items <= 0) return hipSuccess;
  if (!even_supported(n, max_shift)) return hipErrorInvalidValue;
  unsigned char* frag = static_cast<unsigned char*>(frag_v);
#define EBSD_EL(NN)                                                                                                 \
  if (n == NN) {                                                                                                    \
    const auto run = [&](auto f) {                                                                                  \
      return f(spec_p, max_items, spec_l, lib_n, row, cand, count, items, queue, max_shift, frag, consts, scores,   \
               stream);                                                                                             \
    };                                                                                                              \
    if (max_shift >= 16) return split ? run(run_lists<NN, 2, true>) : run(run_lists<NN, 2, false>);                 \
    return split ? run(run_lists<NN, 1, true>) : run(run_lists<NN, 1, false>);                                      \
  }
  EBSD_EVEN_SIZES(EBSD_EL)
#undef EBSD_EL
  return hipErrorInvalidValue;
}

hipError_t launch_xcf_even_rows(int n, bool split, const float2* spec_p, int64_t most, const int32_t* rows,
                                const float2* spec_l, int64_t l, int* queue, int max_shift, const void* frag_v,
                                float* scores, hipStream_t stream) {
  if (most <= 0 || l <= 0) return hipSuccess;
  if (!even_supported(n, max_shift)) return hipErrorInvalidValue;
  const unsigned char* frag = static_cast<const unsigned char*>(frag_v);
#define EBSD_EL(NN)                                                                                              \
  if (n == NN) {                                                                                                 \
    const auto run = [&](auto f) { return f(spec_p, most, rows, spec_l, l, queue, max_shift, frag, scores, stream); }; \
    if (max_shift >= 16)                                                                                         \
      return split ? run(run_rows<NN, 2, even_pb<true, 2>(), true>) : run(run_rows<NN, 2, even_pb<false, 2>(), false>); \
    return split ? run(run_rows<NN, 1, even_pb<true, 1>(), true>) : run(run_rows<NN, 1, even_pb<false, 1>(), false>); \
  }
  EBSD_EVEN_SIZES(EBSD_EL)
#undef EBSD_EL
  return hipErrorInvalidValue;
}

}  // namespace ebsd
