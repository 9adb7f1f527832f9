// Sub-pixel peak of the correlation (gfx950): the largest rho on the grid
//   s = c + (a, b) / kappa,  |a|, |b| <= m = ceil(0.75 kappa),
// around the integer peak c = (x0, y0), by the single-step matrix DFT (Equation 5 and the peak
// upsampling of section "Fast Fourier Transform"); ties to the smallest (b, a) in row-major order.
//
// The grid has (2m + 1)^2 points (22,801 at kappa = 100), but rho is smooth and only the points near
// its top can win.  One block per pair:
//  1  rho at every st-th point, st = ceil(m / 15) (31 x 31 points), with the +-u and +-s symmetries
//     (k_xcf_even.hip) on v_mfma_f32_16x16x4_f32; with it S = sum w |Z| and
//     K = sum w |Z| (2 pi / N)^2 (u^2 + v^2), which bounds |rho_xx| + |rho_yy| everywhere.
//  2  A bilinear interpolant of a cell's corners is off by at most h^2 / 8 (|rho_xx| + |rho_yy|),
//     h = st / kappa px, and never above its largest corner; so a grid point in a cell whose corners
//     all lie below max - K h^2 / 8 (less the rounding of both evaluations, a bound of nk + nv + 16
//     FP32 roundings of S each) is below the coarse maximum and cannot win.  The rows and columns that
//     the remaining cells span are kept: about 11 x 11 points for a clear peak.
//  3  rho at the kept points, in the order of operations of the full-grid evaluation
//     (k_grid_peak.hip), whose values and winner these are bit for bit.  Where the bound excludes
//     nothing (zero spectra, values that are not finite) every point is kept.
// About a tenth of the full grid's multiply-adds; what bounds it now is latency: three phases of a few
// microseconds behind barriers, two blocks per CU.  5,000 pairs at 128, kappa = 100: 0.29 ms (the full grid, one
// block of 1,024 threads per pair: 1.38 ms), at 160 0.43 (1.72), at 64 0.15 (0.64), 1,000 at 256 0.27 (0.76);
// one pair at 128 with its tables 32 us (80).
#include "ebsd_common.hpp"
#include "ebsd_internal.hpp"

#include <math.h>

namespace ebsd {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

template <int N>
struct SubLay {
  static constexpr int B = Plan<N>::B, NV = B + 1, NK = 2 * B + 1, SPEC = NV * NK;
  static constexpr int KC = (B + 32) / 32, VT = (NV + 15) / 16;  // chunks of 32 rows u >= 0, tiles of 16 columns
};

int sub_m(int kappa) { return (3 * kappa + 3) / 4; }
int sub_stride(int m) { return (m + 14) / 15; }
// float2 entries before the constants of the coarse evaluation (16-byte aligned)
int sub_offset(int n, int kappa) { return (grid_table_size(n, kappa, sub_m(kappa)) + 1) & ~1; }

// The full grid's tables (grid_table_entry), then the constants of the coarse evaluation: stage 1
// [KC][cos, sin][2][64 lanes][4] (row u = 32 kc + 8 (lane / 16) + 4 h + i, shift j st / kappa, j = lane % 16),
// stage 2 [VT][w cos, w sin][64 lanes][4] (column v = 16 vt + 4 (lane / 16) + i)
template <int N>
__global__ void k_subpixel_tables(int kappa, int m, int st, int total, float2* __restrict__ tab,
                                  float* __restrict__ out) {
  using L = SubLay<N>;
  constexpr int nw = L::KC * 1024;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < total) {
    tab[t] = grid_table_entry(t, N, L::B, kappa, m);
    return;
  }
  const int i = t - total;
  if (i >= nw + L::VT * 512) return;
  const bool first = i < nw;
  const int c = first ? i : i - nw;
  const int e = c & 3, lane = (c >> 2) & 63, rest = c >> 8;
  const int part = first ? (rest >> 1) & 1 : rest & 1;
  const int f = first ? (rest >> 2) * 32 + 8 * (lane >> 4) + 4 * (rest & 1) + e : (rest >> 1) * 16 + 4 * (lane >> 4) + e;
  double val = 0.0;
  if (f <= L::B) {
    double sn, cs;
    sincospi(2.0 * (double)(f * (lane & 15) * st) / ((double)kappa * N), &sn, &cs);
    val = part ? sn : cs;
    if (!first && f > 0) val *= 2.0;
  }
  out[i] = (float)val;
}

__device__ __forceinline__ int wrap_index(int k, int n) {
  int r = k % n;
  return r < 0 ? r + n : r;
}

template <int N>
__global__ __launch_bounds__(512, 4) void k_subpixel(const cf* __restrict__ spec_p, const cf* __restrict__ spec_l,
                                                     const int32_t* __restrict__ pi, const int32_t* __restrict__ li,
                                                     const int32_t* __restrict__ centre, int kappa, int m, int st,
                                                     const cf* __restrict__ tab, const float* __restrict__ coarse,
                                                     float* __restrict__ h_out, float* __restrict__ s_out) {
  using L = SubLay<N>;
  constexpr int B = L::B, NV = L::NV, NK = L::NK, VJ = (NV + 63) / 64;
  constexpr int UC = N > 160 ? 16 : 32, EL = (UC * NV + 511) / 512;  // rows of Z' per step, values per thread
  __shared__ union {
    float part[8][16][64];  // the waves' coarse sums
    struct {
      cf zc[UC * NV];  // rows of Z'
      cf fc[UC * 16];  // the same rows of F1, 16 shifts
    } s;
  } u1;
  __shared__ cf g[16 * NV];  // rows of G'
  __shared__ cf rn[N];
  __shared__ float grid[31 * 31];
  __shared__ float red[3][8];
  __shared__ int redi[8], box[4];  // first and last kept coarse cell along y, along x
  const int msz = 2 * m + 1;
  const cf* F1 = tab;
  const cf* F2 = tab + NK * msz;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t k = blockIdx.x;
  const cf* E = spec_p + (pi ? (int64_t)pi[k] : k) * L::SPEC;
  const cf* T = spec_l + (li ? (int64_t)li[k] : k) * L::SPEC;
  const int x0 = centre[2 * k], y0 = centre[2 * k + 1];
  for (int i = tid; i < N; i += 512) rn[i] = tab[(NK + NV) * msz + i];
  if (tid < 4) box[tid] = tid & 1 ? -1 : 30;
  __syncthreads();

  // 1: coarse grid; wave w takes the (column tile, row chunk) units w, w + 8, ...
  float sabs = 0.0f, kabs = 0.0f;
  f4 p[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) p[c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int unit = wave; unit < L::KC * L::VT; unit += 8) {
    const int vt = unit / L::KC, kc = unit - vt * L::KC;
    const int v = vt * 16 + r16, vc = min(v, B), u0 = kc * 32 + 8 * q4;
    const cf vph = rn[wrap_index(vc * x0, N)];
    const float wv = v > B ? 0.0f : (v == 0 ? 1.0f : 2.0f);
    cf ep[8], en[8], tp[8], tn[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int up = min(u0 + j, B) * NV + vc, un = (NK - min(max(u0 + j, 1), B)) * NV + vc;
      ep[j] = E[up];
      tp[j] = T[up];
      en[j] = E[un];
      tn[j] = T[un];
    }
    f4 acc[4], w[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      acc[c] = f4{0.f, 0.f, 0.f, 0.f};
      w[c] = reinterpret_cast<const f4*>(coarse)[(kc * 4 + c) * 64 + lane];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int u = u0 + j;
      const cf uph = rn[wrap_index(u * y0, N)];
      const cf zp = cmul(cmulc(ep[j], tp[j]), cmul(vph, uph));
      cf zm = cmul(cmulc(en[j], tn[j]), cmulc(vph, uph));
      if (u == 0) zm = cf{0.f, 0.f};  // there is no row of u = -0
      const float az = (u > B ? 0.0f : wv) * (sqrtf(zp.x * zp.x + zp.y * zp.y) + sqrtf(zm.x * zm.x + zm.y * zm.y));
      sabs += az;
      kabs = __fmaf_rn(az, (float)(u * u + v * v), kabs);
      const float x[4] = {zp.x + zm.x, zp.y + zm.y, zp.x - zm.x, zp.y - zm.y};
#pragma unroll
      for (int c = 0; c < 4; ++c)
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[c], w[(c & 2) + j / 4][j & 3], acc[c], 0, 0, 0);
    }
    const f4* cw = reinterpret_cast<const f4*>(coarse) + L::KC * 256 + vt * 128 + lane;
    const f4 cc = cw[0], cs = cw[64];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(cc[i], acc[0][i], p[0], 0, 0, 0);  // cos C re
      p[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(cc[i], acc[3][i], p[1], 0, 0, 0);  // cos S im
      p[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs[i], acc[1][i], p[2], 0, 0, 0);  // sin C im
      p[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs[i], acc[2][i], p[3], 0, 0, 0);  // sin S re
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) u1.part[wave][4 * c + i][lane] = p[c][i];
  sabs = wave_sum(sabs);
  kabs = wave_sum(kabs);
  if (lane == 0) {
    red[0][wave] = sabs;
    red[1][wave] = kabs;
  }
  __syncthreads();
  float top = -INFINITY;
  if (tid < 256) {
    const int y = tid & 15, x = tid >> 4, at = (x >> 2) * 16 + y, i = x & 3;
    float t[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      t[c] = 0.0f;
#pragma unroll
      for (int w = 0; w < 8; ++w) t[c] += u1.part[w][4 * c + i][at];
    }
    const float a = t[0] - t[1], b = t[0] + t[1], c = t[2] + t[3], d = t[2] - t[3];
    grid[(15 + y) * 31 + 15 + x] = a - c;
    grid[(15 + y) * 31 + 15 - x] = a + c;
    grid[(15 - y) * 31 + 15 + x] = b - d;
    grid[(15 - y) * 31 + 15 - x] = b + d;
    if (x * st <= m && y * st <= m) top = fmaxf(a + fabsf(c), b + fabsf(d));
  }
  top = wave_max(top);
  if (lane == 0) red[2][wave] = top;
  __syncthreads();
  // 2: the cells that can hold the winner
  sabs = kabs = 0.0f;
  top = -INFINITY;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    sabs += red[0][w];
    kabs += red[1][w];
    top = fmaxf(top, red[2][w]);
  }
  const float h = (float)st / (float)kappa, tpn = 6.2831855f / (float)N;
  const float floor_ = top - (1.01f * 0.125f * h * h * tpn * tpn * kabs + (float)(2 * (NK + NV + 16)) * 6.0e-8f * sabs);
  const bool finite = fabsf(floor_) < INFINITY;
  for (int c = tid; c < 900; c += 512) {
    const int i = c / 30, j = c - i * 30;
    const float* q = grid + i * 31 + j;
    if (fmaxf(fmaxf(q[0], q[1]), fmaxf(q[31], q[32])) >= floor_) {
      atomicMin(&box[0], i);
      atomicMax(&box[1], i);
      atomicMin(&box[2], j);
      atomicMax(&box[3], j);
    }
  }
  __syncthreads();
  const bool all = !finite || box[1] < 0;
  const int b_lo = all ? 0 : max(0, m + (box[0] - 15) * st), b_hi = all ? msz - 1 : min(msz - 1, m + (box[1] - 14) * st);
  const int a_lo = all ? 0 : max(0, m + (box[2] - 15) * st), a_hi = all ? msz - 1 : min(msz - 1, m + (box[3] - 14) * st);
  const int na = a_hi - a_lo + 1;

  // 3: the kept points, 16 rows at a time; wave w holds rows w and w + 8, lane = column v
  float best = -INFINITY;
  int bi = 0x7fffffff;
#pragma unroll 1
  for (int b0 = b_lo; b0 <= b_hi; b0 += 16) {
    cf acc[2][VJ];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < VJ; ++j) acc[i][j] = cf{0.f, 0.f};
    // the next step's values are loaded while the current ones are used
    cf ev[EL], tv[EL], fv;
    auto load = [&](int u0) {
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        const int e = min(u0 * NV + tid + 512 * i, L::SPEC - 1);
        ev[i] = E[e];
        tv[i] = T[e];
      }
      fv = F1[min(u0 + (tid >> 4), NK - 1) * msz + min(b0 + (tid & 15), msz - 1)];
    };
    load(0);
#pragma unroll 1
    for (int u0 = 0; u0 < NK; u0 += UC) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < EL; ++i) {
        const int t = tid + 512 * i, kk = u0 + t / NV;
        const int u = kk <= B ? kk : kk - NK;
        if (t < UC * NV) u1.s.zc[t] = cmul(cmulc(ev[i], tv[i]), rn[wrap_index(u * y0, N)]);
      }
      if (tid < UC * 16) u1.s.fc[tid] = fv;
      __syncthreads();
      if (u0 + UC < NK) load(u0 + UC);
      const int uc = min(UC, NK - u0);
#pragma unroll 4
      for (int uu = 0; uu < uc; ++uu) {
        const cf f1 = u1.s.fc[uu * 16 + wave], f2 = u1.s.fc[uu * 16 + wave + 8];
#pragma unroll
        for (int j = 0; j < VJ; ++j) {
          const cf z = u1.s.zc[uu * NV + min(lane + 64 * j, B)];
          acc[0][j].x = __fmaf_rn(f1.x, z.x, __fmaf_rn(-f1.y, z.y, acc[0][j].x));
          acc[0][j].y = __fmaf_rn(f1.x, z.y, __fmaf_rn(f1.y, z.x, acc[0][j].y));
          acc[1][j].x = __fmaf_rn(f2.x, z.x, __fmaf_rn(-f2.y, z.y, acc[1][j].x));
          acc[1][j].y = __fmaf_rn(f2.x, z.y, __fmaf_rn(f2.y, z.x, acc[1][j].y));
        }
      }
    }
#pragma unroll
    for (int j = 0; j < VJ; ++j) {
      const int v = lane + 64 * j;
      if (v < NV) {
        const cf w = cscale(rn[wrap_index(v * x0, N)], v == 0 ? 1.0f : 2.0f);
        g[wave * NV + v] = cmul(acc[0][j], w);
        g[(wave + 8) * NV + v] = cmul(acc[1][j], w);
      }
    }
    __syncthreads();
    const int nb = min(16, b_hi - b0 + 1);
    for (int t = tid; t < nb * na; t += 512) {
      const int r = t / na, a = a_lo + t - r * na;
      const cf* gr = g + r * NV;
      float rho = 0.0f;
#pragma unroll 8
      for (int v = 0; v < NV; ++v) {
        const cf f = F2[v * msz + a];
        rho = __fmaf_rn(gr[v].x, f.x, __fmaf_rn(-gr[v].y, f.y, rho));
      }
      argmax_merge(best, bi, rho, (b0 + r) * msz + a);
    }
  }
  wave_argmax(best, bi);
  if (lane == 0) {
    red[0][wave] = best;
    redi[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 8; ++w) argmax_merge(best, bi, red[0][w], redi[w]);
    if (bi < 0 || bi >= msz * msz) bi = m * msz + m;  // every value NaN
    const int db = bi / msz - m, da = bi - (bi / msz) * msz - m;
    h_out[k] = best;
    s_out[2 * k] = (float)x0 + (float)da / (float)kappa;
    s_out[2 * k + 1] = (float)y0 + (float)db / (float)kappa;
  }
}

}  // namespace

#define EBSD_SUB_SIZES(X) X(64) X(96) X(128) X(160) X(256)

int subpixel_table_size(int n, int kappa) {
  int more = 0;
#define EBSD_SB(NN) \
  if (n == NN) more = SubLay<NN>::KC * 512 + SubLay<NN>::VT * 256;
  EBSD_SUB_SIZES(EBSD_SB)
#undef EBSD_SB
  return sub_offset(n, kappa) + more;
}

// Small grids of many pairs cost less in full (k_grid_peak.hip, the same values and winners), whose small blocks
// share a CU: 5,000 pairs, full / bounded, at kappa = 4 (7 x 7 points) 65 / 145 us at 64, 92 / 200 at 96, 139 / 266
// at 128, 175 / 308 at 160, 1,500 at 256 146 / 338; at kappa = 20 (31 x 31) 90 / 147, 130 / 202, 197 / 270, 282 /
// 314, 261 / 343; at 30 (47 x 47) 118 / 149, 179 / 202, 280 / 270, 389 / 314, 424 / 378.  Few pairs leave the
// bounded form's blocks (512 at a time, 256 at 256) no second round: 512 pairs at 128 cost it 39 us up to kappa =
// 40, in full 38 at 4 and 46 at 20; 600 pairs 53, and 39 at 4; 512 pairs at 256 120 us at 20, 164 at 40, in full 112
// and 153.
static bool full_grid_pays(int n, int m, int64_t k) {
  const int rows = 2 * m + 1;
  if (n == 256) return k > 256 && rows <= (k <= 512 ? 64 : 40);
  return k > 512 && rows <= (k <= 2048 || n == 160 ? 32 : n == 128 ? 40 : 48);
}

// The full grid's evaluation in LDS, which bounds the accepted upsampling factors
size_t subpixel_lds_bytes(int n, int kappa) { return grid_lds_bytes(n, sub_m(kappa)); }

hipError_t launch_subpixel_tables(int n, int kappa, float2* tab, hipStream_t stream) {
  const int m = sub_m(kappa), total = grid_table_size(n, kappa, m);
  float* coarse = reinterpret_cast<float*>(tab + sub_offset(n, kappa));
#define EBSD_SB(NN)                                                                                             \
  if (n == NN) {                                                                                                \
    const int all = total + SubLay<NN>::KC * 1024 + SubLay<NN>::VT * 512;                                      \
    hipLaunchKernelGGL(k_subpixel_tables<NN>, dim3((all + 255) / 256), dim3(256), 0, stream, kappa, m,         \
                       sub_stride(m), total, tab, coarse);                                                      \
    return hipGetLastError();                                                                                   \
  }
  EBSD_SUB_SIZES(EBSD_SB)
#undef EBSD_SB
  return hipErrorInvalidValue;
}

hipError_t launch_subpixel(int n, const float2* spec_p, const float2* spec_l, const int32_t* pi, const int32_t* li,
                           int64_t k, const int32_t* s_int, int kappa, const float2* tab, float* h_sub,
                           float* s_sub, hipStream_t stream) {
  if (k <= 0) return hipSuccess;
  const int bnd = band_of(n), m = sub_m(kappa);
  if (bnd < 0 || subpixel_lds_bytes(n, kappa) > 160 * 1024) return hipErrorInvalidValue;
  if (full_grid_pays(n, m, k))
    return launch_grid(n, spec_p, spec_l, pi, li, k, s_int, kappa, m, 0, tab, h_sub, s_sub, nullptr, stream);
  const int64_t sc = (int64_t)(bnd + 1) * (2 * bnd + 1);
  const int64_t kmax = (int64_t(1) << 31) / 512;  // blocks x threads of one dispatch below 2^31
  const float* coarse = reinterpret_cast<const float*>(tab + sub_offset(n, kappa));
  for (int64_t s = 0; s < k; s += kmax) {
    const int64_t kc = k - s < kmax ? k - s : kmax;
    const cf* sp = (const cf*)(pi ? spec_p : spec_p + s * sc);
    const cf* sl = (const cf*)(li ? spec_l : spec_l + s * sc);
#define EBSD_SB(NN)                                                                                              \
  if (n == NN)                                                                                                   \
    hipLaunchKernelGGL(k_subpixel<NN>, dim3((unsigned)kc), dim3(512), 0, stream, sp, sl, pi ? pi + s : nullptr,  \
                       li ? li + s : nullptr, s_int + 2 * s, kappa, m, sub_stride(m), (const cf*)tab, coarse,    \
                       h_sub + s, s_sub + 2 * s);
    EBSD_SUB_SIZES(EBSD_SB)
#undef EBSD_SB
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ebsd
