// Filtered spectra at 256 x 256 (same definition as k_spectra in
// k_spectra_xcf.hip: contrast normalisation, Hann window, forward 2-D DFT,
// band-pass cut at rho_max, FP64 energy, unit-energy band layout).  A 256^2
// transform does not fit one block's LDS, so it runs as three passes through
// a global intermediate:
//   rows     two real rows packed as one complex 256-point FFT (16 x 16,
//            one LDS exchange), separated into the Hermitian halves v <= B;
//   columns  one block per image: 256-point FFTs along y, 64 columns at a
//            time, the band kept in registers, FP64 energy, band scaled to
//            unit energy and stored once.
// 5,000 images 2,151 -> 1,156 us (columns and scale 495 + 300 -> 254 us per 2,500, by one pass over the band,
// loads along v and roots from constants; statistics by 16-byte loads), one image 62 -> 35 us.
#include "ebsd_common.hpp"
#include "ebsd_internal.hpp"

#include <math.h>

namespace ebsd {

namespace {
constexpr int N = 256, R = 16, B = Plan<256>::B, NV = B + 1, NK = 2 * B + 1;
constexpr int CW = 64, CR = (NV + CW - 1) / CW;  // columns of a wave, rounds of columns

template <int M>
struct Roots {
  cf w[M];
  constexpr Roots() : w() {
    for (int k = 0; k < M; ++k) {
      w[k].x = (float)cx::cos2pi(k, M);
      w[k].y = (float)cx::sin2pi(k, M);
    }
  }
};
__constant__ Roots<N> c_roots256 = Roots<N>();
}  // namespace

// mean and 1/std of each image (FP64 sums; npix a multiple of 4)
__global__ __launch_bounds__(256) void k_img_stats(const float* __restrict__ imgs, int npix, float2* __restrict__ st) {
  const int64_t k = blockIdx.x;
  const float* img = imgs + k * (int64_t)npix;
  double s1 = 0.0, s2 = 0.0;
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));  // images at any float address
#pragma unroll 4
  for (int i = threadIdx.x; i < npix / 4; i += 256) {
    const f4 x = reinterpret_cast<const f4*>(img)[i];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double v = x[j];
      s1 += v;
      s2 += v * v;
    }
  }
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  __shared__ double red[8];
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = s1;
    red[4 + (threadIdx.x >> 6)] = s2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double mean = (red[0] + red[1] + red[2] + red[3]) / npix;
    const double var = (red[4] + red[5] + red[6] + red[7]) / npix - mean * mean;
    st[k] = make_float2((float)mean, var > 0.0 ? (float)(1.0 / sqrt(var)) : 0.0f);
  }
}

// rows: block (image k, group g) handles row pairs (q, q + 128), q in [16 g, 16 g + 16)
__global__ __launch_bounds__(256) void k_rows256(const float* __restrict__ imgs, const float2* __restrict__ st,
                                                 int window, cf* __restrict__ vout) {
  __shared__ cf ys[16 * 16 * 17];  // [pair][c][b], b padded
  __shared__ cf tw[N];
  __shared__ float win[N];
  const int tid = threadIdx.x;
  const int64_t k = blockIdx.x >> 3;
  const int g = blockIdx.x & 7;
  const float* img = imgs + k * (int64_t)N * N;
  const float mean = st[k].x, istd = st[k].y;
  tw[tid] = c_roots256.w[tid];
  {
    const float s = sinpif(((float)tid + 0.5f) / (float)N);
    win[tid] = window ? s * s : 1.0f;
  }
  __syncthreads();
  const int p = tid >> 4, b = tid & 15;
  const int q = 16 * g + p;
  {
    cf x[R];
    const float w0 = win[q] * istd, w1 = win[q + 128] * istd;
#pragma unroll
    for (int a = 0; a < R; ++a) {
      const int col = R * a + b;
      x[a] = cf{(img[q * N + col] - mean) * w0 * win[col], (img[(q + 128) * N + col] - mean) * w1 * win[col]};
    }
    DFT<R, -1>::run(x);
#pragma unroll
    for (int c = 1; c < R; ++c) x[c] = cmulc(x[c], tw[b * c]);
#pragma unroll
    for (int c = 0; c < R; ++c) ys[(p * 16 + c) * 17 + b] = x[c];
  }
  __syncthreads();
  const int c = tid & 15;
  cf z[R];
#pragma unroll
  for (int bb = 0; bb < R; ++bb) z[bb] = ys[(p * 16 + c) * 17 + bb];
  DFT<R, -1>::run(z);  // Z(v = c + 16 d)
  __syncthreads();
  cf* zs = ys;  // [pair][v], 16 x 256
#pragma unroll
  for (int d = 0; d < R; ++d) zs[p * N + c + R * d] = z[d];
  __syncthreads();
  // separate the packed rows: F_q(v) = (Z(v) + conj Z(-v)) / 2, F_{q+128}(v) = (Z(v) - conj Z(-v)) / 2i
  for (int t = tid; t < 16 * NV; t += 256) {
    const int pp = t / NV, v = t - pp * NV;
    const cf z1 = zs[pp * N + v], z2 = zs[pp * N + ((N - v) & (N - 1))];
    const int qq = 16 * g + pp;
    vout[(k * N + qq) * NV + v] = cf{0.5f * (z1.x + z2.x), 0.5f * (z1.y - z2.y)};
    vout[(k * N + qq + 128) * NV + v] = cf{0.5f * (z1.y + z2.y), -0.5f * (z1.x - z2.x)};
  }
}

// columns: block per image; wave b takes the 16-point transforms over a of rows 16 a + b, lanes along 64 columns v,
// then (after one exchange) those over b for outputs u = b + 16 d.  Both rounds' outputs wait in registers for the
// image's energy, so the band is written once, scaled, and loads and stores run along v.
// Bound by memory (199 KB read, 150 KB written an image).
__global__ __launch_bounds__(1024) void k_cols256(const cf* __restrict__ vin, FilterParams fp, cf* __restrict__ spec,
                                                  double* __restrict__ energy) {
  __shared__ cf ys[R * R * CW];  // [c][b][column]
  __shared__ double red[16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int b = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t k = blockIdx.x;
  const cf* in = vin + k * (int64_t)(N * NV);
  cf* out = spec + k * (int64_t)(NK * NV);
  const float inv2hp = 1.0f / (2.0f * fp.sigma_hp * fp.sigma_hp);
  const float inv2lp = 1.0f / (2.0f * fp.sigma_lp * fp.sigma_lp);
  const float rmax2 = fp.rho_max * fp.rho_max;
  cf z[CR][R];
  double en = 0.0;
#pragma unroll
  for (int r = 0; r < CR; ++r) {
    const int v = CW * r + lane;
    const bool vok = v < NV;
    {
      cf x[R];
#pragma unroll
      for (int a = 0; a < R; ++a) x[a] = vok ? in[(R * a + b) * NV + v] : cf{0.f, 0.f};
      DFT<R, -1>::run(x);
#pragma unroll
      for (int c = 1; c < R; ++c) x[c] = cmulc(x[c], c_roots256.w[(b * c) & (N - 1)]);
      if (r) __syncthreads();
#pragma unroll
      for (int c = 0; c < R; ++c) ys[(c * R + b) * CW + lane] = x[c];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R; ++i) z[r][i] = ys[(b * R + i) * CW + lane];
    DFT<R, -1>::run(z[r]);  // X(u = b + 16 d, v)
#pragma unroll
    for (int d = 0; d < R; ++d) {
      const int u = b + R * d;
      const int us = u >= N / 2 ? u - N : u;
      if (u > B && u < N - B) continue;
      const float r2 = (float)(us * us + v * v);
      float h = 0.0f;
      if (vok && r2 <= rmax2) h = (1.0f - expf(-r2 * inv2hp)) * expf(-r2 * inv2lp);
      const cf zz = cscale(z[r][d], h);
      z[r][d] = zz;
      en += (v == 0 ? 1.0 : 2.0) * ((double)zz.x * zz.x + (double)zz.y * zz.y);
    }
  }
  en = wave_sum(en);
  if (lane == 0) red[b] = en;
  __syncthreads();
  double e = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) e += red[w];
  const float sc = e > 0.0 ? (float)(1.0 / sqrt(e)) : 0.0f;
  if (energy && tid == 0) energy[k] = e;
#pragma unroll
  for (int r = 0; r < CR; ++r) {
    const int v = CW * r + lane;
    if (v >= NV) break;
#pragma unroll
    for (int d = 0; d < R; ++d) {
      const int u = b + R * d;
      if (u > B && u < N - B) continue;
      out[(u <= B ? u : u - N + NK) * NV + v] = cscale(z[r][d], sc);
    }
  }
}

size_t spectra256_scratch_bytes(int64_t k) {
  return (size_t)k * (sizeof(float2) + (size_t)N * NV * sizeof(cf));
}

hipError_t launch_spectra256(const float* imgs, int64_t k, const FilterParams& fp, float2* spec, double* energy,
                             void* scratch, hipStream_t stream) {
  if (k <= 0) return hipSuccess;
  if (k > (int64_t(1) << 31) / (13 * 256)) return hipErrorInvalidValue;  // one dispatch below 2^31 items
  float2* st = (float2*)scratch;
  cf* v = (cf*)((char*)scratch + (size_t)k * sizeof(float2));
  hipLaunchKernelGGL(k_img_stats, dim3((unsigned)k), dim3(256), 0, stream, imgs, N * N, st);
  hipLaunchKernelGGL(k_rows256, dim3((unsigned)(k * 8)), dim3(256), 0, stream, imgs, st, fp.window, v);
  hipLaunchKernelGGL(k_cols256, dim3((unsigned)k), dim3(1024), 0, stream, v, fp, (cf*)spec, energy);
  return hipGetLastError();
}

}  // namespace ebsd
