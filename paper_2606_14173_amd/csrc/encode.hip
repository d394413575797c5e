// Phase-only encoding on gfx950: Adam on the SLM phase under complex-amplitude
// supervision on one plane with a phase-shift-invariant scale factor (the
// paper's hologram encoding, Sec. 2 and Sec. 5.3). Per field and step:
//   A = P_z exp(i phi)          k_enc_rows_phase, k_fft_columns, k_enc_ifft_dots
//   s = <V, A> / <V, V>, L = ||A - s V||^2          the dots above, k_enc_scale
//   G = P_{-z} (A - s V)        k_enc_rows_residual, k_fft_columns, k_enc_ifft_adam
//   g = 2 Im(G conj(exp(i phi))); Adam                        the same kernel,
//                               which also starts the next step's A
// The elementwise work runs in the first and last passes of the two
// propagations (asm.hip), on values that are in registers there: exp(i phi)
// is formed from phi where it is read (twice a step) instead of being kept,
// the residual and G are never stored, and A is written once for the
// residual. Fields are [n][h][w] complex64; phases and Adam moments
// [n][h][w] float32; the dot products accumulate in FP64 in a fixed order
// (deterministic).
#include <hip/hip_runtime.h>

#include "asm.hpp"
#include "encode.hpp"
#include "fft.hpp"

namespace hpt {
namespace {

using namespace fft;

constexpr int kEncBlock = 256;

__global__ void __launch_bounds__(kEncBlock) k_enc_init(const float2 *U, float *phi, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float2 u = U[i];
  phi[i] = (u.x == 0.f && u.y == 0.f) ? 0.f : atan2f(u.y, u.x);
}

// Row spectrum of v (v[q], q < E/2: elements t + q TPL) -> row y of field
// blockIdx.y of A [nf][h][Px].
template <int LG, bool TILED>
__device__ __forceinline__ void forward_row(C2 (&v)[Line<LG>::E], float2 *A, uint32_t y, uint32_t h, const float2 *tw,
                                            C2 *lds) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  const uint32_t t = Lines::pos();
  line_fft<LG, false, true, Lines::kStride, Lines::kWave, false>(v, Lines::lds_of(lds), TableTwiddles{tw}, t);
  if (y >= h) return;
  const uint32_t first = Lines::first_of(t, y, h);
  float2 *dst = A + (size_t)blockIdx.y * h * L::N;
#pragma unroll
  for (uint32_t q = 0; q < L::E; ++q) Lines::elem(dst, first, h, q) = make_float2(v[q].x, v[q].y);
}

// Row spectra of the rows [nrows][w] that `elem(i)` gives (i: element of the
// array) -> A [nrows][Px]; grid (rows, fields).
template <int LG, bool TILED, class F>
__device__ __forceinline__ void rows_of(float2 *A, uint32_t w, uint32_t h, const float2 *tw, C2 *lds, F &&elem) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  const uint32_t t = Lines::pos(), y = Lines::group(gridDim.x) * Lines::kLines + Lines::line();
  const size_t row = (size_t)blockIdx.y * h + y;
  C2 v[L::E];
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) {
    const uint32_t i = t + q * L::TPL;
    v[q] = y < h && i < w ? elem(row * w + i) : c2(0.f, 0.f);
  }
  forward_row<LG, TILED>(v, A, y, h, tw, lds);
}

template <int LG, bool TILED>
__global__ void __launch_bounds__((Rows<LG, TILED>::W))
    k_enc_rows_phase(const float *phi, float2 *A, uint32_t w, uint32_t h, const float2 *tw) {
  __shared__ C2 lds[Rows<LG, TILED>::kLdsElems];
  rows_of<LG, TILED>(A, w, h, tw, lds, [&](size_t i) {
    float sn, cs;
    sincosf(phi[i], &sn, &cs);
    return c2(cs, sn);
  });
}

template <int LG, bool TILED>
__global__ void __launch_bounds__((Rows<LG, TILED>::W))
    k_enc_rows_residual(const float2 *R, const float2 *V, const double2 *s, float2 *A, uint32_t w, uint32_t h,
                        const float2 *tw) {
  __shared__ C2 lds[Rows<LG, TILED>::kLdsElems];
  const double2 sf = s[blockIdx.y];
  const float sr = (float)sf.x, si = (float)sf.y;
  rows_of<LG, TILED>(A, w, h, tw, lds, [&](size_t i) {
    const float2 v = V[i], x = R[i];
    return c2(x.x - (sr * v.x - si * v.y), x.y - (sr * v.y + si * v.x));
  });
}

// Inverse FFT of row y of field blockIdx.y of A [nf][h][Px] (tiled), scaled: v[q], q <
// E/2, hold elements t + q TPL (of which the first w are wanted).
template <int LG, bool TILED>
__device__ __forceinline__ void inverse_row(C2 (&v)[Line<LG>::E], const float2 *A, uint32_t y, uint32_t h,
                                            float scale, const float2 *tw, C2 *lds) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  const uint32_t l = Lines::line(), t = Lines::pos();
  const uint32_t first = Lines::first_of(t, y, h);
  const float2 *src = A + (size_t)blockIdx.y * h * L::N;
#pragma unroll
  for (uint32_t q = 0; q < L::E; ++q) {
    const float2 g = y < h ? Lines::elem(src, first, h, q) : make_float2(0.f, 0.f);
    v[q] = c2(g.x, g.y);
  }
  line_fft<LG, true, false, Lines::kStride, Lines::kWave, false>(v, Lines::lds_of(lds), TableTwiddles{tw}, t);
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) v[q] = c2(v[q].x * scale, v[q].y * scale);
}

// R = the inverse row transforms of A; partial sums of conj(V) R (re, im) and
// |R|^2 over the workgroup's rows, in FP64 -> part[(f gridDim.x + group) 3 + k].
// SELF: R is V, and only |R|^2 is wanted (the others are 0).
template <int LG, bool TILED, bool SELF>
__global__ void __launch_bounds__((Rows<LG, TILED>::W)) k_enc_ifft_dots(const float2 *A, float2 *R, const float2 *V,
                                                               double *part, uint32_t w, uint32_t h, float scale,
                                                               const float2 *tw) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  constexpr uint32_t W = Lines::W;
  __shared__ C2 lds[Lines::kLdsElems];
  __shared__ double sums[W / 64][3];
  const uint32_t l = Lines::line(), t = Lines::pos();
  const uint32_t group = Lines::group(gridDim.x), y = group * Lines::kLines + l;
  const size_t row = (size_t)blockIdx.y * h + y;
  const bool ok = y < h;
  C2 v[L::E];
  inverse_row<LG, TILED>(v, A, y, h, scale, tw, lds);
  double dr = 0.0, di = 0.0, aa = 0.0;
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) {
    const uint32_t i = t + q * L::TPL;
    if (ok && i < w) {
      const float2 x = make_float2(v[q].x, v[q].y);
      R[row * w + i] = x;
      if constexpr (!SELF) {
        const float2 u = V[row * w + i];
        dr += (double)u.x * x.x + (double)u.y * x.y;
        di += (double)u.x * x.y - (double)u.y * x.x;
      }
      aa += (double)x.x * x.x + (double)x.y * x.y;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    dr += __shfl_xor(dr, o); di += __shfl_xor(di, o); aa += __shfl_xor(aa, o);
  }
  if (threadIdx.x % 64 == 0) { double *s = sums[threadIdx.x / 64]; s[0] = dr; s[1] = di; s[2] = aa; }
  __syncthreads();
  if (threadIdx.x < 3) {
    double a = 0.0;
    for (uint32_t k = 0; k < W / 64; ++k) a += sums[k][threadIdx.x];
    part[((size_t)blockIdx.y * gridDim.x + group) * 3 + threadIdx.x] = a;
  }
}

// Field blockIdx.x: sum of its nb partials. NORM: vv[f] = <V, V>; else the
// optimal scale s = <V, A> / <V, V> and the relative loss 1 - |<V, A>|^2 /
// (<V, V> <A, A>).
template <bool NORM>
__global__ void __launch_bounds__(kEncBlock) k_enc_scale(const double *part, uint32_t nb, double *vv, double2 *s,
                                                         double *rel) {
  __shared__ double sh[3][kEncBlock];
  const uint32_t f = blockIdx.x, t = threadIdx.x;
  double a[3] = {0.0, 0.0, 0.0};
  for (uint32_t b = t; b < nb; b += kEncBlock)
    for (int k = 0; k < 3; ++k) a[k] += part[((size_t)f * nb + b) * 3 + k];
  for (int k = 0; k < 3; ++k) sh[k][t] = a[k];
  __syncthreads();
  for (uint32_t o = kEncBlock / 2; o > 0; o >>= 1) {
    if (t < o)
      for (int k = 0; k < 3; ++k) sh[k][t] += sh[k][t + o];
    __syncthreads();
  }
  if (t != 0) return;
  const double dr = sh[0][0], di = sh[1][0], aa = sh[2][0];
  if (NORM) { vv[f] = aa; return; }
  const double v = vv[f];
  s[f] = v > 0.0 ? make_double2(dr / v, di / v) : make_double2(0.0, 0.0);
  rel[f] = (v > 0.0 && aa > 0.0) ? 1.0 - (dr * dr + di * di) / (v * aa) : 1.0;
}

// G = the inverse row transforms of A; g = 2 Im(G conj(exp(i phi))); Adam; then
// the row spectra of the new exp(i phi) -> A, which the next step (or the final
// loss) starts with. One kernel for both: the row is in registers, and a step has
// one launch and one reading of phi less (20 steps on 3 fields of 300 x 200 1.07 ->
// 1.015 ms, on 24 of 1920 x 1080 79.7 -> 78.8).
// FIRST: the moments are zero before this step and are not read.
template <int LG, bool TILED, bool FIRST>
__global__ void __launch_bounds__((Rows<LG, TILED>::W))
    k_enc_ifft_adam(float2 *A, float *phi, float *m, float *v2, uint32_t w, uint32_t h, float scale, float lr, float bc1,
                    float bc2, const float2 *tw) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  __shared__ C2 lds[Lines::kLdsElems];
  const uint32_t l = Lines::line(), t = Lines::pos();
  const uint32_t group = Lines::group(gridDim.x), y = group * Lines::kLines + l;
  const size_t row = (size_t)blockIdx.y * h + y;
  const bool ok = y < h;
  C2 v[L::E];
  inverse_row<LG, TILED>(v, A, y, h, scale, tw, lds);
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) {
    const uint32_t x = t + q * L::TPL;
    const C2 G = v[q];
    v[q] = c2(0.f, 0.f);
    if (!ok || x >= w) continue;
    const size_t i = row * w + x;
    const float p0 = phi[i];
    float sn, cs;
    sincosf(p0, &sn, &cs);
    const float g = 2.0f * (G.y * cs - G.x * sn);
    const float m0 = FIRST ? 0.f : m[i], v0 = FIRST ? 0.f : v2[i];
    const float mi = kAdamBeta1 * m0 + (1.0f - kAdamBeta1) * g;
    const float vi = kAdamBeta2 * v0 + (1.0f - kAdamBeta2) * g * g;
    const float p1 = p0 - lr * (mi / bc1) / (sqrtf(vi / bc2) + kAdamEps);
    m[i] = mi;
    v2[i] = vi;
    phi[i] = p1;
    sincosf(p1, &sn, &cs);
    v[q] = c2(cs, sn);
  }
  forward_row<LG, TILED>(v, A, y, h, tw, lds);
}

template <int LG, bool TILED>
dim3 row_grid(uint32_t nf, uint32_t h) { return dim3((h + Rows<LG, TILED>::kLines - 1) / Rows<LG, TILED>::kLines, nf); }

// Rows of w values of h-row fields: f(integral_constant<LG>, bool_constant<TILED>).
template <class F>
hipError_t for_rows(uint32_t w, uint32_t h, F &&f) {
  return with_rows(log2u(asm_padded(w)), asm_tiled(w, h), f) ? hipGetLastError() : hipErrorInvalidValue;
}

float fft_scale(uint32_t w, uint32_t h) { return 1.0f / ((float)asm_padded(w) * (float)asm_padded(h)); }

}  // namespace

uint32_t enc_parts(uint32_t w, uint32_t h) {
  uint32_t n = h;
  (void)for_rows(w, h, [&](auto lg, auto tiled) { n = row_grid<decltype(lg)::value, decltype(tiled)::value>(1, h).x; });
  return n;
}

hipError_t launch_enc_init(const float2 *U, float *phi, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_enc_init, dim3((uint32_t)((n + kEncBlock - 1) / kEncBlock)), dim3(kEncBlock), 0, st, U, phi, n);
  return hipGetLastError();
}

hipError_t launch_enc_target(const float2 *A, float2 *V, double *part, double *vv, const float2 *tw, uint32_t nf,
                             uint32_t w, uint32_t h, hipStream_t st) {
  const float2 *t = tw + 2 * asm_padded(w);
  hipError_t e = for_rows(w, h, [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    const dim3 grid = row_grid<LG, TILED>(nf, h), block(Rows<LG, TILED>::W);
    hipLaunchKernelGGL((k_enc_ifft_dots<LG, TILED, true>), grid, block, 0, st, A, V, nullptr, part,
                       w, h, fft_scale(w, h), t);
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_enc_scale<true>, dim3(nf), dim3(kEncBlock), 0, st, part, enc_parts(w, h), vv, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_enc_rows_phase(const float *phi, float2 *A, const float2 *tw, uint32_t nf, uint32_t w, uint32_t h,
                                 hipStream_t st) {
  return for_rows(w, h, [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    const dim3 grid = row_grid<LG, TILED>(nf, h), block(Rows<LG, TILED>::W);
    hipLaunchKernelGGL((k_enc_rows_phase<LG, TILED>), grid, block, 0, st, phi, A, w, h,
                       tw + 2 * asm_padded(w));
  });
}

hipError_t launch_enc_scale(const float2 *A, float2 *R, const float2 *V, double *part, double *vv, double2 *s,
                            double *rel, const float2 *tw, uint32_t nf, uint32_t w, uint32_t h, hipStream_t st) {
  const float2 *t = tw + 2 * asm_padded(w);
  hipError_t e = for_rows(w, h, [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    const dim3 grid = row_grid<LG, TILED>(nf, h), block(Rows<LG, TILED>::W);
    hipLaunchKernelGGL((k_enc_ifft_dots<LG, TILED, false>), grid, block, 0, st, A, R, V, part, w, h,
                       fft_scale(w, h), t);
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_enc_scale<false>, dim3(nf), dim3(kEncBlock), 0, st, part, enc_parts(w, h), vv, s, rel);
  return hipGetLastError();
}

hipError_t launch_enc_rows_residual(const float2 *R, const float2 *V, const double2 *s, float2 *A, const float2 *tw,
                                    uint32_t nf, uint32_t w, uint32_t h, hipStream_t st) {
  return for_rows(w, h, [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    const dim3 grid = row_grid<LG, TILED>(nf, h), block(Rows<LG, TILED>::W);
    hipLaunchKernelGGL((k_enc_rows_residual<LG, TILED>), grid, block, 0, st, R, V, s, A, w, h,
                       tw + 2 * asm_padded(w));
  });
}

hipError_t launch_enc_adam(float2 *A, float *phi, float *m, float *v, const float2 *tw, uint32_t nf, uint32_t w,
                           uint32_t h, float lr, float bc1, float bc2, bool first, hipStream_t st) {
  const float2 *t = tw + 2 * asm_padded(w);
  return for_rows(w, h, [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    const dim3 grid = row_grid<LG, TILED>(nf, h), block(Rows<LG, TILED>::W);
    if (first)
      hipLaunchKernelGGL((k_enc_ifft_adam<LG, TILED, true>), grid, block, 0, st, A, phi, m, v, w, h,
                         fft_scale(w, h), lr, bc1, bc2, t);
    else
      hipLaunchKernelGGL((k_enc_ifft_adam<LG, TILED, false>), grid, block, 0, st, A, phi, m, v, w, h,
                         fft_scale(w, h), lr, bc1, bc2, t);
  });
}

}  // namespace hpt
