// Angular-spectrum propagation of recorded fields on gfx950: the second
// stage of the two-stage scheme (Sec. 4.4), which carries the field traced
// onto a wave recording plane to the hologram plane; the angular spectrum is
// the field's Fourier transform (Sec. 3).
//
// Per field [h][w] (complex64), zero-padded to [Py][Px] (powers of two,
// >= 2h, >= 2w), with the field in the top-left corner:
//   k_fft_rows     FFT of the h non-zero rows, length Px       [h][w] -> A [h][Px]
//   k_fft_columns  per column: zero-pad to Py, FFT, multiply by the transfer
//                  function, inverse FFT, keep rows [0, h)     A -> A
//   k_ifft_rows    inverse FFT of each row, keep [0, w), scale 1/(Px Py)
// Transfer function H = exp(+i 2 pi z sqrt(1/lambda^2 - f^2)) on propagating
// frequencies (phase reduced in FP64), optionally band-limited
// (Matsushima and Shimobaba, 2009) and cut by a circular pupil, 0 on
// evanescent ones; k_transfer tabulates it once per call over |f_x|, |f_y|
// (H depends on their squares).
//
// Focal stacks (reconstruction): the row spectra of a set of fields are kept;
// k_fft_columns transforms a column forward once and back once per
// observation plane, and k_ifft_rows_intensity sums |u|^2 over the fields
// instead of writing them.
//
// The line FFTs are in fft.hpp. Row spectra whose columns are long (Py >= 2048)
// lie in tiles of eight columns (asm_tiled): a workgroup of two columns then reads
// neighbouring 64-byte pieces, where in plain order it would use 16 bytes of a
// line of the cache per row, and the row passes take two rows at once. Two
// workgroups of two columns run on a CU, one's memory beside the other's
// arithmetic; one of four in plain order had all its waves wait together.
// What bounds the passes, 24 fields of 1920 x 1080 (4096 x 4096 padded): the
// column pass by vector issue (80 % of the cycles; 46 us a field, 60 with one
// workgroup of four columns, 96 with transposes of 12 us each beside it), the row
// passes by memory (13 and 11 us a field for 52 MB; 11 and 9 in plain order, 26
// while their twiddles were gathered). All together 1.56 ms, in plain order 1.71;
// phase encoding of 1920 x 1080, whose fields exceed the last-level cache, 76.1 ms,
// in plain order 94.8 (tiles of 4 and 16 columns 82 and 84 where 8 took 80); a focal
// stack of five planes of 24 fields 6.17 ms, in plain order 6.93, of which 0.6 by the
// transfer functions' tables (one reading a plane). With short columns the plain
// order is as fast or faster (w x h = 1080 x 200: 0.19 ms, tiled 0.20). Several planes
// in workgroups of two 8.1 ms: each plane's transfer function is then read in
// 16-byte pieces. One workgroup of four a CU issues for 60 % of the cycles.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>

#include "asm.hpp"
#include "fft.hpp"

namespace hpt {
namespace {

using namespace fft;

// The transfer function's table T[ky][kx] = H at |f_x| = kx / (Px d), |f_y| = ky /
// (Py d), kx < nx = Px/2 + 1, ky < ny = Py/2 + 1. Its first `tiles` groups of
// kTile columns lie one after the other like the row spectra's (none in plain
// order), what is left of the columns behind them.
struct TransferTable {
  float2 *T;
  uint32_t nx, ny, tiles;
  AsmParams P;
  __device__ __forceinline__ void fill(uint32_t i) const {
    if (i >= nx * ny) return;
    const uint32_t tiled = tiles * ny * kTile;
    uint32_t ky, kx;
    if (i < tiled) {
      const uint32_t j = i / kTile, tile = j / ny;
      ky = j - tile * ny;
      kx = tile * kTile + i % kTile;
    } else {
      const uint32_t rest = nx - tiles * kTile;
      ky = (i - tiled) / rest;
      kx = tiles * kTile + (i - tiled) - ky * rest;
    }
    const double fx = (double)kx * P.dfx, fy = (double)ky * P.dfy;
    const double f2 = fx * fx + fy * fy;
    float2 v = make_float2(0.f, 0.f);
    if ((!P.band_limit || (fx <= P.lim_x && fy <= P.lim_y)) && f2 < P.inv_lam2 && (P.pupil2 <= 0.0 || f2 <= P.pupil2)) {
      // z sqrt(1/lambda^2 - f^2) = z/lambda - z f^2 / (1/lambda + sqrt(1/lambda^2 - f^2)),
      // the first term reduced modulo 1 on the host
      const double rev = P.z_rev_frac - P.z * f2 / (P.inv_lam + sqrt(P.inv_lam2 - f2));
      const double fr = rev - floor(rev);
      double sn, cs;
      sincospi(2.0 * fr, &sn, &cs);
      v = make_float2((float)cs, (float)sn);
    }
    T[i] = v;
  }
};

// Forward FFT of row (f, y) of in [nf][h][w], zero-padded to Px -> A [nf][h][Px], on
// the first `groups` workgroups; the others fill T, which saves a small call a
// launch (two 64 x 64 fields 31 -> 28.5 us).
template <int LG, bool TILED>
__global__ void __launch_bounds__((Rows<LG, TILED>::W))
    k_fft_rows(const float2 *in, float2 *A, uint32_t w, uint32_t h, uint32_t nrows, const float2 *tw, uint32_t groups,
               TransferTable T) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  __shared__ C2 lds[Lines::kLdsElems];
  if (blockIdx.x >= groups) {
    T.fill((blockIdx.x - groups) * Lines::W + threadIdx.x);
    return;
  }
  const uint32_t l = Lines::line(), t = Lines::pos();
  const uint32_t row = Lines::group(groups) * Lines::kLines + l;  // f * h + y
  const bool ok = row < nrows;
  const float2 *src = in + (size_t)row * w;
  C2 v[L::E];
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) {  // w <= Px / 2
    const uint32_t i = t + q * L::TPL;
    const float2 g = ok && i < w ? src[i] : make_float2(0.f, 0.f);
    v[q] = c2(g.x, g.y);
  }
  line_fft<LG, false, true, Lines::kStride, Lines::kWave, false>(v, Lines::lds_of(lds), TableTwiddles{tw}, t);
  if (!ok) return;
  const uint32_t f = TILED ? row / h : row, y = TILED ? row - f * h : 0u, first = Lines::first_of(t, y, h);
  float2 *dst = A + (size_t)f * (TILED ? h : 1u) * L::N;
#pragma unroll
  for (uint32_t q = 0; q < L::E; ++q) Lines::elem(dst, first, h, q) = make_float2(v[q].x, v[q].y);
}

// Columns of a workgroup: kCols neighbouring columns (c fastest in the
// thread index, so that a row's load or store of the workgroup is one
// segment of kCols x 8 bytes), TPL threads each. The lines of the cache that
// neighbouring workgroups share are met in the L2 of the XCD they run on
// (xcd_group), which costs less than the two transposes that contiguous
// columns would need. Of long columns two (LDS of half a CU), four where several
// planes' transfer functions are read and the LDS holds them.
template <int LG, bool PLANES>
struct Cols {
  static constexpr bool kTwo = LG >= 13 || (LG >= 11 && !PLANES);
  static constexpr uint32_t kCols = kTwo ? 2 : LG >= 10 ? 4 : LG == 9 ? 8 : LG >= 6 ? 16 : 32;
  static constexpr uint32_t W = kCols * Line<LG>::TPL;
  static constexpr uint32_t kLdsElems = LG > 4 ? kCols * Line<LG>::kLds : 1;
  static constexpr uint32_t kWaves = LG >= 10 ? 4 : 2;
};

// A loop's index, unknown to the optimiser: it would else keep one 64-bit
// address per access of the body over the iterations (32 registers) instead
// of a scalar base and the shared offsets.
__device__ __forceinline__ uint32_t opaque(uint32_t i) {
  asm volatile("" : "+s"(i));
  return i;
}

// A group of columns of fields [blockIdx.y * fpw, + fpw): src [nf][h][Px]
// holds the row spectra. H: transfer functions of np planes, each [Py/2 +
// 1][Px/2 + 1]. dst [np][nf][h][Px]; may be src when np is 1 (every column
// is read before it is written).
template <int LG, bool PLANES>
__global__ void __launch_bounds__((Cols<LG, PLANES>::W), (Cols<LG, PLANES>::kWaves))
    k_fft_columns(const float2 *src, float2 *dst, const float2 *H, uint32_t np, uint32_t nf, uint32_t fpw, uint32_t h,
                  uint32_t px, uint32_t tile_lg, const float2 *tw) {
  using L = Line<LG>;
  constexpr uint32_t C = Cols<LG, PLANES>::kCols, E = L::E;
  __shared__ C2 lds[Cols<LG, PLANES>::kLdsElems];
  const uint32_t c = threadIdx.x % C, t = threadIdx.x / C;
  // lanes past the last column (px < C) work on column 0 and store nothing
  const uint32_t col = xcd_group(blockIdx.x, gridDim.x) * C + c, kx = col < px ? col : 0u;
  const uint32_t h_store = col < px ? h : 0u;
  C2 *x = lds + c;
  const uint32_t hw = px / 2 + 1, hx = kx <= px / 2 ? kx : px - kx, ny = L::N / 2 + 1;
  const size_t plane = (size_t)hw * ny;
  // this column in the transfer function's tables (see TransferTable): bytes of
  // its first element and between two rows
  const uint32_t tiled = (1u << tile_lg) < px ? hw / kTile * kTile : 0u;
  const uint32_t h_step = (hx < tiled ? kTile : hw - tiled) * 8;
  const uint32_t h_first = hx < tiled ? (hx / kTile * ny * kTile + hx % kTile) * 8 : (tiled * ny + hx - tiled) * 8;
  const size_t field = (size_t)h * px;
  // element (row t + q TPL, column kx) of a field: q steps from a uniform
  // base, plus one byte offset (below 2^32: h <= 4096, px <= 8192)
  // (tiles of 2^tile_lg columns)
  const uint32_t step = L::TPL << tile_lg;
  const uint32_t off = ((((kx >> tile_lg) * h + t) << tile_lg) + (kx & ((1u << tile_lg) - 1u))) * 8;
  auto load_h = [&](C2 (&Hr)[E], const float2 *T) {
    // frequency row i = t + q TPL: |f_y| is i steps, from q = E/2 on N - i
    // (opaque: sixteen offsets kept over the planes would be sixteen registers)
    uint32_t step_h = h_step, up = h_first + t * h_step, down = h_first + (L::N - t) * h_step;
    asm volatile("" : "+v"(step_h), "+v"(up), "+v"(down));
#pragma unroll
    for (uint32_t q = 0; q < E; ++q) {
      const float2 g = at(T, q < E / 2 ? up + q * L::TPL * step_h : down - q * L::TPL * step_h);
      Hr[q] = c2(g.x, g.y);
    }
  };
  auto store = [&](const C2 (&v)[E], float2 *out) {
#pragma unroll
    for (uint32_t q = 0; q < E / 2; ++q) {  // h <= Py / 2
      if (t + q * L::TPL < h_store) at(out + q * step, off) = make_float2(v[q].x, v[q].y);
    }
  };
  using Two = typename std::conditional<C == 2 && (LG <= 12 || PLANES), PairTwiddles<LG>, TableTwiddles>::type;
  typename std::conditional<C % 4 == 0, QuadTwiddles<LG>, Two>::type T;
  T.load(tw, t);
  C2 Hr[E];
  if constexpr (!PLANES) load_h(Hr, H);
  const uint32_t f0 = blockIdx.y * fpw, f1 = min(nf, f0 + fpw);
  // requested before the stores of the current field's last plane are waited for
  float2 next[E / 2];
  auto request = [&](uint32_t f) {
    const float2 *scol = src + opaque(f) * field;
#pragma unroll
    for (uint32_t q = 0; q < E / 2; ++q) {
      // h > Py / 4: the first quarter needs no check
      next[q] = make_float2(0.f, 0.f);
      if (q < E / 4 || t + q * L::TPL < h) next[q] = at(scol + q * step, off);
    }
  };
  request(f0);
  for (uint32_t f = f0; f < f1; ++f) {
    const uint32_t fo = opaque(f);
    C2 v[E];
#pragma unroll
    for (uint32_t q = 0; q < E / 2; ++q) v[q] = c2(next[q].x, next[q].y);
    auto request_next = [&] { if (f + 1 < f1) request(f + 1); };
    line_fft<LG, false, true, C, false, true>(v, x, T, t);
    if constexpr (!PLANES) {
#pragma unroll
      for (uint32_t q = 0; q < E; ++q) v[q] = mul_tw(v[q], Hr[q].x, Hr[q].y);
      line_fft<LG, true, false, C, false, true>(v, x, T, t);
      store(v, dst + fo * field);
      request_next();
    } else {
      C2 S[E];
#pragma unroll
      for (uint32_t q = 0; q < E; ++q) S[q] = v[q];
      for (uint32_t p = 0; p < np; ++p) {
          const uint32_t po = opaque(p);
        load_h(Hr, H + po * plane);
#pragma unroll
        for (uint32_t q = 0; q < E; ++q) v[q] = mul_tw(S[q], Hr[q].x, Hr[q].y);
        line_fft<LG, true, false, C, false, true>(v, x, T, t);
        store(v, dst + ((size_t)po * nf + fo) * field);
      }
      request_next();
    }
  }
}

// Inverse FFT of row (f, y) of A [nf][h][Px]; keep [0, w), scale -> out [nf][h][w].
template <int LG, bool TILED>
__global__ void __launch_bounds__((Rows<LG, TILED>::W))
    k_ifft_rows(const float2 *A, float2 *out, uint32_t w, uint32_t h, uint32_t nrows, float scale, const float2 *tw) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  __shared__ C2 lds[Lines::kLdsElems];
  const uint32_t l = Lines::line(), t = Lines::pos();
  const uint32_t row = Lines::group(gridDim.x) * Lines::kLines + l;
  const bool ok = row < nrows;
  const uint32_t f = TILED ? row / h : row, y = TILED ? row - f * h : 0u, first = Lines::first_of(t, y, h);
  const float2 *src = A + (size_t)f * (TILED ? h : 1u) * L::N;
  C2 v[L::E];
#pragma unroll
  for (uint32_t q = 0; q < L::E; ++q) {
    const float2 g = ok ? Lines::elem(src, first, h, q) : make_float2(0.f, 0.f);
    v[q] = c2(g.x, g.y);
  }
  line_fft<LG, true, false, Lines::kStride, Lines::kWave, false>(v, Lines::lds_of(lds), TableTwiddles{tw}, t);
  float2 *dst = out + (size_t)row * w;
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) {
    const uint32_t i = t + q * L::TPL;
    if (ok && i < w) dst[i] = make_float2(v[q].x * scale, v[q].y * scale);
  }
}

// Summed intensity of row y over nf fields of plane blockIdx.y: inverse FFT
// of row (f, y) of A [np][nf][h][Px] for every f < nf, scaled by 1/(Px Py),
// |.|^2 of the first w values summed over f, times `weight`; written into (or
// added to) I [np][h][w].
template <int LG, bool TILED>
__global__ void __launch_bounds__((Rows<LG, TILED>::W)) k_ifft_rows_intensity(const float2 *A, float *I, uint32_t nf,
                                                                     uint32_t w, uint32_t h, float scale,
                                                                     float weight, uint32_t accumulate,
                                                                     const float2 *tw) {
  using L = Line<LG>;
  using Lines = Rows<LG, TILED>;
  __shared__ C2 lds[Lines::kLdsElems];
  const uint32_t l = Lines::line(), t = Lines::pos();
  const uint32_t y = Lines::group(gridDim.x) * Lines::kLines + l;
  const bool ok = y < h;
  const uint32_t first = Lines::first_of(t, y, h);
  const float2 *Ap = A + (size_t)blockIdx.y * nf * h * L::N;
  float acc[L::E / 2];
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) acc[q] = 0.f;
  for (uint32_t f = 0; f < nf; ++f) {
    const float2 *src = Ap + (size_t)f * h * L::N;
    C2 v[L::E];
#pragma unroll
    for (uint32_t q = 0; q < L::E; ++q) {
      const float2 g = ok ? Lines::elem(src, first, h, q) : make_float2(0.f, 0.f);
      v[q] = c2(g.x, g.y);
    }
    line_fft<LG, true, false, Lines::kStride, Lines::kWave, false>(v, Lines::lds_of(lds), TableTwiddles{tw}, t);
#pragma unroll
    for (uint32_t q = 0; q < L::E / 2; ++q) {
      const float re = v[q].x * scale, im = v[q].y * scale;
      acc[q] += re * re + im * im;
    }
  }
  float *dst = I + ((size_t)blockIdx.y * h + y) * w;
#pragma unroll
  for (uint32_t q = 0; q < L::E / 2; ++q) {
    const uint32_t i = t + q * L::TPL;
    if (ok && i < w) dst[i] = (accumulate ? dst[i] : 0.f) + acc[q] * weight;
  }
}

// Where no row pass goes with it.
__global__ void __launch_bounds__(256) k_transfer(TransferTable T) { T.fill(blockIdx.x * 256 + threadIdx.x); }

// Twiddles of every length, in the order of fft.hpp: entry e of length n =
// 2^lg is exp(-2 pi i m / n) (FP64, rounded).
__global__ void k_twiddles(float2 *tw) {
  const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < 4 || e >= kTwiddleElems) return;
  const uint32_t lg = 30u - (uint32_t)__clz((int)e), n = 1u << lg, i = e - 2 * n;
  const uint32_t rem = lg % 4, ns4 = 1u << (4 * (lg / 4)), off4 = twiddle_off4(lg);
  const uint32_t off2 = off4 + ((rem >= 2 && ns4 > 1) ? 3 * ns4 : 0u);
  uint32_t m = 0;
  if (i < off4) {               // radix 16, span ns = 16, then 256: pairs of factors
    const uint32_t ns = i < 256 ? 16u : 256u, j = i < 256 ? i : i - 256;
    m = (2 * (j / (2 * ns)) + (j & 1u)) * ((j / 2) % ns) * (n / (16 * ns));
  } else if (i < off2) {        // radix 4, span ns4: factors 1 to 3
    const uint32_t j = i - off4;
    m = (j / ns4 + 1) * (j % ns4) * (n / (4 * ns4));
  } else if ((rem & 1u) && i - off2 < n / 2) {  // radix 2, span n / 2
    m = i - off2;
  } else {
    return;
  }
  double sn, cs;
  sincospi(2.0 * (double)m / (double)n, &sn, &cs);
  tw[e] = make_float2((float)cs, (float)-sn);
}

// Fields per column workgroup: all of them (the transfer function's column
// is then read once) unless the launch would have too few workgroups to fill
// the chip's 256 CUs several times over.
uint32_t fields_per_group(uint32_t groups, uint32_t nf) {
  const uint32_t want = (1024 + groups - 1) / groups;  // parts of the fields
  const uint32_t parts = std::min(nf, want);
  return (nf + parts - 1) / parts;
}

}  // namespace

// Scratch of the allocation-free propagation (hpt_asm_propagate_noalloc) and
// the twiddle table: one of each per device, held until the process ends. Host
// code never names them directly (their host-side names are stand-ins, not
// device addresses): the device addresses come from asm_device().
static __device__ __align__(256) float2 scratch[kNoAllocScratchElems];
static __device__ __align__(256) float2 twiddle_table[kTwiddleElems];

hipError_t asm_device(int device, AsmDevice *out) {
  static std::mutex mu;
  static std::map<int, AsmDevice> table;
  std::lock_guard<std::mutex> g(mu);
  auto it = table.find(device);
  if (it != table.end()) { *out = it->second; return hipSuccess; }
  AsmDevice d;
  float2 *tw = nullptr;
  hipError_t e = hipGetSymbolAddress((void **)&d.scratch, HIP_SYMBOL(scratch));
  if (e == hipSuccess) e = hipGetSymbolAddress((void **)&tw, HIP_SYMBOL(twiddle_table));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_twiddles, dim3(kTwiddleElems / 256), dim3(256), 0, 0, tw);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(0);
  if (e != hipSuccess) return e;
  d.tw = tw;
  table[device] = d;
  *out = d;
  return hipSuccess;
}

uint32_t asm_padded(uint32_t n) {
  uint32_t p = 1;
  while (p < 2 * n) p *= 2;
  return p;
}

size_t asm_transfer_elems(uint32_t w, uint32_t h) {
  return (size_t)(asm_padded(w) / 2 + 1) * (asm_padded(h) / 2 + 1);
}

// Whether row spectra are tiled: see the head of this file.
bool asm_tiled(uint32_t w, uint32_t h) { return asm_padded(h) >= 2048 && asm_padded(w) >= 1u << kTiledLg; }

static TransferTable transfer_table(float2 *T, uint32_t w, uint32_t h, const AsmParams &P) {
  const uint32_t nx = asm_padded(w) / 2 + 1;
  return {T, nx, asm_padded(h) / 2 + 1, asm_tiled(w, h) ? nx / kTile : 0u, P};
}

hipError_t launch_asm_transfer(float2 *T, uint32_t w, uint32_t h, const AsmParams &P, hipStream_t st) {
  const TransferTable table = transfer_table(T, w, h, P);
  hipLaunchKernelGGL(k_transfer, dim3((table.nx * table.ny + 255) / 256), dim3(256), 0, st, table);
  return hipGetLastError();
}

// table.nx 0: none.
static hipError_t launch_rows(const float2 *in, float2 *A, const TransferTable &table, const float2 *tw, uint32_t nf,
                              uint32_t w, uint32_t h, hipStream_t st) {
  const uint32_t px = asm_padded(w), nrows = nf * h;
  const bool known = with_rows(log2u(px), asm_tiled(w, h), [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    constexpr uint32_t n = Rows<LG, TILED>::kLines, W = Rows<LG, TILED>::W;
    const uint32_t groups = (nrows + n - 1) / n, more = (table.nx * table.ny + W - 1) / W;
    hipLaunchKernelGGL((k_fft_rows<LG, TILED>), dim3(groups + more), dim3(W), 0, st, in, A, w, h, nrows, tw + 2 * px,
                       groups, table);
  });
  return known ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_asm_rows(const float2 *in, float2 *A, const float2 *tw, uint32_t nf, uint32_t w, uint32_t h,
                           hipStream_t st) {
  return launch_rows(in, A, TransferTable{}, tw, nf, w, h, st);
}

hipError_t launch_asm_columns(const float2 *src, float2 *dst, const float2 *H, uint32_t np, const float2 *tw,
                              uint32_t nf, uint32_t w, uint32_t h, hipStream_t st) {
  const uint32_t px = asm_padded(w), py = asm_padded(h);
  const bool known = with_length(log2u(py), [&](auto lg) {
    constexpr int LG = decltype(lg)::value;
    auto launch = [&](auto kernel, uint32_t cols, uint32_t threads) {
      const uint32_t groups = (px + cols - 1) / cols, fpw = fields_per_group(groups, nf);
      hipLaunchKernelGGL(kernel, dim3(groups, (nf + fpw - 1) / fpw), dim3(threads), 0, st, src, dst, H, np, nf, fpw, h, px,
                         log2u(asm_tiled(w, h) ? kTile : px), tw + 2 * py);
    };
    if (np == 1) launch(k_fft_columns<LG, false>, Cols<LG, false>::kCols, Cols<LG, false>::W);
    else launch(k_fft_columns<LG, true>, Cols<LG, true>::kCols, Cols<LG, true>::W);
  });
  return known ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_asm(const float2 *in, float2 *out, float2 *A, float2 *H, const AsmParams *P, const float2 *tw,
                      uint32_t nf, uint32_t w, uint32_t h, hipStream_t st) {
  if (nf == 0 || w == 0 || h == 0) return hipErrorInvalidValue;
  const uint32_t px = asm_padded(w), py = asm_padded(h), nrows = nf * h;
  hipError_t e = launch_rows(in, A, P ? transfer_table(H, w, h, *P) : TransferTable{}, tw, nf, w, h, st);
  if (e == hipSuccess) e = launch_asm_columns(A, A, H, 1, tw, nf, w, h, st);
  if (e != hipSuccess) return e;
  const bool known = with_rows(log2u(px), asm_tiled(w, h), [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    constexpr uint32_t n = Rows<LG, TILED>::kLines, W = Rows<LG, TILED>::W;
    hipLaunchKernelGGL((k_ifft_rows<LG, TILED>), dim3((nrows + n - 1) / n), dim3(W), 0, st, A, out, w, h, nrows,
                       1.0f / ((float)px * (float)py), tw + 2 * px);
  });
  return known ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_asm_intensity(const float2 *A, const float2 *tw, uint32_t np, uint32_t nf, uint32_t w, uint32_t h,
                                float *I, float weight, bool accumulate, hipStream_t st) {
  const uint32_t px = asm_padded(w), py = asm_padded(h);
  const bool known = with_rows(log2u(px), asm_tiled(w, h), [&](auto lg, auto tiled) {
    constexpr int LG = decltype(lg)::value;
    constexpr bool TILED = decltype(tiled)::value;
    constexpr uint32_t n = Rows<LG, TILED>::kLines, W = Rows<LG, TILED>::W;
    hipLaunchKernelGGL((k_ifft_rows_intensity<LG, TILED>), dim3((h + n - 1) / n, np), dim3(W), 0, st, A, I, nf, w, h,
                       1.0f / ((float)px * (float)py), weight, accumulate ? 1u : 0u, tw + 2 * px);
  });
  return known ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace hpt
