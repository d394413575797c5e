// Line FFTs of the angular-spectrum kernels: lengths N = 2^LG, 2 .. 8192, in
// FP32, one line on N/16 threads with 16 values each in registers (shorter
// lines on one thread).
//
// Stockham stages (Govindaraju et al., SC 2008 formulation) of radix 16 while
// they fit, then radix 4, then radix 2. Thread t of a line holds the elements
// t + (N/16) q, q < 16, before the first stage and after the last one, so
// that both ends stay in registers (a kernel reads and writes global memory
// there, or multiplies by the transfer function); the last radix-4 and
// radix-2 stages work on the thread's own values. LDS is crossed once between
// two radix-16 stages and once before the last, shorter ones: N = 4096 twice,
// N = 128 once.
//
// Twiddles come from a table of each stage's factors in the order its threads
// read them, two to a 16-byte load (radix 16: factors 2j and 2j + 1 of
// butterfly k, 1 <= r < 16, at float4 j Ns + k): a load of a wave takes the
// vector cache 16 cycles whether its lanes read 8 or 16 bytes, and gathers
// exp(-2 pi i m / n) at stride r from one table per length took up to 32.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace hpt {
namespace fft {

constexpr uint32_t kMaxLg = 13;  // longest line: 8192
// Table of all lengths: the factors of length n start at element 2n and take
// at most 2n.
constexpr uint32_t kTwiddleElems = 4u << kMaxLg;

struct C2 { float x, y; };

__device__ __forceinline__ C2 c2(float x, float y) { return {x, y}; }
__device__ __forceinline__ C2 add(C2 a, C2 b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ C2 sub(C2 a, C2 b) { return {a.x - b.x, a.y - b.y}; }
// The complex products of the transforms, with their roundings fixed: each
// part is one product rounded, then a fused multiply-add. Results therefore
// do not depend on what the compiler fuses in one kernel or another.
// a times the table twiddle (c, s).
__device__ __forceinline__ C2 mul_tw(C2 a, float c, float s) {
  return {fmaf(a.x, c, -(a.y * s)), fmaf(a.y, c, a.x * s)};
}
// multiply by -i (forward) or +i (inverse)
__device__ __forceinline__ C2 rot(C2 a, bool inv) { return inv ? c2(-a.y, a.x) : c2(a.y, -a.x); }
__device__ __forceinline__ C2 twiddled(C2 a, const float2 *tw, bool inv) {
  const float2 w = *tw;
  return mul_tw(a, w.x, inv ? -w.y : w.y);
}

// Radix-4 DFT of a0..a3 in place (forward: exp(-2 pi i), inverse: +).
__device__ __forceinline__ void dft4(C2 &a0, C2 &a1, C2 &a2, C2 &a3, bool inv) {
  C2 b0 = add(a0, a2), b1 = sub(a0, a2), b2 = add(a1, a3), b3 = rot(sub(a1, a3), inv);
  a0 = add(b0, b2);
  a1 = add(b1, b3);
  a2 = sub(b0, b2);
  a3 = sub(b1, b3);
}

// Radix-16 DFT of a[0..15] in place, as 4 x 4: DFT-4 over n1 of a[4 n1 + n2]
// for each n2, twiddles exp(-+2 pi i n2 k1 / 16), DFT-4 over n2; output k =
// k1 + 4 k2 lands in a[k]. HALF: a[8..15] are zero (a zero-padded line's
// first stage) and are not read. XR: the inner twiddles m whose imaginary
// part rounds x sin (as mul_tw does) rather than y cos: which product a compiler
// once rounded first, kept because Adam's steps amplify a last bit. With mul_tw
// for all, fields are as exact (2.1e-7 of the RMS from 64 bits either way) and as
// fast, but the phases after 20 steps differ by 6e-6 (300 x 200) and 4e-5
// (1920 x 1080) of their RMS, to either side of the exact ones.
template <bool HALF, uint32_t XR>
__device__ __forceinline__ void dft16(C2 (&a)[16], bool inv) {
  // exp(-2 pi i m / 16), m = 0..9
  constexpr float c1 = 0.923879532511286756f, s1 = 0.382683432365089772f, h = 0.707106781186547524f;
  constexpr float cs[10][2] = {{1.f, 0.f}, {c1, -s1}, {h, -h}, {s1, -c1}, {0.f, -1.f},
                               {-s1, -c1}, {-h, -h}, {-c1, -s1}, {-1.f, 0.f}, {-c1, s1}};
  C2 t[16];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    if constexpr (HALF) {
      const C2 b0 = a[n2], b1 = a[n2 + 4], r1 = rot(b1, inv);
      t[4 * n2 + 0] = add(b0, b1); t[4 * n2 + 1] = add(b0, r1);
      t[4 * n2 + 2] = sub(b0, b1); t[4 * n2 + 3] = sub(b0, r1);
    } else {
      C2 b0 = a[n2], b1 = a[n2 + 4], b2 = a[n2 + 8], b3 = a[n2 + 12];
      dft4(b0, b1, b2, b3, inv);
      t[4 * n2 + 0] = b0; t[4 * n2 + 1] = b1; t[4 * n2 + 2] = b2; t[4 * n2 + 3] = b3;   // t[n2][k1]
    }
  }
#pragma unroll
  for (int n2 = 1; n2 < 4; ++n2)
#pragma unroll
    for (int k1 = 1; k1 < 4; ++k1) {
      const int m = n2 * k1;
      const float c = cs[m][0], s = inv ? -cs[m][1] : cs[m][1];
      C2 &z = t[4 * n2 + k1];
      if (m == 4) z = rot(z, inv);
      else if ((XR >> m) & 1u) z = mul_tw(z, c, s);
      else z = c2(fmaf(z.x, c, -(z.y * s)), fmaf(z.x, s, z.y * c));
    }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    C2 b0 = t[k1], b1 = t[4 + k1], b2 = t[8 + k1], b3 = t[12 + k1];
    dft4(b0, b1, b2, b3, inv);
    a[k1] = b0; a[k1 + 4] = b1; a[k1 + 8] = b2; a[k1 + 12] = b3;
  }
}

// Twiddles of the radix-16 stages of length 2^lg: 16 x 16 for the second
// stage, 16 x 256 for the third (factor 0, always 1, is kept for the pairs).
__host__ __device__ constexpr uint32_t twiddle_off4(uint32_t lg) { return lg >= 12 ? 256 + 4096 : lg >= 8 ? 256 : 0; }

// Shape of the transform of length 2^LG: E values per thread, TPL threads
// per line, S16 radix-16 stages, the rest (1: radix 2, 2: radix 4, 3: radix
// 4 then 2); offsets of the stages' twiddles in the length's table.
template <int LG>
struct Line {
  static constexpr uint32_t N = 1u << LG;
  static constexpr uint32_t E = N < 16 ? N : 16;
  static constexpr uint32_t TPL = N / E;
  static constexpr int S16 = LG / 4, REM = LG % 4;
  static constexpr uint32_t Ns4 = 1u << (4 * S16);                 // span before the radix-4 stage
  static constexpr uint32_t kOff4 = twiddle_off4(LG);              // after 16 x 16, 16 x 256
  static constexpr uint32_t kOff2 = kOff4 + ((REM >= 2 && Ns4 > 1) ? 3 * Ns4 : 0);
  // LDS elements of a line: one pad slot after every 16, which spreads the
  // strided writes of the early stages over the banks
  static constexpr uint32_t kLds = N + N / 16;
};
__device__ __forceinline__ constexpr uint32_t pd(uint32_t i) { return i + (i >> 4); }

// Threads of the group that shares an LDS buffer agree: within one wave the
// LDS pipe keeps its order, so only the compiler has to.
template <bool WAVE>
__device__ __forceinline__ void line_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// v[q] = element t + TPL q of a line after a radix-16 stage of span Ns wrote
// its outputs: through the line's LDS, element e at x[pd(e) * CS].
template <int LG, uint32_t NS, uint32_t CS, bool WAVE>
__device__ __forceinline__ void exchange(C2 (&v)[16], C2 *x, uint32_t t) {
  using L = Line<LG>;
  line_sync<WAVE>();   // the buffer's last reads are done
  C2 *w = x + pd((t / NS) * NS * 16 + t % NS) * CS;
  // element d + r Ns lies r (Ns + Ns/16) slots on (Ns >= 16: d is a multiple
  // of 16 plus less than 16; Ns = 1: all sixteen within one run)
  constexpr uint32_t wstep = (NS < 16 ? NS : NS + NS / 16) * CS;
#pragma unroll
  for (uint32_t r = 0; r < 16; ++r) w[r * wstep] = v[r];
  line_sync<WAVE>();
  if constexpr (L::TPL >= 16) {
    const C2 *rd = x + pd(t) * CS;
#pragma unroll
    for (uint32_t q = 0; q < 16; ++q) v[q] = rd[q * (L::TPL + L::TPL / 16) * CS];
  } else {
#pragma unroll
    for (uint32_t q = 0; q < 16; ++q) v[q] = x[pd(t + q * L::TPL) * CS];
  }
}

// Sources of a line's twiddles: v[r] *= factor r of the radix-16 stage of span
// NS at butterfly k = t mod NS.
// From the table, read where they are used.
struct TableTwiddles {
  const float2 *tw;
  __device__ __forceinline__ void load(const float2 *table, uint32_t) { tw = table; }
  template <uint32_t NS>
  __device__ __forceinline__ void apply(C2 (&v)[16], uint32_t t, bool inv) const {
    const float4 *t4 = reinterpret_cast<const float4 *>(tw + (NS == 16 ? 0 : 256)) + t % NS;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      const float4 w = t4[j * NS];
      if (j) v[2 * j] = mul_tw(v[2 * j], w.x, inv ? -w.y : w.y);
      v[2 * j + 1] = mul_tw(v[2 * j + 1], w.z, inv ? -w.w : w.w);
    }
  }
};

// x of lane L of the caller's quad of lanes (all lanes of the wave active).
template <int L>
__device__ __forceinline__ float quad_lane(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), L * 0x55, 0xF, 0xF, true));
}

// Kept in registers over many transforms by threads of which each quad of
// lanes has the same t: lane l of the quad keeps pairs l and l + 4 of each
// stage (16 registers for both), and the quad's lanes read each other's
// through the DPP unit, mostly as an operand of the multiplication itself.
template <int LG>
struct QuadTwiddles {
  const float2 *tw;
  float4 a[Line<LG>::S16 >= 3 ? 2 : 1][2];
  __device__ __forceinline__ void load(const float2 *table, uint32_t t) {
    tw = table;
    const uint32_t l = threadIdx.x & 3u;
    const float4 *t4 = reinterpret_cast<const float4 *>(table);
    if constexpr (Line<LG>::S16 >= 2)
      for (uint32_t i = 0; i < 2; ++i) a[0][i] = t4[(l + 4 * i) * 16 + t % 16u];
    if constexpr (Line<LG>::S16 >= 3)
      for (uint32_t i = 0; i < 2; ++i) a[1][i] = t4[128 + (l + 4 * i) * 256 + t % 256u];
  }
  template <uint32_t NS, int J>
  __device__ __forceinline__ static void pair(C2 (&v)[16], const float4 &w, bool inv) {
    constexpr int l = J & 3;
    if constexpr (J != 0) {
      const float s = quad_lane<l>(w.y);
      v[2 * J] = mul_tw(v[2 * J], quad_lane<l>(w.x), inv ? -s : s);
    }
    const float s = quad_lane<l>(w.w);
    v[2 * J + 1] = mul_tw(v[2 * J + 1], quad_lane<l>(w.z), inv ? -s : s);
  }
  template <uint32_t NS>
  __device__ __forceinline__ void apply(C2 (&v)[16], uint32_t, bool inv) const {
    float4 w0 = a[NS == 16 ? 0 : 1][0], w1 = a[NS == 16 ? 0 : 1][1];
    // opaque: the lanes' copies are not to be kept instead (60 registers)
    asm volatile("" : "+v"(w0.x), "+v"(w0.y), "+v"(w0.z), "+v"(w0.w), "+v"(w1.x), "+v"(w1.y), "+v"(w1.z), "+v"(w1.w));
    pair<NS, 0>(v, w0, inv); pair<NS, 1>(v, w0, inv); pair<NS, 2>(v, w0, inv); pair<NS, 3>(v, w0, inv);
    pair<NS, 4>(v, w1, inv); pair<NS, 5>(v, w1, inv); pair<NS, 6>(v, w1, inv); pair<NS, 7>(v, w1, inv);
  }
};

// Kept in registers by threads of which each pair of lanes has the same t: the
// last stage's, which fill the L1 (lane l of the pair keeps pairs 2 j + l, 16
// registers); the second's are read from the table.
template <int LG>
struct PairTwiddles {
  TableTwiddles table;
  const float2 *tw;
  float4 a[4];
  __device__ __forceinline__ void load(const float2 *t0, uint32_t t) {
    tw = t0;
    table.tw = t0;
    const uint32_t l = threadIdx.x & 1u;
    const float4 *t4 = reinterpret_cast<const float4 *>(t0);
    if constexpr (Line<LG>::S16 >= 3)
      for (uint32_t j = 0; j < 4; ++j) a[j] = t4[128 + (l + 2 * j) * 256 + t % 256u];
  }
  template <int L>
  __device__ __forceinline__ static float lane(float x) {   // x of lane L of the pair
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), L ? 0xF5 : 0xA0, 0xF, 0xF, true));
  }
  template <int J>
  __device__ __forceinline__ static void pair(C2 (&v)[16], const float4 &w, bool inv) {
    if constexpr (J != 0) {
      const float s = lane<J & 1>(w.y);
      v[2 * J] = mul_tw(v[2 * J], lane<J & 1>(w.x), inv ? -s : s);
    }
    const float s = lane<J & 1>(w.w);
    v[2 * J + 1] = mul_tw(v[2 * J + 1], lane<J & 1>(w.z), inv ? -s : s);
  }
  template <uint32_t NS>
  __device__ __forceinline__ void apply(C2 (&v)[16], uint32_t t, bool inv) const {
    if constexpr (NS == 16) {
      table.template apply<16>(v, t, inv);
    } else {
      float4 w[4];
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {   // opaque: as in QuadTwiddles
        w[j] = a[j];
        asm volatile("" : "+v"(w[j].x), "+v"(w[j].y), "+v"(w[j].z), "+v"(w[j].w));
      }
      pair<0>(v, w[0], inv); pair<1>(v, w[0], inv); pair<2>(v, w[1], inv); pair<3>(v, w[1], inv);
      pair<4>(v, w[2], inv); pair<5>(v, w[2], inv); pair<6>(v, w[3], inv); pair<7>(v, w[3], inv);
    }
  }
};

// The XR of dft16 in the first and third, and in the second radix-16 stage
// (m = 1, 2, 3; in 4096-point columns m = 1, 3, inversely also 9).
template <int LG, bool COLS, bool INV>
struct Roundings {
  static constexpr bool kCol12 = COLS && LG == 12;
  static constexpr uint32_t kMid = kCol12 ? 0x00Au : 0x00Eu, kEnds = kCol12 && INV ? 0x20Au : kMid;
};

// FFT of one line: v[q] = element t + TPL q on entry and on return. HALF: the
// upper half of the input is zero and not read. x: the line's LDS (see
// exchange), T: the length's factors. COLS: a column (see Roundings).
template <int LG, bool INV, bool HALF, uint32_t CS, bool WAVE, bool COLS, class Twiddles>
__device__ __forceinline__ void line_fft(C2 (&v)[Line<LG>::E], C2 *x, const Twiddles &T, uint32_t t) {
  using L = Line<LG>;
  const float2 *tw = T.tw;
  constexpr uint32_t E = L::E;
  if constexpr (L::S16 >= 1) {
    dft16<HALF, Roundings<LG, COLS, INV>::kEnds>(v, INV);
    if constexpr (L::S16 >= 2) {
      exchange<LG, 1, CS, WAVE>(v, x, t);
      T.template apply<16>(v, t, INV);
      dft16<false, Roundings<LG, COLS, INV>::kMid>(v, INV);
    }
    if constexpr (L::S16 >= 3) {
      exchange<LG, 16, CS, WAVE>(v, x, t);
      T.template apply<256>(v, t, INV);
      dft16<false, Roundings<LG, COLS, INV>::kEnds>(v, INV);
    }
    if constexpr (L::REM != 0) exchange<LG, L::Ns4 / 16, CS, WAVE>(v, x, t);
  } else if constexpr (HALF) {
#pragma unroll
    for (uint32_t q = E / 2; q < E; ++q) v[q] = c2(0.f, 0.f);
  }
  if constexpr (L::REM >= 2) {  // radix 4: butterfly j = t + g TPL, g < E/4, of elements j + r N/4
#pragma unroll
    for (uint32_t g = 0; g < E / 4; ++g) {
      if constexpr (L::Ns4 > 1) {
        const uint32_t k = (t + g * L::TPL) % L::Ns4;
#pragma unroll
        for (uint32_t r = 1; r < 4; ++r)
          v[g + r * (E / 4)] = twiddled(v[g + r * (E / 4)], tw + L::kOff4 + (r - 1) * L::Ns4 + k, INV);
      }
      dft4(v[g], v[g + E / 4], v[g + E / 2], v[g + 3 * (E / 4)], INV);
    }
    if constexpr (L::REM == 3) {
      // output r of butterfly j is element (j / Ns) 4 Ns + j % Ns + r Ns, Ns =
      // N/8 = 2 TPL (TPL for N = 8): a permutation of the thread's values
      C2 w[E];
      constexpr uint32_t P = E / 8;  // values per eighth of the line
#pragma unroll
      for (uint32_t g = 0; g < E / 4; ++g)
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) w[(g / P) * (E / 2) + g % P + P * r] = v[g + r * (E / 4)];
#pragma unroll
      for (uint32_t q = 0; q < E; ++q) v[q] = w[q];
    }
  }
  if constexpr ((L::REM & 1) != 0) {  // radix 2 at span N/2
#pragma unroll
    for (uint32_t g = 0; g < E / 2; ++g) {
      if constexpr (L::N > 2) v[g + E / 2] = twiddled(v[g + E / 2], tw + L::kOff2 + t + g * L::TPL, INV);
      const C2 a0 = v[g], a1 = v[g + E / 2];
      v[g] = add(a0, a1);
      v[g + E / 2] = sub(a0, a1);
    }
  }
}

// Element at a byte offset from a uniform base: a scalar base and a 32-bit
// offset register. (The offset goes through an empty asm so that its
// extension to 64 bits stays beside the access; hoisted, every access would
// add two registers' worth of address instead.)
__device__ __forceinline__ const float2 &at(const float2 *p, uint32_t off) {
  asm volatile("" : "+v"(off));
  return *(const float2 *)((const char *)p + off);
}
__device__ __forceinline__ float2 &at(float2 *p, uint32_t off) {
  asm volatile("" : "+v"(off));
  return *(float2 *)((char *)p + off);
}

// Row spectra [h][n] of a field, in the plain order or (TILED) in tiles of kTile
// columns: element (y, x) at ((x / kTile) h + y) kTile + x mod kTile (asm.hip says
// when and why).
constexpr uint32_t kTile = 8;

// Threads of a row kernel's workgroup and the lines it works on. In plain order
// consecutive threads are on consecutive elements of a row; of tiled rows of 2048
// points or more a workgroup takes two, in turn over the threads, so that it has
// whole 128-byte pieces of the tiles.
template <int LG, bool TILED>
struct Rows {
  using L = Line<LG>;
  static constexpr bool kPairs = TILED && (LG == 11 || LG == 12);
  static constexpr uint32_t W = kPairs ? 2 * L::TPL : L::TPL < 64 ? 64 : L::TPL;
  static constexpr uint32_t kLines = W / L::TPL;
  static constexpr uint32_t kStride = kPairs ? kLines : 1;   // of a line's elements in LDS
  static constexpr bool kWave = L::TPL <= 64;
  static constexpr uint32_t kLdsElems = L::S16 >= 1 && LG > 4 ? kLines * L::kLds : 1;
  // this workgroup among its field's: tiled, each XCD takes one range of rows,
  // so that the rows that share a line of the cache meet in one L2
  __device__ __forceinline__ static uint32_t group(uint32_t groups);
  // this thread's line of the workgroup, its place in the line, the line's LDS
  __device__ __forceinline__ static uint32_t line() { return kPairs ? threadIdx.x % kLines : threadIdx.x / L::TPL; }
  __device__ __forceinline__ static uint32_t pos() { return kPairs ? threadIdx.x / kLines : threadIdx.x % L::TPL; }
  __device__ __forceinline__ static C2 *lds_of(C2 *lds) { return lds + line() * (kPairs ? 1 : L::kLds); }
  // element t + q TPL of row y of a field [h][N]: first = first_of(t, y, h)
  __device__ __forceinline__ static uint32_t first_of(uint32_t t, uint32_t y, uint32_t h) {
    return TILED ? ((t / kTile) * h + y) * kTile + t % kTile : y * L::N + t;
  }
  template <class P>
  __device__ __forceinline__ static auto &elem(P *field, uint32_t first, uint32_t h, uint32_t q) {
    if constexpr (TILED) return at(field + (size_t)(q * L::TPL) * h, first * 8);
    else return (field + first)[q * L::TPL];
  }
};

// Workgroup b of g, renumbered so that each of the 8 XCDs (workgroups are
// dealt to them in turn) takes one contiguous range.
__device__ __forceinline__ uint32_t xcd_group(uint32_t b, uint32_t g) {
  return g % 8u ? b : (b % 8u) * (g / 8u) + b / 8u;
}

template <int LG, bool TILED>
__device__ __forceinline__ uint32_t Rows<LG, TILED>::group(uint32_t groups) {
  return TILED ? xcd_group(blockIdx.x, groups) : blockIdx.x;
}

inline uint32_t log2u(uint32_t n) {
  uint32_t l = 0;
  while ((1u << l) < n) ++l;
  return l;
}

// f(integral_constant<LG>) for the line length 2^lg.
template <class F>
inline bool with_length(uint32_t lg, F &&f) {
  switch (lg) {
    case 1: f(std::integral_constant<int, 1>{}); return true;
    case 2: f(std::integral_constant<int, 2>{}); return true;
    case 3: f(std::integral_constant<int, 3>{}); return true;
    case 4: f(std::integral_constant<int, 4>{}); return true;
    case 5: f(std::integral_constant<int, 5>{}); return true;
    case 6: f(std::integral_constant<int, 6>{}); return true;
    case 7: f(std::integral_constant<int, 7>{}); return true;
    case 8: f(std::integral_constant<int, 8>{}); return true;
    case 9: f(std::integral_constant<int, 9>{}); return true;
    case 10: f(std::integral_constant<int, 10>{}); return true;
    case 11: f(std::integral_constant<int, 11>{}); return true;
    case 12: f(std::integral_constant<int, 12>{}); return true;
    case 13: f(std::integral_constant<int, 13>{}); return true;
    default: return false;
  }
}

// f(integral_constant<LG>, bool_constant<TILED>) for rows of length 2^lg.
constexpr int kTiledLg = 9;  // shortest tiled row: kTile divides its TPL, and a tile is a fraction of it
template <class F>
inline bool with_rows(uint32_t lg, bool tiled, F &&f) {
  return with_length(lg, [&](auto l) {
    if constexpr (decltype(l)::value >= kTiledLg) {
      if (tiled) { f(l, std::true_type{}); return; }
    }
    f(l, std::false_type{});
  });
}

}  // namespace fft
}  // namespace hpt
