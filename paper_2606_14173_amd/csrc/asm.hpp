// Angular-spectrum propagation launchers (second stage of the two-stage
// scheme, Sec. 4.4).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace hpt {

// Transfer-function constants of one propagation, computed on the host in FP64.
struct AsmParams {
  double dfx, dfy;        // frequency steps 1 / (Px d), 1 / (Py d)
  double lim_x, lim_y;    // band limits 1 / (lambda sqrt((2 z dfx)^2 + 1)) (and y)
  double inv_lam, inv_lam2;
  double z;
  double z_rev_frac;      // frac(z / lambda)
  double pupil2;          // squared pupil cutoff (NA / lambda)^2; 0: no pupil
  uint32_t band_limit;
};

// Padded length of one axis: the next power of two >= 2 n (1 <= n <= 4096).
uint32_t asm_padded(uint32_t n);

// Complex64 elements of the static scratch of the allocation-free
// propagation (72 MiB: one 1920 x 1080 field, padded to 4096 columns, with
// its work buffer and its transfer function).
constexpr size_t kNoAllocScratchElems = 9437184;
// Device addresses of what each device holds until the process ends: that
// scratch, and the twiddle factors of every line length (built by the first
// call for the device).
struct AsmDevice {
  float2 *scratch = nullptr;
  const float2 *tw = nullptr;
};
hipError_t asm_device(int device, AsmDevice *out);

// Transfer function of P for fields of w x h, tabulated over a quarter of the
// frequency plane (asm_transfer_elems complex64: never more than h Px + Px +
// Py).
size_t asm_transfer_elems(uint32_t w, uint32_t h);
hipError_t launch_asm_transfer(float2 *T, uint32_t w, uint32_t h, const AsmParams &P, hipStream_t st);

// nf fields in [nf][h][w] -> out (may alias in); A: scratch of
// nf * h * asm_padded(w) complex64; H: the table above, which P (if not null) has
// filled on the way.
hipError_t launch_asm(const float2 *in, float2 *out, float2 *A, float2 *H, const AsmParams *P, const float2 *tw,
                      uint32_t nf, uint32_t w, uint32_t h, hipStream_t st);

// Whether the row spectra of w x h fields lie in tiles (fft.hpp).
bool asm_tiled(uint32_t w, uint32_t h);

// The passes by themselves. Row spectra of nf fields [nf][h][w] -> A [nf][h][Px],
// in tiles if asm_tiled, as all row spectra are.
hipError_t launch_asm_rows(const float2 *in, float2 *A, const float2 *tw, uint32_t nf, uint32_t w, uint32_t h,
                           hipStream_t st);
// Column passes of nf fields' row spectra src [nf][h][Px] for np planes, whose
// tables follow each other in H -> dst [np][nf][h][Px] (src itself if np is 1).
hipError_t launch_asm_columns(const float2 *src, float2 *dst, const float2 *H, uint32_t np, const float2 *tw,
                              uint32_t nf, uint32_t w, uint32_t h, hipStream_t st);
// Per plane: weight * sum over the nf fields of |u|^2, u the inverse row
// transforms of A [np][nf][h][Px], written into (accumulate: added to) I
// [np][h][w].
hipError_t launch_asm_intensity(const float2 *A, const float2 *tw, uint32_t np, uint32_t nf, uint32_t w, uint32_t h,
                                float *I, float weight, bool accumulate, hipStream_t st);

}  // namespace hpt
