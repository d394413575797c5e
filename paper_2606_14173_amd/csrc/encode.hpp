// Phase-only encoding launchers (Adam under complex-amplitude supervision).
// A: row spectra [nf][h][Px] (asm.hpp); tw: the device's twiddle table.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace hpt {

// Adam constants (Kingma and Ba, 2015).
constexpr float kAdamBeta1 = 0.9f, kAdamBeta2 = 0.999f, kAdamEps = 1e-8f;

// Partial dot products per field (three doubles each).
uint32_t enc_parts(uint32_t w, uint32_t h);

// phi = arg U (0 where U = 0). n values.
hipError_t launch_enc_init(const float2 *U, float *phi, size_t n, hipStream_t st);
// V = the inverse row transforms of A; vv[f] = <V_f, V_f>.
hipError_t launch_enc_target(const float2 *A, float2 *V, double *part, double *vv, const float2 *tw, uint32_t nf,
                             uint32_t w, uint32_t h, hipStream_t st);
// A = row spectra of exp(i phi).
hipError_t launch_enc_rows_phase(const float *phi, float2 *A, const float2 *tw, uint32_t nf, uint32_t w, uint32_t h,
                                 hipStream_t st);
// R = the inverse row transforms of A; s[f] = <V_f, R_f> / vv[f]; rel[f] = 1 -
// |<V_f, R_f>|^2 / (vv[f] <R_f, R_f>).
hipError_t launch_enc_scale(const float2 *A, float2 *R, const float2 *V, double *part, double *vv, double2 *s,
                            double *rel, const float2 *tw, uint32_t nf, uint32_t w, uint32_t h, hipStream_t st);
// A = row spectra of R_f - s[f] V_f.
hipError_t launch_enc_rows_residual(const float2 *R, const float2 *V, const double2 *s, float2 *A, const float2 *tw,
                                    uint32_t nf, uint32_t w, uint32_t h, hipStream_t st);
// G = the inverse row transforms of A; g = 2 Im(G conj(exp(i phi))); one Adam step
// with bias corrections bc1 = 1 - beta1^k, bc2 = 1 - beta2^k (first: the moments
// are zero before it); then the row spectra of the new exp(i phi) -> A.
hipError_t launch_enc_adam(float2 *A, float *phi, float *m, float *v, const float2 *tw, uint32_t nf, uint32_t w,
                           uint32_t h, float lr, float bc1, float bc2, bool first, hipStream_t st);

}  // namespace hpt
