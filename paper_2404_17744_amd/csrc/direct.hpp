// Elementwise kernels of the GF2 direct (bubble) term; host launchers.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace thcsox {

// Pi[b][Q][S] = Gt[b][Q][S] * Gbt[b][S][Q] for b < nb (naux x naux blocks,
// consecutive blocks aa = naux^2 apart).
hipError_t bubble_pi(const double* Gt, const double* Gbt, double* Pi, int naux, int nb,
                     hipStream_t s);
// H[i] = W[i] * Gt[i], i < len (H may alias W).
hipError_t hadamard64(const double* W, const double* Gt, double* H, int64_t len, hipStream_t s);

// A[b] <- W[b] o A[b] and B[b] <- W[b]^T o B[b] for nb matrices [naux][naux] (A or B
// may be null).
hipError_t hadamard_pair(const double* W, double* A, double* B, int naux, int nb, hipStream_t s);

// *flag is set to 1 if V [naux][naux] is not symmetric to rtol element by element, |V_ij -
// V_ji| <= rtol max(|V_ij|, |V_ji|), or holds a value that is not finite.
hipError_t unsymmetric(const double* V, int naux, double rtol, unsigned long long* flag,
                       hipStream_t s);
}  // namespace thcsox
