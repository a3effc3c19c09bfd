// The pairing of bins k and L - k that turns an L-point complex transform of
// N = 2L reals into their half spectrum and back, shared by the kernels that
// do it in LDS and the launch that does it in HBM.
//
// With Z the transform of z[m] = x[2m] + i x[2m+1], Fe and Fo those of the
// even and odd samples and w = w_N^k:
//   Fe[k] = (Z[k] + conj Z[L-k]) / 2,   Fo[k] = (Z[k] - conj Z[L-k]) / (2i),
//   X[k] = Fe[k] + w Fo[k],   X[L-k] = conj(Fe[k] - w Fo[k]),
// so one twiddle serves both outputs (Fe[L-k] = conj Fe[k], Fo[L-k] = conj
// Fo[k], w_N^{L-k} = -conj w).  k = 0 pairs Z[0] with itself and gives the
// bins 0 and L; for even L, k = L/2 pairs with itself.
#pragma once
#include "fft_common.h"

namespace dpfft {

// Z[k], Z[L-k], w -> X[k], X[L-k]
__device__ __forceinline__ void real_pair_fwd(cf zk, cf zr, cf w, cf &xk, cf &xr) {
  const cf fe = make_float2(0.5f * (zk.x + zr.x), 0.5f * (zk.y - zr.y));
  const cf fo = make_float2(0.5f * (zk.y + zr.y), -0.5f * (zk.x - zr.x));
  const cf t = cmul(w, fo);
  xk = cadd(fe, t);
  xr = make_float2(fe.x - t.x, t.y - fe.y);
}

// X[k], X[L-k], w -> Fe' + i Fo' at k and at L - k (Fe' = 2 Fe, Fo' = 2 Fo),
// whose inverse transform, halved, holds the samples in pairs.  For k = 0 the
// caller clears the imaginary parts of bins 0 and L, which a Hermitian
// spectrum has real.
__device__ __forceinline__ void real_pair_inv(cf xk, cf xr, cf w, cf &zk, cf &zr) {
  const cf fe = make_float2(xk.x + xr.x, xk.y - xr.y);
  const cf fo = cmul(make_float2(xk.x - xr.x, xk.y + xr.y), make_float2(w.x, -w.y));
  zk = make_float2(fe.x - fo.y, fe.y + fo.x);
  zr = make_float2(fe.x + fo.y, fo.x - fe.y);
}

}  // namespace dpfft
