// Spectral preconditioners of the Krylov solves, shared by the vector kernels
// and the fused FFT passes.
#pragma once
#include "kernels.hpp"

namespace tumor {

// The elasticity inverse's two coefficients (below), 1/a and c / (a + c |w|^2),
// from one division by a d and without a branch; m: the coefficient means.  For
// FP64 vectors the factors are first scaled (exactly) by the exponent of a: a d is
// out of range beyond moduli of 1e154 (or 1e-154).  FP32 vectors' coefficients, below
// 1e38, keep it in range.
struct ElastMeans {
  double eta, mu, c;
  __device__ __forceinline__ explicit ElastMeans(const CoefScalars* cs)
      : eta(cs->etabar), mu(cs->mubar), c(cs->lambar + cs->mubar) {}
};
template <typename R>
__device__ __forceinline__ void elast_prec_coefs(double w2, const ElastMeans& m, double& ia, double& f) {
  double a = m.eta + m.mu * w2;
  double d = a + m.c * w2, c = m.c;
  const bool ok = a > 0.0;
  int e = 0;
  if constexpr (sizeof(R) == 8) {
    a = frexp(a, &e);
    d = ldexp(d, -e);
    c = ldexp(c, -e);
  }
  const double inv = 1.0 / (ok ? a * d : 1.0);
  ia = ok ? d * inv : 0.0;
  if constexpr (sizeof(R) == 8) ia = ldexp(ia, -e);
  f = c * a * inv;
}

// Constant-coefficient inverses per Fourier mode (integer wave numbers
// kx, ky, kz with the Nyquist mode already mapped to 0):
//   CN diffusion:  1 / (1 + dt/2 mean(K) |w|^2)
//   elasticity:    (1/a) [I - c w w^T / (a + c |w|^2)], a = mean(eta) + mean(mu)|w|^2,
//                  c = mean(lambda) + mean(mu)  (Sherman-Morrison); a = 0 maps to 0.
template <typename R, int NC>
__device__ __forceinline__ void apply_prec(const cplx<R> (&r)[NC], cplx<R> (&z)[NC], int kx, int ky, int kz,
                                           const CoefScalars* cs, const PrecConsts& pc) {
  const double w2 = (double)kx * kx + (double)ky * ky + (double)kz * kz;
  if constexpr (NC == 1) {
    const R s = R(1.0 / (1.0 + pc.h * cs->Kbar * w2));
    z[0] = cscale(r[0], s);
  } else {
    const double a = cs->etabar + cs->mubar * w2;
    if (a > 0.0) {
      const double c = cs->lambar + cs->mubar;
      const R ia = R(1.0 / a);
      const R f = R(c / (a + c * w2));
      const R wk[3] = {R(kx), R(ky), R(kz)};
      cplx<R> wr;
      wr.x = wk[0] * r[0].x + wk[1] * r[1].x + wk[2] * r[2].x;
      wr.y = wk[0] * r[0].y + wk[1] * r[1].y + wk[2] * r[2].y;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        z[b].x = (r[b].x - f * wk[b] * wr.x) * ia;
        z[b].y = (r[b].y - f * wk[b] * wr.y) * ia;
      }
    } else {
#pragma unroll
      for (int b = 0; b < 3; ++b) z[b] = czero<R>();
    }
  }
}


}  // namespace tumor
