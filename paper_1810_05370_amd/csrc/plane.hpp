// Krylov iterations of small grids (16^3 to 64^3) in three kernels.
//
// On these grids a kernel lasts as long as one block's chain of transforms,
// so an iteration is as fast as its chains are short and its kernels few.
//   inverse: per kx plane and output, z = M^-1 r, then the whole y and z
//            transform of one half array in LDS;
//   x side:  one wave per row transform of the operator;
//   forward: per kx plane and component, A z, then every vector update.
// Both inner products are known before the update (Chronopoulos and Gear's
// arrangement of CG, 1989): gamma = <r, z> and ||r||^2 are summed by the
// inverse kernel, delta = <z, A z> in its energy form by the x side, and
//   beta = gamma / gamma', alpha = gamma / (delta - beta gamma / alpha'),
//   p = z + beta p, s = A z + beta s (= A p), x += alpha p, r -= alpha s.
//
// Measured per elasticity iteration, against five passes, an update and its
// scalars in one kernel each: FP64 32^3 83 -> 20 us, FP32 64^3 93 -> 37 us.  What
// is left per kernel (5 to 14 us) is the launch (2.3 us), one round trip to
// memory and one chain of transforms.  LDS is kept small: the forward kernel
// with its three z transforms side by side in 58 instead of 20 KB lasted 10.5 us
// instead of 7.4 (32^3), nine waves to an x block 11.8 instead of 6.9.
//
// Layouts: spectral vectors [kx][kz][ky] per component, half arrays (after the
// y and z transforms) [kx][z][y].
#pragma once
#include "passes.hpp"

namespace tumor {

// One solve's vectors.  `nc` blocks of S: the three components of the
// elasticity system, or up to three independent diffusion systems.
struct PlaneArgs {
  void *r, *z, *s, *p, *x;
  void* half[9];  // elasticity 8 (as XElastArgs), diffusion 3 per system; x side in place
  const void* prec;  // per mode (1 / a, c / (a + c w^2)), or the diffusion's inverse (launch_plane_start)
  const void* mu;    // elasticity coefficients ([pair][row], launch_plane_coefs); diffusion: K in `lam`
  const void* lam;
  const void* eta;
  const SolveScalars* sv;  // state before this iteration (nc entries for diffusion)
  SolveScalars* svn;       // state after it
  const CoefScalars* cs;
  double* part;   // inverse: per system and plane gamma, ||r||^2, ||z||^2
  double* epart;  // x side: per system (and direction) and block the energy
  double h;       // diffusion: dt / 2
  int nc;
  double thr2[kMaxSys];
  int limit[kMaxSys];
  int fixed[kMaxSys];
};

// One kernel of an iteration: stage 0 inverse, 1 x side, 2 forward.
template <typename R>
void launch_plane(int n, bool elast, int stage, const PlaneArgs& a, const void* tw, hipStream_t st);
// `count` coefficient fields turned into the x side's order.
template <typename R>
void launch_plane_coefs(int n, int count, const void* const* in, void* const* out, hipStream_t st);
// Start: r = scale_k * r64_k (natural order) for the systems in `active`, the
// state of every system reset (inactive ones done).  One `sv` entry per system,
// or one in all for elasticity.
template <typename R>
void launch_plane_start(int n, bool elast, const void* r64, const double (&scale)[kMaxSys], int active,
                        const PlaneArgs& a, SolveScalars* sv, hipStream_t st);
// End: x64_k (natural order) += scale_k x_k for the systems in `active` that iterated.
template <typename R>
void launch_plane_final(int n, bool elast, void* x64, const double (&scale)[kMaxSys], int active, const PlaneArgs& a,
                        const SolveScalars* sv, hipStream_t st);

}  // namespace tumor
