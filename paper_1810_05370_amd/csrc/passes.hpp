// Axis passes of the 3-D real FFT on the periodic N^3 grid, with the spectral
// symbols and pointwise physical-space work of each operator fused in.
//
// Layouts (all C order, x fastest):
//   physical  real    [z][y][x]                        N^3 values
//   spectral  complex [kz][ky][kxp], kxp in [0, N/2)   N^3/2 values
// The spectral array is the x-R2C half spectrum with the real Nyquist
// coefficient (kx = N/2) packed into the imaginary part of the kx = 0
// coefficient.  Both packed planes share w_x = 0 (the Nyquist wave number is
// dropped in every derivative), so every symbol used here acts on the packed
// column exactly as on the two planes separately.  Forward transforms are
// unnormalised, inverse transforms are unnormalised; the 1/N^3 lives in the
// physical-space step of each operator.
//
// Pass kinds:
//   col_pass  : FFT along y or z for a tile of TC adjacent kxp columns.  A
//               small program (ColProg) says which input columns are combined
//               with which axis symbol into each output.
//   xpass_*   : FFT along x (packed R2C / C2R) for a tile of rows, with the
//               operator's physical-space work between the inverse and the
//               forward transform, all in registers.
#pragma once
#include "fft.hpp"
#include "kernels.hpp"

namespace tumor {

constexpr int kMaxCol = 9;
constexpr int kMaxTerms = 3;
// Grids up to this size share the outputs of a pass out over grid layers.  A
// pass at 64^3 or below has at most 64 column tiles or 256 row waves, far too
// few to fill 256 CUs, and lasts as long as one block's chain of transforms.
constexpr int kSplitMaxN = 64;
// Grids whose elasticity iteration runs on the two-kernel transforms (tile.hpp).
// At 256^3 it moves 58 arrays instead of 89 (FP32 1.23 -> 1.13 ms, FP64 2.44 ->
// 2.10).  At 128^3 there are 128 (FP32) or 256 (FP64) spectral tiles for 256 CUs
// and the FP64 x side keeps one wave per SIMD: a solve of 47 iterations takes 15.2
// ms for 13.9 in FP64, one of 48 10.4 for 8.2 in FP32.  A 512^3 tile does not fit
// LDS with 64-byte pieces.
constexpr bool tile_grid(int n) { return n == 256; }
// Grids whose Krylov iterations run in three kernels on kx planes (plane.hpp),
// 8 elements a thread: a plane of 128^2 would take 2048 threads, and in FP64 does
// not fit LDS either (295 KB; in FP32 147 of 160 KB).
constexpr bool plane_grid(int n) { return n <= 64; }

enum ColSym : int { SYM_ONE = 0, SYM_IW = 1, SYM_RAW = 2 };

struct ColTerm {
  int src;
  int sym;      // ColSym
  double coef;  // real multiplier
};

// Inverse pass: out[o] = IFFT_axis( sum_t coef_t * s_t(k) * in[src_t] )
// Forward pass: out[o] = sum_t coef_t * s_t(k) * FFT_axis(in[src_t])
//               (SYM_RAW: the input is read at the output position, untransformed)
struct ColProg {
  const void* in[kMaxCol];
  void* out[kMaxCol];
  int nout;
  int nterm[kMaxCol];
  ColTerm term[kMaxCol][kMaxTerms];
  const int* skip;  // if non-null and *skip != 0 the launch does nothing
  // per output: if non-null and *oskip[o] != 0, output o is not computed
  // (a converged system of a batched solve)
  const int* oskip[kMaxCol];
  // Optional, in the forward y pass of a Krylov apply: the totals per z plane
  // and system of <p, A p>, from the x pass's energies and, with ppart, the
  // first pass's squared norms of p: esum[system * N + plane] =
  // escale * (the plane's epart) + (as many ppart).
  double* esum;
  const double* epart;
  const double* ppart;
  double escale;
  int nes;  // systems
};

// First (inverse z) pass of a Krylov operator apply with the direction update
// fused in: p = M^-1 r + beta p (in place), then out[2a] = IFFT_z(p_a) and
// out[2a+1] = IFFT_z(i w_z p_a) for the NC components.
// With nsys > 0 the vectors hold nsys independent one-component systems
// (scalars sv[0 .. nsys)); a system whose solve is done is left untouched.
struct ZPUpdateArgs {
  const void* r;
  void* p;
  void* x;  // x += alpha p with the previous p and alpha, before p is replaced
  void* out[6];
  SolveScalars* sv;
  const CoefScalars* cs;
  PrecConsts pc;
  int nsys;
  // nsys > 0: each block's part of ||p||^2 at ppart[block * nsys + system]; `first`
  // transforms p as it is (the start has made it)
  double* ppart;
  int first;
};

// Last (forward z) pass of a Krylov operator apply with the residual update
// fused in: q = A p is formed in registers, alpha = rho / <p, q> comes from the N
// plane totals at esum, r -= alpha q in place; each block stores its parts of
// ||r||^2 and <r, M^-1 r> at partials[2 * (system * tiles + tile)].  Elasticity (nsys 0): q_c = F in[c] - i w_z F in[3 + c]; system
// s of a batch: q = p - h (F in[2s] + i w_z F in[2s + 1]).
struct ZUpdateArgs {
  const void* in[6];
  void* r;
  const void* p;  // batch
  SolveScalars* sv;
  const CoefScalars* cs;
  const double* esum;
  double* partials;
  PrecConsts pc;
  int nsys;
};

// Rows of the x pass: generic programs.
//   xinv: phys_out[o] = scale * C2R( sum_t coef_t * s_t(kx) * in[src_t] )
//   xfwd: spec_out[o] = R2C( sum_t coef_t * phys_in[src_t] )
struct XProg {
  const void* in[kMaxCol];
  void* out[kMaxCol];
  int nout;
  int nterm[kMaxCol];
  ColTerm term[kMaxCol][kMaxTerms];
  double scale;
  const int* skip;
};

// Elasticity x pass.  Inputs (packed spectral rows, after the y and z inverse
// passes): U_x, U_y, U_z, dy u_x, dy u_y, (dz u_y + dy u_z), dz u_x, dz u_z.
// Coefficients (physical): mu, lambda, eta.  Outputs (packed spectral rows):
// eta u_x - dx s_xx, eta u_y - dx s_xy, eta u_z - dx s_xz, s_xy, s_yy, s_yz,
// s_xz, s_zz, where s = mu (grad u + grad u^T) + lambda div u I.
struct XElastArgs {
  const void* in[8];
  void* out[8];
  const void* mu;
  const void* lam;
  const void* eta;
  const int* skip;
  double* epart;  // nullable: each row tile's part of <p, A p> (N^3 times its energy)
};

// Diffusion x pass for ns fields (systems) sharing K.  Inputs per field s:
// C, dy c, dz c (packed rows) at in[3s .. 3s+2]; coefficient K.  Outputs:
// i w_x F(K dx c), F(K dy c), F(K dz c) at out[3s .. 3s+2] (each may be its
// own input).  Field s is skipped if skip[s] is non-null and *skip[s] != 0.
struct XDiffArgs {
  const void* in[9];
  void* out[9];
  const void* K;
  const int* skip[3];
  int ns;
  double* epart;  // nullable: epart[tile * ns + s] = the row tile's part of -<c, D c>
};

// Force x pass.  Inputs: T, dy t, dz t (packed rows of tau = p + n).
// Outputs: F(-zeta tanh(tau) d_a tau), a = x, y, z.
struct XForceArgs {
  const void* in[3];
  void* out[3];
  double zeta;
};

// Products in physical space on the x pass (the coefficient sensitivities of
// the adjoint).  A factor is C2R( sum of up to kMaxTerms terms coef * s(kx) *
// in[src] ) of packed rows after the y and z inverse passes; each output is
//   out[o] (=, or += with accumulate) sum_d coef[o][d] * A_od * B_od,
// with B_od = 1 when its factor has no terms.  Outputs are physical FP64.
constexpr int kMaxDotIn = 16;
constexpr int kMaxDotOut = 6;
constexpr int kMaxDotProd = 6;
// compact term (kernel arguments are limited to 4 KiB)
struct DotTerm {
  short src;
  short sym;    // ColSym
  float coef;   // small exact multipliers (1, 2)
};
struct XFactor {
  int nterm;
  DotTerm term[kMaxTerms];
};
struct XDotArgs {
  const void* in[kMaxDotIn];
  double* out[kMaxDotOut];
  int nout;
  int accumulate[kMaxDotOut];
  int nprod[kMaxDotOut];
  XFactor fa[kMaxDotOut][kMaxDotProd];
  XFactor fb[kMaxDotOut][kMaxDotProd];
  double coef[kMaxDotOut][kMaxDotProd];
};
static_assert(sizeof(XDotArgs) <= 3072, "kernel arguments are limited to 4 KiB");

struct PassGeom {
  int n;
};

// Host-side launchers, instantiated for R = double and float.
template <typename R>
void launch_col_pass(int n, int axis /*1 = y, 2 = z*/, bool inverse, const ColProg& prog,
                     const void* tw, hipStream_t st);
template <typename R>
void launch_zinv_pupdate(int n, const ZPUpdateArgs& a, const void* tw, hipStream_t st);
template <typename R>
void launch_xinv(int n, const XProg& prog, const void* tw, hipStream_t st);
template <typename R>
void launch_xfwd(int n, const XProg& prog, const void* tw, hipStream_t st, bool in_fp64);
template <typename R>
void launch_xelast(int n, const XElastArgs& a, const void* tw, hipStream_t st);
template <typename R>
void launch_xdiff(int n, const XDiffArgs& a, const void* tw, hipStream_t st);
template <typename R>
void launch_xforce(int n, const XForceArgs& a, const void* tw, hipStream_t st);
template <typename R>
void launch_xdot(int n, const XDotArgs& a, const void* tw, hipStream_t st);
template <typename R>
void launch_zfwd_update(int n, const ZUpdateArgs& a, const void* tw, hipStream_t st);
// tiles of a fused last pass (the count of its partials)
template <typename R>
int z_tiles(int n);
// row tiles of an x pass (RowCfg: one wave of 64 threads, n / 16 to a row)
constexpr long long x_tiles(long long n) { return n * n * n / 1024; }
// no grid has more tiles of a fused first or last pass
constexpr long long max_z_tiles(long long n) { return n * n / 16; }

}  // namespace tumor
