// Two-kernel transforms for the Krylov iterations of 256^3 grids.
//
// The y transform of length N = 16 * YB is split (decimation): with
// ky = b + YB a and y = jl + 16 jh,
//   inverse: X(y) = sum_b w^(jl b) w_YB^(jh b) [ sum_a x(b + YB a) w_16^(a jl) ],
// so the 16-point part over a, the twiddle and the whole z transform run in
// one kernel on tiles of fixed b, and the YB-point part over b and the whole x
// transform in another on tiles of fixed jl.  A transform of the grid is then
// two passes over memory instead of three.
//
// Layouts (complex elements):
//   spectral vectors ("tile order"): [b][kx / KT][a][kz][kx % KT]
//   spectral to x side:              [b][kx / KT][i][h][jl][kx % KT][z % ZT],
//                                    z = ZT (h + (N / 16 / ZT) i) + z % ZT
//   x to spectral side:              [z / ZT][jl][b][kx][z % ZT]
// A spectral tile (b, kx / KT) and an x tile (z / ZT, jl) share KT * ZT
// adjacent elements (64 bytes).  Between the kernels each writer stores whole
// tiles contiguously and each reader gathers the 64-byte pieces: at 256^3 in
// FP64 stores of scattered pieces reach 2.9 TB/s and loads of them 5.0, against
// 6.0 and 6.3 contiguous.
#pragma once
#include "passes.hpp"

namespace tumor {

template <typename R, int N>
struct TileCfg {
  static constexpr int C = N / 2;
  static constexpr int YB = N / 16;  // second factor of the y transform
  static constexpr int ZB = N / 16;  // second factor of the z transform
  // Columns of a spectral tile and planes of an x tile: 64-byte pieces, and x
  // tiles of 256 threads, two to a CU (FP32 with 512 threads: 0.48 ms for 0.39).
  static constexpr int KT = sizeof(R) == 4 ? 4 : 2;
  static constexpr int ZT = 2;
  // spectral tiles: 16 elements per thread
  static constexpr int TA = N * KT;
  static constexpr int NA = YB * (C / KT);
  // paddings that keep every access of the two exchanges free of bank conflicts
  static constexpr int P1 = KT * ZT, P2 = 1;
  static constexpr int LDSA = 16 * (TA + P1);
  // x tiles: 16 elements per thread (YB values of b for 16 / YB planes)
  static constexpr int L = N / 2, LB = L / 16;
  static constexpr int ZG = ZT * YB / 16;
  static constexpr int TB = C * ZG;
  static constexpr int ROWS = YB * ZT;
  static constexpr int ZH = ZB / ZT;  // x tiles between positions i and i + 1 of a spectral tile
  static constexpr int MS = LB + 1;
  static constexpr int LP = 152;
  static constexpr int NB = (N / ZT) * 16;
  static_assert(LP >= 16 * MS && LP >= L && ZB % ZT == 0 && TB == ROWS * LB, "tile geometry");
};

// tile order index of the spectral element (kz, ky, kx) given as array positions
template <int N, int KT>
__host__ __device__ __forceinline__ long long tile_index(int iz, int iy, int kx) {
  constexpr int YB = N / 16, C = N / 2;
  const int b = iy & (YB - 1), a = iy / YB;
  return (((long long)(b * (C / KT) + kx / KT) * 16 + a) * N + iz) * KT + (kx & (KT - 1));
}

// Spectral side, inverse: with `update`, x += alpha p, p = M^-1 r + beta p
// (tile order, in place); then the nine half arrays of p: U_x, U_y, U_z,
// dy u_x, dy u_y, dz u_y + dy u_z, dz u_x, dz u_z, div u.
struct TileInvArgs {
  const void* r;
  void* p;
  void* x;
  void* out[9];
  const SolveScalars* sv;
  const CoefScalars* cs;
  int update;
};

// x side: the eight half arrays of the stresses (as XElastArgs) from the nine
// of the displacement; each block stores its part of N^3 <p, A p> in epart.
struct TileXArgs {
  const void* in[9];
  void* out[8];
  const void* mu;
  const void* lam;
  const void* eta;
  const SolveScalars* sv;
  double* epart;
};

// Spectral side, forward: q = A p from the eight half arrays, then
// r -= alpha q with alpha = rho / <p, q> totalled from the x side's parts;
// each block stores its part of ||r||^2 and <r, M^-1 r>.
struct TileFwdArgs {
  const void* in[8];
  void* r;
  SolveScalars* sv;
  const CoefScalars* cs;
  const double* epart;
  double* partials;
};

// Start of a solve: r = scale * r64 (natural order, FP64) in tile order,
// p = M^-1 r, x = 0, rho = <r, M^-1 r>; resets the iteration state.
template <typename R>
void launch_tile_start(int n, const void* r64, double scale, void* r, void* p, void* x, const CoefScalars* cs,
                       SolveScalars* sv, double* partials, hipStream_t st);
// End of a solve: x64 (natural order) += scale * (x + alpha p), the last
// iteration's p included; no-op if no iteration ran.
template <typename R>
void launch_tile_final(int n, void* x64, double scale, const void* x, const void* p, const SolveScalars* sv,
                       hipStream_t st);

template <typename R>
void launch_tile_inv(int n, const TileInvArgs& a, const void* tw, hipStream_t st);
template <typename R>
void launch_tile_xelast(int n, const TileXArgs& a, const void* tw, hipStream_t st);
template <typename R>
void launch_tile_fwd(int n, const TileFwdArgs& a, const void* tw, hipStream_t st);
// blocks of launch_tile_fwd (the count of its partials)
template <typename R>
int tile_fwd_blocks(int n);

}  // namespace tumor
