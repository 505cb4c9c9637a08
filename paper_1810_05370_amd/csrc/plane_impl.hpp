// Kernels and launchers of the small grids' Krylov iterations (see plane.hpp).
#pragma once
#include "passes_impl.hpp"
#include "plane.hpp"

namespace tumor {

template <typename R, int N>
struct PlaneCfg {
  static constexpr int C = N / 2, TP = N / 8, TH = N * TP;  // threads of a plane: 8 elements each
  static constexpr int LY = N + N / 8;  // padded line in LDS: no bank conflicts between a wave's lines
  static constexpr int LDS = N * LY;
  // x side: RW rows per wave, TX threads a row
  static constexpr int L = N / 2, TX = L / 8, RW = 64 / TX, LX = (L + L / 8 + 1) | 1, NX = N * N / RW;
  static_assert(RW * LX >= 64 * 8, "a wave's row buffer also holds its 8 values per lane");
};

// Totals over the block (fixed order), valid in every thread; sh: NV * TH / 64
// doubles, rounded up.  A 16^3 plane's block is half a wave.
template <int NV, int TH>
__device__ __forceinline__ void plane_totals(double (&v)[NV], double* sh) {
  constexpr int NW = (TH + 63) / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double s = v[i];
#pragma unroll
    for (int off = (TH < 64 ? TH : 64) / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) sh[i * NW + wv] = s;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double s = 0.0;
    for (int k = 0; k < NW; ++k) s += sh[i * NW + k];
    v[i] = s;
  }
}

// Thread roles in a plane: y lines (position kz, ky = ty + TP j) for spectral
// access, z lines (position y, z = tz + TP j) for half arrays; both contiguous
// in memory across lanes.
template <typename R, int N>
struct PlaneThread {
  using T = PlaneCfg<R, N>;
  int kz, ty, y, tz;
  cplx<R>* buf;
  __device__ __forceinline__ explicit PlaneThread(cplx<R>* b) : buf(b) {
    kz = threadIdx.x / T::TP;
    ty = threadIdx.x % T::TP;
    y = threadIdx.x % N;
    tz = threadIdx.x / N;
  }
  __device__ __forceinline__ int spec(int j) const { return kz * N + ty + T::TP * j; }
  __device__ __forceinline__ int half(int j) const { return (tz + T::TP * j) * N + y; }
  template <bool INV>
  __device__ __forceinline__ void fft_y(cplx<R> (&v)[8], const cplx<R>* tw) const {
    fft_block<R, N, INV, 1>(v, LdsView<R>{buf + kz * T::LY, 1, 1}, ty, tw);
  }
  template <bool INV>
  __device__ __forceinline__ void fft_z(cplx<R> (&v)[8], const cplx<R>* tw) const {
    fft_block<R, N, INV, 1>(v, LdsView<R>{buf + y, N, 0}, tz, tw);
  }
  // y role -> z role and back
  __device__ __forceinline__ void to_z(cplx<R> (&v)[8]) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) buf[kz * T::LY + ty + T::TP * j] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = buf[(tz + T::TP * j) * T::LY + y];
    __syncthreads();
  }
  __device__ __forceinline__ void to_y(cplx<R> (&v)[8]) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) buf[(tz + T::TP * j) * T::LY + y] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = buf[kz * T::LY + ty + T::TP * j];
    __syncthreads();
  }
};

template <typename R>
__device__ __forceinline__ double pdot(cplx<R> a, cplx<R> b) {
  return (double)a.x * (double)b.x + (double)a.y * (double)b.y;
}

// --------------------------------------------------------------- elasticity
// blockIdx.x: kx plane, blockIdx.y: half array.  The first three layers also
// store z, the first the plane's part of gamma and ||r||^2.  Bound by the chain
// (z transform, exchange, y transform): FP64 32^3 5.3 us, FP32 64^3 11.3, FP64
// 64^3 11.6, against two passes of 8 to 13 us.
template <typename R, int N>
__global__ void __launch_bounds__((PlaneCfg<R, N>::TH)) k_plane_inv(PlaneArgs a, const cplx<R>* __restrict__ twg) {
  using T = PlaneCfg<R, N>;
  constexpr long long S = (long long)N * N * T::C;
  __shared__ cplx<R> buf[T::LDS];
  __shared__ cplx<R> stw[N];
  __shared__ double sh[16];
  const PlaneThread<R, N> th(buf);
  const int kx = blockIdx.x, o = blockIdx.y, kz = wavenum<N>(th.kz);
  const long long base = (long long)kx * N * N;
  // the output is (one + i w) z_c, w = ky, kz or 0; dz u_y + dy u_z has a second
  // term (c, w) = (2, ky).  Block-uniform values without branches in the loops.
  const int c0 = o < 3 ? o : (o < 6 ? (o == 3 ? 0 : 1) : (o == 6 ? 0 : 2));
  const R one = R(o < 3 ? 1 : 0), by = R(o == 3 || o == 4 ? 1 : 0), bz = R(o >= 5 ? 1 : 0);
  const R fx = R(c0 == 0 ? kx : 0), fy = R(c0 == 1 ? 1 : 0), fz = R(c0 == 2 ? kz : 0);
  const cplx<R>* r = static_cast<const cplx<R>*>(a.r) + base;
  cplx<R> rv[3][8], rc[8], pc[8], wr[8], v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
#pragma unroll
    for (int c = 0; c < 3; ++c) rv[c][j] = r[c * S + th.spec(j)];
    rc[j] = r[c0 * S + th.spec(j)];
    pc[j] = static_cast<const cplx<R>*>(a.prec)[base + th.spec(j)];
  }
  for (int k = threadIdx.x; k < N; k += T::TH) stw[k] = twg[k];
  hold_loads();
  if (a.sv->done) return;
  R ky[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    ky[j] = R(wavenum<N>(th.ty + T::TP * j));
    wr[j] = {R(kx) * rv[0][j].x + ky[j] * rv[1][j].x + R(kz) * rv[2][j].x,
             R(kx) * rv[0][j].y + ky[j] * rv[1][j].y + R(kz) * rv[2][j].y};
    // z_c = (r_c - f k_c (k . r)) / a
    const R fk = pc[j].y * (fx + fy * ky[j] + fz);
    const cplx<R> z = {(rc[j].x - fk * wr[j].x) * pc[j].x, (rc[j].y - fk * wr[j].y) * pc[j].x};
    const R w = by * ky[j] + bz * R(kz);
    v[j] = {one * z.x - w * z.y, one * z.y + w * z.x};
    rc[j] = z;
  }
  if (o == 5) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const R fk = pc[j].y * R(kz);
      const cplx<R> z = {(rv[2][j].x - fk * wr[j].x) * pc[j].x, (rv[2][j].y - fk * wr[j].y) * pc[j].x};
      v[j] = cadd(v[j], ciw(z, ky[j]));
    }
  }
  double acc[2] = {0.0, 0.0};
  if (o < 3) {
    cplx<R>* zd = static_cast<cplx<R>*>(a.z) + base + c0 * S;
#pragma unroll
    for (int j = 0; j < 8; ++j) zd[th.spec(j)] = rc[j];
  }
  if (o == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const R wk[3] = {R(kx), ky[j], R(kz)};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const cplx<R> x = rv[c][j];
        const cplx<R> z = {(x.x - pc[j].y * wk[c] * wr[j].x) * pc[j].x, (x.y - pc[j].y * wk[c] * wr[j].y) * pc[j].x};
        acc[0] += pdot(x, z);
        acc[1] += pdot(x, x);
      }
    }
  }
  __syncthreads();
  th.template fft_y<true>(v, stw);
  th.to_z(v);
  th.template fft_z<true>(v, stw);
  cplx<R>* dst = static_cast<cplx<R>*>(a.half[o]) + base;
#pragma unroll
  for (int j = 0; j < 8; ++j) dst[th.half(j)] = v[j];
  if (o == 0) {
    // Parseval weight: the packed kx = 0 plane counts once, the others twice
    const double wt = kx == 0 ? 1.0 : 2.0;
    plane_totals<2, T::TH>(acc, sh);
    if (threadIdx.x == 0) {
      a.part[3 * kx] = acc[0] * wt;
      a.part[3 * kx + 1] = acc[1] * wt;
    }
  }
}

// Row access of the x side: RW consecutive rows (lanes) of the wave's tile.
template <typename R, int N>
struct PlaneRow {
  using T = PlaneCfg<R, N>;
  int t, row;  // position in the row, row of the grid
  LdsRowView<R> lds;
  __device__ __forceinline__ PlaneRow(cplx<R>* wbuf, int tile) {
    const int lane = threadIdx.x & 63;
    t = lane / T::RW;
    const int rl = lane % T::RW;
    row = tile * T::RW + rl;
    lds.buf = wbuf + rl * T::LX;
  }
  // the row's values of f at k = t + TX j and at L - k
  __device__ __forceinline__ void load(cplx<R> (&A)[8], cplx<R> (&B)[8], const cplx<R>* f) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = t + T::TX * j;
      A[j] = f[k * (N * N) + row];
      B[j] = f[((T::L - k) & (T::L - 1)) * (N * N) + row];
    }
  }
  __device__ __forceinline__ void iwx(cplx<R> (&A)[8], cplx<R> (&B)[8]) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = t + T::TX * j;
      A[j] = ciw(A[j], R(k));
      B[j] = ciw(B[j], R((T::L - k) & (T::L - 1)));
    }
  }
  // v = C2R of the loaded row, times N^3
  __device__ __forceinline__ void c2r(cplx<R> (&v)[8], const cplx<R> (&A)[8], const cplx<R> (&B)[8],
                                      const cplx<R>* tw) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = c2r_pre<R, N>(A[j], B[j], t + T::TX * j, tw);
    fft_block<R, T::L, true, 2, LdsRowView<R>, false, true>(v, lds, t, tw);
  }
  // coefficient pairs at p = t + TX j ([p][row] order)
  __device__ __forceinline__ void coef(cplx<R> (&c)[8], const void* f) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = static_cast<const cplx<R>*>(f)[(t + T::TX * j) * (N * N) + row];
  }
  __device__ __forceinline__ void store(cplx<R>* dst, const cplx<R> (&v)[8]) const {
#pragma unroll
    for (int j = 0; j < 8; ++j) dst[(t + T::TX * j) * (N * N) + row] = v[j];
  }
};

// blockIdx.x: RW rows; each wave one inverse and one forward row transform.
// blockIdx.y = 0: d_x u_x, d_y u_y, d_z u_z, u_x; 1: the xy shear, u_y, the xz
// shear, u_z; 2: the yz shear (one wave).  In place: a wave that needs another's
// rows has read its own before the block's first barrier.  A wave holds one
// inverse and one forward row, so the chain is two transforms and the trace's
// exchange: FP64 32^3 6.9 us, FP32 64^3 11.9, FP64 64^3 14.2.
template <typename R, int N>
__global__ void __launch_bounds__(256) k_plane_xelast(PlaneArgs a, const cplx<R>* __restrict__ twg) {
  using T = PlaneCfg<R, N>;
  __shared__ cplx<R> buf[4][T::RW * T::LX];
  __shared__ cplx<R> stw[N];
  __shared__ double sh[4];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, role = blockIdx.y * 4 + wv;
  const PlaneRow<R, N> rw(buf[wv], blockIdx.x);
  const R invV = R(1.0) / (R(N) * R(N) * R(N));
  auto half = [&](int f) { return static_cast<cplx<R>*>(a.half[f]); };
  //                        exx eyy ezz u_x s_xy u_y s_xz u_z s_yz
  constexpr int src[12] = {0, 4, 7, 0, 1, 1, 2, 2, 5, 5, 5, 5};
  constexpr int dst[12] = {0, 4, 7, 0, 3, 1, 6, 2, 5, 5, 5, 5};
  const bool diag = role < 3, shear = role == 4 || role == 6, disp = role < 8 && (role & 1) && role != 1;
  // the loads run before the solve's state is known: one round trip to memory
  cplx<R> A[8], B[8], c[8], l[8], v[8];
  rw.load(A, B, half(src[role]));
  for (int k = threadIdx.x; k < N; k += 256) stw[k] = twg[k];
  if (shear) {
    cplx<R> A2[8], B2[8];
    rw.load(A2, B2, half(dst[role]));
    rw.iwx(A, B);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      A[j] = cadd(A[j], A2[j]);
      B[j] = cadd(B[j], B2[j]);
    }
  } else if (role == 0) {
    rw.iwx(A, B);
  }
  rw.coef(c, disp ? a.eta : a.mu);
  if (diag) rw.coef(l, a.lam);
  hold_loads();
  if (a.sv->done) return;
  __syncthreads();
  rw.c2r(v, A, B, stw);  // N^3 times the strain or displacement
  // the trace: the diagonal strains pass through the waves' row buffers
  cplx<R>* mine = buf[wv];
  wave_sync();
  if (diag) {
#pragma unroll
    for (int j = 0; j < 8; ++j) mine[j * 64 + lane] = v[j];
  }
  __syncthreads();
  double acc[1] = {0.0};
  cplx<R> w[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) w[j] = {c[j].x * v[j].x, c[j].y * v[j].y};
  if (diag) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const cplx<R> e0 = buf[0][j * 64 + lane], e1 = buf[1][j * 64 + lane], e2 = buf[2][j * 64 + lane];
      w[j] = {R(2) * w[j].x + l[j].x * (e0.x + e1.x + e2.x), R(2) * w[j].y + l[j].y * (e0.y + e1.y + e2.y)};
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) w[j] = {w[j].x * invV, w[j].y * invV};
  if (role < 9) {
    // <z, A z> of the spectral vectors is N^3 times the physical sum (and products of
    // two physical values would underflow N^3 times as early)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[0] += pdot(w[j], v[j]);
  }
  __syncthreads();
  row_r2c<R, N, false, true>(w, rw.lds, rw.t, stw);
  // s_xx, s_xy, s_xz to the waves of u_x, u_y, u_z
  wave_sync();
  if (role == 0 || shear) {
#pragma unroll
    for (int j = 0; j < 8; ++j) mine[j * 64 + lane] = w[j];
  }
  __syncthreads();
  if (disp) {
    const cplx<R>* other = buf[role == 3 ? 0 : wv - 1];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = csub(w[j], ciw(other[j * 64 + lane], R(rw.t + T::TX * j)));
  }
  if (role != 0 && role < 9) rw.store(half(dst[role]), w);
  plane_totals<1, 256>(acc, sh);
  if (threadIdx.x == 0) a.epart[blockIdx.y * T::NX + blockIdx.x] = acc[0];
}

// The iteration's scalars from gamma, ||r||^2 and delta; false: no update.
// Every block computes them from the same totals; the first one stores them.
// As on the larger grids, the first gamma has to be positive (an indefinite
// preconditioner is refused) and every curvature.
__device__ __forceinline__ bool plane_scalars(const SolveScalars& s, double gamma, double rr, double delta, double thr2,
                                              int limit, int fixed, SolveScalars* out, bool store, double& alpha,
                                              double& beta) {
  SolveScalars n = s;
  n.rr = rr;
  beta = s.it > 0 ? gamma / s.rho : 0.0;
  const double den = s.it > 0 ? delta - beta * gamma / s.alpha : delta;
  alpha = gamma / den;
  bool go = false;
  if (!(isfinite(gamma) && isfinite(rr) && isfinite(delta)) || (s.it == 0 && !(gamma > 0.0))) {
    n.bad = 1;
    n.done = 1;
  } else if (!fixed && rr <= thr2) {
    n.conv = 1;
    n.done = 1;
  } else if (s.it >= limit) {
    n.conv = fixed ? 1 : 0;
    n.done = 1;
  } else if (!(isfinite(alpha) && den > 0.0)) {
    n.bad = 1;
    n.done = 1;
  } else {
    go = true;
    n.it = s.it + 1;
    n.rho = gamma;
    n.alpha = alpha;
    n.beta = beta;
    n.pq = den;
  }
  if (store) *out = n;
  return go;
}

// The update's vectors of one component (or system); off: its plane.
template <typename R, int N>
struct PlaneVecs {
  cplx<R>*r, *s, *p, *x;
  cplx<R> rv[8], sv[8], pv[8], xv[8];
  __device__ __forceinline__ PlaneVecs(const PlaneArgs& a, long long off)
      : r(static_cast<cplx<R>*>(a.r) + off),
        s(static_cast<cplx<R>*>(a.s) + off),
        p(static_cast<cplx<R>*>(a.p) + off),
        x(static_cast<cplx<R>*>(a.x) + off) {}
  // the first iteration starts the recurrences
  __device__ __forceinline__ void load(const PlaneThread<R, N>& th, bool first) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      rv[j] = r[th.spec(j)];
      sv[j] = pv[j] = xv[j] = czero<R>();
    }
    if (!first) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        sv[j] = s[th.spec(j)];
        pv[j] = p[th.spec(j)];
        xv[j] = x[th.spec(j)];
      }
    }
    hold_loads();
  }
  // p, s, x and r from w = A z
  __device__ __forceinline__ void update(const PlaneThread<R, N>& th, const cplx<R> (&w)[8], const cplx<R> (&zv)[8],
                                         R alpha, R beta) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = th.spec(j);
      const cplx<R> sn = {w[j].x + beta * sv[j].x, w[j].y + beta * sv[j].y};
      const cplx<R> pn = {zv[j].x + beta * pv[j].x, zv[j].y + beta * pv[j].y};
      s[e] = sn;
      p[e] = pn;
      x[e] = {xv[j].x + alpha * pn.x, xv[j].y + alpha * pn.y};
      r[e] = {rv[j].x - alpha * sn.x, rv[j].y - alpha * sn.y};
    }
  }
};

// Forward y and z transforms of g + sign (iw_y F(u) + iw_z F(w)) (sign -1 for the
// elasticity, +1 for the diffusion's divergence), left in the y role.
template <typename R, int N>
__device__ __forceinline__ void plane_div(cplx<R> (&g)[8], cplx<R> (&u)[8], cplx<R> (&w)[8],
                                          const PlaneThread<R, N>& th, R sign, const cplx<R>* stw,
                                          PlaneVecs<R, N>& vecs, bool first) {
  using T = PlaneCfg<R, N>;
  th.template fft_z<false>(g, stw);
  th.template fft_z<false>(w, stw);
#pragma unroll
  for (int j = 0; j < 8; ++j) g[j] = cadd(g[j], ciw(w[j], sign * R(wavenum<N>(th.tz + T::TP * j))));
  th.template fft_z<false>(u, stw);
  th.to_y(g);
  th.template fft_y<false>(g, stw);
  th.to_y(u);
  vecs.load(th, first);
  th.template fft_y<false>(u, stw);
#pragma unroll
  for (int j = 0; j < 8; ++j) g[j] = cadd(g[j], ciw(u[j], sign * R(wavenum<N>(th.ty + T::TP * j))));
}

// blockIdx.x: kx plane, blockIdx.y: component; the vector update with the
// plane in registers.  Bound by five transforms in a chain, the vectors' loads
// hidden under the last: FP32 64^3 14.0 us, FP64 32^3 7.4, 64^3 21.3 (its 256
// registers leave the scheduler little to hide with).
template <typename R, int N>
__global__ void __launch_bounds__((PlaneCfg<R, N>::TH)) k_plane_fwd(PlaneArgs a, const cplx<R>* __restrict__ twg) {
  using T = PlaneCfg<R, N>;
  constexpr long long S = (long long)N * N * T::C;
  __shared__ cplx<R> buf[T::LDS];
  __shared__ cplx<R> stw[N];
  __shared__ double sh[32];
  const PlaneThread<R, N> th(buf);
  const int c = blockIdx.y;
  const long long base = (long long)blockIdx.x * N * N, off = base + c * S;
  auto half = [&](int f) { return static_cast<const cplx<R>*>(a.half[f]) + base; };
  // (A z)_x = F0 - dy F3 - dz F6, (A z)_y = F1 - dy F4 - dz F5, (A z)_z = F2 - dy F5 - dz F7;
  // every load at once: one round trip to memory
  cplx<R> g[8], u[8], w[8], zv[8];
  const cplx<R>*fm = half(c), *fy = half(c == 0 ? 3 : c + 3), *fz = half(c == 0 ? 6 : (c == 1 ? 5 : 7)),
               *z = static_cast<const cplx<R>*>(a.z) + off;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    g[j] = fm[th.half(j)];
    w[j] = fz[th.half(j)];
    u[j] = fy[th.half(j)];
    zv[j] = z[th.spec(j)];
  }
  for (int k = threadIdx.x; k < N; k += T::TH) stw[k] = twg[k];
  double tot[3] = {0.0, 0.0, 0.0};
  for (int k = threadIdx.x; k < T::C; k += T::TH) {
    tot[0] += a.part[3 * k];
    tot[1] += a.part[3 * k + 1];
  }
  for (int k = threadIdx.x; k < 3 * T::NX; k += T::TH) tot[2] += a.epart[k];
  const SolveScalars s0 = *a.sv;
  const bool first = blockIdx.x == 0 && blockIdx.y == 0;
  hold_loads();
  if (s0.done) {
    if (first && threadIdx.x == 0) *a.svn = s0;
    return;
  }
  plane_totals<3, T::TH>(tot, sh);
  double alpha, beta;
  if (!plane_scalars(s0, tot[0], tot[1], tot[2], a.thr2[0], a.limit[0], a.fixed[0], a.svn, first && threadIdx.x == 0,
                     alpha, beta))
    return;
  PlaneVecs<R, N> vecs(a, off);
  plane_div<R, N>(g, u, w, th, R(-1), stw, vecs, s0.it == 0);
  vecs.update(th, g, zv, R(alpha), R(beta));
}

// ---------------------------------------------------------------- diffusion
// blockIdx.x: kx plane, blockIdx.y: 3 * system + half array (c, dy c, dz c).
template <typename R, int N>
__global__ void __launch_bounds__((PlaneCfg<R, N>::TH)) k_plane_inv_b(PlaneArgs a, const cplx<R>* __restrict__ twg) {
  using T = PlaneCfg<R, N>;
  const int q = blockIdx.y / 3, o = blockIdx.y % 3;
  constexpr long long S = (long long)N * N * T::C;
  __shared__ cplx<R> buf[T::LDS];
  __shared__ cplx<R> stw[N];
  __shared__ double sh[32];
  const PlaneThread<R, N> th(buf);
  const int kx = blockIdx.x, kz = wavenum<N>(th.kz);
  const long long base = (long long)kx * N * N;
  const cplx<R>* r = static_cast<const cplx<R>*>(a.r) + base + q * S;
  cplx<R>* zd = static_cast<cplx<R>*>(a.z) + base + q * S;
  cplx<R> rv[8], v[8], zv[8];
  const R one = R(o == 0 ? 1 : 0), by = R(o == 1 ? 1 : 0), bz = R(o == 2 ? kz : 0);
#pragma unroll
  for (int j = 0; j < 8; ++j) rv[j] = r[th.spec(j)];
  R m[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) m[j] = static_cast<const cplx<R>*>(a.prec)[base + th.spec(j)].x;
  for (int k = threadIdx.x; k < N; k += T::TH) stw[k] = twg[k];
  hold_loads();
  if (a.sv[q].done) return;
  double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int ky = wavenum<N>(th.ty + T::TP * j);
    zv[j] = cscale(rv[j], m[j]);
    const R w = by * R(ky) + bz;
    v[j] = {one * zv[j].x - w * zv[j].y, one * zv[j].y + w * zv[j].x};
  }
  if (o == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      acc[0] += pdot(rv[j], zv[j]);
      acc[1] += pdot(rv[j], rv[j]);
      acc[2] += pdot(zv[j], zv[j]);
      zd[th.spec(j)] = zv[j];
    }
  }
  __syncthreads();
  th.template fft_y<true>(v, stw);
  th.to_z(v);
  th.template fft_z<true>(v, stw);
  cplx<R>* dst = static_cast<cplx<R>*>(a.half[3 * q + o]) + base;
#pragma unroll
  for (int j = 0; j < 8; ++j) dst[th.half(j)] = v[j];
  if (o == 0) {
    const double wt = kx == 0 ? 1.0 : 2.0;
    plane_totals<3, T::TH>(acc, sh);
    if (threadIdx.x == 0)
      for (int i = 0; i < 3; ++i) a.part[3 * (q * T::C + kx) + i] = acc[i] * wt;
  }
}

// blockIdx.x: row tile of one wave, blockIdx.y: 3 * system + direction; in place.
template <typename R, int N>
__global__ void __launch_bounds__(64) k_plane_xdiff(PlaneArgs a, const cplx<R>* __restrict__ twg) {
  using T = PlaneCfg<R, N>;
  const int q = blockIdx.y / 3, d = blockIdx.y % 3;
  __shared__ cplx<R> buf[T::RW * T::LX];
  __shared__ cplx<R> stw[N];
  __shared__ double sh[4];
  const PlaneRow<R, N> rw(buf, blockIdx.x);
  const R invV = R(1.0) / (R(N) * R(N) * R(N));
  cplx<R>* f = static_cast<cplx<R>*>(a.half[3 * q + d]);
  cplx<R> A[8], B[8], kr[8], v[8];
  rw.load(A, B, f);
  rw.coef(kr, a.lam);
  for (int k = threadIdx.x; k < N; k += 64) stw[k] = twg[k];
  hold_loads();
  if (a.sv[q].done) return;
  __syncthreads();
  if (d == 0) rw.iwx(A, B);
  rw.c2r(v, A, B, stw);
  double acc[1] = {0.0};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const cplx<R> o = v[j];  // N^3 times the physical value
    v[j] = {kr[j].x * o.x * invV, kr[j].y * o.y * invV};
    acc[0] += pdot(v[j], o);
  }
  row_r2c<R, N, false, true>(v, rw.lds, rw.t, stw);
  if (d == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = ciw(v[j], R(rw.t + T::TX * j));
  }
  rw.store(f, v);
  plane_totals<1, 64>(acc, sh);
  if (threadIdx.x == 0) a.epart[(long long)blockIdx.y * T::NX + blockIdx.x] = acc[0];
}

// blockIdx.x: kx plane, blockIdx.y: system.
template <typename R, int N>
__global__ void __launch_bounds__((PlaneCfg<R, N>::TH)) k_plane_fwd_b(PlaneArgs a, const cplx<R>* __restrict__ twg) {
  using T = PlaneCfg<R, N>;
  constexpr long long S = (long long)N * N * T::C;
  const int q = blockIdx.y;
  __shared__ cplx<R> buf[T::LDS];
  __shared__ cplx<R> stw[N];
  __shared__ double sh[32];
  const PlaneThread<R, N> th(buf);
  const long long base = (long long)blockIdx.x * N * N, off = base + q * S;
  auto half = [&](int f) { return static_cast<const cplx<R>*>(a.half[3 * q + f]) + base; };
  cplx<R> g[8], u[8], w[8], zv[8];
  const cplx<R>*f0 = half(0), *f1 = half(1), *f2 = half(2), *z = static_cast<const cplx<R>*>(a.z) + off;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    g[j] = f0[th.half(j)];
    u[j] = f1[th.half(j)];
    w[j] = f2[th.half(j)];
    zv[j] = z[th.spec(j)];
  }
  for (int k = threadIdx.x; k < N; k += T::TH) stw[k] = twg[k];
  double tot[4] = {0.0, 0.0, 0.0, 0.0};
  for (int k = threadIdx.x; k < T::C; k += T::TH)
    for (int i = 0; i < 3; ++i) tot[i] += a.part[3 * (q * T::C + k) + i];
  for (int k = threadIdx.x; k < 3 * T::NX; k += T::TH) tot[3] += a.epart[(long long)q * 3 * T::NX + k];
  const SolveScalars s0 = a.sv[q];
  const bool first = blockIdx.x == 0;
  hold_loads();
  if (s0.done) {
    if (first && threadIdx.x == 0) a.svn[q] = s0;
    return;
  }
  plane_totals<4, T::TH>(tot, sh);
  double alpha, beta;
  // <z, (1 - h D) z> = ||z||^2 + h <K grad z, grad z>
  if (!plane_scalars(s0, tot[0], tot[1], tot[2] + a.h * tot[3], a.thr2[q], a.limit[q], a.fixed[q], a.svn + q,
                     first && threadIdx.x == 0, alpha, beta))
    return;
  PlaneVecs<R, N> vecs(a, off);
  plane_div<R, N>(g, u, w, th, R(1), stw, vecs, s0.it == 0);
  const R h = R(a.h);
#pragma unroll
  for (int j = 0; j < 8; ++j) g[j] = {zv[j].x - h * g[j].x, zv[j].y - h * g[j].y};
  vecs.update(th, g, zv, R(alpha), R(beta));
}

// ------------------------------------------------------------ start and end
// Coefficients [row][pair] -> [pair][row], so the x side's lanes, one a row,
// read neighbours.
struct PlaneCoefs {
  const void* in[3];
  void* out[3];
};
template <typename R, int N>
__global__ void __launch_bounds__(256) k_plane_coef(PlaneCoefs a) {
  constexpr int L = N / 2;
  const int e = blockIdx.x * 256 + threadIdx.x;  // [pair][row]
  const int row = e % (N * N), p = e / (N * N);
  static_cast<cplx<R>*>(a.out[blockIdx.y])[e] = static_cast<const cplx<R>*>(a.in[blockIdx.y])[row * L + p];
}

// (below, nsv states: one per diffusion system, or 0 for the elasticity's one)
struct PlaneScale {
  double s[kMaxSys];
};

template <typename R, int N>
__global__ void __launch_bounds__(256) k_plane_start(const cplx<double>* r64, PlaneScale sc, cplx<R>* r, int nsv,
                                                      int active, SolveScalars* sv, cplx<R>* prec,
                                                      const CoefScalars* cs, double h) {
  constexpr int C = N / 2;
  constexpr long long S = (long long)N * N * C;
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int kx = e % C, zy = e / C, c = blockIdx.y;
  if (nsv == 0 || (active & (1 << c))) {
    const cplx<double> v = r64[c * S + e];
    r[c * S + (long long)kx * N * N + zy] = {R(sc.s[c] * v.x), R(sc.s[c] * v.y)};
  }
  if (c == 0) {
    // the preconditioner per mode: 1 / a and c / (a + c w^2), or the diffusion's inverse
    const int ky = wavenum<N>(zy % N), kz = wavenum<N>(zy / N);
    const double w2 = (double)(kx * kx + ky * ky + kz * kz);
    double ia, f = 0.0;
    if (nsv == 0) elast_prec_coefs<R>(w2, ElastMeans(cs), ia, f);
    else ia = 1.0 / (1.0 + h * cs->Kbar * w2);
    prec[(long long)kx * N * N + zy] = {R(ia), R(f)};
  }
  if (e == 0 && c < max(1, nsv)) {
    sv[c].it = 0;
    sv[c].conv = 0;
    sv[c].bad = 0;
    sv[c].done = (nsv == 0 || (active & (1 << c))) ? 0 : 1;
  }
}

template <typename R, int N>
__global__ void __launch_bounds__(256) k_plane_final(cplx<double>* x64, PlaneScale sc, const cplx<R>* x, int nsv,
                                                      int active, const SolveScalars* sv) {
  constexpr int C = N / 2;
  constexpr long long S = (long long)N * N * C;
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int kx = e % C, zy = e / C, c = blockIdx.y;
  if (nsv > 0 && !(active & (1 << c))) return;
  if (sv[nsv == 0 ? 0 : c].it == 0) return;
  const cplx<R> d = x[c * S + (long long)kx * N * N + zy];
  cplx<double> v = x64[c * S + e];
  v.x += sc.s[c] * (double)d.x;
  v.y += sc.s[c] * (double)d.y;
  x64[c * S + e] = v;
}

// ---------------------------------------------------------------- launchers
#define TUMOR_DISPATCH_PLANE(n, ...)                                                     \
  switch (n) {                                                                           \
    case 16: { constexpr int NN = 16; __VA_ARGS__; } break;                              \
    case 32: { constexpr int NN = 32; __VA_ARGS__; } break;                              \
    case 64: { constexpr int NN = 64; __VA_ARGS__; } break;                              \
    default: throw std::runtime_error("no plane kernels at " + std::to_string(n));       \
  }

template <typename R>
void launch_plane(int n, bool elast, int stage, const PlaneArgs& a, const void* tw, hipStream_t st) {
  const cplx<R>* twp = static_cast<const cplx<R>*>(tw);
  TUMOR_DISPATCH_PLANE(n, {
    using T = PlaneCfg<R, NN>;
    if (elast) {
      if (stage == 0) hipLaunchKernelGGL((k_plane_inv<R, NN>), dim3(T::C, 8), dim3(T::TH), 0, st, a, twp);
      else if (stage == 1) hipLaunchKernelGGL((k_plane_xelast<R, NN>), dim3(T::NX, 3), dim3(256), 0, st, a, twp);
      else hipLaunchKernelGGL((k_plane_fwd<R, NN>), dim3(T::C, 3), dim3(T::TH), 0, st, a, twp);
    } else {
      if (stage == 0) hipLaunchKernelGGL((k_plane_inv_b<R, NN>), dim3(T::C, 3 * a.nc), dim3(T::TH), 0, st, a, twp);
      else if (stage == 1) hipLaunchKernelGGL((k_plane_xdiff<R, NN>), dim3(T::NX, 3 * a.nc), dim3(64), 0, st, a, twp);
      else hipLaunchKernelGGL((k_plane_fwd_b<R, NN>), dim3(T::C, a.nc), dim3(T::TH), 0, st, a, twp);
    }
  });
}

template <typename R>
void launch_plane_coefs(int n, int count, const void* const* in, void* const* out, hipStream_t st) {
  PlaneCoefs a = {};
  for (int k = 0; k < count; ++k) {
    a.in[k] = in[k];
    a.out[k] = out[k];
  }
  TUMOR_DISPATCH_PLANE(n, {
    hipLaunchKernelGGL((k_plane_coef<R, NN>), dim3(NN * NN * NN / 512, count), dim3(256), 0, st, a);
  });
}

template <typename R>
void launch_plane_start(int n, bool elast, const void* r64, const double (&scale)[kMaxSys], int active,
                        const PlaneArgs& a, SolveScalars* sv, hipStream_t st) {
  PlaneScale sc;
  for (int k = 0; k < kMaxSys; ++k) sc.s[k] = scale[elast ? 0 : k];
  TUMOR_DISPATCH_PLANE(n, {
    hipLaunchKernelGGL((k_plane_start<R, NN>), dim3(NN * NN * NN / 512, elast ? 3 : a.nc), dim3(256), 0, st,
                       static_cast<const cplx<double>*>(r64), sc, static_cast<cplx<R>*>(a.r), elast ? 0 : a.nc, active, sv,
                       static_cast<cplx<R>*>(const_cast<void*>(a.prec)), a.cs, a.h);
  });
}

template <typename R>
void launch_plane_final(int n, bool elast, void* x64, const double (&scale)[kMaxSys], int active, const PlaneArgs& a,
                        const SolveScalars* sv, hipStream_t st) {
  PlaneScale sc;
  for (int k = 0; k < kMaxSys; ++k) sc.s[k] = scale[elast ? 0 : k];
  TUMOR_DISPATCH_PLANE(n, {
    hipLaunchKernelGGL((k_plane_final<R, NN>), dim3(NN * NN * NN / 512, elast ? 3 : a.nc), dim3(256), 0, st,
                       static_cast<cplx<double>*>(x64), sc, static_cast<const cplx<R>*>(a.x), elast ? 0 : a.nc, active,
                       sv);
  });
}

}  // namespace tumor
