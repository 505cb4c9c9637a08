// Kernels and launchers of the two-kernel transforms (see tile.hpp).
#pragma once
#include "passes_impl.hpp"
#include "tile.hpp"

namespace tumor {

// Register position of output m of a register transform of length B.
template <int B>
__device__ __forceinline__ constexpr int rpos(int m) { return B == 16 ? 4 * (m & 3) + (m >> 2) : m; }

// 16-point transform in registers, outputs in rpos<16> order.
template <typename R, bool INV>
__device__ __forceinline__ void dft16(cplx<R>* x) {
  const R c1 = R(0.92387953251128675612818318939678829), s1 = R(0.38268343236508977172845998403039887);
  const R h = R(0.70710678118654752440084436210484903928);
  const R sg = INV ? R(1) : R(-1);  // w = exp(sg * 2 pi i / 16)
#pragma unroll
  for (int i = 0; i < 4; ++i) dft4<R, INV>(x[i], x[i + 4], x[i + 8], x[i + 12]);
  // x[i + 4 k] *= w^(i k)
  x[5] = cmul(x[5], {c1, sg * s1});
  x[6] = cmul(x[6], {h, sg * h});
  x[7] = cmul(x[7], {s1, sg * c1});
  x[9] = cmul(x[9], {h, sg * h});
  x[10] = INV ? cplx<R>{-x[10].y, x[10].x} : cplx<R>{x[10].y, -x[10].x};
  x[11] = cmul(x[11], {-h, sg * h});
  x[13] = cmul(x[13], {s1, sg * c1});
  x[14] = cmul(x[14], {-h, sg * h});
  x[15] = cmul(x[15], {-c1, -sg * s1});
#pragma unroll
  for (int k = 0; k < 4; ++k) dft4<R, INV>(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
}

template <typename R, bool INV, int B>
__device__ __forceinline__ void dftB(cplx<R>* x) {
  if constexpr (B == 16) dft16<R, INV>(x);
  else dft_r<R, INV, B>(x);
}

// c2r_pre and the end of row_r2c for a value k that is 0 only if `zero`,
// without branches (the mirrored value is then read from the row's padding and
// dropped).
template <typename R>
__device__ __forceinline__ cplx<R> c2r_mix(cplx<R> A, cplx<R> B, cplx<R> w, bool zero) {
  const cplx<R> s = {A.x + B.x, A.y - B.y}, d = {A.x - B.x, A.y + B.y};
  const cplx<R> e = cmul(cconj(w), d);
  return {zero ? A.x + A.y : s.x - e.y, zero ? A.x - A.y : s.y + e.x};
}
template <typename R>
__device__ __forceinline__ cplx<R> r2c_mix(cplx<R> A, cplx<R> B, cplx<R> w, bool zero) {
  const cplx<R> s = {A.x + B.x, A.y - B.y}, wd = cmul(w, cplx<R>{A.x - B.x, A.y + B.y});
  return {zero ? A.x + A.y : R(0.5) * (s.x + wd.y), zero ? A.x - A.y : R(0.5) * (s.y - wd.x)};
}

// Transform of a line of 16 B points held by B threads: v[j] is position
// t + B j on entry and on return.  buf(m, t): exchange cell.  WAVE: the line's
// threads are lanes of one wave.  TWS: table entries per w_(16 B).
template <typename R, int B, bool INV, int TWS, bool WAVE, typename Buf>
__device__ __forceinline__ void line_fft(cplx<R> (&v)[16], int t, const cplx<R>* __restrict__ tw, const Buf& buf) {
  dft16<R, INV>(v);
  buf(0, t) = v[0];
#pragma unroll
  for (int m = 1; m < 16; ++m) {
    cplx<R> w = tw[t * m * TWS];
    if (INV) w.y = -w.y;
    buf(m, t) = cmul(v[rpos<16>(m)], w);
    if (m % 4 == 3) hold_loads();
  }
  if constexpr (WAVE) wave_sync();
  else __syncthreads();
  constexpr int NS = 16 / B;
  cplx<R> u[16];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int q = 0; q < B; ++q) u[s * B + q] = buf(t + B * s, q);
#pragma unroll
  for (int s = 0; s < NS; ++s) dftB<R, INV, B>(u + s * B);
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int q = 0; q < B; ++q) v[s + NS * q] = u[s * B + rpos<B>(q)];
}

// XCD-aware tile order: workgroups go round-robin to the 8 XCDs, and each XCD
// takes a contiguous range of tiles, so that neighbours (in kx, or in jl),
// whose 64-byte pieces share 128-byte lines, run on one L2.
__device__ __forceinline__ int xcd_tile() {
  const int per = gridDim.x >> 3;
  return ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
}

// Thread roles of a spectral tile.
template <typename R, int N>
struct TileThread {
  using T = TileCfg<R, N>;
  int b, kx0;           // tile
  int iz, kx;           // y role: position kz, column
  int t, jl, kxl, tlo;  // z role: line (jl, kxl), position t
  unsigned zaddr;       // z role: offset of element 0 in an x side's output
  __device__ __forceinline__ TileThread(int tile) {
    const int tid = threadIdx.x;
    b = tile / (T::C / T::KT);
    kx0 = (tile % (T::C / T::KT)) * T::KT;
    iz = tid / T::KT;
    kx = kx0 + tid % T::KT;
    tlo = tid % T::ZT;
    kxl = (tid / T::ZT) % T::KT;
    jl = (tid / (T::ZT * T::KT)) % 16;
    const int thi = tid / (T::ZT * T::KT * 16);
    t = tlo + T::ZT * thi;
    zaddr = ((thi * 16 + jl) * T::YB + b) * (T::C * T::ZT) + (kx0 + kxl) * T::ZT + tlo;
  }
  // stride of that offset from position t + ZB i to t + ZB (i + 1)
  static constexpr int ZSTEP = T::ZH * 16 * T::YB * T::C * T::ZT;
  // exchange cells: (jl, kz, kx) between the roles, (m, t) within a z line
  __device__ __forceinline__ static int x1(int jl_, int pos) { return jl_ * (T::TA + T::P1) + pos; }
  __device__ __forceinline__ int x2(int m, int t_) const {
    return m * (T::TA + T::P2) + (t_ % T::ZT) + T::ZT * (kxl + T::KT * (jl + 16 * (t_ / T::ZT)));
  }
};

// ------------------------------------------------------------ spectral side
// Memory bounds both spectral kernels (256^3, counted): inverse 26 arrays in
// 0.70 ms (FP64) and 0.36 ms (FP32), 5.0 and 4.8 TB/s; forward 18 (FP32 21) arrays in
// 0.59 and 0.36 ms, 4.0 TB/s.  One or two components of p and r are read
// twice: all three in registers would halve the waves, which measured slower.  The
// next half array's loads ahead of a transform spill in the forward kernel: 0.91
// and 0.66 ms.
template <typename R, int N>
__global__ void __launch_bounds__((TileCfg<R, N>::TA), (sizeof(R) == 4 ? 4 : 2)) k_tile_inv(TileInvArgs a, const cplx<R>* __restrict__ twg) {
  if (a.sv->done) return;
  using T = TileCfg<R, N>;
  constexpr long long S = (long long)N * N * (N / 2);
  __shared__ cplx<R> buf[T::LDSA];
  __shared__ cplx<R> stw[N];
  for (int k = threadIdx.x; k < N; k += T::TA) stw[k] = twg[k];
  const int tile = xcd_tile();
  const TileThread<R, N> th(tile);
  const int tid = threadIdx.x;
  // the tile's elements e of component c: block-uniform base, lane offset tid
  const long long tbase = (long long)tile * 16 * T::TA;
  auto at = [&](const void* vec, int c, int e) {
    return static_cast<cplx<R>*>(const_cast<void*>(vec)) + (tbase + c * S + e * T::TA);
  };
  const int kz = wavenum<N>(th.iz);
  const R fkz = R(kz), fkx = R(th.kx);
  auto ky = [&](int e) { return wavenum<N>(th.b + T::YB * e); };

  // z transform of w (y transform done, rpos order over jl) and store
  auto z_store = [&](const cplx<R>(&w)[16], int o) {
    __syncthreads();  // the exchange buffer is free (and the twiddles are staged)
#pragma unroll
    for (int j = 0; j < 16; ++j) buf[th.x1(j, threadIdx.x)] = w[rpos<16>(j)];
    __syncthreads();
    cplx<R> v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = buf[th.x1(th.jl, (th.t + T::ZB * j) * T::KT + th.kxl)];
    __syncthreads();
    line_fft<R, T::ZB, true, 1, false>(v, th.t, stw, [&](int m, int t_) -> cplx<R>& { return buf[th.x2(m, t_)]; });
    cplx<R>* dst = static_cast<cplx<R>*>(a.out[o]) + tbase;
#pragma unroll
    for (int i = 0; i < 16; ++i, dst += T::TA) dst[tid] = v[i];
  };
  // 16-point part of the y transform with its twiddle w^(jl b)
  auto y_part = [&](cplx<R>(&w)[16]) {
    dft16<R, true>(w);
#pragma unroll
    for (int j = 1; j < 16; ++j) w[rpos<16>(j)] = cmul(w[rpos<16>(j)], cconj(twg[j * th.b]));
  };

  cplx<R> u[16], w[16];  // p_x; i k . p
  if (a.update) {
    const ElastMeans em(a.cs);
    const R beta = R(a.sv->beta), alpha = R(a.sv->alpha);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const R wk[3] = {fkx, R(ky(e)), fkz};
      const int kzo = opaque(kz);
      double ia, f;
      elast_prec_coefs<R>((double)(th.kx * th.kx + ky(e) * ky(e) + kzo * kzo), em, ia, f);
      cplx<R> rv[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) rv[c] = at(a.r, c, e)[tid];
      const R ff = R(f), fia = R(ia);
      const cplx<R> wr = {wk[0] * rv[0].x + wk[1] * rv[1].x + wk[2] * rv[2].x,
                          wk[0] * rv[0].y + wk[1] * rv[1].y + wk[2] * rv[2].y};
      cplx<R> d = czero<R>();
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const cplx<R> pv = at(a.p, c, e)[tid], xv = at(a.x, c, e)[tid];
        at(a.x, c, e)[tid] = {xv.x + alpha * pv.x, xv.y + alpha * pv.y};
        const cplx<R> pn = {(rv[c].x - ff * wk[c] * wr.x) * fia + beta * pv.x,
                            (rv[c].y - ff * wk[c] * wr.y) * fia + beta * pv.y};
        at(a.p, c, e)[tid] = pn;
        if (c == 0) u[e] = pn;
        d = cadd(d, ciw(pn, wk[c]));
      }
      w[e] = d;
      if (e % 2 == 1) hold_loads();
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      u[e] = at(a.p, 0, e)[tid];
      w[e] = cadd(ciw(u[e], fkx), cadd(ciw(at(a.p, 1, e)[tid], R(ky(e))), ciw(at(a.p, 2, e)[tid], fkz)));
    }
  }
  // div u
  y_part(w);
  z_store(w, 8);
  // x: dy u_x, U_x, dz u_x (the last two share the y part)
#pragma unroll
  for (int e = 0; e < 16; ++e) w[e] = ciw(u[e], R(ky(e)));
  y_part(w);
  z_store(w, 3);
  y_part(u);
  z_store(u, 0);
#pragma unroll
  for (int e = 0; e < 16; ++e) u[e] = ciw(u[e], fkz);
  z_store(u, 6);
  // y: dy u_y, U_y, and dz u_y + dy u_z (the other components come back from
  // memory: three at once would cost half the waves)
#pragma unroll
  for (int e = 0; e < 16; ++e) u[e] = at(a.p, 1, e)[tid];
#pragma unroll
  for (int e = 0; e < 16; ++e) w[e] = ciw(u[e], R(ky(e)));
  y_part(w);
  z_store(w, 4);
  y_part(u);
  z_store(u, 1);
  cplx<R> v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = at(a.p, 2, e)[tid];
#pragma unroll
  for (int e = 0; e < 16; ++e) w[e] = ciw(v[e], R(ky(e)));
  y_part(w);
#pragma unroll
  for (int e = 0; e < 16; ++e) w[e] = cadd(w[e], ciw(u[e], fkz));
  z_store(w, 5);
  // z: U_z, dz u_z
  y_part(v);
  z_store(v, 2);
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = ciw(v[e], fkz);
  z_store(v, 7);
}

template <typename R, int N>
__global__ void __launch_bounds__((TileCfg<R, N>::TA), (sizeof(R) == 4 ? 4 : 2)) k_tile_fwd(TileFwdArgs a, const cplx<R>* __restrict__ twg) {
  using T = TileCfg<R, N>;
  if (a.sv->done) return;
  constexpr long long S = (long long)N * N * (N / 2);
  __shared__ cplx<R> buf[T::LDSA];
  __shared__ cplx<R> stw[N];
  const int tile = xcd_tile();
  const TileThread<R, N> th(tile);
  const int tid = threadIdx.x;
  const long long tbase = (long long)tile * 16 * T::TA;
  auto at = [&](void* vec, int c, int e) { return static_cast<cplx<R>*>(vec) + (tbase + c * S + e * T::TA); };
  double al;
  if (!block_alpha<T::TA>(a.sv, a.epart, T::NB, blockIdx.x == 0, reinterpret_cast<double*>(buf), al)) return;
  const R alpha = R(al);
  for (int k = tid; k < N; k += T::TA) stw[k] = twg[k];
  const int kz = wavenum<N>(th.iz);
  const R fkz = R(kz), fkx = R(th.kx);
  auto ky = [&](int e) { return wavenum<N>(th.b + T::YB * e); };
  const ElastMeans em(a.cs);
  // forward z transform of a half array, handed to the y role (index jl)
  auto z_load = [&](cplx<R>(&w)[16], int f) {
    const cplx<R>* src = static_cast<const cplx<R>*>(a.in[f]);
    cplx<R> v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i, src += th.ZSTEP) v[i] = src[th.zaddr];
    __syncthreads();
    line_fft<R, T::ZB, false, 1, false>(v, th.t, stw, [&](int m, int t_) -> cplx<R>& { return buf[th.x2(m, t_)]; });
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) buf[th.x1(th.jl, (th.t + T::ZB * i) * T::KT + th.kxl)] = v[i];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) w[j] = buf[th.x1(j, threadIdx.x)];
  };
  // twiddle and 16-point part of the y transform (outputs in rpos order)
  auto y_part = [&](cplx<R>(&w)[16]) {
#pragma unroll
    for (int j = 1; j < 16; ++j) w[j] = cmul(w[j], twg[j * th.b]);
    dft16<R, false>(w);
  };
  cplx<R> g[16], w[16];
  double acc[2] = {0.0, 0.0};
  // q_x = F0 - dy F3 - dz F6, q_y = F1 - dy F4 - dz F5, q_z = F2 - dy F5 - dz F7
#pragma unroll 1
  for (int c = 0; c < 3; ++c) {
    const int fy = c == 0 ? 3 : (c == 1 ? 4 : 5), fz = c == 0 ? 6 : (c == 1 ? 5 : 7);
    z_load(g, c);
    z_load(w, fz);
#pragma unroll
    for (int j = 0; j < 16; ++j) g[j] = csub(g[j], ciw(w[j], fkz));
    y_part(g);
    z_load(w, fy);
    y_part(w);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const cplx<R> q = csub(g[rpos<16>(e)], ciw(w[rpos<16>(e)], R(ky(e))));
      cplx<R> rv = at(a.r, c, e)[tid];
      rv.x -= alpha * q.x;
      rv.y -= alpha * q.y;
      at(a.r, c, e)[tid] = rv;
      if (e % 4 == 3) hold_loads();
      acc[0] += (double)rv.x * (double)rv.x + (double)rv.y * (double)rv.y;
    }
  }
  // <r, M^-1 r>: the three components come back from memory
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const R wk[3] = {fkx, R(ky(e)), fkz};
    if (e % 4 == 0) hold_loads();
    const int kzo = opaque(kz);
    double ia, f;
    elast_prec_coefs<R>((double)(th.kx * th.kx + ky(e) * ky(e) + kzo * kzo), em, ia, f);
    cplx<R> rv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) rv[c] = at(a.r, c, e)[tid];
    const R ff = R(f), fia = R(ia);
    const cplx<R> wr = {wk[0] * rv[0].x + wk[1] * rv[1].x + wk[2] * rv[2].x,
                        wk[0] * rv[0].y + wk[1] * rv[1].y + wk[2] * rv[2].y};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const R zx = (rv[c].x - ff * wk[c] * wr.x) * fia, zy = (rv[c].y - ff * wk[c] * wr.y) * fia;
      acc[1] += (double)rv[c].x * (double)zx + (double)rv[c].y * (double)zy;
    }
    pin(acc[1]);
  }
  // Parseval weight: the packed kx = 0 column counts once, the others twice
  const double wt = th.kx == 0 ? 1.0 : 2.0;
  acc[0] *= wt;
  acc[1] *= wt;
  block_totals<2, T::TA>(acc, reinterpret_cast<double*>(buf));
  if (threadIdx.x == 0) {
    a.partials[2 * (long long)blockIdx.x] = acc[0];
    a.partials[2 * (long long)blockIdx.x + 1] = acc[1];
  }
}

// ------------------------------------------------------------------ x side
// Ten row transforms in and nine out per row.  FP32 (0.38 ms at 256^3) keeps mu,
// eta and the next inputs in registers and is bound by its instructions and LDS
// accesses; FP64 (0.82 ms) has no room for them and moves 33 arrays at 5.4 TB/s,
// the coefficient re-reads among them.
template <typename R, int N>
__global__ void __launch_bounds__((TileCfg<R, N>::TB), 2) k_tile_xelast(TileXArgs a, const cplx<R>* __restrict__ twg) {
  if (a.sv->done) return;
  using T = TileCfg<R, N>;
  constexpr bool RICH = sizeof(R) == 4;
  constexpr int L = T::L, LB = T::LB, YB = T::YB, NS = 16 / T::YB;
  __shared__ cplx<R> buf[T::ROWS * T::LP];
  __shared__ cplx<R> stw[N];
  for (int k = threadIdx.x; k < N; k += T::TB) stw[k] = twg[k];
  const int tid = threadIdx.x;
  const R invV = R(1.0) / (R(N) * R(N) * R(N));
  // column role: kx with YB values of b (or jh) on NS planes
  const int zg = tid % T::ZG, kx = tid / T::ZG;
  const int tile = xcd_tile(), zt = tile / 16, jl = tile % 16;
  const long long oblk = (long long)tile * (YB * T::C * T::ZT);
  const unsigned ooff = kx * T::ZT + zg;
  const int iblk = (zt / T::ZH) * T::TA + T::ZT * T::KT * (jl + 16 * (zt % T::ZH));
  const unsigned ioff = (kx / T::KT) * (16 * T::TA) + (kx % T::KT) * T::ZT + zg;
  const R fkx = R(kx);
  // row role: row = jh * ZT + plane, LB threads a row (lanes of one wave)
  const int row = tid / LB, t = tid % LB;
  // physical pairs: plane z = zt ZT + row % ZT, y = jl + 16 (row / ZT)
  const long long pblk = ((long long)zt * T::ZT * N + jl) * L;
  const unsigned poff = ((row % T::ZT) * N + 16 * (row / T::ZT)) * L + t;
  const cplx<R>* mu = static_cast<const cplx<R>*>(a.mu) + pblk;
  const cplx<R>* lam = static_cast<const cplx<R>*>(a.lam) + pblk;
  const cplx<R>* eta = static_cast<const cplx<R>*>(a.eta) + pblk;
  cplx<R>* rbuf = buf + row * T::LP;
  // row role: the row's values at k = t + LB j, at L - k, and their twiddles
  const cplx<R>*rk = rbuf + t, *rm = rbuf + (L - t - 15 * LB), *tk = stw + t;
  // column role: the column's values in the block's rows at kx and L - kx
  const cplx<R>*ck = buf + zg * T::LP + kx, *cm = buf + zg * T::LP + (L - kx);
  auto cell = [&](int m, int t_) -> cplx<R>& { return rbuf[m * T::MS + t_]; };
  double en = 0.0;

  auto load = [&](cplx<R>(&v)[16], int f) {
    const cplx<R>* src = static_cast<const cplx<R>*>(a.in[f]) + iblk;
#pragma unroll
    for (int q = 0; q < YB; ++q, src += (T::C / T::KT) * 16 * T::TA)
#pragma unroll
      for (int s = 0; s < NS; ++s) v[s * YB + q] = src[ioff + s * T::ZG];
  };
  auto store = [&](const cplx<R>(&v)[16], int f) {
    cplx<R>* dst = static_cast<cplx<R>*>(a.out[f]) + oblk;
#pragma unroll
    for (int q = 0; q < YB; ++q, dst += T::C * T::ZT)
#pragma unroll
      for (int s = 0; s < NS; ++s) dst[ooff + s * T::ZG] = v[s * YB + rpos<YB>(q)];
  };
  // column role (spectral, index b) -> row role (physical pairs at t + LB i,
  // times N^3).  `fetch` issues the next inputs' loads once v is in LDS.
  auto to_rows = [&](cplx<R>(&v)[16], auto&& fetch) {
#pragma unroll
    for (int s = 0; s < NS; ++s) dftB<R, true, YB>(v + s * YB);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int q = 0; q < YB; ++q) buf[(q * T::ZT + zg + T::ZG * s) * T::LP + kx] = v[s * YB + rpos<YB>(q)];
    fetch();
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      v[j] = c2r_mix(rk[LB * j], rm[LB * (15 - j)], tk[LB * j], j == 0 && t == 0);
      if (j % 4 == 3) hold_loads();
    }
    wave_sync();
    line_fft<R, LB, true, 2, true>(v, t, stw, cell);
  };
  // row role -> column role, index jh, packed R2C done
  auto to_cols = [&](cplx<R>(&v)[16]) {
    wave_sync();
    line_fft<R, LB, false, 2, true>(v, t, stw, cell);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) rbuf[t + LB * i] = v[i];
    __syncthreads();
    const cplx<R> w = stw[kx];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int q = 0; q < YB; ++q) {
        constexpr int QS = T::ZT * T::LP;
        v[s * YB + q] = r2c_mix(ck[q * QS + T::ZG * s * T::LP], cm[q * QS + T::ZG * s * T::LP], w, kx == 0);
        if (q % 4 == 3) hold_loads();
      }
  };
  // YB-point part of the forward y transform (index b, rpos order)
  auto y_part = [&](cplx<R>(&v)[16]) {
#pragma unroll
    for (int s = 0; s < NS; ++s) dftB<R, false, YB>(v + s * YB);
  };
  // coefficient rows: FP32 holds mu and eta for the whole tile; FP64 reads them
  // where they are used
  cplx<R> mur[RICH ? 16 : 1], etar[RICH ? 16 : 1];
  if constexpr (RICH) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      mur[i] = mu[poff + LB * i];
      etar[i] = eta[poff + LB * i];
    }
  }
  auto mu_at = [&](int i) -> cplx<R> {
    if constexpr (RICH) return mur[i];
    else return mu[poff + LB * i];
  };
  auto eta_at = [&](int i) -> cplx<R> {
    if constexpr (RICH) return etar[i];
    else return eta[poff + LB * i];
  };
  // c v / N^3, the same bits in any order: in FP32 c v first (v / N^3 alone is out of
  // range for moduli above 1e33), in FP64 c / N^3, which spills less and is 2 % of a
  // split step faster
  auto scaled = [&](R c, R v) { return RICH ? c * v * invV : (c * invV) * v; };
  // v <- c * v / N^3 per pair, adding its product with v to the energy: <p, A p> of
  // the spectral vectors is N^3 times the physical sum (and products of two
  // physical values would underflow N^3 times as early)
  auto scale_by = [&](cplx<R>(&v)[16], auto&& coef) {
    hold_loads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const cplx<R> c = coef(i), o = v[i];
      v[i] = {scaled(c.x, o.x), scaled(c.y, o.y)};
      en += (double)v[i].x * (double)o.x + (double)v[i].y * (double)o.y;
    }
    pin(en);
  };
  auto none = [] {};

  // inputs in flight: FP32 fetches each during the row work before its use
  cplx<R> nx[16], nu[16];
  auto want = [&](cplx<R>(&v)[16], int f) {
    if constexpr (!RICH) load(v, f);
  };
  cplx<R> v[16], xs[16];
  {
    // lambda div u, kept for the three diagonal stresses
    cplx<R> lt[16];
    load(lt, 8);
    to_rows(lt, [&] { if constexpr (RICH) load(nx, 4); });
    scale_by(lt, [&](int i) { return lam[poff + LB * i]; });
    auto diagonal = [&](cplx<R>(&w)[16]) {
      hold_loads();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const cplx<R> m = mu_at(i);
        const cplx<R> me = {scaled(R(2) * m.x, w[i].x), scaled(R(2) * m.y, w[i].y)};
        en += (double)me.x * (double)w[i].x + (double)me.y * (double)w[i].y;
        w[i] = cadd(me, lt[i]);
      }
      pin(en);
    };
#pragma unroll 1
    for (int f = 4; f < 8; f += 3) {
      want(nx, f);
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = nx[e];
      to_rows(v, [&] { if constexpr (RICH) load(nx, f == 4 ? 7 : 0); });
      diagonal(v);
      to_cols(v);
      y_part(v);
      store(v, f);
    }
    // s_xx
    want(nx, 0);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      nu[e] = nx[e];
      xs[e] = ciw(nx[e], fkx);
    }
    to_rows(xs, [&] { if constexpr (RICH) load(nx, 3); });
    diagonal(xs);
    to_cols(xs);
  }
  // eta u_x - dx s_xx; then s_xy with eta u_y - dx s_xy, s_xz with eta u_z - dx s_xz
#pragma unroll 1
  for (int c = 0; c < 3; ++c) {
    const int fs = c == 1 ? 3 : 6;  // s_xy, s_xz
    if (c > 0) {
      want(nx, fs);
      want(nu, c);
#pragma unroll
      for (int e = 0; e < 16; ++e) xs[e] = cadd(nx[e], ciw(nu[e], fkx));
      to_rows(xs, [&] { if constexpr (RICH) load(nx, c == 1 ? 6 : 5); });
      scale_by(xs, mu_at);
      to_cols(xs);
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = xs[e];
      y_part(v);
      store(v, fs);
    }
    if constexpr (!RICH) load(nu, c);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      xs[e] = ciw(xs[e], fkx);
      v[e] = nu[e];
    }
    to_rows(v, [&] { if constexpr (RICH) { if (c < 2) load(nu, c + 1); } });
    scale_by(v, eta_at);
    to_cols(v);
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = csub(v[e], xs[e]);
    y_part(v);
    store(v, c);
  }
  // s_yz
  want(nx, 5);
  to_rows(nx, none);
  scale_by(nx, mu_at);
  to_cols(nx);
  y_part(nx);
  store(nx, 5);

  double e1[1] = {en};
  block_totals<1, T::TB>(e1, reinterpret_cast<double*>(buf));
  if (tid == 0) a.epart[blockIdx.x] = e1[0];
}

// ---------------------------------------------------------------- launchers
#define TUMOR_DISPATCH_TILE(n, ...)                                                          \
  if ((n) == 256) { constexpr int NN = 256; __VA_ARGS__; }                                  \
  else throw std::runtime_error("no two-kernel transform at " + std::to_string(n));

template <typename R>
void launch_tile_inv(int n, const TileInvArgs& a, const void* tw, hipStream_t st) {
  TUMOR_DISPATCH_TILE(n, {
    using T = TileCfg<R, NN>;
    hipLaunchKernelGGL((k_tile_inv<R, NN>), dim3(T::NA), dim3(T::TA), 0, st, a, static_cast<const cplx<R>*>(tw));
  });
}

template <typename R>
void launch_tile_xelast(int n, const TileXArgs& a, const void* tw, hipStream_t st) {
  TUMOR_DISPATCH_TILE(n, {
    using T = TileCfg<R, NN>;
    hipLaunchKernelGGL((k_tile_xelast<R, NN>), dim3(T::NB), dim3(T::TB), 0, st, a, static_cast<const cplx<R>*>(tw));
  });
}

template <typename R>
void launch_tile_fwd(int n, const TileFwdArgs& a, const void* tw, hipStream_t st) {
  TUMOR_DISPATCH_TILE(n, {
    using T = TileCfg<R, NN>;
    hipLaunchKernelGGL((k_tile_fwd<R, NN>), dim3(T::NA), dim3(T::TA), 0, st, a, static_cast<const cplx<R>*>(tw));
  });
}

template <typename R>
int tile_fwd_blocks(int n) {
  int nb = 0;
  TUMOR_DISPATCH_TILE(n, nb = (TileCfg<R, NN>::NA));
  return nb;
}

}  // namespace tumor
