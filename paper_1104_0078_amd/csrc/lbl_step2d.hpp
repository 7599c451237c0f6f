// lbl_step2d.hpp -- the coupled Heun step on D2Q9 in two launches.
//
// The general path takes five launches a step and passes mu, u^n, the stage
// velocity u-bar^1 and the stage input through memory between them: 49 values
// of b bytes per site and step.  In 2-D the halos are cheap, so two kernels on
// 32 x 8 or 64 x 8 tiles keep those fields on the chip:
//   half 1: mu(psi^n) (LDS), the pulls, force, u^n on the tile and a one-site
//           ring, the collision with its noise on the tile, the SMOL noise
//           N^n, and the first stage phi^1 = psi^n + R + N^n; writes f*^n,
//           phi^1 and the rate R (the frozen noise cancels in Heun's mean);
//   half 2: mu(psi^n) and mu(phi^1) (LDS), the pulls of the streamed
//           populations, u-bar^1 on the tile and the ring, and the second
//           stage; writes psi^{n+1} = phi^1 + (R^1 - R)/2.
// 34 values per site and step.  The ring costs 84 more pulls and force
// evaluations per 256 sites (148 per 512) but no collision and no mode noise; a
// single kernel would have to collide (and draw) on a two-site ring as well.
//
// A block is a chain of loads, three barriers and stores, with few blocks
// resident (FP64: 3 or 4), so every load of a block is issued before its first
// barrier: the fields, the pulls, then the ring's pulls, which used to start
// after the tile's sites and held the whole block for one more latency
// (4096^2 FP64, 64 x 8, half 1 + half 2: 714 + 477 -> 675 + 380 us; FP32
// 357 + 263 -> 328 + 215; 64^2 FP64, 32 x 8, 13.7 -> 11.8 us a step).  The
// pulls are cached, as a ring is part of four other tiles.
// Measured (half 1 + half 2, us): 64^2 FD FP64 9.1 + 6.8 timed singly (11.4 a
// step back to back), 1000^2 FD FP64 47 + 22, 4096^2 FD FP64 693 + 376 (4.3
// and 5.4 TB/s of 92 + 88 and 113 + 8 B a site), FP32 334 + 214.  What is left of
// half 1 in FP64 is issue: 1922 instructions a thread, VALU 75% busy.
#pragma once

#include "lbl_kernels.hpp"

namespace lbl {

template <typename S>
struct HalfArgs {
  LBArgs<S> lb;  // f_in, f_out, u_out (half 1: u^n, or nullptr), rates, noise key
  Coef<S> c;
  S amp;           // sqrt(2 kT M)
  int smol_noise;  // 0: kT == 0
  const S* psi;    // psi^n
  S* phi;          // phi^1
  S* rate;         // R
  S* out;          // psi^{n+1}
};

// Tile of R rows per thread on 256 threads: 32 x 8 sites (R = 1) or 64 x 8
// (R = 2), thread (tx, ty) with the rows R ty ... R ty + R - 1.  LDS regions
// around it: psi and phi with halo 3, mu with halo 2, fluxes and node normals
// with halo 1.
template <int R>
struct Tile2 {
  static constexpr int TX = R == 1 ? 32 : 64, NT = 256, RY = NT / TX, TY = RY * R;
  static constexpr int W3 = TX + 6, H3 = TY + 6;
  static constexpr int W2 = TX + 4, H2 = TY + 4;
  static constexpr int W1 = TX + 2, H1 = TY + 2;
  static constexpr int kRing = 2 * W1 + 2 * TY;  // sites of the one-site ring
  static_assert(kRing <= NT, "ring sites in one pass");
};

// Position in the halo-1 region of ring element r: its two rows, then its two
// columns.
template <int R>
__device__ __forceinline__ void ring_pos(int r, int& i, int& j) {
  using T = Tile2<R>;
  if (r < 2 * T::W1) {
    j = r < T::W1 ? 0 : T::H1 - 1;
    i = r < T::W1 ? r : r - T::W1;
  } else {
    const int q = r - 2 * T::W1;
    i = q < T::TY ? 0 : T::W1 - 1;
    j = 1 + (q < T::TY ? q : q - T::TY);
  }
}

// The elements of a halo-3 region that a thread loads: its column of the tile
// at every RY-th row, then one element of the six side columns.
template <int R>
struct Region3 {
  using T = Tile2<R>;
  static constexpr int NK = (T::H3 + T::RY - 1) / T::RY;
  static_assert(6 * T::H3 <= T::NT, "side columns in one pass");
  int src[NK + 1], dst[NK + 1];
  bool on[NK + 1];
  __device__ __forceinline__ Region3(const Geom& g, int x0, int y0, bool near, int tid) {
    const int tx = tid % T::TX, ty = tid / T::TX;
    const int x = wrap_r(x0 + tx, g.nx, near);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int j = ty + T::RY * k;
      on[k] = j < T::H3;
      src[k] = x + g.nx * wrap_r(y0 - 3 + j, g.ny, near);
      dst[k] = (tx + 3) + T::W3 * j;
    }
    const int j = tid / 6, c = tid % 6, i = c < 3 ? c : c + T::TX;
    on[NK] = j < T::H3;
    src[NK] = wrap_r(x0 - 3 + i, g.nx, near) + g.nx * wrap_r(y0 - 3 + j, g.ny, near);
    dst[NK] = i + T::W3 * j;
  }
  template <typename S>
  __device__ __forceinline__ void fetch(const S* __restrict__ v, S (&e)[NK + 1]) const {
#pragma unroll
    for (int k = 0; k <= NK; ++k) e[k] = on[k] ? v[src[k]] : S(0);
  }
  template <typename S>
  __device__ __forceinline__ void store(const S (&e)[NK + 1], S* __restrict__ to) const {
#pragma unroll
    for (int k = 0; k <= NK; ++k)
      if (on[k]) to[dst[k]] = e[k];
  }
};

// The streamed populations of ring element tid, asked for with the tile's own.
template <typename S, int R, bool WALLS>
struct RingPull {
  int i = 0, j = 0, y = 0;  // position in the halo-1 region; row
  S f[9];
  __device__ __forceinline__ RingPull(const LBArgs<S>& a, int x0, int y0, bool near, int tid) {
    if (tid < Tile2<R>::kRing) {
      ring_pos<R>(tid, i, j);
      y = wrap_r(y0 - 1 + j, a.g.ny, near);
      const Nbr nr(a.g, wrap_r(x0 - 1 + i, a.g.nx, near), y, 0);
      lb_pull<S, 9, kCached, WALLS>(a, nr, y, 0, f);
    }
  }
};

// mu of the field in the halo-3 region `src` on the halo-2 region: each thread
// its own R points from the row sums of one column, then its points of the
// frame around the tile.  WALLS: a neighbour row beyond a wall reads the centre.
template <typename S, int R, bool WALLS>
__device__ __forceinline__ void mu_region2(const Geom& g, const Coef<S>& c, int y0, int tid,
                                           const S* __restrict__ src, S* __restrict__ dst) {
  using T = Tile2<R>;
  // mu from the centre and side sums of rows below (0), at (1) and above (2);
  // yr: the row of the point
  auto mu = [&](const S (&cc)[3], const S (&ss)[3], int yr) {
    S c0 = cc[0], c2 = cc[2], s0 = ss[0], s2 = ss[2];
    if (WALLS && yr - 1 < 0) {
      c0 = cc[1];
      s0 = S(2) * cc[1];
    }
    if (WALLS && yr + 1 >= g.ny) {
      c2 = cc[1];
      s2 = S(2) * cc[1];
    }
    const S p = cc[1];
    const S lap = S(0.5) * (ss[1] + (c0 + c2)) + S(0.25) * (s0 + s2) - S(3.0) * p;
    return c.a * p + c.b * p * p * p - c.kappa * lap;
  };
  const int tx = tid % T::TX, ty = tid / T::TX;
  {
    const S* P = src + (tx + 3) + T::W3 * (R * ty + 2);
    S cc[R + 2], ss[R + 2];
#pragma unroll
    for (int m = 0; m < R + 2; ++m) {
      cc[m] = P[T::W3 * m];
      ss[m] = P[T::W3 * m - 1] + P[T::W3 * m + 1];
    }
#pragma unroll
    for (int m = 0; m < R; ++m) {
      const S c3[3] = {cc[m], cc[m + 1], cc[m + 2]}, s3[3] = {ss[m], ss[m + 1], ss[m + 2]};
      dst[(tx + 2) + T::W2 * (R * ty + m + 2)] = mu(c3, s3, y0 + R * ty + m);
    }
  }
  constexpr int kRows = 4 * T::W2;  // two rows below the tile and two above
  constexpr int kFrame = kRows + 4 * T::TY;
#pragma unroll
  for (int f = tid; f < kFrame; f += T::NT) {
    int i, j;
    if (f < kRows) {
      i = f % T::W2;
      j = f / T::W2;
      if (j >= 2) j += T::TY;
    } else {
      const int q = f - kRows;
      i = (q & 3) < 2 ? (q & 3) : (q & 3) + T::TX;
      j = 2 + (q >> 2);
    }
    const S* P = src + (i + 1) + T::W3 * j;
    const S c3[3] = {P[0], P[T::W3], P[2 * T::W3]};
    const S s3[3] = {P[-1] + P[1], P[T::W3 - 1] + P[T::W3 + 1],
                     P[2 * T::W3 - 1] + P[2 * T::W3 + 1]};
    dst[i + T::W2 * j] = mu(c3, s3, y0 - 2 + j);
  }
}

// The variant's gradient of m at the centre P in a halo-2 region (row yr).
template <typename S, int SMOL, bool WALLS, int W2>
__device__ __forceinline__ void grad2(const Geom& g, const S* P, int yr, S& gx, S& gy) {
  using L = Lat<9>;
  if constexpr (SMOL == kFD) {
    gx = S(0.5) * (P[1] - P[-1]);
    gy = S(0.5) * (P[W2] - P[-W2]);
  } else {
    gx = gy = S(0);
#pragma unroll
    for (int q = 1; q < 9; ++q) {
      const bool cut = WALLS && (yr + L::cy[q] < 0 || yr + L::cy[q] >= g.ny);
      const S t = S(L::w[q]) * (cut ? P[0] : P[L::cx[q] + W2 * L::cy[q]]);
      if (L::cx[q]) gx += L::cx[q] * t;
      if (L::cy[q]) gy += L::cy[q] * t;
    }
    gx *= S(3);
    gy *= S(3);
  }
}

// Gamma . X at the centre e of two halo-1 component planes (FV, row yr): a
// link across a wall takes minus the centre's X.
template <typename S, bool WALLS, int W1>
__device__ __forceinline__ S div2_fv(const Geom& g, const S* X, const S* Y, int e, int yr) {
  using L = Lat<9>;
  S G = 0;
#pragma unroll
  for (int q = 1; q < 9; ++q) {
    const bool cut = WALLS && (yr + L::cy[q] < 0 || yr + L::cy[q] >= g.ny);
    const int k = cut ? e : e + L::cx[q] + W1 * L::cy[q];
    S v = 0;
    if (L::cx[q]) v += L::cx[q] * X[k];
    if (L::cy[q]) v += L::cy[q] * Y[k];
    G += S(L::w[q]) * (cut ? -v : v);
  }
  return S(3) * G;
}

// What a stage advects and diffuses at one point of the halo-1 region: FD the
// products u phi, FV the node flux J = -u phi + M Gamma mu.
template <typename S, int SMOL>
__device__ __forceinline__ void stage_flux2(const Coef<S>& c, const S (&u)[2], S ph, S gx, S gy,
                                            S& fx, S& fy) {
  if constexpr (SMOL == kFD) {
    fx = u[0] * ph;
    fy = u[1] * ph;
  } else {
    fx = -u[0] * ph + c.M * gx;
    fy = -u[1] * ph + c.M * gy;
  }
}

// G without the noise at the tile point (tx, t): FD -D.(u phi) + M L mu from
// the flux region and mu, FV Gamma . J.
template <typename S, int SMOL, bool WALLS, int R>
__device__ __forceinline__ S stage_rate2(const Geom& g, const Coef<S>& c, const S* sx, const S* sy,
                                         const S* smu, int tx, int t, int y) {
  constexpr int W1 = Tile2<R>::W1, W2 = Tile2<R>::W2;
  const int e = (tx + 1) + W1 * (t + 1);
  if constexpr (SMOL == kFD) {
    const S adv = S(0.5) * (sx[e + 1] - sx[e - 1]) + S(0.5) * (sy[e + W1] - sy[e - W1]);
    const S* P = smu + (tx + 2) + W2 * (t + 2);
    const S lap = lap_so<S, 2>([&](int dx, int dy, int) { return P[dx + W2 * dy]; });
    return -adv + c.M * lap;
  } else {
    return div2_fv<S, WALLS, W1>(g, sx, sy, e, y);
  }
}

template <typename S, bool DEV, int SMOL, bool GHOST, int NT, bool WALLS, int R>
__device__ __forceinline__ void half1_body(const HalfArgs<S>& a, int bx, int by) {
  using L = Lat<9>;
  using T = Tile2<R>;
  constexpr int WZ = SMOL == kFD ? T::TX + 1 : T::W1;  // FD reads no normals at x0 + TX
  constexpr int NZ = SMOL == kFD ? 4 : 2;
  __shared__ S spsi[T::W3 * T::H3], smu[T::W2 * T::H2];
  __shared__ S sx[T::W1 * T::H1], sy[T::W1 * T::H1];
  __shared__ S sz[NZ][WZ * T::H1];
  __shared__ NormalTables<S> tables;
  const Geom& g = a.lb.g;
  const int tid = threadIdx.x, tx = tid % T::TX, ty = tid / T::TX;
  const int x0 = bx * T::TX, y0 = by * T::TY;
  const bool near = g.nx >= T::TX + 8 && g.ny >= T::TY + 8;
  const int x = x0 + tx;

  // Points past the edge of a ragged tile stand for their periodic images:
  // the ring of the live points may reach them.
  const int xw = wrap_r(x, g.nx, near);
  int yw[R], s[R];
  bool live[R];
  S fv[R][9];
  const bool fill = NormalTables<S>::kUsed && (a.lb.noise || a.smol_noise);
  typename NormalTables<S>::Part part{};
  if (fill) part = NormalTables<S>::fetch(tid);
  const Region3<R> reg(g, x0, y0, near, tid);
  S ep[Region3<R>::NK + 1];
  reg.fetch(a.psi, ep);
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const int y = y0 + R * ty + m;
    live[m] = x < g.nx && y < g.ny;
    yw[m] = wrap_r(y, g.ny, near);
    const Nbr nb(g, xw, yw[m], 0);
    s[m] = nb.at(0, 0, 0);
    lb_pull<S, 9, kCached, WALLS>(a.lb, nb, yw[m], 0, fv[m]);
  }
  RingPull<S, R, WALLS> ring(a.lb, x0, y0, near, tid);
  reg.store(ep, spsi);
  if (fill) tables.store(tid, part);
  __syncthreads();
  mu_region2<S, R, WALLS>(g, a.c, y0, tid, spsi, smu);

  // one site of the halo-1 normals
  auto draw = [&](uint32_t site, int e) {
    S zz[4];
    if constexpr (SMOL == kFD)
      Normal4<S>::gen(site, a.lb.step, 0, kTagSMOL, a.lb.k0, a.lb.k1, tables, zz);
    else
      Normal4<S>::gen2(site, a.lb.step, 0, kTagSMOL, a.lb.k0, a.lb.k1, tables, zz);
#pragma unroll
    for (int c = 0; c < NZ; ++c) sz[c][e] = zz[c];
  };
  if (a.smol_noise) {
#pragma unroll
    for (int m = 0; m < R; ++m)
      draw(static_cast<uint32_t>(s[m]), (tx + 1) + WZ * (R * ty + m + 1));
  }
  __syncthreads();

  S nk[kModeSlots<9>] = {};
  S u[2], gx, gy;
  auto keep_u = [&](S ux, S uy, S) {
    u[0] = ux;
    u[1] = uy;
  };
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const int t = R * ty + m;
    const S ps = spsi[(tx + 3) + T::W3 * (t + 3)];
    grad2<S, SMOL, WALLS, T::W2>(g, smu + (tx + 2) + T::W2 * (t + 2), yw[m], gx, gy);
    const S F[3] = {-ps * gx, -ps * gy, S(0)};
    if (live[m]) {
      if (a.lb.noise) lb_mode_noise<S, 9>(a.lb, s[m], tables, nk);
      lb_update<S, DEV, 9, GHOST, true, NT>(a.lb, s[m], fv[m], F, nk, [&](S ux, S uy, S) {
        u[0] = ux;
        u[1] = uy;
        if (a.lb.u_out) store_vec<S, 2, NT>(a.lb.u_out, g.N, s[m], ux, uy, S(0));
      });
    } else {
      lb_update<S, DEV, 9, false, false, NT>(a.lb, s[m], fv[m], F, nk, keep_u);
    }
    const int e = (tx + 1) + T::W1 * (t + 1);
    stage_flux2<S, SMOL>(a.c, u, ps, gx, gy, sx[e], sy[e]);
  }
  // The ring's velocities from the first thread on, the halo's normals from the
  // last one down.
  if (tid < T::kRing) {
    const int i = ring.i, j = ring.j;
    const S ps = spsi[(i + 2) + T::W3 * (j + 2)];
    grad2<S, SMOL, WALLS, T::W2>(g, smu + (i + 1) + T::W2 * (j + 1), ring.y, gx, gy);
    const S F[3] = {-ps * gx, -ps * gy, S(0)};
    lb_update<S, DEV, 9, false, false, false>(a.lb, s[0], ring.f, F, nk, keep_u);
    const int e = i + T::W1 * j;
    stage_flux2<S, SMOL>(a.c, u, ps, gx, gy, sx[e], sy[e]);
  }
  if (a.smol_noise && T::NT - 1 - tid < T::kRing) {
    int i, j;
    ring_pos<R>(T::NT - 1 - tid, i, j);
    if (i < WZ)
      draw(static_cast<uint32_t>(wrap_r(x0 - 1 + i, g.nx, near) +
                                 g.nx * wrap_r(y0 - 1 + j, g.ny, near)),
           i + WZ * j);
  }
  __syncthreads();

#pragma unroll
  for (int m = 0; m < R; ++m) {
    if (!live[m]) continue;
    const int t = R * ty + m;
    S N = 0;
    if (a.smol_noise) {
      if constexpr (SMOL == kFD) {
        // one flux per undirected link: N = sum_l A_l [zeta_l(x - c_l) - zeta_l(x)]
        const int own = (tx + 1) + WZ * (t + 1);
        static_for<L::NLINKS>([&](auto lc) {
          constexpr int l = decltype(lc)::value;
          constexpr double rt = ce_sqrt(L::lw[l]);
          const S A = a.amp * S(rt);
          N -= A * sz[l][own];
          N += A * sz[l][(tx + 1 - L::lx[l]) + WZ * (t + 1 - L::ly[l])];
        });
      } else {
        N = a.amp *
            div2_fv<S, WALLS, T::W1>(g, sz[0], sz[1], (tx + 1) + T::W1 * (t + 1), y0 + t);
      }
    }
    const S rate = stage_rate2<S, SMOL, WALLS, R>(g, a.c, sx, sy, smu, tx, t, y0 + t);
    a.rate[s[m]] = rate;
    a.phi[s[m]] = spsi[(tx + 3) + T::W3 * (t + 3)] + (rate + N);
  }
}

template <typename S, bool DEV, int SMOL, bool WALLS, int R>
__device__ __forceinline__ void half2_body(const HalfArgs<S>& a, int bx, int by) {
  using T = Tile2<R>;
  __shared__ S spsi[T::W3 * T::H3], sphi[T::W3 * T::H3];
  __shared__ S smu[T::W2 * T::H2], snu[T::W2 * T::H2];  // mu(psi^n), mu(phi^1)
  __shared__ S sx[T::W1 * T::H1], sy[T::W1 * T::H1];
  const Geom& g = a.lb.g;
  const int tid = threadIdx.x, tx = tid % T::TX, ty = tid / T::TX;
  const int x0 = bx * T::TX, y0 = by * T::TY;
  const bool near = g.nx >= T::TX + 8 && g.ny >= T::TY + 8;
  const int x = x0 + tx;
  const int xw = wrap_r(x, g.nx, near);
  int yw[R], s[R];
  bool live[R];
  S fv[R][9], rate[R];
  const Region3<R> reg(g, x0, y0, near, tid);
  S ep[Region3<R>::NK + 1], eh[Region3<R>::NK + 1];
  reg.fetch(a.psi, ep);
  reg.fetch(static_cast<const S*>(a.phi), eh);
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const int y = y0 + R * ty + m;
    live[m] = x < g.nx && y < g.ny;
    yw[m] = wrap_r(y, g.ny, near);
    const Nbr nb(g, xw, yw[m], 0);
    s[m] = nb.at(0, 0, 0);
    lb_pull<S, 9, kCached, WALLS>(a.lb, nb, yw[m], 0, fv[m]);
    rate[m] = live[m] ? a.rate[s[m]] : S(0);
  }
  RingPull<S, R, WALLS> ring(a.lb, x0, y0, near, tid);
  reg.store(ep, spsi);
  reg.store(eh, sphi);
  __syncthreads();
  mu_region2<S, R, WALLS>(g, a.c, y0, tid, spsi, smu);
  mu_region2<S, R, WALLS>(g, a.c, y0, tid, sphi, snu);
  __syncthreads();

  S nk[kModeSlots<9>] = {};
  // the velocity of the streamed populations, (jbar^{n+1} + F^n/2)/rho^{n+1},
  // and the stage's flux at one point of the halo-1 region
  auto point = [&](const S (&f)[9], int i, int j, int yr) {
    S gx, gy, u[2];
    grad2<S, SMOL, WALLS, T::W2>(g, smu + (i + 1) + T::W2 * (j + 1), yr, gx, gy);
    const S ps = spsi[(i + 2) + T::W3 * (j + 2)];
    const S F[3] = {-ps * gx, -ps * gy, S(0)};
    lb_update<S, DEV, 9, false, false, false>(a.lb, s[0], f, F, nk, [&](S ux, S uy, S) {
      u[0] = ux;
      u[1] = uy;
    });
    if constexpr (SMOL == kFV)
      grad2<S, SMOL, WALLS, T::W2>(g, snu + (i + 1) + T::W2 * (j + 1), yr, gx, gy);
    const int e = i + T::W1 * j;
    stage_flux2<S, SMOL>(a.c, u, sphi[(i + 2) + T::W3 * (j + 2)], gx, gy, sx[e], sy[e]);
  };
#pragma unroll
  for (int m = 0; m < R; ++m) point(fv[m], tx + 1, R * ty + m + 1, yw[m]);
  if (tid < T::kRing) point(ring.f, ring.i, ring.j, ring.y);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < R; ++m) {
    if (!live[m]) continue;
    const int t = R * ty + m;
    const S r1 = stage_rate2<S, SMOL, WALLS, R>(g, a.c, sx, sy, snu, tx, t, y0 + t);
    a.out[s[m]] = sphi[(tx + 3) + T::W3 * (t + 3)] + S(0.5) * (r1 - rate[m]);
  }
}

// The tile of a launch: the wide one once its tiles fill the chip six times over
// and it covers at most a tenth more sites than the narrow one.  Below that
// there are too few blocks to hide a block's serial chain (FP64 FD, R = 2
// against 1: 64^2 16.3 against 11.8 us a step, 724^2 46.4 against 46.5); above,
// the longer rows and fewer ring sites count (1000^2 67.1 against 68.6, 4096^2
// 1053 against 1120, FP32 546 against 621).
constexpr long kWideTiles = 6 * 256;
struct HalfTiles {
  long narrow = 0, wide = 0;
  void add(int nx, int ny) {
    narrow += tiles<1>(nx, ny);
    wide += tiles<2>(nx, ny);
  }
  bool use_wide() const { return wide >= kWideTiles && 20 * wide <= 11 * narrow; }

 private:
  template <int R>
  static long tiles(int nx, int ny) {
    using T = Tile2<R>;
    return static_cast<long>((nx + T::TX - 1) / T::TX) * ((ny + T::TY - 1) / T::TY);
  }
};

template <int R>
__host__ inline TileMap make_half_map(int nx, int ny, bool swizzle) {
  TileMap m{};
  m.ntx = (nx + Tile2<R>::TX - 1) / Tile2<R>::TX;
  m.nty = (ny + Tile2<R>::TY - 1) / Tile2<R>::TY;
  m.nt = m.ntx * m.nty;
  m.per = swizzle ? (m.nt + 7) / 8 : 0;
  return m;
}

template <typename S, bool DEV, int SMOL, bool GHOST, int NT, bool WALLS, int R>
__global__ __launch_bounds__(Tile2<R>::NT) void k_half1(HalfArgs<S> a, TileMap m) {
  int bx, by, bz;
  if (tile_of(m, bx, by, bz)) half1_body<S, DEV, SMOL, GHOST, NT, WALLS, R>(a, bx, by);
}

template <typename S, bool DEV, int SMOL, bool WALLS, int R>
__global__ __launch_bounds__(Tile2<R>::NT) void k_half2(HalfArgs<S> a, TileMap m) {
  int bx, by, bz;
  if (tile_of(m, bx, by, bz)) half2_body<S, DEV, SMOL, WALLS, R>(a, bx, by);
}

}  // namespace lbl
