// msl_stream2s.hpp -- stream-collide of the 2D sets whose windows do not fit
// in LDS: thermal D2Q25 and D2Q36 in FP64 (50 and 72 planes).
//
// A wave per x node: lanes are 64 cells of a row, wave a of a workgroup streams
// the 2 N planes of x node a (f and g, every y node) for its cells, straight
// from memory into registers, and the workgroup's waves exchange only the
// moments (four partial sums per cell, through LDS).  A wave so holds 2 N R
// values where a lane that held all planes of its cells spilled 3 KB, and its
// loads are all independent: that form took a plane at a time from LDS behind
// a barrier, 89 us on an 8192 x 4 tube with a few live tiles, all of it
// latency; this one 11 us (2048^2 D2Q36: 10.24 -> 2.89 ms a step, the rate of
// the L1 reads: a value is read nine times, 3 columns of R + 2 rows for R rows
// of cells).
#pragma once
#include "msl_device.hpp"

template <int N, int R, bool QE>
__global__ void __launch_bounds__(64 * N)
k_sc2d_split(const Tab *__restrict__ tab, int lat, Geo g, const double *__restrict__ in, double *__restrict__ out,
             const uint8_t *__restrict__ cls, const uint8_t *__restrict__ tflag, int faces) {
  constexpr int Q = N * N;
  __shared__ double red[N][R][4][64];
  __shared__ double redq[QE ? N : 1][QE ? R : 1][6][64];
  const LatTab &L = tab->lat[lat];
  const int lin = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  const int tile = msl_xcd_tile(lin, (int)(gridDim.x * gridDim.y));
  const int x0 = (tile % (int)gridDim.x) * MSL_TX, y0 = (tile / (int)gridDim.x) * R;
  if (!(tflag[(y0 / MSL_MTY) * g.ntx + x0 / MSL_TX] & (1 << lat))) return;
  const int lane = threadIdx.x & 63;
  const int a = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);   // x node
  const int x = x0 + lane;
  // ghost points mapped by their faces' rules (two bits per face: 1 periodic,
  // 2 zero-gradient, 0 stored); a stored ghost row keeps its own x ghosts
  auto mapped = [&](int ax, int p, int n) {
    if (p >= 0 && p < n) return p;
    const int rule = (faces >> (4 * ax + (p < 0 ? 0 : 2))) & 3;
    return rule == 1 ? (p < 0 ? p + n : p - n) : (rule == 2 ? (p < 0 ? 0 : n - 1) : p);
  };
  int xr[3], xm[3];   // columns of the departure stencil, lanes outside at the last ghost
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int X = min(x + L.n0[0][a] - 1 + k, g.nx + MSL_G - 1);
    xr[k] = g.xo + X;
    xm[k] = g.xo + mapped(0, X, g.nx);
  }
  const double wx0 = L.a[0][a][0], wx2 = L.a[0][a][2], cx = L.v[0][a];
  double v[2][N][R];   // streamed f and g of (a, b)
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int b = 0; b < N; ++b) {
      const double *pl = in + (long long)(p * Q + a + N * b) * g.plane;
      const double wy0 = L.a[1][b][0], wy2 = L.a[1][b][2];
      double h[R + 2];
#pragma unroll
      for (int r = 0; r < R + 2; ++r) {
        const int Y = mapped(1, y0 + L.n0[1][b] - 1 + r, g.ny);
        const double *row = pl + (long long)(Y + MSL_G) * g.pitch;
        const bool raw = Y < 0 || Y >= g.ny;
        const double l = row[raw ? xr[0] : xm[0]], m = row[raw ? xr[1] : xm[1]], q = row[raw ? xr[2] : xm[2]];
        // differenced form: the centre weight is 1 - w0 - w2 exactly, so a
        // uniform field is reproduced without a rounding bias in the weights
        h[r] = m + wx0 * (l - m) + wx2 * (q - m);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) v[p][b][r] = h[r + 1] + wy0 * (h[r] - h[r + 1]) + wy2 * (h[r + 2] - h[r + 1]);
    }
  // moments (Sec. II.B): this wave's part, then the sum over the waves
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double s = 0, jy = 0, e = 0;
#pragma unroll
    for (int b = 0; b < N; ++b) {
      const double cy = L.v[1][b], f = v[0][b][r];
      s += f;
      jy += cy * f;
      e += 0.5 * (cx * cx + cy * cy) * f + v[1][b][r];
    }
    red[a][r][0][lane] = s;
    red[a][r][1][lane] = cx * s;
    red[a][r][2][lane] = jy;
    red[a][r][3][lane] = e;
  }
  __syncthreads();
  double om = tab->omega, tl = tab->tau, rho[R], ux[R], uy[R], T[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double m[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int w = 0; w < N; ++w) m[k] += red[w][r][k][lane];
    const double ird = 1.0 / m[0];
    rho[r] = m[0];
    ux[r] = m[1] * ird;
    uy[r] = m[2] * ird;
    T[r] = (m[3] - 0.5 * m[0] * (ux[r] * ux[r] + uy[r] * uy[r])) / (tab->cv * m[0]);
  }
  // x factor of this wave's node: falling factorials k of its Hermite series
  // (k = 0: the equilibrium factor)
  auto xfactor = [&](double u, double theta, int k) {
    double b[N], s = 0;
    b[0] = 1.0;
    b[1] = u;
#pragma unroll
    for (int j = 1; j + 1 < N; ++j) b[j + 1] = u * b[j] + (double)j * (theta - 1.0) * b[j - 1];
#pragma unroll
    for (int j = k; j < N; ++j) {
      double fall = 1.0;
      for (int m = 0; m < k; ++m) fall *= (double)(j - m);
      s += L.hw[a][j] * fall * b[j - k];
    }
    return s;
  };
  if constexpr (QE) {
    // two-relaxation model: this wave's part of Qbar, qbar (eqs. Pond_f/g)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double Py[N], q[6] = {0, 0, 0, 0, 0, 0};
      eq_axis<double, N>(L, (uy[r] - L.ur[1]) * L.isq, T[r] * L.iTr, Py);
      const double Px = rho[r] * xfactor((ux[r] - L.ur[0]) * L.isq, T[r] * L.iTr, 0);
      const double dx = cx - ux[r], gf = tab->gfac * T[r];
#pragma unroll
      for (int b = 0; b < N; ++b) {
        const double dy = L.v[1][b] - uy[r], feq = Px * Py[b], nf = v[0][b][r] - feq, ng = v[1][b][r] - gf * feq;
        q[0] += dx * dx * dx * nf;
        q[1] += dx * dx * dy * nf;
        q[2] += dx * dy * dy * nf;
        q[3] += dy * dy * dy * nf;
        q[4] += dx * ng;
        q[5] += dy * ng;
      }
#pragma unroll
      for (int k = 0; k < 6; ++k) redq[a][r][k][lane] = q[k];
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int y = y0 + r;
    const bool inside = x < g.nx && y < g.ny;
    const bool mine = inside && (cls[inside ? (long long)y * g.nx + x : 0] & 1) == lat;
    if (tab->tau_mode == 1) {
      const double mu = tab->mu_ref * pow(T[r] / tab->tau_ref_T, tab->mu_exp);
      tl = mu / (rho[r] * T[r] * tab->dt) + 0.5;
      om = 1.0 / tl;
    }
    const double hx = (ux[r] - L.ur[0]) * L.isq, hy = (uy[r] - L.ur[1]) * L.isq, th = T[r] * L.iTr;
    double Py[N];
    eq_axis<double, N>(L, hy, th, Py);
    const double Px = rho[r] * xfactor(hx, th, 0), gf = tab->gfac * T[r];
    // quasi-equilibrium terms, folded with (omega1 - omega2) and constants
    double Ax[4], Ay[QE ? 4 : 1][N], Qb[6];
    if constexpr (QE) {
#pragma unroll
      for (int k = 0; k < 4; ++k) Ax[k] = xfactor(hx, th, k);
      qe_axis<double, N>(L, hy, th, Ay);
      const double dom = 1.0 / tl - 1.0 / (0.5 + (tl - 0.5) * tab->qe_ratio);
      const double cf = L.isq * L.isq * L.isq / 6.0 * dom, cg = L.isq * dom;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        Qb[k] = 0;
#pragma unroll
        for (int w = 0; w < N; ++w) Qb[k] += redq[w][r][k][lane];
        Qb[k] *= k > 3 ? cg : (k == 1 || k == 2 ? 3.0 * cf : cf);
      }
    }
    double *po = out + (long long)a * g.plane + g.idx(inside ? x : 0, inside ? y : 0, 0);
#pragma unroll
    for (int b = 0; b < N; ++b) {
      const double feq = Px * Py[b];
      double fo = v[0][b][r] + om * (feq - v[0][b][r]);
      double go = v[1][b][r] + om * (gf * feq - v[1][b][r]);
      if constexpr (QE) {
        fo += Qb[0] * Ax[3] * Ay[0][b] + Qb[1] * Ax[2] * Ay[1][b] + Qb[2] * Ax[1] * Ay[2][b] + Qb[3] * Ax[0] * Ay[3][b];
        go += Qb[4] * Ax[1] * Ay[0][b] + Qb[5] * Ax[0] * Ay[1][b];
      }
      if (mine) {
        po[(long long)(N * b) * g.plane] = fo;
        po[(long long)(Q + N * b) * g.plane] = go;
      }
    }
  }
}
