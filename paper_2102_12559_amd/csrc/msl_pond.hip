// msl_pond.hip -- the step in co-moving reference frames (PonD, Sec. II.C.1),
// one or two velocity sets, 2D, FP64.
//
// Every cell keeps its post-collision populations in its own frame
// lambda = {u, T} (eq. reference; particle velocities sqrt(T) c_i + u, eq. vi,
// with T_L = 1).  A group of lanes owns one cell, one lane per x node of the
// velocity set; a workgroup's cells are an x segment of four rows, and the
// neighbourhood of the tile (populations and frames, boundary rules applied)
// is staged in LDS once.  Per iteration of the predictor-corrector:
// each lane finds its populations' departure points x - v_i dt in the current
// frame, and for each of the 3 x 3 collocation points around the nearest node
// transfers that point's population vector from its own frame to the current
// one and keeps its own components (eqs. reconstructionPond, fll).  The
// transfer G = M_target^{-1} M_source of the moment matrices of eq. momf
// factorises per axis, and its one-axis factor is the Lagrange basis of the
// lattice nodes evaluated at the source nodes mapped into the target frame:
//   G_x[a][a'] = l_a((sqrt(T_s) c_a' + u_s,x - u_x) / sqrt(T)),
// because the inverse of a Vandermonde matrix holds the Lagrange basis
// polynomials of its nodes.  The group then sums rho, j, E of the
// reconstructed populations (shuffles over the cell's lanes), which define the
// next frame (eqs. correctorfields), until neither a velocity component nor T
// changes by more than 1e-14 (at most 60 passes).  The collision runs in the
// converged frame, where f^eq = rho W_i and g^eq = (cv - 1) T rho W_i (eqs.
// feqPond, geqPond), BGK or two-relaxation (eqs. fqeq, gqeq in the co-moving
// frame).
// With two velocity sets (Sec. III) the step launches once per set, over the
// cells of that set; afterwards every band cell (within two cells of the other
// set) converts its new state into the other set in its own new frame
// (lifting or projection, Sec. III.B-C), so a collocation point of the other
// set holds this set's populations in its own frame when the next step reads
// it.  The Knudsen-number criterion re-selects the sets every crit_every
// steps from each cell's own state; a cell whose set changes converts its
// state in its own frame.
#include <hip/hip_runtime.h>
#include <math.h>

#include "msl_band.hpp"

#define POND_MAXIT 60
#define POND_TOL 1e-14

struct PondArgs {
  int nx, ny;
  long long ncell;
  int bc[4];
  double st[4][5];   // fixed-equilibrium face states rho, ux, uy, uz, T
};

// sum over a cell's lanes (CW apart within the wave)
template <int CW>
__device__ __forceinline__ double cell_sum(double v) {
#pragma unroll
  for (int o = CW; o < 64; o <<= 1) v += __shfl_xor(v, o);
  return v;
}

// Lane layout of the step kernel.  A cell has GS lanes, one per x node a of its
// velocity set (GS = 4 or 8; lanes with a >= N idle), each of which carries the
// populations (a, b) of every y node b.  The stencil of a population is the
// product of an x offset that depends on a alone and a y offset that depends
// on b alone, so the transfer along x of a collocation point's populations is
// done once per (point, a) and shared by the y nodes, and the y rows of the
// transfer come from shared partial products.  (One lane per population, which
// repeats both for every population, issued about seven times the
// instructions.)  SPX: the three point columns of a stencil go to lanes of
// their own as well (16 lanes per cell, 3 N of them at work), whose partial
// populations are added once the frame has converged; the sums that define the
// next frame are linear, so they need no such step.  A third of the serial
// work per lane, for grids that leave the chip idle, and a better fit of
// N = 5 (15 of 16 lanes against 5 of 8).  A wave holds one row segment of CW
// cells, node-major (lane = index CW + cell), a workgroup four rows of it.
template <int N, bool TH, bool SPX>
struct PondTraits {
  static constexpr int Q = N * N;
  static constexpr int NP = TH ? 2 * Q : Q;
  static_assert(!SPX || 3 * N <= 16, "16 lanes per cell");
  static constexpr int GS = SPX ? 16 : (N <= 4 ? 4 : 8);   // lanes per cell
  static constexpr int PTS = SPX ? 1 : 3;     // point columns per lane
  static constexpr int CW = 64 / GS;          // cells of a wave: one x segment of a row
  static constexpr int TY = 4;                // rows of a workgroup
  static constexpr int SW = CW + 4;           // staged columns (two on each side)
  static constexpr int SP = SW * (TY + 4);    // staged collocation points
  // doubles per staged point: populations, frame velocity, sqrt of its
  // temperature; an odd number of 16-byte units, so that 16 consecutive points
  // start in different LDS banks
  static constexpr int EV = (NP + 3 + 1) / 2 * 2;
  static constexpr int STRIDE = EV / 2 % 2 ? EV : EV + 2;
};

// unnormalised Lagrange basis at z: l[b] = prod_{c != b} (z - x_c), from shared
// products of pairs
template <int N>
__host__ __device__ __forceinline__ void lagrange_products(double z, const double *xn, double *l) {
  double d[N];
#pragma unroll
  for (int m = 0; m < N; ++m) d[m] = z - xn[m];
  if constexpr (N == 3) {
    l[0] = d[1] * d[2];
    l[1] = d[0] * d[2];
    l[2] = d[0] * d[1];
  } else if constexpr (N == 4) {
    const double p = d[0] * d[1], q = d[2] * d[3];
    l[0] = d[1] * q;
    l[1] = d[0] * q;
    l[2] = d[3] * p;
    l[3] = d[2] * p;
  } else if constexpr (N == 5) {
    const double p = d[0] * d[1], q = d[2] * d[3], p4 = p * d[4], q4 = q * d[4];
    l[0] = d[1] * q4;
    l[1] = d[0] * q4;
    l[2] = d[3] * p4;
    l[3] = d[2] * p4;
    l[4] = p * q;
  } else {
    static_assert(N == 6, "velocity sets of 3 to 6 nodes per axis");
    const double p = d[0] * d[1], q = d[2] * d[3], r = d[4] * d[5], qr = q * r, pr = p * r, pq = p * q;
    l[0] = d[1] * qr;
    l[1] = d[0] * qr;
    l[2] = d[3] * pr;
    l[3] = d[2] * pr;
    l[4] = d[5] * pq;
    l[5] = d[4] * pq;
  }
}

// the collocation point (x, y) (possibly outside the domain): the cell index
// whose state it takes, -1 - face for a fixed-equilibrium face state, or
// -5 - (side nx + x) for the diffuse wall point of column x on the low (side
// 0) or high y face
__device__ __forceinline__ long long pond_resolve(const PondArgs &pa, int x, int y) {
  if (x < 0 && pa.bc[0] == MSL_BC_FIXED_EQ) return -1;
  if (x >= pa.nx && pa.bc[1] == MSL_BC_FIXED_EQ) return -2;
  if (y < 0 && pa.bc[2] == MSL_BC_FIXED_EQ) return -3;
  if (y >= pa.ny && pa.bc[3] == MSL_BC_FIXED_EQ) return -4;
  if (x < 0 || x >= pa.nx) x = pa.bc[0] == MSL_BC_PERIODIC ? (x + pa.nx) % pa.nx : (x < 0 ? 0 : pa.nx - 1);
  if (y < 0 && pa.bc[2] == MSL_BC_DIFFUSE_WALL) return -5 - (long long)x;
  if (y >= pa.ny && pa.bc[3] == MSL_BC_DIFFUSE_WALL) return -5 - ((long long)pa.nx + x);
  if (y < 0 || y >= pa.ny) y = pa.bc[2] == MSL_BC_PERIODIC ? (y + pa.ny) % pa.ny : (y < 0 ? 0 : pa.ny - 1);
  return (long long)y * pa.nx + x;
}

// Bound by FP64 issue (the VALU issues about 80 % of the time).  A step of
// 1024^2 thermal D2Q16, 3 passes: 6.7 ms with one lane per population and
// pass counts by atomics, 0.78 ms now; 512^2: 1692 us, 225 us now (432 us with
// the atomics).  The 4096 x 4 two-set shock, bound by latency: 139 and 122 us
// for its D2Q16 and D2Q25 launches, 29 and 45 us now.
template <int N, bool TH, bool QE, bool SPX>
__global__ void __launch_bounds__(256)
k_pond_step(const Tab *__restrict__ tab, int lat, const uint8_t *__restrict__ cls, PondArgs pa,
            const double *__restrict__ fin, const double *__restrict__ frin, double *__restrict__ fout,
            double *__restrict__ frout, int *__restrict__ flag, unsigned long long *__restrict__ stats,
            const double *__restrict__ wrho) {
  using Tr = PondTraits<N, TH, SPX>;
  constexpr int Q = Tr::Q, NP = Tr::NP, PTS = Tr::PTS, CW = Tr::CW, SW = Tr::SW, SP = Tr::SP, STRIDE = Tr::STRIDE;
  __shared__ __align__(16) double stg[SP * STRIDE];
  __shared__ int wstat[Tr::TY][2];
  const LatTab &L = tab->lat[lat];
  const int x0 = blockIdx.x * CW, y0 = blockIdx.y * Tr::TY;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // the lane's cell, x node and (SPX) point column
  const int c = lane % CW, li = lane / CW;
  const int a = SPX ? li % N : li, col = SPX ? (li / N < 3 ? li / N : 0) : 0;
  const int px = x0 + c, py = y0 + w;
  const bool inside = px < pa.nx && py < pa.ny;
  const long long k = inside ? (long long)py * pa.nx + px : 0;
  // cells of this launch's velocity set (with two sets); a tile without any
  // leaves before it stages its neighbourhood
  const bool cell_ok = inside && (cls[k] & 1) == lat;
  if (!__syncthreads_or(cell_ok)) return;
  const double dt = tab->dt, cv = tab->cv;
  // the collocation points around the tile, two on every side (populations and
  // frames, boundary rules applied): a thread takes one point, so that
  // neighbouring threads read neighbouring cells of a plane
  constexpr int NG = 256 / SP;
  static_assert(NG >= 1, "one staged point per thread");
  static_assert(CW >= MSL_POND_SLOT_X && Tr::TY == MSL_POND_SLOT_Y, "a statistics slot per workgroup");
  if ((int)threadIdx.x < NG * SP) {
    const int sp = threadIdx.x % SP, m0 = threadIdx.x / SP;
    const long long q = pond_resolve(pa, x0 - 2 + sp % SW, y0 - 2 + sp / SW);
    double *dst = stg + sp * STRIDE;
    if (q >= 0) {
#pragma unroll
      for (int m = 0; m < NP; m += NG)
        if (m + m0 < NP) dst[m + m0] = fin[(long long)(m + m0) * pa.ncell + q];
      if (m0 == 0) {
        dst[NP] = frin[q];
        dst[NP + 1] = frin[pa.ncell + q];
        dst[NP + 2] = sqrt(frin[3 * pa.ncell + q]);
      }
    } else {
      // a fixed-equilibrium face state, or a diffuse wall point at the wall
      // state with the column's wall density: rho W_i (and (cv - 1) T rho W_i)
      // in its own frame
      const bool wall = q <= -5;
      const long long wi = wall ? -5 - q : 0;
      const double *st = wall ? pa.st[wi < pa.nx ? 2 : 3] : pa.st[-1 - q];
      const double rs = wall ? wrho[wi] : st[0];
      const double Ts = TH ? st[4] : 1.0;
      for (int m = m0; m < NP; m += NG) {
        const int j = m % Q;
        dst[m] = (m < Q ? 1.0 : (cv - 1.0) * Ts) * rs * L.w[j % N] * L.w[j / N];
      }
      if (m0 == 0) {
        dst[NP] = st[1];
        dst[NP + 1] = st[2];
        dst[NP + 2] = sqrt(Ts);
      }
    }
  }
  __syncthreads();
  const bool act = cell_ok && (SPX ? li < 3 * N : li < N);   // lanes at work
  const bool own_f = cell_ok && li < N;                      // lanes that write populations
  // lattice nodes; the lane's node, the other nodes, and the Lagrange
  // denominators 1 / prod_{c != a} (x_a - x_c) along x (dena) and y (den)
  double xn[N], den[N], xo[N - 1], xa = L.cr[0], wa = L.w[0], dena = L.den[0];
#pragma unroll
  for (int m = 0; m < N; ++m) {
    xn[m] = L.cr[m];
    den[m] = L.deny[m];
  }
#pragma unroll
  for (int m = 0; m < N - 1; ++m) xo[m] = a <= m ? xn[m + 1] : xn[m];
#pragma unroll
  for (int m = 1; m < N; ++m)
    if (a == m) {
      xa = xn[m];
      wa = L.w[m];
      dena = L.den[m];
    }
  const double *own = stg + ((w + 2) * SW + c + 2) * STRIDE;
  double ux = inside ? frin[k] : 0.0, uy = inside ? frin[pa.ncell + k] : 0.0,
         T = inside ? frin[3 * pa.ncell + k] : 1.0;
  double ft[N], gt[TH ? N : 1], rho = 0.0, Tn = 1.0;
#pragma unroll
  for (int b = 0; b < N; ++b) {
    ft[b] = 0.0;
    if (TH) gt[TH ? b : 0] = 0.0;
  }
  bool done = !cell_ok;
  int it = 0;
  for (int pass = 1; pass <= POND_MAXIT; ++pass) {
    double r = 0.0, jx = 0.0, jy = 0.0, e = 0.0;
    if (!done) {
      it = pass;
      const double sT = sqrt(T), isT = 1.0 / sT;
      const double vx = sT * xa + ux, dx = -vx * dt;
      const int nx0 = (int)floor(dx + 0.5);
      bool out = nx0 < -1 || nx0 > 1;
      const double xi = dx - nx0;
      // 3-point Lagrange weights through -1, 0, 1, with the denominator of the
      // lane's transfer row
      const double w3[3] = {dena * (0.5 * xi * (xi - 1.0)), dena * (1.0 - xi * xi), dena * (0.5 * xi * (xi + 1.0))};
      double wx[PTS];
#pragma unroll
      for (int m = 0; m < PTS; ++m) wx[m] = SPX ? (col == 0 ? w3[0] : (col == 1 ? w3[1] : w3[2])) : w3[m];
      int ny0[N];
      double yi[N];
#pragma unroll
      for (int b = 0; b < N; ++b) {
        const double dy = -(sT * xn[b] + uy) * dt;
        ny0[b] = (int)floor(dy + 0.5);
        yi[b] = dy - ny0[b];
        out |= ny0[b] < -1 || ny0[b] > 1;
      }
      if (act && out) atomicOr(flag, 1);
      // (a lane whose stencil left the reach reads the nearest staged points
      // instead; its cell is reported and its result is not used)
      const int ox = nx0 < -1 ? -1 : (nx0 > 1 ? 1 : nx0);
#pragma unroll
      for (int b = 0; b < N; ++b) {
        ny0[b] = ny0[b] < -1 ? -1 : (ny0[b] > 1 ? 1 : ny0[b]);
        ft[b] = 0.0;
        if (TH) gt[TH ? b : 0] = 0.0;
      }
#pragma unroll 1
      for (int sr = -2; sr <= 2; ++sr) {
        // the y weights of this row of points for every node b (zero outside
        // its stencil); a cell leaves out the rows that none of its nodes needs,
        // also where another cell of the wave needs them: their weights are zero,
        // but a point without a finite state would reach the cell all the same
        bool use = false;
        double wy[N];
#pragma unroll
        for (int b = 0; b < N; ++b) {
          const int s = sr - ny0[b];
          const bool in = s >= -1 && s <= 1;
          const double w0 = 1.0 - yi[b] * yi[b], w1 = 0.5 * yi[b] * (yi[b] + (double)s);
          use |= in;
          wy[b] = in ? (s == 0 ? w0 : w1) : 0.0;
        }
        if (!use) continue;
        double vf[N], vg[TH ? N : 1];
#pragma unroll
        for (int b = 0; b < N; ++b) {
          vf[b] = 0.0;
          if (TH) vg[TH ? b : 0] = 0.0;
        }
        const double *prow = own + (sr * SW + ox - 1 + col) * STRIDE;
        // the lane's points of the row, their populations read one y node ahead
        // of their use: with three waves per SIMD the LDS latency is otherwise
        // exposed at every node (the scheduling barriers keep the reads there)
        double cf[N], cg[TH ? N : 1], nf[N], ng[TH ? N : 1], fr[3];
        auto read = [&](int st, double (&f)[N], double (&g)[TH ? N : 1]) {
          const double *pt = prow + st / N * STRIDE + st % N * N;
#pragma unroll
          for (int ma = 0; ma < N; ++ma) {
            f[ma] = pt[ma];
            if (TH) g[TH ? ma : 0] = pt[Q + ma];
          }
        };
#pragma unroll
        for (int m = 0; m < 3; ++m) fr[m] = prow[NP + m];
        read(0, cf, cg);
        double s = 0.0, by = 0.0, gx[N];
#pragma unroll
        for (int st = 0; st < PTS * N; ++st) {
          const int sx = st / N, mb = st % N;
          if (mb == 0) {
            // the point's nodes in the current frame: z = s x + (u_s - u) / sqrt(T),
            // and the x row of the lane's node a
            s = fr[2] * isT;
            by = (fr[1] - uy) * isT;
            const double bx = (fr[0] - ux) * isT;
#pragma unroll
            for (int m = 0; m < N; ++m) {
              const double z = s * xn[m] + bx;
              double p = wx[sx] * (z - xo[0]);
#pragma unroll
              for (int cc = 1; cc < N - 1; ++cc) p *= z - xo[cc];
              gx[m] = p;
            }
          }
          if (st + 1 < PTS * N) read(st + 1, nf, ng);
          if (mb == N - 2 && sx < PTS - 1) {
#pragma unroll
            for (int m = 0; m < 3; ++m) fr[m] = prow[(sx + 1) * STRIDE + NP + m];
          }
          __builtin_amdgcn_sched_barrier(0);
          double sf = 0.0, sg = 0.0;
#pragma unroll
          for (int ma = 0; ma < N; ++ma) {
            sf += gx[ma] * cf[ma];
            if (TH) sg += gx[ma] * cg[TH ? ma : 0];
          }
          double gy[N];   // the y rows of every node at the point's node mb
          lagrange_products<N>(s * xn[mb] + by, xn, gy);
#pragma unroll
          for (int b = 0; b < N; ++b) {
            vf[b] += gy[b] * sf;
            if (TH) vg[TH ? b : 0] += gy[b] * sg;
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int ma = 0; ma < N; ++ma) {
            cf[ma] = nf[ma];
            if (TH) cg[TH ? ma : 0] = ng[TH ? ma : 0];
          }
        }
#pragma unroll
        for (int b = 0; b < N; ++b) {
          ft[b] += wy[b] * vf[b];
          if (TH) gt[TH ? b : 0] += wy[b] * vg[TH ? b : 0];
        }
      }
#pragma unroll
      for (int b = 0; b < N; ++b) {
        ft[b] *= den[b];
        if (TH) gt[TH ? b : 0] *= den[b];
        if (act) {
          const double vy = sT * xn[b] + uy;
          r += ft[b];
          jy += vy * ft[b];
          e += 0.5 * (vx * vx + vy * vy) * ft[b];
          if (TH) e += gt[TH ? b : 0];
        }
      }
      jx = vx * r;
    }
    // corrector: the cell's sums (every lane of the wave takes part)
    r = cell_sum<CW>(r);
    jx = cell_sum<CW>(jx);
    jy = cell_sum<CW>(jy);
    e = cell_sum<CW>(e);
    if (!done) {
      const double nux = jx / r, nuy = jy / r;
      const double nT = TH ? (e / r - 0.5 * (nux * nux + nuy * nuy)) / cv : 1.0;
      if (!(r > 0.0) || !(nT > 0.0) || !isfinite(r)) {
        if (li == 0) atomicOr(flag, 2);
        done = true;
      } else {
        const double delta = fmax(fabs(nT - T), fmax(fabs(nux - ux), fabs(nuy - uy)));
        rho = r;
        Tn = nT;
        if (delta <= POND_TOL || pass == POND_MAXIT) {
          done = true;
        } else {
          ux = nux;
          uy = nuy;
          T = nT;
        }
      }
    }
    if (__all(done)) break;
  }
  if constexpr (SPX) {
    // the three point columns' parts of each population
#pragma unroll
    for (int b = 0; b < N; ++b) {
      ft[b] += __shfl(ft[b], lane + N * CW) + __shfl(ft[b], lane + 2 * N * CW);
      if (TH) gt[TH ? b : 0] += __shfl(gt[TH ? b : 0], lane + N * CW) + __shfl(gt[TH ? b : 0], lane + 2 * N * CW);
    }
  }
  // collision in the converged frame {ux, uy, T}
  double tl = tab->tau;
  if (tab->tau_mode == 1) tl = tab->mu_ref * pow(Tn / tab->tau_ref_T, tab->mu_exp) / (rho * Tn * dt) + 0.5;
  const double om = 1.0 / tl, gq = (cv - 1.0) * T;
  double Qxxx = 0.0, Qxxy = 0.0, Qxyy = 0.0, Qyyy = 0.0, qx = 0.0, qy = 0.0, dom = 0.0;
  if constexpr (QE) {
    // quasi-equilibria in the co-moving frame (v - u = sqrt(T) c):
    // Qbar = T^{3/2} sum c c c (f - f^eq), qbar = T^{1/2} sum c (g - g^eq)
    dom = om - 1.0 / (0.5 + (tl - 0.5) * tab->qe_ratio);
#pragma unroll
    for (int b = 0; b < N; ++b) {
      const double cx = xa, cy = xn[b], feq = rho * (wa * L.w[b]);
      const double nf = own_f ? ft[b] - feq : 0.0, ng = own_f && TH ? gt[TH ? b : 0] - gq * feq : 0.0;
      Qxxx += cx * cx * cx * nf;
      Qxxy += cx * cx * cy * nf;
      Qxyy += cx * cy * cy * nf;
      Qyyy += cy * cy * cy * nf;
      qx += cx * ng;
      qy += cy * ng;
    }
    Qxxx = cell_sum<CW>(Qxxx);
    Qxxy = cell_sum<CW>(Qxxy);
    Qxyy = cell_sum<CW>(Qxyy);
    Qyyy = cell_sum<CW>(Qyyy);
    qx = cell_sum<CW>(qx);
    qy = cell_sum<CW>(qy);
  }
#pragma unroll
  for (int b = 0; b < N; ++b) {
    const double W = wa * L.w[b], feq = rho * W;
    double fo = ft[b] + om * (feq - ft[b]), go = 0.0;
    if (TH) go = gt[TH ? b : 0] + om * (gq * feq - gt[TH ? b : 0]);
    if constexpr (QE) {
      // f* - f^eq = W T^{-3/2}/6 Qbar : He3(c), Qbar = T^{3/2} (sums above)
      const double cx = xa, cy = xn[b];
      const double h = Qxxx * (cx * cx * cx - 3.0 * cx) + 3.0 * Qxxy * (cx * cx * cy - cy) +
                       3.0 * Qxyy * (cx * cy * cy - cx) + Qyyy * (cy * cy * cy - 3.0 * cy);
      fo += dom * W * h / 6.0;
      if (TH) go += dom * W * (qx * cx + qy * cy);
    }
    if (own_f) {
      fout[(long long)(a + N * b) * pa.ncell + k] = fo;
      if (TH) fout[(long long)(Q + a + N * b) * pa.ncell + k] = go;
    }
  }
  if (cell_ok && li == 0) {
    frout[k] = ux;
    frout[pa.ncell + k] = uy;
    frout[2 * pa.ncell + k] = 0.0;
    frout[3 * pa.ncell + k] = T;
  }
  // passes of the workgroup's cells, added to its own slot of the statistics
  // (launches that share a slot follow one another on the stream).  Atomics of
  // every wave on one counter took 385 us of a 432 us launch (512^2): updates of
  // one address are served one after the other, at about 12 ns each.
  int ws = cell_ok && li == 0 ? it : 0, wm = ws;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ws += __shfl_xor(ws, o);
    wm = max(wm, __shfl_xor(wm, o));
  }
  if (lane == 0) {
    wstat[w][0] = ws;
    wstat[w][1] = wm;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long *st = stats + 2 * ((size_t)blockIdx.y * gridDim.x + blockIdx.x);
    unsigned long long m = st[1];
    int sum = 0;
#pragma unroll
    for (int v = 0; v < Tr::TY; ++v) {
      sum += wstat[v][0];
      m = m > (unsigned)wstat[v][1] ? m : (unsigned)wstat[v][1];
    }
    st[0] += sum;
    st[1] = m;
  }
}

// pass counts of every workgroup: out[0] their sum, out[1] the maximum
__global__ void __launch_bounds__(256)
k_pond_stats(const unsigned long long *__restrict__ slots, long long n, unsigned long long *__restrict__ out) {
  __shared__ unsigned long long ss[256], sx[256];
  unsigned long long s = 0, m = 0;
  for (long long t = threadIdx.x; t < n; t += 256) {
    s += slots[2 * t];
    m = max(m, slots[2 * t + 1]);
  }
  ss[threadIdx.x] = s;
  sx[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      ss[threadIdx.x] += ss[threadIdx.x + w];
      sx[threadIdx.x] = max(sx[threadIdx.x], sx[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = ss[0];
    out[1] = sx[0];
  }
}

// every cell at the co-moving equilibrium of (rho, u, T) in its own frame, in
// each set (an equilibrium is the same state in both)
__global__ void k_pond_init(const Tab *__restrict__ tab, long long ncell, int thermal, int nlat,
                            const double *rho, const double *u, const double *T, double *f0, double *f1,
                            double *fr) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ncell) return;
  const double Tk = thermal ? T[k] : 1.0;
  for (int l = 0; l < nlat; ++l) {
    const LatTab &L = tab->lat[l];
    double *f = l ? f1 : f0;
    for (int i = 0; i < L.Q; ++i) {
      const double W = L.w[i % L.n] * L.w[i / L.n];
      f[(long long)i * ncell + k] = rho[k] * W;
      if (thermal) f[(long long)(L.Q + i) * ncell + k] = (tab->cv - 1.0) * Tk * rho[k] * W;
    }
  }
  fr[k] = u[k];
  fr[ncell + k] = u[ncell + k];
  fr[2 * ncell + k] = 0.0;
  fr[3 * ncell + k] = Tk;
}

// rho, u, T of cell k from its populations (set l) in its own frame
__device__ __forceinline__ void pond_cell_macros(const Tab *tab, int l, long long ncell, int thermal,
                                                 const double *f, const double *fr, long long k, double &r,
                                                 double &ux, double &uy, double &T) {
  const LatTab &L = tab->lat[l];
  const double sT = sqrt(fr[3 * ncell + k]), fx = fr[k], fy = fr[ncell + k];
  double jx = 0, jy = 0, e = 0;
  r = 0;
  for (int i = 0; i < L.Q; ++i) {
    const double fi = f[(long long)i * ncell + k];
    const double vx = sT * L.cr[i % L.n] + fx, vy = sT * L.cr[i / L.n] + fy;
    r += fi;
    jx += vx * fi;
    jy += vy * fi;
    e += 0.5 * (vx * vx + vy * vy) * fi;
    if (thermal) e += f[(long long)(L.Q + i) * ncell + k];
  }
  ux = jx / r;
  uy = jy / r;
  T = thermal ? (e / r - 0.5 * (ux * ux + uy * uy)) / tab->cv : 1.0;
}

// rho, u, T of every cell from its own set's populations in its own frame
__global__ void k_pond_macros(const Tab *__restrict__ tab, long long ncell, int thermal, const double *f0,
                              const double *f1, const uint8_t *__restrict__ cls, const double *fr, double *rho,
                              double *u, double *T) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ncell) return;
  const int l = cls[k] & 1;
  double r, ux, uy, t;
  pond_cell_macros(tab, l, ncell, thermal, l ? f1 : f0, fr, k, r, ux, uy, t);
  if (rho) rho[k] = r;
  if (u) {
    u[k] = ux;
    u[ncell + k] = uy;
  }
  if (T) T[k] = t;
}

// Knudsen-number criterion (Sec. IV.A.3), pass 1 on the co-moving state: each
// cell's density and hard-sphere mean free path
// lambda = 16/(5 sqrt(2 pi gamma)) mu a / p from its own set in its own frame
__global__ void k_pond_kn_fields(const Tab *__restrict__ tab, long long ncell, int thermal, const double *f0,
                                 const double *f1, const uint8_t *__restrict__ cls, const double *fr,
                                 double *__restrict__ rho, double *__restrict__ lam) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ncell) return;
  const int l = cls[k] & 1;
  double r, ux, uy, T;
  pond_cell_macros(tab, l, ncell, thermal, l ? f1 : f0, fr, k, r, ux, uy, T);
  const double mu = tab->tau_mode == 1 ? tab->mu_ref * pow(T / tab->tau_ref_T, tab->mu_exp)
                                       : (tab->tau - 0.5) * r * T * tab->dt;
  const double gam = (tab->cv + 1.0) / tab->cv;
  rho[k] = r;
  lam[k] = 16.0 / (5.0 * sqrt(2.0 * M_PI * gam)) * mu * sqrt(gam * T) / (r * T);
}

// Raw completion along one axis in the frame v = s c + u: the degree < NL
// part of each high-order Lagrange basis polynomial written in the particle
// velocity v, evaluated at the low-order velocities.  The basis in c has the
// monomial coefficients Vi (the inverse Vandermonde matrix of the high-order
// nodes); ((v - u)/s)^k = s^-k sum_p C(k, p) v^p (-u)^(k-p) re-expands it in v.
template <int NL, int NH>
__device__ __forceinline__ void frame_completion(const Tab *tab, double s, double u, double (*K)[NL]) {
  const LatTab &Lq = tab->lat[0];
  double C[NH][NH], mu[NH];
#pragma unroll
  for (int k = 0; k < NH; ++k)
#pragma unroll
    for (int p = 0; p < NH; ++p) C[k][p] = (p == 0 || p == k) ? 1.0 : (p > k ? 0.0 : C[k - 1][p - 1] + C[k - 1][p]);
  mu[0] = 1.0;
#pragma unroll
  for (int k = 1; k < NH; ++k) mu[k] = mu[k - 1] * (-u);
  const double is = 1.0 / s;
#pragma unroll
  for (int A = 0; A < NH; ++A) {
    double beta[NL];
#pragma unroll
    for (int p = 0; p < NL; ++p) beta[p] = 0.0;
    double isk = 1.0;
#pragma unroll
    for (int k = 0; k < NH; ++k) {
      const double ck = tab->Vi[A][k] * isk;
#pragma unroll
      for (int p = 0; p < NL; ++p)
        if (p <= k) beta[p] += ck * C[k][p] * mu[k - p];
      isk *= is;
    }
#pragma unroll
    for (int a = 0; a < NL; ++a) {
      const double v = s * Lq.cr[a] + u;
      double acc = 0.0, vp = 1.0;
#pragma unroll
      for (int p = 0; p < NL; ++p) {
        acc += beta[p] * vp;
        vp *= v;
      }
      K[A][a] = acc;
    }
  }
}

// One cell's state of one set, given in its own frame {ufx, ufy, Tf}, in the
// other set in the same frame (Sec. III.B-C, App. C).  Lifting keeps the
// moments of the low-order set taken at the frame's particle velocities and
// completes the others from the high-order equilibrium: the low-order
// non-equilibrium part through the frame's completion matrices on top of the
// high-order equilibrium, both equilibria at the cell's rho, u, T taken in the
// frame (equilibrium factors at the reduced velocity (u - u_f)/sqrt(T_f) and
// temperature T/T_f); the Hermite variant keeps Hermite coefficients in the
// reduced velocities, whose matrix serves every frame.  Projection applies
// the low-order Lagrange basis at the high-order nodes (the moments it keeps
// span the same polynomials in every frame).
template <int NL, int NH, bool TH>
__device__ void pond_lift(const Tab *tab, const double *f, const double *g, double ufx, double ufy, double Tf,
                          double *fo, double *go) {
  constexpr int q = NL * NL;
  const LatTab &Lq = tab->lat[0], &LQ = tab->lat[1];
  const double sT = sqrt(Tf);
  double r = 0, jx = 0, jy = 0, e = 0;
#pragma unroll
  for (int i = 0; i < q; ++i) {
    const double vx = sT * Lq.cr[i % NL] + ufx, vy = sT * Lq.cr[i / NL] + ufy;
    r += f[i];
    jx += vx * f[i];
    jy += vy * f[i];
    e += 0.5 * (vx * vx + vy * vy) * f[i];
    if (TH) e += g[i];
  }
  const double ux = jx / r, uy = jy / r;
  const double T = TH ? (e / r - 0.5 * (ux * ux + uy * uy)) / tab->cv : 1.0;
  const double uxr = (ux - ufx) / sT, uyr = (uy - ufy) / sT, th = T / Tf;
  double pxl[NL], pyl[NL], pxh[NH], pyh[NH];
  eq_axis<double, NL>(Lq, uxr, th, pxl);
  eq_axis<double, NL>(Lq, uyr, th, pyl);
  eq_axis<double, NH>(LQ, uxr, th, pxh);
  eq_axis<double, NH>(LQ, uyr, th, pyh);
  double Kx[NH][NL], Ky[NH][NL];
  if (tab->lift_mode == MSL_LIFT_GRAD_HERMITE) {
#pragma unroll
    for (int A = 0; A < NH; ++A)
#pragma unroll
      for (int a = 0; a < NL; ++a) Kx[A][a] = Ky[A][a] = tab->KH[A][a];
  } else {
    frame_completion<NL, NH>(tab, sT, ufx, Kx);
    frame_completion<NL, NH>(tab, sT, ufy, Ky);
  }
#pragma unroll
  for (int h = 0; h < (TH ? 2 : 1); ++h) {
    const double s = h ? tab->gfac * T : 1.0;
    const double *in = h ? g : f;
    double *out = h ? go : fo;
    double neq[q];
#pragma unroll
    for (int i = 0; i < q; ++i) neq[i] = in[i] - s * r * pxl[i % NL] * pyl[i / NL];
#pragma unroll
    for (int A = 0; A < NH; ++A) {
      double t[NL];
#pragma unroll
      for (int b = 0; b < NL; ++b) {
        double sum = 0.0;
#pragma unroll
        for (int a = 0; a < NL; ++a) sum += Kx[A][a] * neq[a + NL * b];
        t[b] = sum;
      }
#pragma unroll
      for (int B = 0; B < NH; ++B) {
        double cr = 0.0;
#pragma unroll
        for (int b = 0; b < NL; ++b) cr += Ky[B][b] * t[b];
        out[A + NH * B] = s * r * pxh[A] * pyh[B] + cr;
      }
    }
  }
}

template <int NL, int NH, bool TH>
__device__ void pond_project(const Tab *tab, const double *f, const double *g, double *fo, double *go) {
#pragma unroll
  for (int h = 0; h < (TH ? 2 : 1); ++h) {
    const double *in = h ? g : f;
    double *out = h ? go : fo;
#pragma unroll
    for (int bp = 0; bp < NL; ++bp) {
      double t[NH];   // along y first: t[A] = sum_B P[bp][B] f[A + NH B]
#pragma unroll
      for (int A = 0; A < NH; ++A) {
        double sum = 0.0;
#pragma unroll
        for (int B = 0; B < NH; ++B) sum += tab->P[bp][B] * in[A + NH * B];
        t[A] = sum;
      }
#pragma unroll
      for (int ap = 0; ap < NL; ++ap) {
        double sum = 0.0;
#pragma unroll
        for (int A = 0; A < NH; ++A) sum += tab->P[ap][A] * t[A];
        out[ap + NL * bp] = sum;
      }
    }
  }
}

// mode 0: every band cell of buffer (f0, f1, fr) converts its own set's state
// into the other set; mode 1: every cell whose set differs from mask[] converts
// its state into the new set (conv = 0: only its set changes) and takes it
template <int NL, int NH, bool TH>
__global__ void __launch_bounds__(256)
k_pond_convert(const Tab *__restrict__ tab, long long ncell, int mode, int conv, double *f0, double *f1,
               const double *__restrict__ fr, uint8_t *__restrict__ cls, const uint8_t *__restrict__ mask) {
  constexpr int q = NL * NL, Q = NH * NH;
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= ncell) return;
  const uint8_t cb = cls[k];
  const int o = cb & 1;
  int to;
  if (mode == 0) {
    if (!(cb & 2)) return;
    to = o ^ 1;
  } else {
    to = mask[k] & 1;
    if (to == o) return;
    cls[k] = (uint8_t)to;
    if (!conv) return;
  }
  const double ufx = fr[k], ufy = fr[ncell + k], Tf = fr[3 * ncell + k];
  if (o == 0) {
    double f[q], g[TH ? q : 1], fo[Q], go[TH ? Q : 1];
#pragma unroll
    for (int i = 0; i < q; ++i) {
      f[i] = f0[(long long)i * ncell + k];
      if (TH) g[i] = f0[(long long)(q + i) * ncell + k];
    }
    pond_lift<NL, NH, TH>(tab, f, g, ufx, ufy, Tf, fo, go);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      f1[(long long)i * ncell + k] = fo[i];
      if (TH) f1[(long long)(Q + i) * ncell + k] = go[i];
    }
  } else {
    double f[Q], g[TH ? Q : 1], fo[q], go[TH ? q : 1];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      f[i] = f1[(long long)i * ncell + k];
      if (TH) g[i] = f1[(long long)(Q + i) * ncell + k];
    }
    pond_project<NL, NH, TH>(tab, f, g, fo, go);
#pragma unroll
    for (int i = 0; i < q; ++i) {
      f0[(long long)i * ncell + k] = fo[i];
      if (TH) f0[(long long)(q + i) * ncell + k] = go[i];
    }
  }
}

// Diffuse y walls: per column, the density rho_w of the wall state's co-moving
// equilibrium {u_w, T_w} that balances the wall-normal particle flux of the
// adjacent fluid cell, both fluxes counted in the wall's frame: the cell's
// populations (its own set, its own frame) are transferred to the wall's frame
// with the per-axis Lagrange rows of the step kernel.
template <int N>
__device__ double pond_wall_density(const Tab *tab, int l, const double *f, long long ncell, long long k,
                                    const double *fr, const double *ws, int side, int thermal) {
  constexpr int Q = N * N;
  const LatTab &L = tab->lat[l];
  double xn[N], den[N];
#pragma unroll
  for (int m = 0; m < N; ++m) xn[m] = L.cr[m];
#pragma unroll
  for (int m = 0; m < N; ++m) {
    double p = 1.0;
#pragma unroll
    for (int cc = 0; cc < N; ++cc)
      if (cc != m) p *= xn[m] - xn[cc];
    den[m] = 1.0 / p;
  }
  const double Tw = thermal ? ws[4] : 1.0, sTw = sqrt(Tw), isTw = 1.0 / sTw;
  const double sTk = sqrt(fr[3 * ncell + k]), ukx = fr[k], uky = fr[ncell + k];
  // G[a][a'] = l_a((sqrt(T_k) c_a' + u_k - u_w) / sqrt(T_w)) along x and y
  double Gx[N][N], Gy[N][N];
#pragma unroll
  for (int m = 0; m < N; ++m) {
    const double zx = (sTk * xn[m] + ukx - ws[1]) * isTw, zy = (sTk * xn[m] + uky - ws[2]) * isTw;
#pragma unroll
    for (int a = 0; a < N; ++a) {
      double px = den[a], py = den[a];
#pragma unroll
      for (int cc = 0; cc < N; ++cc)
        if (cc != a) {
          px *= zx - xn[cc];
          py *= zy - xn[cc];
        }
      Gx[a][m] = px;
      Gy[a][m] = py;
    }
  }
  double in = 0.0, out = 0.0;
#pragma unroll
  for (int b = 0; b < N; ++b) {
    // the wall-normal (y) velocity of the wall frame's node b
    const double vw = sTw * xn[b] + ws[2];
    const bool towall = side ? vw > 0.0 : vw < 0.0, fromwall = side ? vw < 0.0 : vw > 0.0;
    if (!towall && !fromwall) continue;
#pragma unroll
    for (int a = 0; a < N; ++a) {
      if (towall) {
        double s = 0.0;
#pragma unroll
        for (int bp = 0; bp < N; ++bp) {
          double t = 0.0;
#pragma unroll
          for (int ap = 0; ap < N; ++ap) t += Gx[a][ap] * f[(long long)(ap + N * bp) * ncell + k];
          s += Gy[b][bp] * t;
        }
        in += fabs(vw) * s;
      } else {
        out += fabs(vw) * L.w[a] * L.w[b];
      }
    }
  }
  (void)Q;
  return in / out;
}

__global__ void k_pond_wall(const Tab *__restrict__ tab, PondArgs pa, int thermal, int faces, const double *f0,
                            const double *f1, const uint8_t *__restrict__ cls, const double *__restrict__ fr,
                            double *__restrict__ wrho) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int nx = pa.nx, ny = pa.ny;
  const long long ncell = pa.ncell;
  if (t >= 2 * nx) return;
  const int side = t / nx, x = t % nx;
  if (!(faces & (1 << side))) return;
  const long long k = (long long)(side ? ny - 1 : 0) * nx + x;
  const int l = cls[k] & 1;
  const double *f = l ? f1 : f0;
  const double *ws = pa.st[2 + side];
  double r = 0.0;
  switch (tab->lat[l].n) {
    case 3: r = pond_wall_density<3>(tab, l, f, ncell, k, fr, ws, side, thermal); break;
    case 4: r = pond_wall_density<4>(tab, l, f, ncell, k, fr, ws, side, thermal); break;
    case 5: r = pond_wall_density<5>(tab, l, f, ncell, k, fr, ws, side, thermal); break;
    case 6: r = pond_wall_density<6>(tab, l, f, ncell, k, fr, ws, side, thermal); break;
  }
  wrho[t] = r;
}

// Lagrange denominators of a set's nodes, from the products as the step kernel
// forms them at the nodes themselves, with which they round to 1: the rows of
// the transfer between equal frames are then unit rows.  (Denominators rounded
// from the exact products leave an error of every node's row that is the same in
// each step: the error of rho after 4 steps 2.6e-15 with them, 1.8e-15 now, in
// D2Q9, and 2.0e-15, 9.8e-16 in D2Q36.)
static double unit_denominator(double p) {
  const double r = 1.0 / p, near[3] = {r, nextafter(r, INFINITY), nextafter(r, -INFINITY)};
  for (int k = 0; k < 3; ++k)
    if (p * near[k] == 1.0) return near[k];
  return r;
}

template <int N>
static void pond_denominators(LatTab &L) {
  for (int a = 0; a < N; ++a) {
    double p = 1.0, l[N];
    for (int c = 0; c < N; ++c)
      if (c != a) p *= L.cr[a] - L.cr[c];
    lagrange_products<N>(L.cr[a], L.cr, l);
    L.den[a] = unit_denominator(p);
    L.deny[a] = unit_denominator(l[a]);
  }
}

void msl_pond_tables(LatTab &L) {
  switch (L.n) {
    case 3: pond_denominators<3>(L); break;
    case 4: pond_denominators<4>(L); break;
    case 5: pond_denominators<5>(L); break;
    case 6: pond_denominators<6>(L); break;
  }
}

static PondArgs pond_args(const msl_ctx *c) {
  PondArgs pa;
  pa.nx = c->geo.nx;
  pa.ny = c->geo.ny;
  pa.ncell = c->ncell;
  for (int f = 0; f < 4; ++f) {
    pa.bc[f] = c->cfg.bc[f];
    for (int m = 0; m < 5; ++m) pa.st[f][m] = c->cfg.bc_state[f][m];
  }
  return pa;
}

static unsigned pond_blocks(const msl_ctx *c) { return (unsigned)((c->ncell + 255) / 256); }

int msl_pond_launch_init(msl_ctx *c, const double *rho, const double *u, const double *T) {
  hipLaunchKernelGGL(k_pond_init, dim3(pond_blocks(c)), dim3(256), 0, c->stream, c->dtab, c->ncell,
                     c->cfg.thermal, c->nlat, rho, u, T, c->pond_f[0][c->cur],
                     c->nlat > 1 ? c->pond_f[1][c->cur] : nullptr, c->pond_fr[c->cur]);
  return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
}

int msl_pond_launch_macros(msl_ctx *c, double *rho, double *u, double *T) {
  hipLaunchKernelGGL(k_pond_macros, dim3(pond_blocks(c)), dim3(256), 0, c->stream, c->dtab, c->ncell,
                     c->cfg.thermal, c->pond_f[0][c->cur], c->nlat > 1 ? c->pond_f[1][c->cur] : nullptr,
                     c->cls, c->pond_fr[c->cur], rho, u, T);
  return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
}

// conversion launch over buffer `buf` (mode and mask as in k_pond_convert)
static int pond_convert(msl_ctx *c, int buf, int mode, int conv, const uint8_t *mask) {
  return msl_pair_dispatch(2, c->htab.lat[0].n, c->htab.lat[1].n, [&]<int D, int NL, int NH>() {
    if (c->cfg.thermal)
      hipLaunchKernelGGL((k_pond_convert<NL, NH, true>), dim3(pond_blocks(c)), dim3(256), 0, c->stream, c->dtab,
                         c->ncell, mode, conv, c->pond_f[0][buf], c->pond_f[1][buf], c->pond_fr[buf], c->cls, mask);
    else
      hipLaunchKernelGGL((k_pond_convert<NL, NH, false>), dim3(pond_blocks(c)), dim3(256), 0, c->stream, c->dtab,
                         c->ncell, mode, conv, c->pond_f[0][buf], c->pond_f[1][buf], c->pond_fr[buf], c->cls, mask);
    return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
  });
}

// new sets from `mask` (converting the cells that change when conv), then the
// band of the current buffer
int msl_pond_launch_set_mask(msl_ctx *c, const uint8_t *mask, int conv) {
  if (c->nlat < 2) return MSL_OK;   // the mask check admits only zeros
  int rc = pond_convert(c, c->cur, 1, conv, mask);
  if (!rc) rc = msl_launch_classify(c);
  if (!rc && conv) rc = pond_convert(c, c->cur, 0, 1, nullptr);
  return rc;
}

template <int N, bool TH, bool QE, bool SPX>
static int pond_step_n(msl_ctx *c, int lat) {
  using Tr = PondTraits<N, TH, SPX>;
  const PondArgs pa = pond_args(c);
  const dim3 grid((unsigned)((pa.nx + Tr::CW - 1) / Tr::CW), (unsigned)((pa.ny + Tr::TY - 1) / Tr::TY));
  hipLaunchKernelGGL((k_pond_step<N, TH, QE, SPX>), grid, dim3(256), 0, c->stream, c->dtab, lat, c->cls, pa,
                     c->pond_f[lat][c->cur], c->pond_fr[c->cur], c->pond_f[lat][c->cur ^ 1],
                     c->pond_fr[c->cur ^ 1], c->flag, c->pond_slots, c->pond_wall);
  return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
}

template <bool TH, bool QE>
static int pond_step_th(msl_ctx *c, int lat) {
  // Point columns on lanes of their own: N = 5 always (the two-set shock's
  // D2Q25 launch 94 us without, 45 us with); N = 3, 4 while the plain layout's
  // 64-cell workgroups leave three CUs in four idle (12 or 9 of 16 lanes work).
  // us a step, with against without: thermal D2Q16 15.3, 21.5 at 4 workgroups
  // (16 x 16), 16.8, 24.4 at 64 (64 x 64), 36.6, 35.1 at 144, 89, 61 at 650;
  // athermal D2Q9 10.9, 12.0 and 11.3, 12.4 at 4 and 64.  N = 6 has no room for
  // them in 16 lanes.
  const long long wgs = (long long)((c->geo.nx + 15) / 16) * ((c->geo.ny + 3) / 4);
  const bool spx = wgs <= 64;
  switch (c->htab.lat[lat].n) {
    case 3: return spx ? pond_step_n<3, TH, QE, true>(c, lat) : pond_step_n<3, TH, QE, false>(c, lat);
    case 4: return spx ? pond_step_n<4, TH, QE, true>(c, lat) : pond_step_n<4, TH, QE, false>(c, lat);
    case 5: return pond_step_n<5, TH, QE, true>(c, lat);
    case 6: return pond_step_n<6, TH, QE, false>(c, lat);
  }
  return MSL_EINVAL;
}

// the pass counts since the slots were cleared into pond_stats
int msl_pond_launch_stats(msl_ctx *c) {
  hipLaunchKernelGGL(k_pond_stats, dim3(1), dim3(256), 0, c->stream, c->pond_slots, c->pond_nslot, c->pond_stats);
  return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
}

// one step: [the Knudsen-number criterion pass], one launch per set, the band
// of the new buffer; the new buffers become current
int msl_pond_launch_step(msl_ctx *c) {
  int rc;
  if (c->nlat > 1 && c->cfg.crit_kind == MSL_CRIT_KN && c->cfg.crit_every > 0 &&
      c->step % c->cfg.crit_every == 0) {
    hipLaunchKernelGGL(k_pond_kn_fields, dim3(pond_blocks(c)), dim3(256), 0, c->stream, c->dtab, c->ncell,
                       c->cfg.thermal, c->pond_f[0][c->cur], c->pond_f[1][c->cur], c->cls, c->pond_fr[c->cur],
                       c->kn_rho, c->kn_lam);
    if (hipGetLastError() != hipSuccess) return MSL_EHIP;
    if ((rc = msl_launch_kn_mask(c))) return rc;
    if ((rc = msl_launch_dilate(c))) return rc;
    if ((rc = msl_pond_launch_set_mask(c, c->newmask, 1))) return rc;
  }
  const int faces = (c->cfg.bc[2] == MSL_BC_DIFFUSE_WALL ? 1 : 0) | (c->cfg.bc[3] == MSL_BC_DIFFUSE_WALL ? 2 : 0);
  if (faces) {
    // the wall densities from the current state (the wall states travel in
    // the kernel arguments)
    const PondArgs pa = pond_args(c);
    hipLaunchKernelGGL(k_pond_wall, dim3((unsigned)((2 * pa.nx + 255) / 256)), dim3(256), 0, c->stream, c->dtab,
                       pa, c->cfg.thermal, faces, c->pond_f[0][c->cur],
                       c->nlat > 1 ? c->pond_f[1][c->cur] : nullptr, c->cls, c->pond_fr[c->cur], c->pond_wall);
    if (hipGetLastError() != hipSuccess) return MSL_EHIP;
  }
  for (int l = 0; l < c->nlat; ++l) {
    if (c->cfg.thermal) rc = c->htab.qe ? pond_step_th<true, true>(c, l) : pond_step_th<true, false>(c, l);
    else rc = c->htab.qe ? pond_step_th<false, true>(c, l) : pond_step_th<false, false>(c, l);
    if (rc) return rc;
  }
  if (c->nlat > 1 && (rc = pond_convert(c, c->cur ^ 1, 0, 1, nullptr))) return rc;
  c->cur ^= 1;
  return MSL_OK;
}
