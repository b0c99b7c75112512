// msl_stream3z.hpp -- the 3D stream-and-collide kernels that march along z, for
// athermal sets: D3Q27 in FP32 storage (first), D3Q27 and D3Q64 in 16-bit
// storage (below).  FP64, thermal and FP32 D3Q64 runs use the chunked kernel of
// msl_stream3.hpp.
//
// A workgroup owns a column of 64 x 4 x zc cells and walks it from its lowest
// z cell upwards.  Its nine waves share out the populations: a wave holds the
// three planes of one z and one y node for all four rows of the column, one x
// cell per lane.  At each step of the walk a wave brings one z
// slab of each of its planes' departure windows into LDS (direct-to-LDS
// buffer loads of 6 rows x 66 cells: the departure offset x - v_i dt is the
// same for every cell of a plane, so the slab is the column's cross-section
// shifted by the plane's base offset), interpolates the slab along x (six
// rows) and y (four cells; eq. reconstructionPond, 3-point Lagrange weights),
// and combines it with the two slabs before it, which each lane keeps in
// registers, into the populations streamed to its cells (the z interpolation).
// Every slab of a column's window is read once per column.  No wave reads
// another's slabs, so the loads need no barrier, only the wave's own wait;
// the loads of the next slab are in flight while the cells collide.
//
// The cells collide in registers: the waves exchange their partial moments
// through LDS; one wave per row adds them in wave order and evaluates the
// FP64 equilibrium factors in the run's frame; every wave relaxes its own
// populations (BGK, eqs. Pond_f/g, feqL, geqL) and stores them with buffer
// stores whose out-of-range offset drops the writes of foreign or outside
// cells.  Two barriers per step.
//
// What bounds it: on large grids the stores (a step's burst of R PW stores per
// wave is issued at 16 to 30 cycles each), VALU issue at about a third; on small
// grids the chain of a step's phases.  The form before (one wave per row with
// every plane of its cells, columns of 32) interpolated each row three times
// and read nine LDS values per population and cell; six rows shared by four
// cells take 4.5 reads, and the factors are formed once per cell.
// 150 x 130 x 141: 367 us before, 267 us now; 64^3: 240 us before, 24 us now.
#pragma once
#include <utility>

#include "msl_stream3.hpp"

// s_waitcnt for the vector memory counter only (gfx9 encoding: vmcnt in bits
// 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at their maxima): wait until
// at most NV vector memory operations of this wave are outstanding
template <int NV>
__device__ __forceinline__ void msl_wait_vm() {
  static_assert(NV >= 0 && NV <= 63, "vmcnt is a 6-bit field");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((NV & 15) | (7 << 4) | (15 << 8) | ((NV >> 4) << 14));
  asm volatile("" ::: "memory");
}

// this wave's LDS operations have completed (lgkmcnt 0), and no memory
// operation moves across
__device__ __forceinline__ void msl_wait_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
  asm volatile("" ::: "memory");
}

// workgroup barrier for LDS traffic only; unlike __syncthreads() it does not
// wait for outstanding global stores
__device__ __forceinline__ void msl_lds_barrier() {
  msl_wait_lds();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// a 16-bit stored element (the low 16 bits of u) as float
template <typename S>
__device__ __forceinline__ float half_elem(uint32_t u);
template <>
__device__ __forceinline__ float half_elem<_Float16>(uint32_t u) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)u);
}
template <>
__device__ __forceinline__ float half_elem<bf16_t>(uint32_t u) { return __uint_as_float(u << 16); }
template <typename S>
__device__ __forceinline__ float half_elem(uint32_t) { return 0.0f; }

// columns of the high-order set beyond which its launch runs over the list of
// live columns: 32 per CU, of which a criterion's set fills a part
#define MSL_WALK_LIST_MIN 8192
#define MSL_WALK_ZC 8   // most cells of a column along z

struct SC3ZTraits {
  static constexpr int N = 3, Q = N * N * N;
  // one z and one y node per wave (all three y nodes, in three waves of 178
  // registers, measured 82 against 54 us on 64^3 and 644 against 598 us on 200^3)
  static constexpr int NWV = N * N;            // waves per workgroup
  static constexpr int NT = 64 * NWV;
  static constexpr int PW = N;                 // planes of a wave
  static constexpr int R = MSL_MTY;            // rows
  // a window row is loaded in 16-byte chunks
  static constexpr int CPR = (66 * 4 + 15) / 16;
  static constexpr int ROWB = 16 * CPR;
  static constexpr int CPP = (R + 2) * CPR;    // chunks of a plane's slab
  static constexpr int M = (CPP + 63) / 64;    // DMA instructions per plane
  static constexpr int SLAB = 16 * CPP;
  static constexpr int NPS = 2;                // partial sums of a wave: rho, j_x
  static constexpr int NFAC = 3 * N + 1;       // equilibrium factors, omega
  static constexpr int LDS_BYTES = Q * SLAB + ((NWV - 1) * NPS + NFAC) * 256 * 4;
  // waves per SIMD that the registers have to allow (two workgroups of nine
  // waves take five on some SIMD)
  static constexpr int WAVES = 5;
};

// OWN: stored ghost slabs keep their own ghost rows (a slot on a z face: its
// profile goes on beyond the y edges, as the highest axis out of range decides);
// otherwise a stored slab is uniform or follows the y faces' rules, and its rows
// are mapped like every other slab's.  A variant of its own: the choice inside
// the walk cost 1 to 4 % of every run (16-bit D3Q27 64^3 30.1 us a step, 31.1).
template <bool OWN>
__global__ void __launch_bounds__(SC3ZTraits::NT) __attribute__((amdgpu_waves_per_eu(SC3ZTraits::WAVES)))
k_sc3d_zm(const Tab *__restrict__ tab, int lat, Geo g, const float *__restrict__ in,
          float *__restrict__ out, const uint8_t *__restrict__ cls,
          const uint8_t *__restrict__ tflag, int remap, int xmir, int faces, int zc) {
  using Tr = SC3ZTraits;
  typedef float C;
  constexpr int N = Tr::N, Q = Tr::Q, NWV = Tr::NWV, PW = Tr::PW, R = Tr::R, M = Tr::M;
  constexpr int SZ = 4, ROWB = Tr::ROWB, CPR = Tr::CPR, CPP = Tr::CPP, SLAB = Tr::SLAB, NPS = Tr::NPS;
  __shared__ __align__(16) char sm[Q * SLAB];
  __shared__ float s_part[(NWV - 1) * NPS][256];   // partial moments of the waves that do not own the row
  __shared__ float s_fac[Tr::NFAC][256];           // equilibrium factors per axis (x with rho), omega
  const LatTab &L = tab->lat[lat];
  // the column (XCD-aware order; the low-order set's launches are dense)
  const int lin = (int)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
  const int tile = remap ? msl_xcd_tile(lin, (int)(gridDim.x * gridDim.y * gridDim.z)) : lin;
  const int bx = tile % g.ntx, by = (tile / g.ntx) % g.nty;
  const int z0 = tile / (g.ntx * g.nty) * zc;
  const int x0 = bx * MSL_TX, y0 = by * MSL_MTY;
  const int zn = g.nz - z0 < zc ? g.nz - z0 : zc;   // cells of the column (>= 1)
  {
    uint8_t any = 0;
    for (int k = 0; k < zn; ++k) any |= tflag[((long long)(z0 + k) * g.nty + by) * g.ntx + bx];
    if (!(any & (1 << lat))) return;
  }
  // the wave's z node cc, y node b0 and first plane kb, as scalars
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cc = wv / N, b0 = wv % N, kb = wv * N;
  const unsigned pitch_b = (unsigned)g.pitch * SZ;
  const unsigned plane_b = (unsigned)g.plane * SZ;
  const unsigned slab_b = (unsigned)g.rows * pitch_b;
  // the cells of this velocity set along the column, as bits per cell (bit k:
  // z0 + k), through LDS
  uint32_t mine[R];
  {
    static_assert(MSL_WALK_ZC <= 8, "a byte per cell of the cross-section");
    uint8_t *bits = (uint8_t *)s_fac;
    if (threadIdx.x < 256) {
      const int x = x0 + (threadIdx.x & 63), y = y0 + (threadIdx.x >> 6);
      unsigned m = 0;
      if (x < g.nx && y < g.ny)
#pragma unroll
        for (int j = 0; j < MSL_WALK_ZC; ++j)
          if (j < zn) m |= (unsigned)((cls[((long long)(z0 + j) * g.ny + y) * g.nx + x] & 1) == lat) << j;
      bits[threadIdx.x] = (uint8_t)m;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) mine[r] = bits[64 * r + lane];
  }
  // interpolation weights and window offsets of the departure stencil
  C wx[3][N], wy[3], wz[3];
  int offx[N];
#pragma unroll
  for (int s = 0; s < 3; ++s) {
#pragma unroll
    for (int a = 0; a < N; ++a) wx[s][a] = L.af[0][a][s];
    wy[s] = L.af[1][b0][s];
    wz[s] = L.af[2][cc][s];
  }
#pragma unroll
  for (int a = 0; a < N; ++a) offx[a] = L.n0[0][a] - 1;
  // Ghost rows and slabs.  A y or z coordinate of the window outside the domain
  // is mapped by its face's rule (two bits of `faces` per face: 1 periodic,
  // wrapped; 2 zero-gradient, clamped; 0 fixed or diffuse, the stored ghost
  // layer) when the slab is loaded, rows by the lanes' addresses and slabs by
  // the scalar offset, so no pass copies those ghost layers (41 to 46 us a step
  // at 150 x 130 x 141 FP32 and 256^3 FP16).  Ghost columns are stored: written as
  // images below, or by the ghost fill.  (Loading them per plane into the
  // staged rows, 24 lanes a plane, cost more than the images: the D3Q64 launch
  // of the 256^3 run 505 against 475 us.)
  auto mapped = [&](int ax, int p, int n) {
    if (p >= 0 && p < n) return p;
    const int rule = (faces >> (4 * ax + (p < 0 ? 0 : 2))) & 3;
    return rule == 1 ? (p < 0 ? p + n : p - n) : (rule == 2 ? (p < 0 ? 0 : n - 1) : p);
  };
  // byte offsets inside a slab of this lane's chunks; lanes past the slab's CPP
  // chunks issue no load
  unsigned voff[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int d = lane + 64 * m, row = d / CPR;
    voff[m] = (unsigned)(mapped(1, y0 + L.n0[1][b0] - 1 + row, g.ny) + MSL_G) * pitch_b +
              (unsigned)(d - row * CPR) * 16u;
  }
  const unsigned row0b = (unsigned)(g.xo + x0) * SZ;   // byte of x0 in a row
  const int zw = z0 + L.n0[2][cc] - 1;                 // z of step 0's slab
  // DMA of step t's slab of the wave's planes into LDS: slab z0 + n0_z - 1 + t.
  // Each plane has its own buffer descriptor (the range of one plane); the
  // base offsets pass through an empty asm at every call, so the per-plane
  // descriptors and offsets are formed here rather than hoisted out of the
  // walk (4 + 1 scalar registers per plane)
  const long long plane_b64 = g.plane * SZ;
  auto issue = [&](const int t) {
    const int zm = mapped(2, zw + t, g.nz);
    unsigned ob = (unsigned)(zm + MSL_G) * slab_b;
    const char *pp = (const char *)in + kb * plane_b64;
    asm volatile("" : "+s"(ob), "+s"(pp));
    const bool own = OWN && (zm < 0 || zm >= g.nz);
    msl_for_planes<PW>([&]<int K>() {
      const unsigned so = ob + row0b + (unsigned)(offx[K] * SZ);
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc((void *)pp, (short)0, (int)plane_b, MSL_RSRC_WORD3);
#pragma unroll
      for (int m = 0; m < M; ++m)
        if ((m + 1) * 64 <= CPP || lane + 64 * m < CPP) {
          const int d = lane + 64 * m, row = d / CPR;
          const unsigned vo = own ? (unsigned)(y0 + L.n0[1][b0] - 1 + row + MSL_G) * pitch_b + (unsigned)(d - row * CPR) * 16u
                                  : voff[m];
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (msl_lds_t *)(sm + (kb + K) * SLAB + 1024 * m), 16, (int)vo,
                                                   (int)so, 0, 0);
        }
      pp += plane_b64;
    });
  };
  // LDS byte offset of the lane's first element in the first window row of the
  // wave's first plane
  unsigned rb = (unsigned)(kb * SLAB + lane * SZ);
  // per plane and row: the x, y interpolated values of the two slabs before the
  // new one (ha: slab t - 2, hb: slab t - 1) and the streamed value
  C ha[PW][R], hb[PW][R], ftk[PW][R];
#pragma unroll
  for (int k = 0; k < PW; ++k)
#pragma unroll
    for (int r = 0; r < R; ++r) ha[k][r] = hb[k][r] = C(0);
  // the lane's window values of three rows of plane K (H: the lower or upper
  // three): three of each row
  static_assert(R == 4, "a slab's six rows are read three at a time");
  auto fetch = [&]<int K, int H>(C (&v)[3][3]) {
    typedef volatile const __attribute__((address_space(3))) float lds_f32;
    const char *base = (const char *)sm + rb + K * SLAB + 3 * H * ROWB;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int e = 0; e < 3; ++e) v[dy][e] = *(lds_f32 *)(base + dy * ROWB + SZ * e);
  };
  // x interpolation of three rows
  // (differenced form, centre weight 1 - w0 - w2 exactly)
  auto xrows = [&]<int K>(const C (&v)[3][3], C *hx) {
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
      hx[dy] = v[dy][1] + wx[0][K] * (v[dy][0] - v[dy][1]) + wx[2][K] * (v[dy][2] - v[dy][1]);
  };
  // the new slab of plane K: y interpolation, then the z interpolation of the
  // three slabs into the streamed values of cells z0 + t - 2
  auto yz = [&]<int K>(const C (&hx)[R + 2]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const C hn = hx[r + 1] + wy[0] * (hx[r] - hx[r + 1]) + wy[2] * (hx[r + 2] - hx[r + 1]);
      ftk[K][r] = hb[K][r] + wz[0] * (ha[K][r] - hb[K][r]) + wz[2] * (hn - hb[K][r]);
      ha[K][r] = hb[K][r];
      hb[K][r] = hn;
      asm("" : "+v"(ftk[K][r]), "+v"(hb[K][r]));
    }
    // (the empty asm statements fix the final values: without them the
    // interpolation would be sunk into the collision, keeping the LDS values
    // of every plane alive until then)
  };
  // every plane of the wave, the LDS reads of three rows issued before the
  // arithmetic of the three rows before them (the scheduling barriers keep
  // them there: left to itself the compiler reads six values at a time and
  // waits for them)
  auto slab = [&]() {
    C lo[3][3], hi[3][3];
    fetch.template operator()<0, 0>(lo);
    msl_for_planes<PW>([&]<int K>() {
      C hx[R + 2];
      fetch.template operator()<K, 1>(hi);
      __builtin_amdgcn_sched_barrier(0);
      xrows.template operator()<K>(lo, hx);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (K + 1 < PW) fetch.template operator()<K + 1, 0>(lo);
      __builtin_amdgcn_sched_barrier(0);
      xrows.template operator()<K>(hi, hx + 3);
      yz.template operator()<K>(hx);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // periodic x (xmir, nx >= 4): the cells x < 2 and x >= nx - 2 are also
  // stored into the ghost columns of the other side, which the next step's
  // windows read; only the columns at the two x ends take the second store
  const int x = x0 + lane;
  const bool xedge = xmir && (x0 < MSL_G || x0 + MSL_TX > g.nx - MSL_G);
  // byte offset of the lane's cell in the first row at z0, and of its image
  const unsigned cell0 = (unsigned)g.idx(x < g.nx ? x : 0, y0, z0) * SZ;
  const unsigned img0 = x < MSL_G ? cell0 + (unsigned)g.nx * SZ : cell0 - (unsigned)g.nx * SZ;
  const uint32_t imask = x < MSL_G || x >= g.nx - MSL_G ? ~0u : 0u;   // lanes with an image
  // moments, equilibrium, collision and stores of the lane's cells at z0 + k
  auto finish = [&]<bool XE>(const int k) {
    // the per-plane scales and velocities are loaded here at every cell
    // (scalar loads) rather than hoisted out of the walk into scalar registers
    // (through the constant address space: the table is read-only for the
    // kernel's lifetime, which the empty asm would otherwise hide, turning
    // the scalar loads into vector loads)
    typedef const __attribute__((address_space(4))) LatTab cLatTab;
    typedef const __attribute__((address_space(4))) Tab cTab;
    cLatTab *Lp = (cLatTab *)&L;
    cTab *tp = (cTab *)tab;
    // plane K's base, advanced plane by plane (from the wave's first plane)
    const char *op = (const char *)out + (long long)kb * plane_b64;
    asm volatile("" : "+s"(Lp), "+s"(tp), "+s"(op));
    auto &L = *Lp;
    // partial moments of the wave's planes
    C rp[R], xp[R];
#pragma unroll
    for (int r = 0; r < R; ++r) rp[r] = xp[r] = C(0);
    msl_for_planes<PW>([&]<int K>() {
      const C cx = L.vf[0][K];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        rp[r] += ftk[K][r];
        xp[r] = __builtin_fmaf(cx, ftk[K][r], xp[r]);
      }
    });
    // row r belongs to wave r (mod the number of waves): the others hand it
    // their partial sums
#pragma unroll
    for (int r = 0; r < R; ++r) {
      constexpr auto owner = [](int row) { return row % NWV; };
      if (wv != owner(r)) {
        const int slot = (wv < owner(r) ? wv : wv - 1) * NPS;
        s_part[slot][64 * r + lane] = rp[r];
        s_part[slot + 1][64 * r + lane] = xp[r];
      }
    }
    msl_lds_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int ow = r % NWV;
      if (wv == ow) {
        const int ci = 64 * r + lane;
        // (the owner's nodes are constants here)
        C rho = rp[r], jx = xp[r], jy = L.vf[1][ow % N] * rp[r], jz = L.vf[2][ow / N] * rp[r];
#pragma unroll
        for (int s = 0; s < NWV - 1; ++s) {
          const int w = s < ow ? s : s + 1;
          const C pr = s_part[s * NPS][ci];
          rho += pr;
          jx += s_part[s * NPS + 1][ci];
          jy += L.vf[1][w % N] * pr;
          jz += L.vf[2][w / N] * pr;
        }
        // equilibrium factors in FP64 (no rounding bias in the equilibrium's
        // mass and momentum), kept in the compute precision; athermal: T = 1
        const double rd = (double)rho, dx = (double)jx, dy = (double)jy, dz = (double)jz;
        const double ird = 1.0 / rd;
        C om = tp->omegaf;
        if (tp->tau_mode == 1) om = (C)(1.0 / (tp->mu_T1 / (rd * tp->dt) + 0.5));
        double p[N];
        eq_axis<double, N>(L, (dx * ird - L.ur[0]) * L.isq, L.iTr, p);
#pragma unroll
        for (int q = 0; q < N; ++q) s_fac[q][ci] = (float)(p[q] * rd);
        eq_axis<double, N>(L, (dy * ird - L.ur[1]) * L.isq, L.iTr, p);
#pragma unroll
        for (int q = 0; q < N; ++q) s_fac[N + q][ci] = (float)p[q];
        eq_axis<double, N>(L, (dz * ird - L.ur[2]) * L.isq, L.iTr, p);
#pragma unroll
        for (int q = 0; q < N; ++q) s_fac[2 * N + q][ci] = (float)p[q];
        s_fac[3 * N][ci] = om;
      }
    }
    msl_lds_barrier();
    C Px[R][N], Pyz[R], om[R];
    unsigned vo[R], vi[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int ci = 64 * r + lane;
#pragma unroll
      for (int a = 0; a < N; ++a) Px[r][a] = s_fac[a][ci];
      Pyz[r] = s_fac[N + b0][ci] * s_fac[2 * N + cc][ci];
      om[r] = s_fac[3 * N][ci];
      // (the row's offset goes into the scalar offset of the stores; cells that
      // are not this set's get an offset beyond the plane)
      vo[r] = (mine[r] >> k) & 1u ? cell0 : 0x80000000u;
      if constexpr (XE) vi[r] = ((mine[r] & imask) >> k) & 1u ? img0 : 0x80000000u;
    }
    const unsigned so = (unsigned)k * slab_b;
    msl_for_planes<PW>([&]<int K>() {
      const __amdgpu_buffer_rsrc_t rsout =
          __builtin_amdgcn_make_buffer_rsrc((void *)op, (short)0, (int)plane_b, MSL_RSRC_WORD3);
      op += plane_b64;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const C feq = Px[r][K] * Pyz[r], h = ftk[K][r];
        const C f = __builtin_fmaf(om[r], feq - h, h);
        const int sr = (int)(so + (unsigned)r * pitch_b);
        auto put = [&](unsigned o) {
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, f), rsout, (int)o, sr, 0);
        };
        put(vo[r]);
        if constexpr (XE) put(vi[r]);
      }
    });
  };

  // the walk: slabs t = 0 .. zn + 1; from t = 2 on, cells z0 + t - 2 are
  // complete.  The next slab is loaded while they collide: vector memory
  // operations complete in issue order, so waiting until no more than the
  // cells' stores are outstanding waits for exactly the slab (vmcnt holds at
  // most 63: with more stores per step the wait also takes the oldest of them)
  constexpr int VW1 = R * PW < 63 ? R * PW : 63, VW2 = 2 * R * PW < 63 ? 2 * R * PW : 63;
  issue(0);
  msl_wait_vm<0>();
  for (int t = 0; t < zn + 2; ++t) {
    // the LDS offset passes through an empty asm at every step, so that the
    // per-plane LDS addresses are formed in the walk, not hoisted out of it
    asm volatile("" : "+v"(rb));
    slab();
    msl_wait_lds();   // the slab's LDS values are read; the next load may overwrite them
    if (t + 1 < zn + 2) issue(t + 1);
    if (t >= 2) {
      if (xedge) {
        finish.template operator()<true>(t - 2);
        msl_wait_vm<VW2>();
      } else {
        finish.template operator()<false>(t - 2);
        msl_wait_vm<VW1>();
      }
    } else {
      msl_wait_vm<0>();
    }
  }
}

// ---------------------------------------------------------------------------
// The walk of 16-bit storage: one wave per row of cells with all planes of its
// cells (D3Q64: four waves, each with the 16 planes of one z node).  The
// deviations are rounded to 16 bits every step, so a different order of the
// FP32 sums over a cell's populations would change a few of those roundings,
// and with them, after some steps, all of them: this form keeps each sum in
// population order within a wave, which the split over y and z nodes above
// does not.  What it shares with that walk: ghost rows and slabs mapped when a
// slab is loaded, short columns, 16-byte DMA chunks (each wave loads its share
// of the planes: a quarter of the load instructions of 4-byte chunks by all
// waves), LDS reads one plane ahead of their use.
// One stream, D3Q27 / D3Q64: 256^3 705 / 645 us in the form before, 644 / 635 us
// now; 64^3 166 / 229 us before, 32 / 42 us now.  (The split form of D3Q64, with
// other sums, ran 256^3 in 396 us.)
// ---------------------------------------------------------------------------
template <typename S, int N>
struct SC3RTraits {
  using T = StoreTraits<S>;
  static constexpr int Q = N * N * N;
  static constexpr int NHW = N == 4 ? 4 : 1;   // waves per row of cells
  static constexpr int NWV = MSL_MTY * NHW;
  static constexpr int NT = 64 * NWV;
  static constexpr int NPW = Q / NHW;          // planes of a wave's cells
  static constexpr int NLD = (Q + NWV - 1) / NWV;   // planes that a wave loads
  static constexpr int CPR = (66 * 2 + 2 + 15) / 16;
  static constexpr int ROWB = 16 * CPR;
  static constexpr int CPP = (MSL_MTY + 2) * CPR;   // chunks of a plane's slab (54 lanes)
  static_assert(CPP <= 64, "one DMA instruction per plane");
  static constexpr int SLAB = 16 * CPP;
  static constexpr int WAVES = N == 4 ? 4 : 3;
};

// (OWN: as in the walk above)
template <typename S, int N, bool LIST, bool OWN>
__global__ void __launch_bounds__((SC3RTraits<S, N>::NT)) __attribute__((amdgpu_waves_per_eu(SC3RTraits<S, N>::WAVES)))
k_sc3d_zr(const Tab *__restrict__ tab, int lat, Geo g, const S *__restrict__ in, S *__restrict__ out,
          const uint8_t *__restrict__ cls, const uint8_t *__restrict__ tflag, int remap, int xmir, int faces, int zc,
          const int *__restrict__ tlist, const int *__restrict__ tcount) {
  using Tr = SC3RTraits<S, N>;
  using T = typename Tr::T;
  typedef float C;
  constexpr int Q = Tr::Q, NHW = Tr::NHW, NPW = Tr::NPW, NLD = Tr::NLD, ROWB = Tr::ROWB, CPR = Tr::CPR, CPP = Tr::CPP,
                SLAB = Tr::SLAB;
  constexpr bool SPL = NHW > 1;
  __shared__ __align__(16) char sm[Q * SLAB];
  __shared__ float smom[SPL ? NHW : 1][SPL ? 4 : 1][SPL ? 256 : 1];   // partial moments per part
  const LatTab &L = tab->lat[lat];
  int tile;
  if constexpr (LIST) {
    const int n = *tcount;
    if ((int)blockIdx.x >= n) return;
    tile = tlist[msl_xcd_tile((int)blockIdx.x, n)];
  } else {
    const int lin = (int)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
    tile = remap ? msl_xcd_tile(lin, (int)(gridDim.x * gridDim.y * gridDim.z)) : lin;
  }
  const int bx = tile % g.ntx, by = (tile / g.ntx) % g.nty;
  const int z0 = tile / (g.ntx * g.nty) * zc;
  const int x0 = bx * MSL_TX, y0 = by * MSL_MTY;
  const int zn = g.nz - z0 < zc ? g.nz - z0 : zc;   // cells of the column (>= 1)
  {
    uint8_t any = 0;
    for (int k = 0; k < zn; ++k) any |= tflag[((long long)(z0 + k) * g.nty + by) * g.ntx + bx];
    if (!(any & (1 << lat))) return;
  }
  // w: the wave's row of cells; hf: its part of the planes, which starts at
  // plane kb and z node hf
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = wv & 3, hf = SPL ? wv >> 2 : 0, kb = hf * NPW;
  const unsigned pitch_b = (unsigned)g.pitch * 2;
  const unsigned plane_b = (unsigned)g.plane * 2;
  const unsigned slab_b = (unsigned)g.rows * pitch_b;
  // ghost rows and slabs by their faces' rules, as in the walk above
  auto mapped = [&](int ax, int p, int n) {
    if (p >= 0 && p < n) return p;
    const int rule = (faces >> (4 * ax + (p < 0 ? 0 : 2))) & 3;
    return rule == 1 ? (p < 0 ? p + n : p - n) : (rule == 2 ? (p < 0 ? 0 : n - 1) : p);
  };
  // the planes that this wave loads, wv NLD + j: byte offsets of the lane's
  // chunk inside a slab (D3Q27: 0, 1 or 2 y nodes among them, one register each)
  const int kl = wv * NLD;
  unsigned voff[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int K = kl + j < Q ? kl + j : Q - 1, a = K % N, b = (K / N) % N;
    const int row = lane / CPR;
    voff[j] = (unsigned)(mapped(1, y0 + L.n0[1][b] - 1 + row, g.ny) + MSL_G) * pitch_b +
              (unsigned)(lane - row * CPR) * 16u + ((unsigned)((g.xo + x0 + L.n0[0][a] - 1) * 2) & ~3u);
  }
  int n0z[N];
#pragma unroll
  for (int c = 0; c < N; ++c) n0z[c] = L.n0[2][c];
  const long long plane_b64 = g.plane * 2;
  // DMA of step t's slab of the wave's share of the planes: slab z0 + n0_z - 1 + t
  auto issue = [&](const int t) {
    unsigned oz[N];
#pragma unroll
    for (int c = 0; c < N; ++c) oz[c] = (unsigned)(mapped(2, z0 + n0z[c] - 1 + t, g.nz) + MSL_G) * slab_b;
    const char *pp = (const char *)in + kl * plane_b64;
    asm volatile("" : "+s"(pp));
    if (lane < CPP)
#pragma unroll
      for (int j = 0; j < NLD; ++j) {
        const int K = kl + j;
        if (Q % Tr::NWV == 0 || K < Q) {
          const int c = K / (N * N);
          unsigned so = oz[0];
#pragma unroll
          for (int q = 1; q < N; ++q) so = c == q ? oz[q] : so;
          const __amdgpu_buffer_rsrc_t rs =
              __builtin_amdgcn_make_buffer_rsrc((void *)pp, (short)0, (int)plane_b, MSL_RSRC_WORD3);
          unsigned vo = voff[j];
          if constexpr (OWN) {
            const int zm = mapped(2, z0 + L.n0[2][c] - 1 + t, g.nz), row = lane / CPR;
            if (zm < 0 || zm >= g.nz)
              vo = (unsigned)(y0 + L.n0[1][(K / N) % N] - 1 + row + MSL_G) * pitch_b + (unsigned)(lane - row * CPR) * 16u +
                   ((unsigned)((g.xo + x0 + L.n0[0][K % N] - 1) * 2) & ~3u);
          }
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (msl_lds_t *)(sm + K * SLAB), 16, (int)vo, (int)so, 0, 0);
        }
        pp += plane_b64;
      }
  };
  // per-node tables of each axis: interpolation weights (z from the wave's
  // first z node on)
  C wlo[3][N], wmid[3][N], whi[3][N];
  unsigned rb[N];   // LDS byte of the lane's first element in its row, per x node
#pragma unroll
  for (int a = 0; a < N; ++a) {
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const int q = SPL && ax == 2 ? hf : a;   // (split walk: every plane of the wave has z node hf)
      wlo[ax][a] = L.af[ax][q][0];
      wmid[ax][a] = L.af[ax][q][1];
      whi[ax][a] = L.af[ax][q][2];
    }
    rb[a] = (unsigned)(kb * SLAB + w * ROWB + lane * 2) + (unsigned)((L.n0[0][a] - 1) & 1) * 2u;
  }
  // per plane: the z interpolation's partial sums of the next two cells and the
  // streamed value
  C ha[NPW], hb[NPW], ftk[NPW];
#pragma unroll
  for (int k = 0; k < NPW; ++k) ha[k] = hb[k] = C(0);
  auto fetch = [&]<int K>(uint32_t (&v)[3][3]) {
    typedef volatile const __attribute__((address_space(3))) uint16_t lds_u16;
    const char *base = (const char *)sm + rb[K % N] + K * SLAB;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int e = 0; e < 3; ++e) v[dy][e] = *(lds_u16 *)(base + dy * ROWB + 2 * e);
  };
  auto recon = [&]<int K>(const uint32_t (&v)[3][3]) {
    constexpr int a = K % N, b = (K / N) % N, cc = K / (N * N);
    C hy[3];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
      hy[dy] = __builtin_fmaf(wlo[0][a], (C)half_elem<S>(v[dy][0]),
                              __builtin_fmaf(wmid[0][a], (C)half_elem<S>(v[dy][1]),
                                             __builtin_fmaf(whi[0][a], (C)half_elem<S>(v[dy][2]), 0.0f)));
    const C hn = wlo[1][b] * hy[0] + wmid[1][b] * hy[1] + whi[1][b] * hy[2];
    // (three-address FMAs: no register moves as the walk advances)
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(ftk[K]) : "s"(whi[2][cc]), "v"(hn), "v"(ha[K]));
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(ha[K]) : "s"(wmid[2][cc]), "v"(hn), "v"(hb[K]));
    hb[K] = wlo[2][cc] * hn;
    asm("" : "+v"(hb[K]));
  };
  auto slab = [&]() {
    uint32_t cur[3][3], nxt[3][3];
    fetch.template operator()<0>(cur);
    msl_for_planes<NPW>([&]<int K>() {
      if constexpr (K + 1 < NPW) fetch.template operator()<K + 1>(nxt);
      __builtin_amdgcn_sched_barrier(0);
      recon.template operator()<K>(cur);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (K + 1 < NPW)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int e = 0; e < 3; ++e) cur[dy][e] = nxt[dy][e];
    });
  };
  const int x = x0 + lane, y = y0 + w;
  // the lane's cells of this velocity set along the column (bit k: z0 + k)
  uint32_t mine_bits = 0;
  if (x < g.nx && y < g.ny)
    for (int k = 0; k < zn; ++k)
      mine_bits |= (uint32_t)((cls[((long long)(z0 + k) * g.ny + y) * g.nx + x] & 1) == lat) << k;
  const bool xedge = xmir && (x0 < MSL_G || x0 + MSL_TX > g.nx - MSL_G);
  const unsigned cell0 = (unsigned)g.idx(x < g.nx ? x : 0, y < g.ny ? y : 0, z0) * 2;
  auto finish = [&]<bool XE>(const int k) {
    const bool mine = (mine_bits >> k) & 1u;
    // (scales and velocities by scalar loads here, as in the walk above)
    typedef const __attribute__((address_space(4))) LatTab cLatTab;
    typedef const __attribute__((address_space(4))) Tab cTab;
    cLatTab *Lp = (cLatTab *)&L;
    cTab *tp = (cTab *)tab;
    const char *op = (const char *)out + (long long)kb * plane_b64;
    asm volatile("" : "+s"(Lp), "+s"(tp), "+s"(op));
    auto &L = *Lp;
    C rho = C(0), jx = C(0), jy = C(0), jz = C(0);
    msl_for_planes<NPW>([&]<int K>() {
      constexpr int a = K % N, b = (K / N) % N, cc = K / (N * N);
      const C f = L.scf[kb + K] * (C(1) + ftk[K]);
      ftk[K] = f;   // the population itself from here on
      rho += f;
      jx += L.vf[0][a] * f;
      jy += L.vf[1][b] * f;
      jz += L.vf[2][hf + cc] * f;
    });
    if constexpr (SPL) {
      const int ci = w * 64 + lane;
      smom[hf][0][ci] = rho;
      smom[hf][1][ci] = jx;
      smom[hf][2][ci] = jy;
      smom[hf][3][ci] = jz;
      msl_lds_barrier();
      rho = smom[0][0][ci];
      jx = smom[0][1][ci];
      jy = smom[0][2][ci];
      jz = smom[0][3][ci];
#pragma unroll
      for (int h = 1; h < NHW; ++h) {
        rho += smom[h][0][ci];
        jx += smom[h][1][ci];
        jy += smom[h][2][ci];
        jz += smom[h][3][ci];
      }
    }
    // equilibrium factors in FP64, kept in FP32; athermal: T = 1
    const double rd = (double)rho, ird = 1.0 / rd;
    const double ux = (double)jx * ird, uy = (double)jy * ird, uz = (double)jz * ird;
    C om = tp->omegaf;
    if (tp->tau_mode == 1) om = (C)(1.0 / (tp->mu_T1 / (rd * 1.0 * tp->dt) + 0.5));
    C Px[N], Py[N], Pz[N];
    {
      double px[N], py[N], pz[N];
      eq_axis<double, N>(L, (ux - L.ur[0]) * L.isq, L.iTr, px);
      eq_axis<double, N>(L, (uy - L.ur[1]) * L.isq, L.iTr, py);
      eq_axis<double, N>(L, (uz - L.ur[2]) * L.isq, L.iTr, pz);
#pragma unroll
      for (int q = 0; q < N; ++q) {
        Px[q] = (C)(px[q] * rd);
        Py[q] = (C)py[q];
        Pz[q] = (C)pz[q];
      }
      if constexpr (SPL) {   // the z factor of the wave's node
#pragma unroll
        for (int q = 1; q < N; ++q)
          if (q == hf) Pz[0] = (C)pz[q];
      }
    }
    const unsigned soff = mine ? cell0 + (unsigned)k * slab_b : 0x80000000u;
    const unsigned ioff = (mine && x < MSL_G) ? soff + (unsigned)g.nx * 2
                          : (mine && x >= g.nx - MSL_G) ? soff - (unsigned)g.nx * 2 : 0x80000000u;
    msl_for_planes<NPW>([&]<int K>() {
      constexpr int a = K % N, b = (K / N) % N, cc = K / (N * N);
      const C isc = L.iscf[kb + K];
      const C feq = Px[a] * Py[b] * Pz[cc];
      const C v = ftk[K];
      const C vo = v + om * (feq - v);
      const S sv = T::store(vo * isc - C(1));
      const __amdgpu_buffer_rsrc_t rsout =
          __builtin_amdgcn_make_buffer_rsrc((void *)op, (short)0, (int)plane_b, MSL_RSRC_WORD3);
      op += plane_b64;
      __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, sv), rsout, (int)soff, 0, 0);
      if constexpr (XE) __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, sv), rsout, (int)ioff, 0, 0);
    });
  };
  // the walk, as above; a row's window rows are loaded by several waves, so
  // two barriers bracket the reads of a slab
  constexpr int VW1 = NPW < 63 ? NPW : 63, VW2 = 2 * NPW < 63 ? 2 * NPW : 63;
  issue(0);
  msl_wait_vm<0>();
  for (int t = 0; t < zn + 2; ++t) {
#pragma unroll
    for (int a = 0; a < N; ++a) asm volatile("" : "+v"(rb[a]));
    msl_lds_barrier();   // every wave's share of the slab is in LDS
    slab();
    msl_lds_barrier();   // the slab's LDS values are read; the next load may overwrite them
    if (t + 1 < zn + 2) issue(t + 1);
    if (t >= 2) {
      if (xedge) {
        finish.template operator()<true>(t - 2);
        msl_wait_vm<VW2>();
      } else {
        finish.template operator()<false>(t - 2);
        msl_wait_vm<VW1>();
      }
    } else {
      msl_wait_vm<0>();
    }
  }
}
