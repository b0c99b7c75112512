// msl_stream.hpp -- dispatch of the fused stream-and-collide launches, by
// dimension, velocity-set order, storage precision and thermal model:
//   2D  every plane's window resident in LDS (msl_stream2.hpp), which also
//       converts the band cells of two-set runs, both sets in one launch on small
//       grids; thermal FP64 D2Q25 and D2Q36, whose windows do not fit, a wave per
//       x node (msl_stream2s.hpp)
//   3D  column walks along z for athermal 16-bit storage and FP32 D3Q27
//       (msl_stream3z.hpp); planes streamed through LDS in chunks otherwise
//       (msl_stream3.hpp)
// Cells of the other velocity set are skipped; tiles without a cell of this set
// exit before loading anything.
#pragma once
#include <utility>

#include "msl_device.hpp"
#include "msl_stream2.hpp"
#include "msl_stream2s.hpp"
#include "msl_stream3.hpp"
#include "msl_stream3z.hpp"

// 2D, every plane resident in LDS (k_sc2d_res); NO > 0: the launch also
// converts its band cells into the other set's planes `oth` (NO nodes per axis)
template <typename S, bool TH, int N, bool QE, int NO>
static int launch_sc2(msl_ctx *c, int lat, const char *in, char *out, char *oth) {
  const Geo &g = c->geo;
  dim3 block(256);
  S *os = (S *)oth;
  // non-temporal stores for FP32 / FP64 D2Q9 planes when the set's buffer
  // exceeds the 256 MB last-level cache
  const int nt = N == 3 && sizeof(S) >= 4 &&
                 (double)g.plane * sizeof(S) * c->Q[lat] * (c->cfg.thermal ? 2 : 1) > 256.0 * (1 << 20);
  const long long tiles8 = (long long)((g.nx + MSL_TX - 1) / MSL_TX) * ((g.ny + 7) / 8);
  bool small = false;
  if constexpr (N == 3) {
    // D2Q9 on a grid of fewer than 8 tiles of 8 rows per CU: 4-row tiles,
    // twice as many workgroups
    using T2 = SC2Traits<S, TH, N, true>;
    static_assert(T2::fits && T2::TY == 4, "4-row D2Q9 tile");
    small = tiles8 < 2048;
    if (small) {
      dim3 grid((g.nx + MSL_TX - 1) / MSL_TX, (g.ny + T2::TY - 1) / T2::TY);
      hipLaunchKernelGGL((k_sc2d_res<S, TH, N, true, false, QE, NO>), grid, block, 0, c->stream, c->dtab, lat, g,
                         (const S *)in, (S *)out, c->cls, c->tflag, lat == 0, nt, nullptr, nullptr, os, c->faces);
    }
  }
  if constexpr (N > 3 && NO < N) {
    using T2 = SC2Traits<S, TH, N>;
    const long long tiles = (long long)g.ntx * ((g.ny + T2::TY - 1) / T2::TY);
    const long long fit = 256LL * (T2::WGS < 1 ? 1 : T2::WGS);
    if (!small && lat != 0 && tiles > 4 * fit) {
      // the high-order set on a large grid: one workgroup per live tile of
      // the compact list, whose length is read back (one stream
      // synchronisation each time the tile flags change, i.e. once per
      // criterion pass); smaller grids launch the whole tile grid, where
      // tiles without cells of the set exit at once
      if (c->capturing) return MSL_ESTATE;   // the list length is read by the host
      if (!c->tl_ok) {
        if (msl_launch_tile_list(c, lat, T2::R, 1)) return MSL_EHIP;
        int n = 0;
        if (hipMemcpyAsync(&n, c->tcount, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
            hipStreamSynchronize(c->stream) != hipSuccess)
          return MSL_EHIP;
        c->tl_n = n;
        c->tl_ok = 1;
      }
      if (c->tl_n == 0) return MSL_OK;
      dim3 grid((unsigned)c->tl_n);
      hipLaunchKernelGGL((k_sc2d_res<S, TH, N, false, true, QE, NO>), grid, block, 0, c->stream, c->dtab, lat,
                         g, (const S *)in, (S *)out, c->cls, c->tflag, 0, nt, c->tlist, c->tcount, os, c->faces);
      return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
    }
  }
  if (!small) {
    using T2 = SC2Traits<S, TH, N>;
    dim3 grid((g.nx + MSL_TX - 1) / MSL_TX, (g.ny + T2::TY - 1) / T2::TY);
    hipLaunchKernelGGL((k_sc2d_res<S, TH, N, false, false, QE, NO>), grid, block, 0, c->stream, c->dtab, lat, g,
                       (const S *)in, (S *)out, c->cls, c->tflag, lat == 0, nt, nullptr, nullptr, os, c->faces);
  }
  return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
}

// whether the launches of set `lat` can convert its band cells themselves
// (2D kernels with every plane resident in LDS)
template <typename S, bool TH, int N>
static bool fusable_n(int D) {
  return D == 2 && SC2Traits<S, TH, N>::fits;
}

// 3D sets that run a column walk
template <typename S, bool TH>
constexpr bool msl_walk_set(int n) { return !TH && (sizeof(S) == 2 || (sizeof(S) == 4 && n == 3)); }

template <typename S, bool TH, int N, int D, bool QE = false>
static int launch_one(msl_ctx *c, int lat, const char *in, char *out, char *oth) {
  const Geo &g = c->geo;
  dim3 block(256);
  if constexpr (D == 2 && SC2Traits<S, TH, N>::fits) {
    switch (oth ? c->htab.lat[lat ^ 1].n : 0) {
      case 0: return launch_sc2<S, TH, N, QE, 0>(c, lat, in, out, nullptr);
      case 3: if constexpr (N != 3) return launch_sc2<S, TH, N, QE, 3>(c, lat, in, out, oth); break;
      case 4: if constexpr (N != 4) return launch_sc2<S, TH, N, QE, 4>(c, lat, in, out, oth); break;
      case 5: if constexpr (N != 5) return launch_sc2<S, TH, N, QE, 5>(c, lat, in, out, oth); break;
      case 6: if constexpr (N != 6) return launch_sc2<S, TH, N, QE, 6>(c, lat, in, out, oth); break;
    }
    return MSL_EINVAL;
  } else if constexpr (D == 2) {
    // thermal D2Q25, D2Q36 in FP64
    static_assert(sizeof(S) == 8 && TH);
    if (oth) return MSL_EINVAL;
    auto run = [&]<int R>() {
      hipLaunchKernelGGL((k_sc2d_split<N, R, QE>), dim3(g.ntx, (g.ny + R - 1) / R), dim3(64 * N), 0, c->stream,
                         c->dtab, lat, g, (const S *)in, (S *)out, c->cls, c->tflag, c->faces);
    };
    // one row of cells per workgroup; two for D2Q25 where that leaves 8
    // workgroups per CU (2048^2: 1640 us a step, one row 2021).  D2Q36 spills
    // with two (3368, one row 2895; 512^2 207 and 170)
    if constexpr (N == 5) {
      if ((long long)g.ntx * g.ny >= 4096) {
        run.template operator()<2>();
        return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
      }
    }
    run.template operator()<1>();
  } else {
    if (oth) return MSL_EINVAL;
    if constexpr (msl_walk_set<S, TH>(N)) {
      // 3D, athermal 16-bit storage and FP32 D3Q27: columns of 64 x 4 x zc cells
      // walked along z; the high-order set of a large grid runs over the
      // compact list of its live columns.
      // Column length: a column loads two slabs more than it has cells, and the
      // launch takes as long as its columns have steps.  8 cells (FP16 D3Q27
      // and D3Q64, one stream: 200^3 396 + 371 us against 415 + 403 at 16; 256^3
      // 644 + 635 against 631 + 643), 4 where 8 leave CUs idle (64^3 FP16: a step
      // of 118 against 84 us)
      const long long cols = (long long)g.ntx * g.nty;
      const int zc = cols * ((g.nz + 7) / 8) >= 256 ? MSL_WALK_ZC : 4;
      const int ncz = (g.nz + zc - 1) / zc;
      const dim3 grid((g.nx + MSL_TX - 1) / MSL_TX, (g.ny + MSL_MTY - 1) / MSL_MTY, ncz);
      auto walk = [&]<bool OWN>() -> int {
        if constexpr (sizeof(S) == 4) {
          hipLaunchKernelGGL((k_sc3d_zm<OWN>), grid, dim3(SC3ZTraits::NT), 0, c->stream, c->dtab, lat, g, (const S *)in,
                             (S *)out, c->cls, c->tflag, lat == 0, c->xmir, c->faces, zc);
        } else {
          const dim3 nt(SC3RTraits<S, N>::NT);
          if constexpr (N > 3) {
            if (lat != 0 && cols * ncz > MSL_WALK_LIST_MIN) {
              if (c->capturing) return MSL_ESTATE;   // the list length is read by the host
              if (!c->tl_ok) {
                if (msl_launch_tile_list(c, lat, 1, zc)) return MSL_EHIP;
                int n = 0;
                if (hipMemcpyAsync(&n, c->tcount, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
                    hipStreamSynchronize(c->stream) != hipSuccess)
                  return MSL_EHIP;
                c->tl_n = n;
                c->tl_ok = 1;
              }
              if (c->tl_n == 0) return MSL_OK;
              hipLaunchKernelGGL((k_sc3d_zr<S, N, true, OWN>), dim3((unsigned)c->tl_n), nt, 0, c->stream, c->dtab, lat, g,
                                 (const S *)in, (S *)out, c->cls, c->tflag, 0, c->xmir, c->faces, zc, c->tlist, c->tcount);
              return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
            }
          }
          hipLaunchKernelGGL((k_sc3d_zr<S, N, false, OWN>), grid, nt, 0, c->stream, c->dtab, lat, g, (const S *)in, (S *)out,
                             c->cls, c->tflag, lat == 0, c->xmir, c->faces, zc, (const int *)nullptr, (const int *)nullptr);
        }
        return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
      };
      // a slot on a fixed z face between y faces that map ghost rows: the stored
      // slabs keep their own ghost rows
      bool own = false;
      for (int f = 4; f < 6; ++f) own |= c->cfg.bc[f] == MSL_BC_FIXED_EQ && c->cfg.slot[f][0] < c->cfg.slot[f][1];
      return own && ((c->faces >> 4) & 15) ? walk.template operator()<true>() : walk.template operator()<false>();
    } else {
    // the other 3D sets (FP64, thermal, FP32 D3Q64): planes streamed through LDS
    // in chunks; the high-order set of a large grid runs over the compact list of
    // its live tiles (as in 2D)
    using T3 = SC3Traits<S, TH, N>;
    if constexpr (N > 3) {
      const long long tiles = (long long)g.ntx * g.nty * ((g.ntz + T3::RZ - 1) / T3::RZ);
      const long long fit = 256LL * ((160 * 1024) / T3::LDS_BYTES);
      if (lat != 0 && tiles > 4 * fit) {
        if (c->capturing) return MSL_ESTATE;   // the list length is read by the host
        if (!c->tl_ok) {
          if (msl_launch_tile_list(c, lat, 1, T3::RZ)) return MSL_EHIP;
          int n = 0;
          if (hipMemcpyAsync(&n, c->tcount, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
              hipStreamSynchronize(c->stream) != hipSuccess)
            return MSL_EHIP;
          c->tl_n = n;
          c->tl_ok = 1;
        }
        if (c->tl_n == 0) return MSL_OK;
        hipLaunchKernelGGL((k_sc3d_res<S, TH, N, true>), dim3((unsigned)c->tl_n), block, 0, c->stream,
                           c->dtab, lat, g, (const S *)in, (S *)out, c->cls, c->tflag, 0, c->xmir,
                           c->tlist, c->tcount);
        return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
      }
    }
    dim3 grid((g.nx + MSL_TX - 1) / MSL_TX, (g.ny + MSL_MTY - 1) / MSL_MTY, (g.nz + T3::RZ - 1) / T3::RZ);
    hipLaunchKernelGGL((k_sc3d_res<S, TH, N>), grid, block, 0, c->stream, c->dtab, lat, g,
                       (const S *)in, (S *)out, c->cls, c->tflag, lat == 0, c->xmir, nullptr, nullptr);
    }
  }
  return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
}

template <typename S, bool TH>
static int launch_n(msl_ctx *c, int lat, const char *in, char *out, char *oth) {
  const int n = c->htab.lat[lat].n;
  if (c->D == 2) {
    if (c->htab.qe) {
      switch (n) {
        case 3: return launch_one<S, TH, 3, 2, true>(c, lat, in, out, oth);
        case 4: return launch_one<S, TH, 4, 2, true>(c, lat, in, out, oth);
        case 5: return launch_one<S, TH, 5, 2, true>(c, lat, in, out, oth);
        case 6: return launch_one<S, TH, 6, 2, true>(c, lat, in, out, oth);
      }
      return MSL_EINVAL;
    }
    switch (n) {
      case 3: return launch_one<S, TH, 3, 2>(c, lat, in, out, oth);
      case 4: return launch_one<S, TH, 4, 2>(c, lat, in, out, oth);
      case 5: return launch_one<S, TH, 5, 2>(c, lat, in, out, oth);
      case 6: return launch_one<S, TH, 6, 2>(c, lat, in, out, oth);
    }
  } else {
    switch (n) {
      case 3: return launch_one<S, TH, 3, 3>(c, lat, in, out, oth);
      case 4: return launch_one<S, TH, 4, 3>(c, lat, in, out, oth);
    }
  }
  return MSL_EINVAL;
}

// stream-and-collide of set `lat` for one storage type and energy variant;
// oth: the other set's new planes when the launch converts its band cells
template <typename S, bool TH>
int msl_launch_store_th(msl_ctx *c, int lat, const char *in, char *out, char *oth) {
  return launch_n<S, TH>(c, lat, in, out, oth);
}

// both sets of a fused 2D run in one launch; MSL_ESTATE: not for this grid (the
// caller launches them one after the other).  The line: what the CUs hold by the
// launch's LDS four times over, at most 8 workgroups per CU.  us per step with a
// sixteenth of the grid high-order, one launch against two: FP64 D2Q9+D2Q16 64^2
// 6.4, 12.8, 256^2 7.3, 12.2, 512^2 (1536 workgroups) 16.4, 19.2; FP32 D2Q9+D2Q36
// 64^2 9.9, 17.7, 512^2 (2048) 17.0, 19.7, but 768^2 (4608) 26.9, 25.2 and 1024^2
// 51.1, 33.1: the low-order tiles hold the other set's LDS.  FP64 D2Q9+D2Q25
// 512^2 (2048, where the CUs hold 256 at a time), a tenth high-order: 54, 35.  Up
// to 1024 workgroups one launch wins in that class too: D2Q9+D2Q25 256^2 (512)
// 13.2, 15.5, 320^2 (800) 14.4, 16.2; the closest of its pairs, thermal FP64
// D2Q9+D2Q16, 320^2 19.2, 20.7 (a sixteenth of the grid high-order; half: 1.17 to
// 1.6 times).
template <typename S, bool TH, int NL, int NH>
static int launch_pair(msl_ctx *c, int cur) {
  using P = SC2PairTraits<S, TH, NL, NH>;
  if constexpr (P::fits) {
    const Geo &g = c->geo;
    const long long nlo = (long long)g.ntx * ((g.ny + P::TL::TY - 1) / P::TL::TY);
    const long long nhi = (long long)g.ntx * ((g.ny + P::TH_::TY - 1) / P::TH_::TY);
    if (nlo + nhi > (P::WGS < 2 ? 1024 : 2048)) return MSL_ESTATE;
    auto run = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)(nlo + nhi)), dim3(256), 0, c->stream, c->dtab, g,
                         (const S *)c->planes[0][cur], (S *)c->planes[0][cur ^ 1], (const S *)c->planes[1][cur],
                         (S *)c->planes[1][cur ^ 1], c->cls, c->tflag, (int)nlo, c->faces);
    };
    if (c->htab.qe) run(k_sc2d_pair<S, TH, NL, NH, true>);
    else run(k_sc2d_pair<S, TH, NL, NH, false>);
    return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
  }
  return MSL_ESTATE;
}

template <typename S, bool TH>
int msl_launch_pair_th(msl_ctx *c, int cur) {
  const int nl = c->htab.lat[0].n, nh = c->htab.lat[1].n;
  if (nl == 3 && nh == 4) return launch_pair<S, TH, 3, 4>(c, cur);
  if (nl == 3 && nh == 5) return launch_pair<S, TH, 3, 5>(c, cur);
  if (nl == 3 && nh == 6) return launch_pair<S, TH, 3, 6>(c, cur);
  if (nl == 4 && nh == 5) return launch_pair<S, TH, 4, 5>(c, cur);
  if (nl == 4 && nh == 6) return launch_pair<S, TH, 4, 6>(c, cur);
  if (nl == 5 && nh == 6) return launch_pair<S, TH, 5, 6>(c, cur);
  return MSL_ESTATE;
}

// every set of a 2D context runs the kernel with all planes resident in LDS
// (which can convert band cells itself)
template <typename S, bool TH>
int msl_sc2_all_th(const msl_ctx *c) {
  if (c->D != 2) return 0;
  for (int l = 0; l < c->nlat; ++l) {
    bool ok = false;
    switch (c->htab.lat[l].n) {
      case 3: ok = fusable_n<S, TH, 3>(2); break;
      case 4: ok = fusable_n<S, TH, 4>(2); break;
      case 5: ok = fusable_n<S, TH, 5>(2); break;
      case 6: ok = fusable_n<S, TH, 6>(2); break;
    }
    if (!ok) return 0;
  }
  return 1;
}
