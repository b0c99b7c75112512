// msl_fields.hip -- the passes between a state and its macroscopic fields:
// equilibrium initialisation from rho, u, T and the fields of every cell from
// its own populations, with compile-time velocity-set sizes.
#include "msl_band.hpp"
#include "msl_device.hpp"

#define FLD_BLOCK 256

// Both kernels are bound by memory: one thread per cell reads (or writes) each
// population of the cell's own set once and the FP64 fields once.  With the
// set sizes known at compile time the populations stay in registers and their
// loads are all in flight together; with run-time sizes they went through
// arrays in scratch memory, which cost several times the planes themselves.
// 8192^2 D2Q9 FP32 fields: 3781 us before, 800 us (5.8 TB/s) now;
// 3001 x 2003 D2Q36 FP16: 1155 us before, 128 us now.
// NH = 0: one velocity set.
template <typename S, int D, int N, bool TH>
__device__ __forceinline__ void cell_fields(const Tab *tab, const Geo &g, const char *base, int l, int off,
                                            double &rho, double *u, double &T) {
  constexpr int Q = Pow<D, N>::v;
  double f[Q], gg[TH ? Q : 1];
  read_cell_t<S, D, N, TH>(tab, g, base, l, off, f, gg);
  macros_t<D, N>(tab->lat[l], TH, tab->cv, f, gg, rho, u, T);
}

template <typename S, int D, int NL, int NH, bool TH>
__global__ void __launch_bounds__(FLD_BLOCK)
k_macros_t(const Tab *__restrict__ tab, Geo g, const char *__restrict__ bl, const char *__restrict__ bh,
           const uint8_t *__restrict__ cls, double *__restrict__ rho, double *__restrict__ u,
           double *__restrict__ T) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= g.ncell) return;
  int x, y, z;
  cell_coords(g, k, x, y, z);
  const int off = g.idx(x, y, z);
  double r, uu[3], t;
  if (NH > 0 && (cls[k] & 1)) cell_fields<S, D, (NH > 0 ? NH : NL), TH>(tab, g, bh, 1, off, r, uu, t);
  else cell_fields<S, D, NL, TH>(tab, g, bl, 0, off, r, uu, t);
  if (rho) rho[k] = r;
  if (u) {
#pragma unroll
    for (int a = 0; a < D; ++a) u[a * g.ncell + k] = uu[a];
  }
  if (T) T[k] = t;
}

template <typename S, int D, int N, bool TH>
__device__ __forceinline__ void cell_init(const Tab *tab, const Geo &g, char *base, int l, int off, double rho,
                                          const double *u, double T) {
  constexpr int Q = Pow<D, N>::v;
  double f[Q], gg[TH ? Q : 1];
  feq_t<D, N>(tab->lat[l], rho, u, T, f);
  if (TH) {
    const double s = tab->gfac * T;
#pragma unroll
    for (int i = 0; i < Q; ++i) gg[TH ? i : 0] = s * f[i];
  }
  write_cell_t<S, D, N, TH>(tab, g, base, l, off, f, gg);
}

// lattice equilibrium of each cell's own velocity set
template <typename S, int D, int NL, int NH, bool TH>
__global__ void __launch_bounds__(FLD_BLOCK)
k_init_eq_t(const Tab *__restrict__ tab, Geo g, char *bl, char *bh, const uint8_t *__restrict__ cls,
            const double *__restrict__ rho, const double *__restrict__ u, const double *__restrict__ T) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= g.ncell) return;
  int x, y, z;
  cell_coords(g, k, x, y, z);
  const int off = g.idx(x, y, z);
  double uu[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int a = 0; a < D; ++a) uu[a] = u[a * g.ncell + k];
  const double Tk = TH ? T[k] : 1.0;
  if (NH > 0 && (cls[k] & 1)) cell_init<S, D, (NH > 0 ? NH : NL), TH>(tab, g, bh, 1, off, rho[k], uu, Tk);
  else cell_init<S, D, NL, TH>(tab, g, bl, 0, off, rho[k], uu, Tk);
}

// a functor templated on (D, NL, NH) for the context's sets (NH = 0: one set)
template <typename F>
static int sets_dispatch(const msl_ctx *c, F &&f) {
  const int n = c->htab.lat[0].n;
  if (c->nlat > 1) return msl_pair_dispatch(c->D, n, c->htab.lat[1].n, f);
  if (c->D == 2) {
    switch (n) {
      case 3: return f.template operator()<2, 3, 0>();
      case 4: return f.template operator()<2, 4, 0>();
      case 5: return f.template operator()<2, 5, 0>();
      case 6: return f.template operator()<2, 6, 0>();
    }
  } else {
    switch (n) {
      case 3: return f.template operator()<3, 3, 0>();
      case 4: return f.template operator()<3, 4, 0>();
    }
  }
  return MSL_EINVAL;
}

template <typename S, bool TH>
static int macros_st(msl_ctx *c, double *rho, double *u, double *T) {
  return sets_dispatch(c, [&]<int D, int NL, int NH>() {
    hipLaunchKernelGGL((k_macros_t<S, D, NL, NH, TH>), dim3((unsigned)((c->ncell + FLD_BLOCK - 1) / FLD_BLOCK)),
                       dim3(FLD_BLOCK), 0, c->stream, c->dtab, c->geo, c->planes[0][c->cur],
                       c->nlat > 1 ? c->planes[1][c->cur] : nullptr, c->cls, rho, u, T);
    return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
  });
}

template <typename S, bool TH>
static int init_st(msl_ctx *c, const double *rho, const double *u, const double *T) {
  return sets_dispatch(c, [&]<int D, int NL, int NH>() {
    hipLaunchKernelGGL((k_init_eq_t<S, D, NL, NH, TH>), dim3((unsigned)((c->ncell + FLD_BLOCK - 1) / FLD_BLOCK)),
                       dim3(FLD_BLOCK), 0, c->stream, c->dtab, c->geo, c->planes[0][c->cur],
                       c->nlat > 1 ? c->planes[1][c->cur] : nullptr, c->cls, rho, u, T);
    return hipGetLastError() == hipSuccess ? MSL_OK : MSL_EHIP;
  });
}

int msl_launch_macros(msl_ctx *c, double *rho, double *u, double *T) {
  const bool th = c->cfg.thermal;
  switch (c->cfg.store) {
    case MSL_FP64: return th ? macros_st<double, true>(c, rho, u, T) : macros_st<double, false>(c, rho, u, T);
    case MSL_FP32: return th ? macros_st<float, true>(c, rho, u, T) : macros_st<float, false>(c, rho, u, T);
    case MSL_FP16_DEV: return th ? macros_st<_Float16, true>(c, rho, u, T) : macros_st<_Float16, false>(c, rho, u, T);
    case MSL_BF16_DEV: return th ? macros_st<bf16_t, true>(c, rho, u, T) : macros_st<bf16_t, false>(c, rho, u, T);
  }
  return MSL_EINVAL;
}

int msl_launch_init_eq(msl_ctx *c, const double *rho, const double *u, const double *T) {
  const bool th = c->cfg.thermal;
  switch (c->cfg.store) {
    case MSL_FP64: return th ? init_st<double, true>(c, rho, u, T) : init_st<double, false>(c, rho, u, T);
    case MSL_FP32: return th ? init_st<float, true>(c, rho, u, T) : init_st<float, false>(c, rho, u, T);
    case MSL_FP16_DEV: return th ? init_st<_Float16, true>(c, rho, u, T) : init_st<_Float16, false>(c, rho, u, T);
    case MSL_BF16_DEV: return th ? init_st<bf16_t, true>(c, rho, u, T) : init_st<bf16_t, false>(c, rho, u, T);
  }
  return MSL_EINVAL;
}
