// Launchers of the y transforms. A workgroup takes one z plane and 2*LPW
// adjacent x slots and transforms the LPW complex columns formed by pairing
// neighbouring slots; each row access is 2*LPW contiguous values. The x<->y
// permutation of the pencil method is therefore never materialised: the
// kernel gathers its columns straight from the x-packed array and writes
// them back in place.
#include "fft_y.hpp"
#include "pf_internal.hpp"

namespace pf {

namespace {
template <typename T>
int y_lines_of(int n, bool inv, int yw, bool xr, long slots, long planes) {
  if (!y_in_regs<T>(n) || y_lds_mode<T>(n, inv, yw, xr)) return 0;
  const int lpw = yr_lpw<T>(n);
  const long wgs = slots * planes / (2 * lpw);
  if (wgs <= y_lds_wgs<T>(n, inv, yw, xr)) return 0;
  // 48 slots (an x-face field of the shortest lines) need the narrow ones
  return wgs <= y_narrow_wgs<T>(n) || slots % (2 * lpw) ? yr_narrow<T>(n) : lpw;
}
template <typename T, int N, int LPW, bool INV, int YW, bool XR>
hipError_t yr_launch(int nx, int nz, T *data, size_t sp, const cplx<double> *tw, const cplx<double> *ctw,
                     const PlaneMean &pm, hipStream_t st) {
  if (nx % (2 * LPW)) return hipErrorInvalidValue;
  const int nib = nx / (2 * LPW);
  hipLaunchKernelGGL((k_yr<T, N, LPW, INV, YW, XR>), dim3((unsigned)((long)nib * nz)),
                     dim3(LinePlan<N>::tpl * LPW), 0, st, data, tw, ctw, nx, nib, sp, pm);
  return hipGetLastError();
}
// Kernels of one length: the register engine (k_yr) or the LDS engine (k_yfwd,
// k_yinv).
template <typename T, int N, bool INV, int YW, bool XR>
hipError_t y_launch(int nx, int nz, T *data, size_t sp, const cplx<double> *tw, const cplx<double> *ctw,
                    const PlaneMean &pm, hipStream_t st) {
  if constexpr (y_in_regs<T>(N) && !y_lds_mode<T>(N, INV, YW, XR)) {
    constexpr int LPW = yr_lpw<T>(N), LN = yr_narrow<T>(N);
    const int lines = y_lines_of<T>(N, INV, YW, XR, nx, nz);
    if (lines == LPW) return yr_launch<T, N, LPW, INV, YW, XR>(nx, nz, data, sp, tw, ctw, pm, st);
    if (lines) return yr_launch<T, N, LN, INV, YW, XR>(nx, nz, data, sp, tw, ctw, pm, st);
  }
  if constexpr (!y_in_regs<T>(N) || y_lds_mode<T>(N, INV, YW, XR) || y_lds_wgs<T>(N, INV, YW, XR) > 0) {
    constexpr int TPL = y_tpl(N), LPW = y_lpw<T>(N);
    if (nx % (2 * LPW)) return hipErrorInvalidValue;
    const int nib = nx / (2 * LPW);
    const dim3 g((unsigned)((long)nib * nz)), b(TPL * LPW);
    if constexpr (INV)
      hipLaunchKernelGGL((k_yinv<T, N, TPL, LPW, YW, XR>), g, b, 0, st, data, tw, ctw, nx, nib, sp);
    else
      hipLaunchKernelGGL((k_yfwd<T, N, TPL, LPW, YW, XR>), g, b, 0, st, data, tw, ctw, nx, nib, sp, pm);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <typename T, bool INV>
hipError_t y_any(int nx, int ny, int nz, T *data, size_t sp, const cplx<double> *tw, const cplx<double> *ctw,
                 int yw, bool xr, const PlaneMean &pm, hipStream_t st) {
  if ((yw == 1 || yw == 2) && !ctw) return hipErrorInvalidValue;
  switch (yw == 3 ? 2 * ny : ny) {  // a field on the y faces: one FFT of twice the rows per column
#define PF_CASE(N)                                                                                \
  case N:                                                                                         \
    if (yw == 3) return y_launch<T, N, INV, 3, false>(nx, nz, data, sp, tw, ctw, PlaneMean{}, st); \
    if (yw == 2) return y_launch<T, N, INV, 2, false>(nx, nz, data, sp, tw, ctw, pm, st);         \
    if (yw == 1) return y_launch<T, N, INV, 1, false>(nx, nz, data, sp, tw, ctw, pm, st);         \
    if (xr) return y_launch<T, N, INV, 0, true>(nx, nz, data, sp, tw, ctw, pm, st);               \
    return y_launch<T, N, INV, 0, false>(nx, nz, data, sp, tw, ctw, pm, st);
    PF_FOR_FFT_SIZES_Y(PF_CASE)
#undef PF_CASE
    default:
      return hipErrorInvalidValue;
  }
}
}  // namespace

int y_lines(bool fp64, int n, bool inv, int yw, bool xr, int nx, int nz) {
  return fp64 ? y_lines_of<double>(n, inv, yw, xr, nx, nz) : y_lines_of<float>(n, inv, yw, xr, nx, nz);
}

template <typename T>
hipError_t launch_yfwd(int nx, int ny, int nz, T *data, size_t sp, const cplx<double> *tw,
                       const cplx<double> *ctw, int yw, hipStream_t st, bool xr, int shape,
                       const PlaneMean &pm) {
  if (shape != 0) {
    if (yw != 0 || xr) return hipErrorInvalidValue;
    if (shape == kYPersistShape) return launch_y_persist<T>(false, nx, ny, nz, data, sp, tw, st, pm);
    return launch_y_alt<T>(false, shape, nx, ny, nz, data, sp, tw, st, pm);
  }
  return y_any<T, false>(nx, ny, nz, data, sp, tw, ctw, yw, xr, pm, st);
}

template <typename T>
hipError_t launch_yinv(int nx, int ny, int nz, T *data, size_t sp, const cplx<double> *tw,
                       const cplx<double> *ctw, int yw, hipStream_t st, bool xr, int shape) {
  if (shape != 0) {
    if (yw != 0 || xr) return hipErrorInvalidValue;
    if (shape == kYPersistShape) return launch_y_persist<T>(true, nx, ny, nz, data, sp, tw, st);
    return launch_y_alt<T>(true, shape, nx, ny, nz, data, sp, tw, st);
  }
  return y_any<T, true>(nx, ny, nz, data, sp, tw, ctw, yw, xr, PlaneMean{}, st);
}

// ------------------------------------------------------------ grouped
__device__ __forceinline__ PlaneMean grp_mean(const GJob &J) {
  return PlaneMean{J.sums, static_cast<const double *>(J.in2), const_cast<double *>(J.zm), J.scale};
}
template <int N, int TPL, int LPW, bool INV>
__global__ __launch_bounds__(TPL *LPW) void k_y_grp(const GJobs g) {
  const GJob &J = g.j[blockIdx.y];
  if (blockIdx.x >= J.nblk) return;  // uniform per block
  float *W = static_cast<float *>(J.out);
  const int nib = J.nx / (2 * LPW);
  if constexpr (y_in_regs<float>(N))
    yr_body<float, N, LPW, INV, 0, false>(W, J.tw, nullptr, J.nx, nib, J.sp, grp_mean(J), blockIdx.x, J.nblk);
  else if constexpr (INV)
    yinv_body<float, N, TPL, LPW, 0, false>(W, J.tw, nullptr, J.nx, nib, J.sp, blockIdx.x, J.nblk);
  else
    yfwd_body<float, N, TPL, LPW, 0, false>(W, J.tw, nullptr, J.nx, nib, J.sp, grp_mean(J), blockIdx.x, J.nblk);
}

template <int N, int TPL, int LPW, bool INV>
static hipError_t y_grp_run(GJobs &g, hipStream_t st) {
  for (int k = 0; k < g.count; ++k) {
    if (g.j[k].ny != N || g.j[k].nx % (2 * LPW)) return hipErrorInvalidValue;
    g.j[k].nblk = (unsigned)(g.j[k].nx / (2 * LPW) * g.j[k].nz);
  }
  hipLaunchKernelGGL((k_y_grp<N, TPL, LPW, INV>), grp_grid(g), dim3(TPL * LPW), 0, st, g);
  return hipGetLastError();
}
// the lines of a group's workgroups by all its jobs
template <int N, bool INV>
static hipError_t y_grp_launch(GJobs &g, hipStream_t st) {
  if constexpr (y_in_regs<float>(N)) {
    static_assert(!y_lds_mode<float>(N, INV, 0, false) && y_lds_wgs<float>(N, INV, 0, false) == 0, "periodic float32");
    constexpr int LPW = yr_lpw<float>(N), LN = yr_narrow<float>(N);
    long slots = 0;
    for (int k = 0; k < g.count; ++k) slots += (long)g.j[k].nx * g.j[k].nz;
    if (y_lines_of<float>(N, INV, 0, false, slots, 1) == LPW) return y_grp_run<N, rx_tpl(N), LPW, INV>(g, st);
    return y_grp_run<N, rx_tpl(N), LN, INV>(g, st);
  } else {
    return y_grp_run<N, y_tpl(N), y_lpw<float>(N), INV>(g, st);
  }
}
template <bool INV>
static hipError_t launch_y_grp(int ny, GJobs &g, hipStream_t st) {
  if (!grp_ok(g)) return hipErrorInvalidValue;
  switch (ny) {
#define PF_CASE(N) \
  case N:          \
    return y_grp_launch<N, INV>(g, st);
    PF_FOR_FFT_SIZES_Y(PF_CASE)
#undef PF_CASE
    default:
      return hipErrorInvalidValue;
  }
}
hipError_t launch_yfwd_grp(int ny, GJobs &g, hipStream_t st) { return launch_y_grp<false>(ny, g, st); }
hipError_t launch_yinv_grp(int ny, GJobs &g, hipStream_t st) { return launch_y_grp<true>(ny, g, st); }

template hipError_t launch_yfwd<double>(int, int, int, double *, size_t, const cplx<double> *,
                                        const cplx<double> *, int, hipStream_t, bool, int, const PlaneMean &);
template hipError_t launch_yfwd<float>(int, int, int, float *, size_t, const cplx<double> *,
                                       const cplx<double> *, int, hipStream_t, bool, int, const PlaneMean &);
template hipError_t launch_yinv<double>(int, int, int, double *, size_t, const cplx<double> *,
                                        const cplx<double> *, int, hipStream_t, bool, int);
template hipError_t launch_yinv<float>(int, int, int, float *, size_t, const cplx<double> *,
                                       const cplx<double> *, int, hipStream_t, bool, int);

}  // namespace pf
