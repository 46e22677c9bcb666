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
// Kernels of one length: the register engine (k_yr) or the LDS engine (k_yfwd,
// k_yinv).
template <typename T, int N, bool INV, int YW, bool XR>
hipError_t y_launch(int nx, int nz, T *data, size_t sp, const cplx<double> *tw, const cplx<double> *ctw,
                    const PlaneMean &pm, hipStream_t st) {
  if constexpr (y_in_regs<T>(N)) {
    constexpr int LPW = yr_lpw<T>(N), TPL = LinePlan<N>::tpl;
    if (nx % (2 * LPW) == 0) {
      const int nib = nx / (2 * LPW);
      hipLaunchKernelGGL((k_yr<T, N, LPW, INV, YW, XR>), dim3((unsigned)((long)nib * nz)), dim3(TPL * LPW), 0, st,
                         data, tw, ctw, nx, nib, sp, pm);
      return hipGetLastError();
    }
    // half the columns (48 slots, an x-face field of the shortest lines)
    if constexpr (LPW > 8) {
      if (nx % LPW) return hipErrorInvalidValue;
      const int nib = nx / LPW;
      hipLaunchKernelGGL((k_yr<T, N, LPW / 2, INV, YW, XR>), dim3((unsigned)((long)nib * nz)), dim3(TPL * LPW / 2),
                         0, st, data, tw, ctw, nx, nib, sp, pm);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  } else {
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

template <int N, bool INV>
static hipError_t y_grp_launch(GJobs &g, hipStream_t st) {
  constexpr bool kRegs = y_in_regs<float>(N);
  constexpr int TPL = kRegs ? rx_tpl(N) : y_tpl(N), LPW = kRegs ? yr_lpw<float>(N) : y_lpw<float>(N);
  for (int k = 0; k < g.count; ++k) {
    if (g.j[k].ny != N || g.j[k].nx % (2 * LPW)) return hipErrorInvalidValue;
    g.j[k].nblk = (unsigned)(g.j[k].nx / (2 * LPW) * g.j[k].nz);
  }
  hipLaunchKernelGGL((k_y_grp<N, TPL, LPW, INV>), grp_grid(g), dim3(TPL * LPW), 0, st, g);
  return hipGetLastError();
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
