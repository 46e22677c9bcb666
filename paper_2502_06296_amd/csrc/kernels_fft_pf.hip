// Persistent launches of the periodic y transforms: one round of resident
// workgroups that walk the blocks (k_yr_persist of fft_y.hpp; k_y_persist of
// fft_kernels.hpp, which prefetches the next block's rows during the current
// block's passes). The autotuner's y transform shape kYPersistShape.
#include "fft_y.hpp"
#include "pf_internal.hpp"

namespace pf {

namespace {
template <typename T, int N, bool INV>
hipError_t y_persist_one(int nx, int nz, T *data, size_t sp, const cplx<double> *tw, hipStream_t st,
                         const PlaneMean &pm) {
  constexpr bool kRegs = y_in_regs<T>(N);
  constexpr int TPL = kRegs ? rx_tpl(N) : y_tpl(N), LPW = kRegs ? yr_lpw<T>(N) : y_lpw<T>(N);
  if (nx % (2 * LPW)) return hipErrorInvalidValue;
  const int nib = nx / (2 * LPW);
  const long nblk = (long)nib * nz;
  if (nblk <= 0) return hipSuccess;
  int occ = 0;
  hipError_t e;
  if constexpr (kRegs)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_yr_persist<T, N, LPW, INV>, TPL * LPW, 0);
  else
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_y_persist<T, N, TPL, LPW, INV>, TPL * LPW, 0);
  if (e != hipSuccess) return e;
  const int cus = device_cus();
  if (occ < 1 || cus < 1) return hipErrorInvalidValue;
  const long G = nblk < (long)cus * occ ? nblk : (long)cus * occ;
  if constexpr (kRegs)
    hipLaunchKernelGGL((k_yr_persist<T, N, LPW, INV>), dim3((unsigned)G), dim3(TPL * LPW), 0, st, data, tw, nx, nib,
                       sp, (unsigned)nblk, pm);
  else
    hipLaunchKernelGGL((k_y_persist<T, N, TPL, LPW, INV>), dim3((unsigned)G), dim3(TPL * LPW), 0, st, data, tw, nx,
                       nib, sp, nblk, pm);
  return hipGetLastError();
}
}  // namespace

template <typename T>
hipError_t launch_y_persist(bool inv, int nx, int ny, int nz, T *data, size_t sp, const cplx<double> *tw,
                            hipStream_t st, const PlaneMean &pm) {
  switch (ny) {
#define PF_CASE(N)                                                                               \
  case N:                                                                                        \
    return inv ? y_persist_one<T, N, true>(nx, nz, data, sp, tw, st, pm)                         \
               : y_persist_one<T, N, false>(nx, nz, data, sp, tw, st, pm);
    PF_FOR_FFT_SIZES_Y(PF_CASE)
#undef PF_CASE
    default:
      return hipErrorInvalidValue;
  }
}

template hipError_t launch_y_persist<double>(bool, int, int, int, double *, size_t, const cplx<double> *,
                                             hipStream_t, const PlaneMean &);
template hipError_t launch_y_persist<float>(bool, int, int, int, float *, size_t, const cplx<double> *,
                                            hipStream_t, const PlaneMean &);

}  // namespace pf
