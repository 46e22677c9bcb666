// The y transforms on the register engine (fft_regs.hpp): one workgroup per
// z plane and 2 LPW adjacent slots, LPW complex lines, lanes over the lines
// first. The same transforms and layouts as k_yfwd / k_yinv of
// fft_kernels.hpp (see there for the spectra, the walls' transforms and the
// slots 0 and 1).
//
// What bounds it: HBM where the rows are 64 bytes or more and two workgroups
// share a compute unit; for the long lines one workgroup's loads, exchanges
// and stores in sequence, and the short row segments (32 float32 bytes). The 864
// threads of 3456 points leave 128 registers each, of which the forward spills
// 18-20 (its radix 18 beside the slots 0 and 1), the others 2-22, and the
// walls' forward of 3200 points 5: 12-76 bytes of scratch a thread.
// Forward / inverse in ms on MI355X, before (LDS engine) and now:
//   float32  1024 points, 1024 x 1024 x 512   1.37 / 1.24 -> 0.90 / 0.93  (4.7 TB/s)
//   float32   512 points, 1024 x 512 x 512    0.49 / 0.48 -> 0.43 / 0.42  (5.0)
//   float32  3072 points, 3456 x 3072 x 30    1.53 / 1.54 -> 0.99 / 0.98  (2.6)
//   float32  3456 points, 3200 x 3456 x 28    1.54 / 1.50 -> 1.10 / 1.00  (2.3)
//   float64  3456 points, 3200 x 3456 x 28    1.83 / 1.81 -> 1.40 / 1.22  (3.8)
//   float64  2048 points, 1024 x 2048 x 128   1.17 / 1.16 -> 0.94 / 0.94  (4.6)
// Walls, the inverse with both rows of a mirror pair read twice and with every
// row read once (UnpairPlan; yr_unpair):
//   float32   512 points, 1024 x 512 x 512    0.568 -> 0.487
//   float64  1024 points, 1024 x 1024 x 256   0.919 -> 0.828, sine 1.164 -> 0.826
//   float64  3072 points, 3456 x 3072 x 30    1.55 -> 1.45
#pragma once
#include "fft_kernels.hpp"
#include "fft_regs.hpp"

namespace pf {

// The wall inverses that read every row once (ms at the head of this file).
// They start with radix 8 instead of 16, which takes a pass more at 192, 256
// and from 3072 points: 192, 384, 2048 and 3200 points lose by it (float32
// 0.189 -> 0.212, 0.497 -> 0.546, 0.757 -> 0.851, 0.800 -> 0.844 ms), and 3456
// float32 points (1.21 -> 1.24; float64 1.60 -> 1.54).
template <typename T>
constexpr bool yr_unpair(int n) {
  return n != 192 && n != 384 && n != 2048 && n != 3200 && (n != 3456 || sizeof(T) == 8);
}

// WALK: one of many blocks of a persistent workgroup. The thread's number is then
// made anew for each block, or the compiler keeps every address of the passes
// across the loop (up to 139 registers spilled).
template <typename T, int N, int LPW, bool INV, int YW, bool XR, bool WALK = false>
__device__ __forceinline__ void yr_body(T *data, const cplx<double> *__restrict__ tw,
                                        const cplx<double> *__restrict__ ctw, int nx, int nib, size_t sp,
                                        const PlaneMean &pm, unsigned bx_, unsigned gx_) {
  using C = cplx<double>;
  using L = LinePlan<N>;
  constexpr int NT = L::tpl * LPW, S = rx_stride(N, LPW);
  static_assert(NT >= 64, "a whole wave takes the plane mean");
  __shared__ double lds[LPW * S];
  int tid = threadIdx.x;
  if constexpr (WALK) asm volatile("" : "+v"(tid));
  const int l = tid % LPW, t = tid / LPW;
  const unsigned blk = xcd_block(bx_, gx_);
  const int ib = blk % nib;
  const long k = blk / nib;
  if (!INV && ib == 0) plane_mean(pm, (int)k, N);
  T *base = data + (size_t)k * sp + (size_t)ib * 2 * LPW;
  double *buf = lds + l * S;
  // row j + c: the part of the address that differs between the lanes is a
  // 32-bit offset from the row c of the workgroup's slots, which is uniform
  const unsigned nxu = (unsigned)nx, l2 = 2 * (unsigned)l;
  auto at = [&](int j, int c) { return ld2<T>(base + (size_t)c * nxu + ((unsigned)j * nxu + l2)); };
  auto put = [&](int j, int c, double x, double y) {
    st2<T>(base + (size_t)c * nxu + ((unsigned)j * nxu + l2), x, y);
  };
  if constexpr (YW == 3) {
    // the odd extension of rows 0..NR-2 (faces 1..NR-1), its own inverse
    constexpr int NR = N / 2;
    auto src = [&](int j, int c) {
      const int i = j + c;
      if (i == 0 || i == NR) return mkc<double>(0.0, 0.0);
      if (i < NR) return at(i - 1, 0);
      const C v = at(N - 1 - i, 0);
      return mkc<double>(-v.x, -v.y);
    };
    auto dst = [&](int j, int c, const C &v, int, int) {
      const int q = j + c;
      if (q >= 1 && q < NR) put(q - 1, 0, -v.y, v.x);
      else if (q == NR) put(NR - 1, 0, 0.0, 0.0);
    };
    typename RxFirst<L>::Regs v;
    rx_load<L>(v, t, src);
    rx_passes<L, 0, false>(buf, tw, t, v, false, dst);
    return;
  } else {
    if constexpr (YW == 0 && !XR) {
      // Slots 0 and 1, line 0 of the first workgroup of a plane (ib 0): the
      // line goes through the LDS as a whole (the arrays of two lines) to be
      // split into, or joined from, two packed real spectra. The passes are
      // the other workgroups' own code: a second copy of them took 9
      // registers more.
      static_assert(LPW >= 2, "a complex line in the LDS of two");
      double *zx = lds, *zy = lds + S;
      typename RxFirst<L>::Regs v;
      if constexpr (!INV) {
        rx_load<L>(v, t, at);
        const bool line0 = ib == 0 && l == 0;
        rx_passes<L, 0, false>(buf, tw, t, v, ib == 0, [&](int j, int c, const C &x, int, int) {
          if (line0) {
            zx[j + c] = x.x;
            zy[j + c] = x.y;
          } else {
            put(j, c, x.x, x.y);
          }
        });
        if (ib != 0) return;
        __syncthreads();
        for (int q = tid; q < N / 2; q += NT) {
          C r0 = mkc<double>(zx[0], zy[0]), r1 = mkc<double>(zx[N / 2], zy[N / 2]);
          if (q != 0) {
            C A, B;
            split_pair<double>(mkc<double>(zx[q], zy[q]), mkc<double>(zx[N - q], zy[N - q]), A, B);
            r0 = mkc<double>(A.x, B.x);
            r1 = mkc<double>(A.y, B.y);
          }
          st2<T>(base + (size_t)(2 * q) * nxu, r0.x, r0.y);
          st2<T>(base + (size_t)(2 * q + 1) * nxu, r1.x, r1.y);
        }
      } else {
        if (ib != 0) {
          rx_load<L>(v, t, at);
        } else {
          for (int q = tid; q < N / 2; q += NT) {
            const C r0 = ld2<T>(base + (size_t)(2 * q) * nxu), r1 = ld2<T>(base + (size_t)(2 * q + 1) * nxu);
            C zq = r0, zn = r1;
            if (q != 0) join_pair<double>(mkc<double>(r0.x, r1.x), mkc<double>(r0.y, r1.y), zq, zn);
            const int n = q == 0 ? N / 2 : N - q;
            zx[q] = zq.x;
            zy[q] = zq.y;
            zx[n] = zn.x;
            zy[n] = zn.y;
          }
          __syncthreads();
          if (l == 0) rx_load<L>(v, t, [&](int j, int c) { return mkc<double>(zx[j + c], zy[j + c]); });
          else rx_load<L>(v, t, at);
          __syncthreads();
        }
        rx_passes<L, 0, true>(buf, tw, t, v, false,
                              [&](int j, int c, const C &x, int, int) { put(j, c, x.x, x.y); });
      }
      return;
    } else {
    // walls in y (or in x, XR): every line's spectrum is folded with its
    // mirror image. Forward, a thread of the PAIR transform holds both
    // positions; inverse, a thread of the UNPAIR transform does, or it reads
    // both rows (the second time from cache; packed spectra always).
    if constexpr (!INV) {
      using Q = PairPlan<N>;
      typename RxFirst<Q>::Regs v;
      rx_load<Q>(v, t, [&](int j, int c) {
        if constexpr (YW == 0) {
          return at(j, c);
        } else {
          const int n = j + c, y = n < N / 2 ? 2 * n : 2 * N - 1 - 2 * n;
          const C x = at(y, 0);
          return (YW == 2 && (y & 1)) ? mkc<double>(-x.x, -x.y) : x;
        }
      });
      rx_passes<Q, 0, false, kPair>(buf, tw, t, v, false, [&](int j, int c, const C &x, const C &m, int, int r) {
        const int q = j + c;
        if constexpr (YW == 0) {
          constexpr int H = 4;  // positions q <= N/2, the half of the last pass's radix
          if (r > H) return;
          if (q == 0 || 2 * q == N) {
            put(q == 0 ? 0 : 1, 0, x.x, x.y);
          } else if (r < H) {
            C A, B;
            split_pair<double>(x, m, A, B);
            put(2 * q, 0, A.x, B.x);
            put(2 * q + 1, 0, A.y, B.y);
          }
        } else {
          const C w = ctw[q];
          put(YW == 2 ? N - 1 - q : q, 0, w.x * x.x - w.y * x.y + w.x * m.x + w.y * m.y,
              w.x * x.y + w.y * x.x + w.x * m.y - w.y * m.x);
        }
      });
    } else if constexpr (YW == 0) {
      typename RxFirst<L>::Regs v;
      rx_load<L>(v, t, [&](int j, int c) {
        // position n of the joined packed real spectra
        const int n = j + c, q = n <= N / 2 ? n : N - n;
        if (q == 0 || 2 * q == N) return at(q == 0 ? 0 : 1, 0);
        const C r0 = at(2 * q, 0), r1 = at(2 * q + 1, 0);
        const double s = 2 * n < N ? 1.0 : -1.0;
        return mkc<double>(r0.x - s * r1.y, r0.y + s * r1.x);
      });
      rx_passes<L, 0, true>(buf, tw, t, v, false, [&](int j, int c, const C &x, int, int) { put(j, c, x.x, x.y); });
    } else {
      // the wall's rows: position n takes conj(c_n) (X_n - i X_{N-n}) / 2, X_N = 0
      auto dst = [&](int j, int c, const C &x, int, int) {
        const int n = j + c, y = n < N / 2 ? 2 * n : 2 * N - 1 - 2 * n;
        const double sg = (YW == 2 && (y & 1)) ? -1.0 : 1.0;
        put(y, 0, sg * x.x, sg * x.y);
      };
      if constexpr (!yr_unpair<T>(N)) {
        typename RxFirst<L>::Regs v;
        rx_load<L>(v, t, [&](int j, int c) {
          const int n = j + c;
          const C x = at(YW == 2 ? N - 1 - n : n, 0), w = ctw[n];
          const C z = n == 0 ? mkc<double>(0.0, 0.0) : at(YW == 2 ? n - 1 : N - n, 0);
          const double ur = 0.5 * (x.x + z.y), ui = 0.5 * (x.y - z.x);
          return mkc<double>(w.x * ur + w.y * ui, w.x * ui - w.y * ur);
        });
        rx_passes<L, 0, true>(buf, tw, t, v, false, dst);
      } else {
        // every row read once: the mirror image of butterfly j, position r, is
        // N/8 - j, position 7 - r; that of butterfly 0 is its own position
        // 8 - r, that of N/16 (the other one of thread 0) its own 7 - r
        using Q = UnpairPlan<N>;
        constexpr int NB = N / 8;
        cplx<T> X[2][8];
        typename RxFirst<Q>::Regs v;
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int j = rx_butterfly<Q, 0, kUnpair>(t, it);
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const C x = YW == 2 ? at(NB - 1 - j, (7 - r) * NB) : at(j, r * NB);
            X[it][r] = mkc<T>((T)x.x, (T)x.y);
          }
        }
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int j = rx_butterfly<Q, 0, kUnpair>(t, it);
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const cplx<T> x = X[it][r], m = X[1 - it][7 - r], o = X[it][(it ? 7 - r : 8 - r) % 8];
            const bool none = it == 0 && r == 0 && t == 0;
            const T zx = none ? T(0) : t ? m.x : o.x, zy = none ? T(0) : t ? m.y : o.y;
            const C w = ctw[j + r * NB];
            const double ur = 0.5 * ((double)x.x + zy), ui = 0.5 * ((double)x.y - zx);
            v[it][r] = mkc<double>(w.x * ur + w.y * ui, w.x * ui - w.y * ur);
          }
        }
        rx_passes<Q, 0, true, kUnpair>(buf, tw, t, v, false, dst);
      }
    }
    }
  }
}

template <typename T, int N, int LPW, bool INV, int YW, bool XR>
__global__ __launch_bounds__(LinePlan<N>::tpl *LPW) void k_yr(T *data, const cplx<double> *__restrict__ tw,
                                                               const cplx<double> *__restrict__ ctw, int nx,
                                                               int nib, size_t sp, PlaneMean pm) {
  yr_body<T, N, LPW, INV, YW, XR>(data, tw, ctw, nx, nib, sp, pm, blockIdx.x, gridDim.x);
}
// The same for a grid of at most one round of resident workgroups, which
// walk the blocks; nothing of a block outlives its turn, and nothing is loaded
// ahead. The plane means come before the walk, whose registers they would add
// to.
template <typename T, int N, int LPW, bool INV>
__global__ __launch_bounds__(LinePlan<N>::tpl *LPW) void k_yr_persist(T *data, const cplx<double> *__restrict__ tw,
                                                                       int nx, int nib, size_t sp, unsigned nblk,
                                                                       PlaneMean pm) {
  if (!INV) plane_means(pm, (int)(nblk / nib), N);
  for (unsigned b = blockIdx.x; b < nblk; b += gridDim.x) {  // uniform
    yr_body<T, N, LPW, INV, 0, false, true>(data, tw, nullptr, nx, nib, sp, PlaneMean{}, b, nblk);
    __syncthreads();
  }
}

}  // namespace pf
