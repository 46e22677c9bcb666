// The x transforms (periodic) and the refinement residual on the register
// engine (fft_regs.hpp): LPW pairs of lines per workgroup, the lanes along the
// line. The same transforms and layouts as k_xfwd, k_resid_spec and k_xinv of
// fft_kernels.hpp (see there for the spectra). The forward ends with the
// positions q and N - q in one thread (PairPlan), so the split into the two
// lines' spectra needs no further exchange, and the inverse starts with both
// in one thread (UnpairPlan).
//
// Bound by HBM at the copy rate, but for the longest lines (4 passes) and the
// residual (the latency of its neighbour loads). ms on MI355X, LDS engine and
// this one (float32 inverse: of two spectra; x_fwd_in_regs, x_inv_in_regs and
// resid_in_regs say which lengths are left to the LDS engine):
//   forward  float32  1024 x 512 x 512  0.625 -> 0.600 (5.4 TB/s)   3456 x 3072 x 30  1.16 -> 0.85
//            float64  3200 x 3456 x 28  1.20 -> 0.98                2048 x 1024 x 128  0.757 -> 0.764
//   inverse  float32  1024 x 512 x 512  0.806 -> 0.739 (5.8 TB/s)   3456 x 3072 x 30  1.50 -> 1.07
//            float64  3200 x 3456 x 28  1.05 -> 0.93                1024 x 512 x 512  0.742 -> 0.798
//   divergence float64  1024 x 512 x 256  1.152 -> 0.816 (5.3 TB/s)   3200 x 3456 x 28  5.68 -> 2.32
//            refined  512 x 512 x 512  1.326 -> 0.928 (5.2 TB/s)   3456 x 1024 x 30  1.76 -> 0.82
//            (192 x 96 x 100 0.025 -> 0.028, refined 0.025 -> 0.031: the LDS engine stays there)
//   residual          512 x 512 x 512   0.580 -> 0.513              3456 x 3072 x 30  2.22 -> 1.59
//                     1024 x 512 x 512  1.049 -> 1.042              1536 x 512 x 256  0.846 -> 0.876
#pragma once
#include "fft_kernels.hpp"
#include "fft_regs.hpp"

namespace pf {

// LDS stride between lines: two lines within 32 lanes (16 threads a line) in
// different halves of the bank pairs
constexpr int xr_stride(int n) {
  int s = rx_idx(n);
  while (n / 16 < 32 && s % 32 != 16) ++s;
  return s;
}

// The forward transform of a line pair from src(i) (position i of the two
// lines as one complex value), handed on as out(q, Z_q, Z_{N-q}, r), q the
// positions 0..N-1 of the thread, r below 4 for q < N/2.
template <int N, class Src, class Out>
__device__ __forceinline__ void xr_forward(double *buf, const cplx<double> *__restrict__ tw, int t, Src src, Out out) {
  using Q = PairPlan<N>;
  typename RxFirst<Q>::Regs v;
  rx_load<Q>(v, t, [&](int j, int c) { return src(j + c); });
  rx_passes<Q, 0, false, kPair>(buf, tw, t, v, false,
                                [&](int j, int c, const cplx<double> &x, const cplx<double> &m, int, int r) {
                                  out(j + c, x, m, r);
                                });
}

// The two spectra of pair c from src, packed as in k_xfwd, into out; c past
// the last pair (ok false) stores nothing.
template <typename T, int N, class Src>
__device__ __forceinline__ void xr_pair(double *buf, T *__restrict__ out, const cplx<double> *__restrict__ tw,
                                        double *__restrict__ sums, long c, int ny, size_t sp, int t, bool ok,
                                        Src src) {
  using C = cplx<double>;
  T *oa = out + (size_t)(2 * c / ny) * sp + (size_t)(2 * c % ny) * N;
  T *ob = oa + N;
  xr_forward<N>(buf, tw, t, src, [&](int q, const C &z, const C &m, int r) {
    if (!ok) return;
    if (r < 4 && q != 0) {
      C A, B;
      split_pair<double>(z, m, A, B);
      st2<T>(oa + 2 * q, A.x, A.y);
      st2<T>(ob + 2 * q, B.x, B.y);
    } else if (q == 0) {
      oa[0] = (T)z.x;
      ob[0] = (T)z.y;
      // the float64 zero mode of each line is its sum
      sums[2 * c] = z.x;
      sums[2 * c + 1] = z.y;
    } else if (2 * q == N) {
      oa[1] = (T)z.x;
      ob[1] = (T)z.y;
    }
  });
}

template <typename T, int N, int LPW>
__device__ __forceinline__ void xr_fwd_body(const double *__restrict__ in, T *__restrict__ out,
                                            const cplx<double> *__restrict__ tw, double *__restrict__ sums, long ncl,
                                            int ny, size_t sp, unsigned bx_) {
  constexpr int TPL = LinePlan<N>::tpl;
  __shared__ double lds[LPW * xr_stride(N)];
  const int l = threadIdx.x / TPL, t = threadIdx.x % TPL;
  const long c = (long)bx_ * LPW + l;
  const bool ok = c < ncl;
  // a workgroup's lines past the last pair transform the last pair again
  const long cc = ok ? c : ncl - 1;
  const double *a = in + (size_t)(2 * cc) * N, *b = a + N;
  xr_pair<T, N>(lds + l * xr_stride(N), out, tw, sums, cc, ny, sp, t, ok,
                [&](int i) { return mkc<double>(a[i], b[i]); });
}
template <typename T, int N, int LPW>
__global__ __launch_bounds__(LinePlan<N>::tpl *LPW) void k_xr_fwd(const double *__restrict__ in,
                                                                   T *__restrict__ out,
                                                                   const cplx<double> *__restrict__ tw,
                                                                   double *__restrict__ sums, long ncl, int ny,
                                                                   size_t sp) {
  xr_fwd_body<T, N, LPW>(in, out, tw, sums, ncl, ny, sp, blockIdx.x);
}

// The forward of a projection's right-hand side, formed as the positions are
// read (as k_xfwd_div, periodic x). It has eleven reads per position pair:
// half the LDS of k_xfwd_div gives twice the waves, and all of a position's
// reads are unconditional (past a wall the line itself is read and its value
// dropped), so they are in flight together; the pass then runs at the copy
// rate of its 32 (refined 36) bytes a point, but for the longest lines.
template <typename T, int N, int LPW, bool STASH>
__global__ __launch_bounds__(LinePlan<N>::tpl *LPW) void k_xr_div(DivArgs d, T *__restrict__ out,
                                                                   const cplx<double> *__restrict__ tw,
                                                                   double *__restrict__ sums, long ncl, int ny,
                                                                   int nz, size_t sp) {
  constexpr int TPL = LinePlan<N>::tpl;
  __shared__ double lds[LPW * xr_stride(N)];
  const int l = threadIdx.x / TPL, t = threadIdx.x % TPL;
  const long c = (long)blockIdx.x * LPW + l;
  const bool ok = c < ncl;
  const long cc = ok ? c : ncl - 1;
  const int k = (int)(2 * cc / ny), j = (int)(2 * cc % ny);
  const size_t o = (size_t)(2 * cc) * N;
  const bool top = k < nz - 1, bot = k > 0, south = !(d.ywalls && j == 0), north = !(d.ywalls && j + 2 == ny);
  const double *u = d.u + o, *v = d.v + o;
  const double *vm = d.v + ((size_t)k * ny + (j == 0 ? ny - 1 : j - 1)) * N;
  const double *wt = top ? d.w + o : u, *wb = bot ? d.w + (o - (size_t)ny * N) : u;
  const double rz = d.rdzf[k];
  double *f = STASH ? d.stash + o : nullptr;
  xr_pair<T, N>(lds + l * xr_stride(N), out, tw, sums, cc, ny, sp, t, ok, [&](int i) {
    const int im = i == 0 ? N - 1 : i - 1;
    const double v0 = v[i], vs = vm[i], vn = v[N + i], ta = wt[i], tb = wt[N + i], ba = wb[i], bb = wb[N + i];
    double fa = (u[i] - u[im]) * d.idx + (v0 - (south ? vs : 0.0)) * d.idy;
    double fb = (u[N + i] - u[N + im]) * d.idx + ((north ? vn : 0.0) - v0) * d.idy;
    fa = (fa + (top ? ta : 0.0) * rz - (bot ? ba : 0.0) * rz) * d.igdt;
    fb = (fb + (top ? tb : 0.0) * rz - (bot ? bb : 0.0) * rz) * d.igdt;
    if (STASH && ok) {
      f[i] = fa;
      f[N + i] = fb;
    }
    return mkc<double>(fa, fb);
  });
}

// ------------------------------------------------------------- x inverse
// in and out may be the same array: a workgroup reads its lines before the
// first exchange and writes them after the last.
template <typename TS, typename TO, int N, int LPW, bool SUM2>
__device__ __forceinline__ void xr_inv_body(const TS *in, TO *out, const cplx<double> *__restrict__ tw,
                                            const double *__restrict__ zm, const TS *in2, double scale, int ny,
                                            long ncl, size_t sp, unsigned long long *__restrict__ stat,
                                            unsigned bx_) {
  using C = cplx<double>;
  using L = UnpairPlan<N>;
  constexpr int TPL = L::tpl, NB = N / 8;
  __shared__ double lds[LPW * xr_stride(N)];
  const int l = threadIdx.x / TPL, t = threadIdx.x % TPL;
  const long c = (long)bx_ * LPW + l;
  const bool ok = c < ncl;
  const long cc = ok ? c : ncl - 1;
  const size_t o = (size_t)(2 * cc / ny) * sp + (size_t)(2 * cc % ny) * N;
  double m0 = 0.0, m1 = 0.0;  // largest |iterate| and |correction| seen (SUM2)
  // slots s, s + 1 of line h of the pair (two spectra summed in float64)
  auto two = [&](int h, int s) {
    C v = ld2<TS>(in + o + h * N + s);
    if constexpr (SUM2) {
      const C w = ld2<TS>(in2 + o + h * N + s);
      m0 = fmax(m0, fmax(fabs(v.x), fabs(v.y)));
      m1 = fmax(m1, fmax(fabs(w.x), fabs(w.y)));
      v = mkc<double>(v.x + w.x, v.y + w.y);
    }
    return v;
  };
  // Z_q = A_q + i B_q and Z_{N-q} from the conjugates, q the thread's four
  // lower positions of each of its two butterflies; the pair of slots 0 and 1
  // (q = 0) holds the positions 0 and N/2
  typename RxFirst<L>::Regs v;
  C zn[2][4];
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int j = rx_butterfly<L, 0, kUnpair>(t, it);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const C A = two(0, 2 * (j + r * NB)), B = two(1, 2 * (j + r * NB));
      join_pair<double>(A, B, v[it][r], zn[it][r]);
      if (it == 0 && r == 0 && t == 0) {
        v[0][0] = mkc<double>(A.x, B.x);
        zn[0][0] = mkc<double>(A.y, B.y);
      }
    }
  }
  // the mirror image of butterfly j, position r, is N/8 - j, position 7 - r;
  // that of butterfly 0 is its own position 8 - r
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const C own = zn[0][(r + 1) % 4];
    v[1][7 - r] = mkc<double>(t ? zn[0][r].x : zn[1][r].x, t ? zn[0][r].y : zn[1][r].y);
    v[0][7 - r] = mkc<double>(t ? zn[1][r].x : own.x, t ? zn[1][r].y : own.y);
  }
  if (SUM2 && stat) {  // uniform: the a-posteriori estimate of the refinement
    for (int s = 32; s > 0; s >>= 1) {
      m0 = fmax(m0, __shfl_xor(m0, s));
      m1 = fmax(m1, __shfl_xor(m1, s));
    }
    if ((threadIdx.x & 63) == 0) {
      atomicMax(stat, (unsigned long long)__double_as_longlong(m0));
      atomicMax(stat + 1, (unsigned long long)__double_as_longlong(m1));
    }
  }
  const double add = zm[(2 * cc) / ny];
  TO *oa = out + (size_t)(2 * cc) * N;
  TO *ob = oa + N;
  rx_passes<L, 0, true, kUnpair>(lds + l * xr_stride(N), tw, t, v, false, [&](int j, int k, const C &z, int, int) {
    if (!ok) return;
    oa[j + k] = (TO)(z.x * scale + add);
    ob[j + k] = (TO)(z.y * scale + add);
  });
}
template <typename TS, typename TO, int N, int LPW, bool SUM2>
__global__ __launch_bounds__(LinePlan<N>::tpl *LPW) void k_xr_inv(const TS *in, TO *out,
                                                                   const cplx<double> *__restrict__ tw,
                                                                   const double *__restrict__ zm, const TS *in2,
                                                                   double scale, int ny, long ncl, size_t sp,
                                                                   unsigned long long *__restrict__ stat) {
  xr_inv_body<TS, TO, N, LPW, SUM2>(in, out, tw, zm, in2, scale, ny, ncl, sp, stat, blockIdx.x);
}

// ------------------------------ residual of the correction in x-spectral space
// One position's neighbour loads at a time (kFence) for the lengths up to 512
// and the powers of two, whose registers then leave a wave more; the longer
// mixed lengths lose by it (3456 points 1.59 -> 1.75 ms).
template <int N, int LPW>
__device__ __forceinline__ void xr_resid_body(const double *__restrict__ f, const double *__restrict__ fbar,
                                              const float *__restrict__ W, float *__restrict__ out,
                                              const cplx<double> *__restrict__ tw, double *__restrict__ sums_p,
                                              const double *__restrict__ sx, const double *__restrict__ zal,
                                              const double *__restrict__ zga, const double *__restrict__ zex, int ny,
                                              int nz, double idy2, double inv_ny, int ywalls, size_t sp,
                                              unsigned bx_, unsigned gx_) {
  using C = cplx<double>;
  constexpr int TPL = LinePlan<N>::tpl;
  constexpr bool kFence = N <= 512 || (N & (N - 1)) == 0;
  __shared__ double lds[LPW * xr_stride(N)];
  const int l = threadIdx.x / TPL, t = threadIdx.x % TPL;
  // block order, ghost rows: as in resid_spec_body
  const unsigned b = xcd_block(bx_, gx_);
  const int njg = ny / (2 * LPW);
  const long per = (long)kResidPlanes * njg;
  const int k0 = (int)(b / per) * kResidPlanes;
  const int sz = nz - k0 < kResidPlanes ? nz - k0 : kResidPlanes;
  const long rem = (long)b - (long)(k0 / kResidPlanes) * per;
  const int k = k0 + (int)(rem % sz), j = (int)(rem / sz) * 2 * LPW + 2 * l;
  const double *fa = f + ((size_t)k * ny + j) * N, *fb = fa + N;
  const double ak = zal[k], gk = zga[k], dk = ak + gk + zex[k], fk = (double)N * fbar[k];
  const int jm = j == 0 ? (ywalls ? 0 : ny - 1) : j - 1;
  const int jp = j + 2 == ny ? (ywalls ? ny - 1 : 0) : j + 2;
  const double gm = j == 0 ? (ywalls == 2 ? -1.0 : ywalls == 3 ? 0.0 : 1.0) : 1.0;
  const double gp = j + 2 == ny ? (ywalls == 2 ? -1.0 : ywalls == 3 ? 0.0 : 1.0) : 1.0;
  const float *w0 = W + (size_t)k * sp + (size_t)j * N;
  // the planes below and above; past a wall the plane itself, whose
  // coefficient is zero there (alpha_0 = gamma_{nz-1} = 0)
  const float *wd = k > 0 ? w0 - sp : w0, *wu = k < nz - 1 ? w0 + sp : w0;
  const float *wm = W + (size_t)k * sp + (size_t)jm * N, *wp = W + (size_t)jp * N + (size_t)k * sp;
  float *oa = out + (size_t)k * sp + (size_t)j * N;
  // R of one slot of the two lines: (A, B) the transform of f, s the shift,
  // the iterate's rows j, j+1 (c), j-1 and j+2 (m, p), planes k-1 (a), k+1 (g)
  struct Row {
    double c0, c1, m, p, a0, a1, g0, g1;
  };
  auto line = [&](double A, double B, double s, const Row &w, double &ra, double &rb) {
    ra = A - inv_ny * ((gm * w.m - 2.0 * w.c0 + w.c1) * idy2 + (ak * w.a0 + gk * w.g0) - (dk + s) * w.c0);
    rb = B - inv_ny * ((w.c0 - 2.0 * w.c1 + gp * w.p) * idy2 + (ak * w.a1 + gk * w.g1) - (dk + s) * w.c1);
  };
  auto put1 = [&](int s, double A, double B) {
    const Row w{w0[s], w0[N + s], wm[s], wp[s], wd[s], wd[N + s], wu[s], wu[N + s]};
    double ra, rb;
    line(A, B, sx[s], w, ra, rb);
    oa[s] = (float)ra;
    oa[N + s] = (float)rb;
    if (s == 0) {  // the iterate's line sums
      sums_p[(size_t)k * ny + j] = w.c0 * inv_ny;
      sums_p[(size_t)k * ny + j + 1] = w.c1 * inv_ny;
    }
  };
  xr_forward<N>(
      lds + l * xr_stride(N), tw, t, [&](int i) { return mkc<double>(fa[i], fb[i]); },
      [&](int q, const C &z, const C &m, int r) {
        if (r < 4 && q != 0) {
          C A, B;
          split_pair<double>(z, m, A, B);
          const int s = 2 * q;
          const C c0 = ld2<float>(w0 + s), c1 = ld2<float>(w0 + N + s), cm = ld2<float>(wm + s),
                  cp = ld2<float>(wp + s), a0 = ld2<float>(wd + s), a1 = ld2<float>(wd + N + s),
                  g0 = ld2<float>(wu + s), g1 = ld2<float>(wu + N + s);
          double ra0, ra1, rb0, rb1;
          line(A.x, B.x, sx[s], Row{c0.x, c1.x, cm.x, cp.x, a0.x, a1.x, g0.x, g1.x}, ra0, rb0);
          line(A.y, B.y, sx[s + 1], Row{c0.y, c1.y, cm.y, cp.y, a0.y, a1.y, g0.y, g1.y}, ra1, rb1);
          st2<float>(oa + s, ra0, ra1);
          st2<float>(oa + N + s, rb0, rb1);
          if (kFence) __builtin_amdgcn_sched_barrier(0);
        } else if (q == 0) {
          put1(0, z.x - fk, z.y - fk);
        } else if (2 * q == N) {
          put1(1, z.x, z.y);
        }
      });
}
template <int N, int LPW>
__global__ __launch_bounds__(LinePlan<N>::tpl *LPW) void k_xr_resid(
    const double *__restrict__ f, const double *__restrict__ fbar, const float *__restrict__ W,
    float *__restrict__ out, const cplx<double> *__restrict__ tw, double *__restrict__ sums_p,
    const double *__restrict__ sx, const double *__restrict__ zal, const double *__restrict__ zga,
    const double *__restrict__ zex, int ny, int nz, double idy2, double inv_ny, int ywalls, size_t sp) {
  xr_resid_body<N, LPW>(f, fbar, W, out, tw, sums_p, sx, zal, zga, zex, ny, nz, idy2, inv_ny, ywalls, sp, blockIdx.x,
                        gridDim.x);
}

}  // namespace pf
