// Wall-normal solves (paper Sec. 2.2.3 steps 4-6, Sec. 2.2.4, Algorithm 2).
//
// Both the Poisson z solve and the Helmholtz apply use the partition method
// of the paper inside one workgroup: each column of N_z unknowns is cut into
// P chunks, one thread per chunk holds its m = N_z/P values in registers,
// reduces them to the two boundary rows of the chunk, the 2P boundary rows of
// every column form a tridiagonal system that is solved by parallel cyclic
// reduction in LDS, and each thread rebuilds its interior. Where the paper
// exchanges the boundary rows between GPUs with an all-to-all, here they only
// cross the LDS of one compute unit.
//
// All rows are sign-normalised M-matrix rows
//   -alpha x[k-1] + (alpha + gamma + eps) x[k] - gamma x[k+1] = d,
// alpha, gamma, eps >= 0, and every elimination keeps each diagonal as a sum
// of non-negative parts (a forward excess, a backward excess), so no pivot is
// ever formed by subtraction.
#include "pf_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace pf {

// ----------------------------------------------------------- zero mode
// The (0,0) slot of the transformed problem is the plane-mean profile of p:
// the plane means fbar projected onto the range of L_z (zero dzf-weighted
// mean c removed), the singular Neumann system, zero dzf-weighted mean. Its
// rows have no excess, so each of them is a flux balance,
//   gamma_k dzf_k (m[k+1] - m[k]) = sum_{i<=k} dzf_i (fbar_i - c),
// and the solve is two running sums: the fluxes, then m from its
// differences. One wave does both, 16 rows a lane at most (nz <= 1024),
// with shuffles and no LDS, in a workgroup of its own in front of the z
// solve's. What bounds it is latency: as a launch of one thread's serial
// sweeps it took 16 us at 64 planes and 60 us at 512 (and the plane means
// another launch of 3-5 us); inside the z solve its few microseconds run
// beside the columns.
__device__ __forceinline__ double lane_sum(double v, int lanes) {
  for (int o = lanes / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
// the sum of v over the lanes below this one
__device__ __forceinline__ double lane_before(double v, int lanes) {
  const int lane = threadIdx.x;
  double s = v;
  for (int o = 1; o < lanes; o <<= 1) {
    const double t = __shfl_up(s, o);
    if (lane >= o) s += t;
  }
  const double b = __shfl_up(s, 1);
  return lane ? b : 0.0;
}
// Rows of a lane at most: nz <= 1024 over 64 lanes, and the z solve's smaller
// workgroups (P chunks of M <= 16 rows, P TP threads with TP >= 4) leave half
// of their threads or more: at most 2 M / TP rows each.
constexpr int kZeroRows = 16;
__device__ __forceinline__ void zero_solve(const ZeroJob &z, const double *zga, int nz) {
  // the first 64 threads, or as many as a power of two of a smaller workgroup
  int lanes = 64;
  while (lanes > (int)blockDim.x) lanes >>= 1;
  if ((int)threadIdx.x >= lanes) return;
  const int rows = (nz + lanes - 1) / lanes, r0 = (int)threadIdx.x * rows;
  double w = 0.0, wf = 0.0;
  for (int q = 0; q < rows; ++q)
    if (r0 + q < nz) {
      w += z.dzf[r0 + q];
      wf += z.dzf[r0 + q] * z.fbar[r0 + q];
    }
  const double wt = lane_sum(w, lanes), c = lane_sum(wf, lanes) / wt;
  double fl = 0.0;
  for (int q = 0; q < rows; ++q)
    if (r0 + q < nz) fl += z.dzf[r0 + q] * (z.fbar[r0 + q] - c);
  double g = lane_before(fl, lanes), x = 0.0, wm = 0.0;
  double xs[kZeroRows];
#pragma unroll
  for (int q = 0; q < kZeroRows; ++q) {
    xs[q] = x;
    const int r = r0 + q;
    if (q < rows && r < nz) {
      const double d = z.dzf[r];
      wm += d * x;
      g += d * (z.fbar[r] - c);
      if (r + 1 < nz) x += g / (zga[r] * d);
    }
  }
  const double x0 = lane_before(x, lanes);
  const double shift = lane_sum(wm + w * x0, lanes) / wt;
#pragma unroll
  for (int q = 0; q < kZeroRows; ++q)
    if (q < rows && r0 + q < nz) z.m[r0 + q] = x0 + xs[q] - shift;
}

// ------------------------------------------------------- Poisson z solve
// Thread (col, ch): column i = ib*TI + col of plane j, rows [ch*M, ch*M+M)
// of the column. Columns are padded to P*M rows with identity rows (alpha =
// gamma = 0, excess = 1), which decouple exactly because the last real row
// has gamma = 0; the padding keeps every loop and register index a compile-
// time constant. The chunk's Step 1 coefficients depend on the column's
// shift lambda = sx[i] + sy[j] (the modified wavenumbers; sy holds the
// packed-slot values for the x slots 0 and 1 and, from index ny on, the
// values of the natural-order complex y modes of the other slot pairs), so
// they are
// rebuilt in registers: an upward sweep gives the reduced first row, a
// downward sweep (Algorithm 2, Step 1 and the forward half of Step 2, fused)
// gives the reduced last row and leaves the forward-reduced d and the pivots
// 1/b. After the reduced solve the interior follows from one forward and one
// backward substitution with the chunk's end values as Dirichlet data.
// 1/b for the positive, normal pivots of the eliminations: the hardware
// reciprocal refined by two Newton steps (about 1 ulp), a third of the
// instructions of an IEEE division.
__device__ __forceinline__ double rcp64(double b) {
  double r = __builtin_amdgcn_rcp(b);
  double e = __builtin_fma(-b, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-b, r, 1.0);
  return __builtin_fma(r, e, r);
}
// A compiler memory fence every fourth row of an unrolled sweep: the
// compiler would otherwise issue every table and field read of the sweep up
// front and run out of registers. It emits no instruction.
__device__ __forceinline__ void sched_fence(int q) {
  if ((q & 3) == 3) asm volatile("" ::: "memory");
}

template <bool FAST>
__device__ __forceinline__ double qdiv(double a, double b) {
  if constexpr (FAST) return a * rcp64(b);
  else return a / b;
}

template <typename TS, int M, int TI, int WAVES, bool FAST>
__global__ __launch_bounds__(512, WAVES) void k_zsolve(TS *__restrict__ data, int nx, int ny, int nz, int P,
                                                 const double *__restrict__ zal,
                                                 const double *__restrict__ zga,
                                                 const double *__restrict__ zex,
                                                 const double *__restrict__ sx,
                                                 const double *__restrict__ sy, size_t sp, ZeroJob zj) {
  unsigned bx_ = blockIdx.x, gx_ = gridDim.x;
  if (zj.m) {  // the first workgroup takes the zero mode
    if (bx_ == 0) return zero_solve(zj, zga, nz);
    --bx_;
    --gx_;
  }
  extern __shared__ double red[];  // [4][2P][TI]: alpha, gamma, eps, d of the reduced rows
  const int nr = 2 * P;
  double *RA = red, *RG = red + nr * TI, *RE = red + 2 * nr * TI, *RD = red + 3 * nr * TI;
  const int nib = nx / TI;
  const int blk = (int)xcd_block(bx_, gx_);
  const int ib = blk % nib;
  const int j = blk / nib;
  const int col = threadIdx.x % TI;
  const int ch = threadIdx.x / TI;
  const int i = ib * TI + col;
  const int r0 = ch * M;
  const size_t plane = sp;
  TS *cp = data + (size_t)j * nx + i + (size_t)r0 * plane;
  // the singular column is the one with no shift at all (Poisson's (0,0);
  // the 3-D Helmholtz has 1/s in every entry of sx)
  const double lam0 = sx[i] + sy[(i >= 2 ? ny : 0) + j];
  const bool zero_col = lam0 == 0.0;
  const double lam = zero_col ? 1.0 : lam0;
  const double *al = zal + r0, *ga = zga + r0, *ex = zex + r0;

  double d[M], ib_[M];
#pragma unroll
  for (int q = 0; q < M; ++q) {
    d[q] = (r0 + q < nz) ? -(double)cp[(size_t)q * plane] : 0.0;
    ib_[q] = 0.0;
  }

  // upward sweep: the first row reduced to couple x_{-1}, x_0, x_{M-1}
  double uc = ga[M - 2];
  double ue = ex[M - 2] + lam;
  double ud = d[M - 2];
  double ub = al[M - 2] + uc + ue;
#pragma unroll
  for (int q = M - 3; q >= 0; --q) {
    const double tq = qdiv<FAST>(ga[q], ub);
    uc = tq * uc;
    ue = (ex[q] + lam) + tq * ue;
    ud = d[q] + tq * ud;
    ub = al[q] + uc + ue;
  }
  // downward sweep: pivots b_q = gamma_q + |a_q| + e'_q, forward-reduced d
  double fa = al[1];
  double fe = ex[1] + lam;
  ib_[1] = qdiv<FAST>(1.0, ga[1] + fa + fe);
#pragma unroll
  for (int q = 2; q < M; ++q) {
    const double tq = al[q] * ib_[q - 1];
    fa = tq * fa;
    fe = (ex[q] + lam) + tq * fe;
    d[q] = d[q] + tq * d[q - 1];
    ib_[q] = qdiv<FAST>(1.0, ga[q] + fa + fe);
  }

  // reduced rows 2ch (first) and 2ch+1 (last) of this column
  double ra0 = al[0], rg0 = uc, re0 = ue, rd0 = ud;
  double ra1 = fa, rg1 = ga[M - 1], re1 = fe, rd1 = d[M - 1];
  const int w0 = (2 * ch) * TI + col, w1 = (2 * ch + 1) * TI + col;
  // parallel cyclic reduction over the 2P rows: after the step of stride s
  // every row couples only to rows 2s away; the sums stay subtraction-free
  for (int s = 1; s < nr; s *= 2) {
    RA[w0] = ra0; RG[w0] = rg0; RE[w0] = re0; RD[w0] = rd0;
    RA[w1] = ra1; RG[w1] = rg1; RE[w1] = re1; RD[w1] = rd1;
    __syncthreads();
    double na[2], ng[2], ne[2], nd[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 2 * ch + h;
      const double a = h ? ra1 : ra0, g = h ? rg1 : rg0, e = h ? re1 : re0, dd = h ? rd1 : rd0;
      double k1 = 0.0, k2 = 0.0, am = 0.0, em = 0.0, dm = 0.0, gp = 0.0, ep = 0.0, dp = 0.0;
      if (r - s >= 0) {
        const int o = (r - s) * TI + col;
        am = RA[o]; em = RE[o]; dm = RD[o];
        k1 = qdiv<FAST>(a, am + RG[o] + em);
      }
      if (r + s < nr) {
        const int o = (r + s) * TI + col;
        gp = RG[o]; ep = RE[o]; dp = RD[o];
        k2 = qdiv<FAST>(g, RA[o] + gp + ep);
      }
      na[h] = k1 * am;
      ng[h] = k2 * gp;
      ne[h] = e + k1 * em + k2 * ep;
      nd[h] = dd + k1 * dm + k2 * dp;
    }
    __syncthreads();
    ra0 = na[0]; rg0 = ng[0]; re0 = ne[0]; rd0 = nd[0];
    ra1 = na[1]; rg1 = ng[1]; re1 = ne[1]; rd1 = nd[1];
  }
  const double x0 = qdiv<FAST>(rd0, ra0 + rg0 + re0);
  const double xl = qdiv<FAST>(rd1, ra1 + rg1 + re1);

  // interior: y_q = (d_q + |a_q| x0) / b_q forward, x_q = y_q + gamma_q x_{q+1} / b_q backward
  double a = al[1];
#pragma unroll
  for (int q = 1; q < M - 1; ++q) {
    if (q >= 2) a = al[q] * ib_[q - 1] * a;
    d[q] = (d[q] + a * x0) * ib_[q];
  }
  d[M - 1] = xl;
#pragma unroll
  for (int q = M - 2; q >= 1; --q) d[q] = d[q] + ga[q] * ib_[q] * d[q + 1];
  d[0] = x0;
#pragma unroll
  for (int q = 0; q < M; ++q)
    if (r0 + q < nz) cp[(size_t)q * plane] = (TS)(zero_col ? 0.0 : d[q]);
}

// Paired variant: each thread takes two adjacent slot columns (i, i+1), i
// even. Slots 2q and 2q+1 carry the real and imaginary parts of the same x
// mode, so the two columns share the shift lambda and the whole Step 1
// (pivots, reciprocals, reduced-row coefficients, the cyclic-reduction
// multipliers): only the right-hand sides are doubled. The one pair whose
// slots differ in mode (slots 0 and 1: the mean and the Nyquist mode) lives
// in the workgroups with ib == 0; those run two passes, pass p solving
// column p of every pair with that column's own shift.
template <int NR>
__device__ __forceinline__ double rcpn(double b) {
  double r = __builtin_amdgcn_rcp(b);
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const double e = __builtin_fma(-b, r, 1.0);
    r = __builtin_fma(r, e, r);
  }
  return r;
}

// The z tables are deliberately not restrict-qualified: the workgroup
// barriers then force them to be re-read (from L1) after the reduced solve
// instead of being held in registers through it.
// LDS slot of reduced row `row` of thread pair pc: consecutive pairs are
// adjacent, and with fewer than 8 pairs per workgroup every row pair is
// followed by a gap of TP slots, so the 8 lanes of one 128-bit LDS access
// (two chunks) fall in different banks.
__host__ __device__ constexpr int zskew(int tp, bool sk) { return sk && tp < 8 ? tp : 0; }
template <int TP, bool SK>
__device__ __forceinline__ int zslot(int row, int pc) {
  return (row >> 1) * (2 * TP + zskew(TP, SK)) + (row & 1) * TP + pc;
}

template <typename TS, int M, int TP, int NR, int WAVES, bool SK>
__global__ __launch_bounds__(512, WAVES) void k_zsolve2(TS *data, int nx, int ny, int nz, int P,
                                               const double *zal, const double *zga,
                                               const double *zex, const double *sx,
                                               const double *sy, size_t sp, int xr, ZeroJob zj) {
  unsigned bx_ = blockIdx.x, gx_ = gridDim.x;
  if (zj.m) {  // the first workgroup takes the zero mode
    if (bx_ == 0) return zero_solve(zj, zga, nz);
    --bx_;
    --gx_;
  }
  using V = cplx<TS>;  // the pair (column i, column i+1) of one row
  // LDS: the z tables of the column, (alpha, gamma) and eps of row
  // ch*M + q at [q*P + ch] (the chunks of one wave read consecutive
  // entries), then three double2 arrays of the 2P reduced rows (zslot)
  extern __shared__ double red[];
  using D2 = cplx<double>;
  const int nr = 2 * P;
  D2 *tag = reinterpret_cast<D2 *>(red);
  double *tex = reinterpret_cast<double *>(tag + P * M);
  for (int e = threadIdx.x; e < P * M; e += blockDim.x) {
    const int o = (e % M) * P + e / M;
    tag[o] = mkc<double>(zal[e], zga[e]);
    tex[o] = zex[e];
  }
  const int nib = nx / (2 * TP);
  const int blk = (int)xcd_block(bx_, gx_);
  const int ib = blk % nib;
  const int j = blk / nib;
  const int pc = threadIdx.x % TP;
  const int ch = threadIdx.x / TP;
  const int i = 2 * (ib * TP + pc);
  const int r0 = ch * M;
  const size_t plane = sp;
  V *cp = reinterpret_cast<V *>(data + (size_t)j * nx + i + (size_t)r0 * plane);
  const size_t vplane = plane / 2;
  const D2 *agc = tag + ch;
  const double *exc = tex + ch;
  auto al = [&](int q) { return agc[q * P].x; };
  auto ga = [&](int q) { return agc[q * P].y; };
  auto ex = [&](int q) { return exc[q * P]; };
  __syncthreads();
  // xr (x walls): every slot is its own real x mode, so the two columns of
  // a pair have different shifts and every pair takes both passes
  const int npass = ib == 0 || xr ? 2 : 1;  // uniform per workgroup
  for (int pass = 0; pass < npass; ++pass) {
    // pass 1 exists only for the pair of slots 0 and 1; other lanes redo
    // pass 0's work on already solved data and store nothing
    const int ci = i + pass;
    const double lam0 = sx[ci] + sy[(ci >= 2 ? ny : 0) + j];
    const bool zero_col = lam0 == 0.0;  // Poisson's (0,0) only
    const double lam = zero_col ? 1.0 : lam0;
    // pass 0 stores both columns of every pair except column 1 of the pair
    // (0, 1); pass 1 stores only that column (with xr: pass 0 column 0 and
    // pass 1 column 1 of every pair)
    const bool st0 = pass == 0;
    const bool st1 = xr ? pass == 1
                        : (pass == 0 && (npass == 1 || i != 0)) || (pass == 1 && i == 0);

    double d0[M], d1[M], ib_[M];
#pragma unroll
    for (int q = 0; q < M; ++q) {
      V v = V{};
      if (r0 + q < nz) v = cp[(size_t)q * vplane];
      d0[q] = -(double)v.x;
      d1[q] = -(double)v.y;
    }
    // upward sweep (reduced first row) and downward sweep (pivots, reduced last row)
    double uc = ga(M - 2);
    double ue = ex(M - 2) + lam;
    double ud0 = d0[M - 2], ud1 = d1[M - 2];
    double ub = al(M - 2) + uc + ue;
#pragma unroll
    for (int q = M - 3; q >= 0; --q) {
      const double tq = ga(q) * rcpn<NR>(ub);
      uc = tq * uc;
      ue = (ex(q) + lam) + tq * ue;
      ud0 = d0[q] + tq * ud0;
      ud1 = d1[q] + tq * ud1;
      ub = al(q) + uc + ue;
    }
    double fa = al(1);
    double fe = ex(1) + lam;
    ib_[1] = rcpn<NR>(ga(1) + fa + fe);
#pragma unroll
    for (int q = 2; q < M; ++q) {
      const double tq = al(q) * ib_[q - 1];
      fa = tq * fa;
      fe = (ex(q) + lam) + tq * fe;
      d0[q] = d0[q] + tq * d0[q - 1];
      d1[q] = d1[q] + tq * d1[q - 1];
      ib_[q] = rcpn<NR>(ga(q) + fa + fe);
    }
    // The reduced rows 2ch (first row of the chunk) and 2ch+1 (last row),
    // each kept divided by its own diagonal: coupling below A, above G,
    // excess E (A + G + E = 1) and the right-hand sides D0, D1. A cyclic-
    // reduction step on normalised rows needs no division by a neighbour's
    // pivot: row r takes A' D[r-s] and G' D[r+s] into its parts, sums its
    // new diagonal from non-negative terms and divides once. A row with no
    // neighbour at distance s already has A (or G) exactly zero, so the
    // clamped read contributes nothing.
    D2 *X1 = reinterpret_cast<D2 *>(tex + P * M);  // (A, E)
    const int span = (nr / 2) * (2 * TP + zskew(TP, SK));
    D2 *X2 = X1 + span;                    // (D0, D1)
    D2 *X3 = X2 + span;                    // (G, E)
    double A[2], G[2], E[2], D0[2], D1[2];
    {
      const double b0 = rcpn<NR>(al(0) + uc + ue), b1 = rcpn<NR>(fa + ga(M - 1) + fe);
      A[0] = al(0) * b0; G[0] = uc * b0; E[0] = ue * b0; D0[0] = ud0 * b0; D1[0] = ud1 * b0;
      A[1] = fa * b1; G[1] = ga(M - 1) * b1; E[1] = fe * b1; D0[1] = d0[M - 1] * b1; D1[1] = d1[M - 1] * b1;
    }
    for (int s = 1; s < nr; s *= 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int o = zslot<TP, SK>(2 * ch + h, pc);
        X1[o] = mkc<double>(A[h], E[h]);
        X2[o] = mkc<double>(D0[h], D1[h]);
        X3[o] = mkc<double>(G[h], E[h]);
      }
      __syncthreads();
      double na[2], ng[2], ne[2], n0[2], n1[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = 2 * ch + h;
        const int lo = zslot<TP, SK>(r - s < 0 ? 0 : r - s, pc);
        const int hi = zslot<TP, SK>(r + s >= nr ? nr - 1 : r + s, pc);
        const D2 ae = X1[lo], dl = X2[lo], ge = X3[hi], dh = X2[hi];
        na[h] = A[h] * ae.x;
        ng[h] = G[h] * ge.x;
        ne[h] = E[h] + A[h] * ae.y + G[h] * ge.y;
        n0[h] = D0[h] + A[h] * dl.x + G[h] * dh.x;
        n1[h] = D1[h] + A[h] * dl.y + G[h] * dh.y;
      }
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double ib = rcpn<NR>(na[h] + ng[h] + ne[h]);
        A[h] = na[h] * ib; G[h] = ng[h] * ib; E[h] = ne[h] * ib;
        D0[h] = n0[h] * ib; D1[h] = n1[h] * ib;
      }
    }
    // decoupled: every diagonal is 1
    const double x00 = D0[0], x01 = D1[0], xl0 = D0[1], xl1 = D1[1];
    // interior: forward y_q = (d_q + |a_q| x0) / b_q, backward x_q = y_q + gamma_q x_{q+1} / b_q
    double a = al(1);
#pragma unroll
    for (int q = 1; q < M - 1; ++q) {
      if (q >= 2) a = al(q) * ib_[q - 1] * a;
      d0[q] = (d0[q] + a * x00) * ib_[q];
      d1[q] = (d1[q] + a * x01) * ib_[q];
    }
    d0[M - 1] = xl0;
    d1[M - 1] = xl1;
#pragma unroll
    for (int q = M - 2; q >= 1; --q) {
      const double c = ga(q) * ib_[q];
      d0[q] = d0[q] + c * d0[q + 1];
      d1[q] = d1[q] + c * d1[q + 1];
    }
    d0[0] = x00;
    d1[0] = x01;
    if (st0 || st1) {
#pragma unroll
      for (int q = 0; q < M; ++q) {
        if (r0 + q < nz) {
          TS *e = reinterpret_cast<TS *>(cp + (size_t)q * vplane);
          if (st0 && st1) {
            cp[(size_t)q * vplane] = V{(TS)(zero_col ? 0.0 : d0[q]), (TS)d1[q]};
          } else if (st0) {
            e[0] = (TS)(zero_col ? 0.0 : d0[q]);
          } else {
            e[1] = (TS)d1[q];
          }
        }
      }
    }
  }
}

// Separator form of the paired solve. The last row of every chunk is a
// separator; the other M-1 rows of the chunk are interior to it. A downward
// sweep from the chunk's first row (which couples to the previous separator
// by its alpha) reduces the chunk to its separator row; an upward sweep over
// the interior rows reduces the chunk's first row to its couplings with the
// previous and the own separator. The separator row then eliminates the
// next chunk's first row (read from LDS), which leaves one tridiagonal row
// per chunk in the separators alone: P rows instead of the 2P of the first-
// and-last-row reduction, one row per thread, and one cyclic-reduction step
// fewer. Every pivot is still a sum of non-negative parts:
//   separator row:  -SA x[s-1] + (SA + SG + SE) x[s] - SG x[s+1] = SD,
//   SA = fa, SG = t ug', SE = fe + t ue', SD = D + t U', t = gamma / C',
// with (fa, fe, D) from the downward sweep and (ug', ue', U', C') the next
// chunk's reduced first row.
//
// TILE: the workgroup's R*2*TP columns (128 bytes of every row) are staged
// through LDS: the whole column tile is read row by row with 16-byte loads
// (whole 128-byte lines, instead of 2*TP*sizeof(TS) bytes per row and
// thread group), every thread takes its rows from LDS, and the results go
// back the same way, after the last round. The threads take the tile's
// columns in R rounds of 2*TP; each round's columns are a region of their
// own, [P*M rows][2*TP], whose first bytes the reduced-row arrays share
// once every thread holds its rows. Only single-pass workgroups tile; the
// two-pass ones (the pair of slots 0 and 1, x walls) read and write their
// columns directly.
// DB: the three reduced-row arrays are doubled, and the steps of the cyclic
// reduction alternate between the two sets: a step writes one set while the
// previous step's reads of the other may still be in flight, so a step
// takes one barrier instead of two.
// Hides a per-lane column pointer from common-subexpression elimination:
// with chunks narrower than a wave the row addresses are per-lane 64-bit
// values, and keeping all of them from the loads to the stores of a sweep
// took as many registers as the column itself; they are recomputed instead.
template <typename TS>
__device__ __forceinline__ TS *fresh(TS *p) {
  uintptr_t a = reinterpret_cast<uintptr_t>(p);
  asm volatile("" : "+v"(a));
  // as a global address: through a plain integer the accesses become flat
  // ones, whose waits are the LDS accesses' too
  return (TS *)(TS __attribute__((address_space(1))) *)a;
}

// One column pair's solve in separator form, in place on the right-hand sides
// d0, d1 (negated) of the thread's chunk. tag / agc / exc: the z tables in LDS
// (of the workgroup, and from the chunk's rows on); X1: the reduced-row
// arrays, three of [P][TP], six with DB.
// PS: chunks the arrays are laid out for, a constant that saves the address
// registers of a run-time count (0: P).
template <int M, int TP, int NR, bool DB, bool kFence, int PS = 0>
__device__ __forceinline__ void sep_solve(double (&d0)[M], double (&d1)[M], double lam, const cplx<double> *tag,
                                          const cplx<double> *agc, const double *exc, cplx<double> *X1,
                                          int P, int ch, int pc) {
  using D2 = cplx<double>;
  const int ps = PS ? PS : P;
  auto al = [&](int q) { return agc[q * ps].x; };
  auto ga = [&](int q) { return agc[q * ps].y; };
  auto ex = [&](int q) { return exc[q * ps]; };
  D2 *const X2 = X1 + ps * TP, *const X3 = X2 + ps * TP;
  const int me = ch * TP + pc;
  const int nch = ch + 1 < P ? ch + 1 : ch;  // the last chunk's gamma is 0
  const int nb = nch * TP + pc;
  double ib_[M];
  // upward sweep over the interior: the chunk's first row in terms of the
  // previous separator (alpha_0) and the own separator (ug)
  {
    double ug = ga(M - 2), ue = ex(M - 2) + lam, u0 = d0[M - 2], u1 = d1[M - 2];
    double cb = al(M - 2) + ug + ue;
#pragma unroll
    for (int q = M - 3; q >= 0; --q) {
      const double t = ga(q) * rcpn<NR>(cb);
      ug = t * ug;
      ue = (ex(q) + lam) + t * ue;
      u0 = d0[q] + t * u0;
      u1 = d1[q] + t * u1;
      cb = al(q) + ug + ue;
      if constexpr (kFence) sched_fence(q);
    }
    X1[me] = mkc<double>(ug, ue);
    X2[me] = mkc<double>(u0, u1);
  }
  // downward sweep from the first row (coupled to the previous separator)
  double fa = al(0), fe = ex(0) + lam;
  ib_[0] = rcpn<NR>(fa + ga(0) + fe);
#pragma unroll
  for (int q = 1; q < M; ++q) {
    const double t = al(q) * ib_[q - 1];
    fa = t * fa;
    fe = (ex(q) + lam) + t * fe;
    d0[q] = d0[q] + t * d0[q - 1];
    d1[q] = d1[q] + t * d1[q - 1];
    if (q < M - 1) ib_[q] = rcpn<NR>(fa + ga(q) + fe);
    if constexpr (kFence) sched_fence(q);
  }
  __syncthreads();
  double A, G, E, S0, S1;
  {
    const D2 gu = X1[nb], uu = X2[nb];
    const double t = ga(M - 1) * rcpn<NR>(tag[nch].x + gu.x + gu.y);
    const double sa = fa, sg = t * gu.x, se = fe + t * gu.y;
    const double s0 = d0[M - 1] + t * uu.x, s1 = d1[M - 1] + t * uu.y;
    const double b = rcpn<NR>(sa + sg + se);
    A = sa * b; G = sg * b; E = se * b; S0 = s0 * b; S1 = s1 * b;
  }
  __syncthreads();
  // cyclic reduction on the P separator rows (normalised, see k_zsolve2)
  D2 *F2 = X2;  // the set the separator values go to
  if constexpr (DB) {
    D2 *const Y1 = X3 + ps * TP, *const Y2 = Y1 + ps * TP, *const Y3 = Y2 + ps * TP;
    bool odd = false;
    for (int s = 1; s < P; s *= 2) {
      D2 *const Z1 = odd ? Y1 : X1, *const Z2 = odd ? Y2 : X2, *const Z3 = odd ? Y3 : X3;
      Z1[me] = mkc<double>(A, E);
      Z2[me] = mkc<double>(S0, S1);
      Z3[me] = mkc<double>(G, E);
      __syncthreads();
      const int lo = (ch - s < 0 ? 0 : ch - s) * TP + pc;
      const int hi = (ch + s >= P ? P - 1 : ch + s) * TP + pc;
      const D2 ae = Z1[lo], dl = Z2[lo], ge = Z3[hi], dh = Z2[hi];
      const double na = A * ae.x, ng = G * ge.x, ne = E + A * ae.y + G * ge.y;
      const double n0 = S0 + A * dl.x + G * dh.x, n1 = S1 + A * dl.y + G * dh.y;
      const double b = rcpn<NR>(na + ng + ne);
      A = na * b; G = ng * b; E = ne * b; S0 = n0 * b; S1 = n1 * b;
      odd = !odd;
    }
    // the set the last step did not read
    F2 = odd ? Y2 : X2;
  } else {
    for (int s = 1; s < P; s *= 2) {
      X1[me] = mkc<double>(A, E);
      X2[me] = mkc<double>(S0, S1);
      X3[me] = mkc<double>(G, E);
      __syncthreads();
      const int lo = (ch - s < 0 ? 0 : ch - s) * TP + pc;
      const int hi = (ch + s >= P ? P - 1 : ch + s) * TP + pc;
      const D2 ae = X1[lo], dl = X2[lo], ge = X3[hi], dh = X2[hi];
      const double na = A * ae.x, ng = G * ge.x, ne = E + A * ae.y + G * ge.y;
      const double n0 = S0 + A * dl.x + G * dh.x, n1 = S1 + A * dl.y + G * dh.y;
      __syncthreads();
      const double b = rcpn<NR>(na + ng + ne);
      A = na * b; G = ng * b; E = ne * b; S0 = n0 * b; S1 = n1 * b;
    }
  }
  // separator values: the own one and the previous chunk's
  F2[me] = mkc<double>(S0, S1);
  __syncthreads();
  const D2 xl = ch > 0 ? F2[me - TP] : mkc<double>(0.0, 0.0);
  __syncthreads();
  // interior: forward y_q = (D_q + fa_q x_lo) / b_q, backward x_q = y_q + gamma_q x_{q+1} / b_q
  double a = al(0);
#pragma unroll
  for (int q = 0; q < M - 1; ++q) {
    if (q >= 1) a = al(q) * ib_[q - 1] * a;
    d0[q] = (d0[q] + a * xl.x) * ib_[q];
    d1[q] = (d1[q] + a * xl.y) * ib_[q];
    if constexpr (kFence) sched_fence(q);
  }
  d0[M - 1] = S0;
  d1[M - 1] = S1;
#pragma unroll
  for (int q = M - 2; q >= 0; --q) {
    const double c = ga(q) * ib_[q];
    d0[q] = d0[q] + c * d0[q + 1];
    d1[q] = d1[q] + c * d1[q + 1];
    if constexpr (kFence) sched_fence(q);
  }
}

template <typename TS, int M, int TP, int NR, int WAVES, int MAXT = 512, bool TILE = false, int R = 1,
          bool DB = false>
__device__ __forceinline__ void zsolve3_body(TS *data, int nx, int ny, int nz, int P,
                                                      const double *zal, const double *zga,
                                                      const double *zex, const double *sx,
                                                      const double *sy, size_t sp, int xr,
                                             unsigned bx_, unsigned gx_) {
  static_assert(M >= 3, "a chunk needs interior rows");
  static_assert(TILE || R == 1, "rounds need the tile");
  using V = cplx<TS>;
  using D2 = cplx<double>;
  // LDS: the z tables as in k_zsolve2, then three double2 arrays [P][TP]
  // (TILE: then R tile regions, the first bytes of the current one shared
  // with the three arrays)
  extern __shared__ double red[];
  D2 *tag = reinterpret_cast<D2 *>(red);
  double *tex = reinterpret_cast<double *>(tag + P * M);
  for (int e = threadIdx.x; e < P * M; e += blockDim.x) {
    const int o = (e % M) * P + e / M;
    tag[o] = mkc<double>(zal[e], zga[e]);
    tex[o] = zex[e];
  }
  constexpr int TC = 2 * TP;  // columns of one round
  // one tile region: P*M rows of TC values, at least the three arrays
  constexpr int NX = DB ? 6 : 3;  // reduced-row arrays
  const size_t region = ((size_t)P * M * TC * sizeof(TS) > (size_t)NX * P * TP * sizeof(D2)
                             ? (size_t)P * M * TC * sizeof(TS)
                             : (size_t)NX * P * TP * sizeof(D2)) / sizeof(double);
  double *const reg0 = tex + P * M;
  D2 *X1 = reinterpret_cast<D2 *>(reg0);
  TS *tile = reinterpret_cast<TS *>(reg0);
  const int nib = nx / (R * TC);
  const int blk = (int)xcd_block(bx_, gx_);
  const int ib = blk % nib;
  const int j = blk / nib;
  const int pc = threadIdx.x % TP;
  const int ch = threadIdx.x / TP;
  int i = 2 * (ib * R * TP + pc);
  const int r0 = ch * M;
  const size_t plane = sp;
  V *cp = reinterpret_cast<V *>(data + (size_t)j * nx + i + (size_t)r0 * plane);
  const size_t vplane = plane / 2;
  const D2 *agc = tag + ch;
  const double *exc = tex + ch;
  const int npass = ib == 0 || xr ? 2 : 1;  // uniform per workgroup
  // 16-byte vectors of a round's row segment and of a tile row, and the
  // tile's first row in global memory
  constexpr int EPV = 16 / (int)sizeof(TS);
  constexpr int VPR = TC / EPV;
  static_assert(!TILE || TC % EPV == 0, "tile rows are whole 16-byte vectors");
  TS *const gt = data + (size_t)j * nx + (size_t)ib * R * TC;
  const bool tiled = TILE && npass == 1;
  auto tile_io = [&](bool load) {
    for (int e = threadIdx.x; e < nz * R * VPR; e += blockDim.x) {
      const int r = e / (R * VPR), c = e % (R * VPR);
      uint4 *l = reinterpret_cast<uint4 *>(reinterpret_cast<TS *>(reg0 + (c / VPR) * region) + r * TC +
                                           (c % VPR) * EPV);
      uint4 *g = reinterpret_cast<uint4 *>(gt + (size_t)r * plane + c * EPV);
      if (load)
        *l = *g;
      else
        *g = *l;
    }
  };
  if (tiled) tile_io(true);
  __syncthreads();
  // the tiled and the direct path as separate instances of the pass loop,
  // so that neither keeps the other's addresses live
  auto passes = [&](auto tl) {
  constexpr bool TL = decltype(tl)::value;
  for (int pass = 0; pass < npass; ++pass) {
    // as in k_zsolve2: pass 1 only for column 1 of the pair of slots 0, 1,
    // or (xr) for column 1 of every pair
    const int ci = i + pass;
    const double lam0 = sx[ci] + sy[(ci >= 2 ? ny : 0) + j];
    const bool zero_col = lam0 == 0.0;  // Poisson's (0,0) only
    const double lam = zero_col ? 1.0 : lam0;
    const bool st0 = pass == 0;
    const bool st1 = xr ? pass == 1
                        : (pass == 0 && (npass == 1 || i != 0)) || (pass == 1 && i == 0);

    double d0[M], d1[M];
    // the 1024-thread shapes have half the registers: compiler fences keep
    // their unrolled sweeps from issuing every read up front
    constexpr bool kFence = MAXT > 512 || M >= 32;
#pragma unroll
    for (int q = 0; q < M; ++q) {
      V v = V{};
      if (r0 + q < nz)
        v = TL ? *reinterpret_cast<const V *>(tile + (r0 + q) * TC + 2 * pc) : cp[(size_t)q * vplane];
      d0[q] = -(double)v.x;
      d1[q] = -(double)v.y;
    }
    // every thread holds its rows before the reduced-row arrays reuse the tile
    if constexpr (TL) __syncthreads();
    sep_solve<M, TP, NR, DB, kFence>(d0, d1, lam, tag, agc, exc, X1, P, ch, pc);
    if constexpr (TL) {
      // single pass: both columns, into the round's region (its reduced-row
      // arrays are read by now); the tile goes out after the last round
      __syncthreads();
#pragma unroll
      for (int q = 0; q < M; ++q)
        if (r0 + q < nz)
          *reinterpret_cast<V *>(tile + (r0 + q) * TC + 2 * pc) = V{(TS)d0[q], (TS)d1[q]};
      __syncthreads();
    } else if (st0 || st1) {
#pragma unroll
      for (int q = 0; q < M; ++q) {
        if (r0 + q < nz) {
          TS *e = reinterpret_cast<TS *>(cp + (size_t)q * vplane);
          if (st0 && st1) {
            cp[(size_t)q * vplane] = V{(TS)(zero_col ? 0.0 : d0[q]), (TS)d1[q]};
          } else if (st0) {
            e[0] = (TS)(zero_col ? 0.0 : d0[q]);
          } else {
            e[1] = (TS)d1[q];
          }
        }
      }
    }
  }
  };
  for (int rd = 0; rd < R; ++rd) {
    if (rd > 0) {
      // the next round: its columns, its tile region (which the three
      // arrays share now)
      i += 2 * TP;
      cp += TP;
      X1 = reinterpret_cast<D2 *>(reg0 + rd * region);
      tile = reinterpret_cast<TS *>(reg0 + rd * region);
    }
    if (tiled)
      passes(std::true_type{});
    else
      passes(std::false_type{});
  }
  if (tiled) tile_io(false);
}
template <typename TS, int M, int TP, int NR, int WAVES, int MAXT = 512, bool TILE = false, int R = 1,
          bool DB = false>
__global__ __launch_bounds__(MAXT, WAVES) void k_zsolve3(TS *data, int nx, int ny, int nz, int P,
                                                      const double *zal, const double *zga,
                                                      const double *zex, const double *sx,
                                                      const double *sy, size_t sp, int xr, ZeroJob zj) {
  unsigned bx = blockIdx.x, gx = gridDim.x;
  if (zj.m) {  // the first workgroup takes the zero mode
    if (bx == 0) return zero_solve(zj, zga, nz);
    --bx;
    --gx;
  }
  zsolve3_body<TS, M, TP, NR, WAVES, MAXT, TILE, R, DB>(data, nx, ny, nz, P, zal, zga, zex, sx, sy, sp, xr,
                                                        bx, gx);
}

// The separator form in persistent workgroups: one round of resident
// workgroups walks the tiles of 2 TP columns, and each loads its next tile's
// rows into registers before it solves the current one, so that those loads
// travel during the elimination. The z tables are staged once per workgroup.
// PS: chunks of a column at most.
//
// What bounds it: the elimination itself at 1024 rows (one workgroup of 128
// chunks a compute unit; about 13 us a tile, some 4 each of float64
// arithmetic and of LDS accesses), HBM for the short columns. Float32 ms on
// MI355X against the best of the shapes that load, solve and store in turn:
//   1024 x 512 x 1024  2.06 -> 1.40     512 x 512 x 256  0.153 -> 0.144
//   1024 x 512 x 512   0.72 -> 0.57     256 x 256 x 96   0.0275 -> 0.0201
//   3456 x 3072 x 30   0.67 -> 0.53 (4.8 TB/s)
// In float64 the next tile's rows take 32 registers, which leaves 12 waves a
// compute unit instead of 16: slower than the direct shapes (1024 x 512 x 512
// 1.21 against 1.05 ms) except on small planes of short columns (64 x 64 x 64
// 8.1 against 10 us).
template <typename TS, int M, int TP, int PS>
__device__ __forceinline__ void zsolve4_body(TS *data, int nx, int ny, int nz, int P, const double *zal,
                                             const double *zga, const double *zex, const double *sx,
                                             const double *sy, size_t sp, int xr, unsigned bx, unsigned G) {
  using V = cplx<TS>;
  using D2 = cplx<double>;
  extern __shared__ double red[];
  D2 *tag = reinterpret_cast<D2 *>(red);
  double *tex = reinterpret_cast<double *>(tag + PS * M);
  for (int e = threadIdx.x; e < P * M; e += blockDim.x) {
    const int o = (e % M) * PS + e / M;
    tag[o] = mkc<double>(zal[e], zga[e]);
    tex[o] = zex[e];
  }
  D2 *X1 = reinterpret_cast<D2 *>(tex + PS * M);
  const unsigned nib = nx / (2 * TP);
  const int pc = threadIdx.x % TP, ch = threadIdx.x / TP, r0 = ch * M;
  const size_t vplane = sp / 2;
  // the tiles of first passes, then those of second passes (the pair of slots
  // 0 and 1 in every row j; with x walls every pair, see zsolve3_body), which
  // read and write columns of their own
  const unsigned n1 = nib * ny, ntiles = n1 + (xr ? n1 : ny);
  auto tile_of = [&](unsigned i) {
    const unsigned b0 = i * G;
    return b0 + G <= ntiles ? b0 + xcd_block(bx, G) : b0 + bx;
  };
  struct Tile {
    int j, i, pass;
  };
  auto place = [&](unsigned t) {
    const bool second = t >= n1;
    const unsigned u = second ? t - n1 : t;
    const unsigned ib = second && !xr ? 0 : u % nib;
    return Tile{(int)(second && !xr ? u : u / nib), 2 * (int)(ib * TP + pc), second ? 1 : 0};
  };
  // Nothing may touch a value of the next tile before its turn, nor a load
  // be issued in a branch: the wait for either would be a wait for them all.
  // So the two parts of the shift are kept apart, and rows past nz read the
  // last row.
  V nxt[M];
  double sxn, syn;
  auto load = [&](unsigned t) {
    const Tile p = place(t);
    const int ci = p.i + p.pass;
    sxn = sx[ci];
    syn = sy[(ci >= 2 ? ny : 0) + p.j];
    const V *c = fresh(reinterpret_cast<const V *>(data + (size_t)p.j * nx + p.i + (size_t)r0 * sp));
    const int last = nz - 1 - r0;  // >= 0
#pragma unroll
    for (int q = 0; q < M; ++q) nxt[q] = c[(size_t)(q < last ? q : last) * vplane];
  };
  unsigned t = tile_of(0);
  if (t >= ntiles) return;  // uniform
  load(t);
  __syncthreads();
  for (unsigned it = 0;;) {
    const Tile p = place(t);
    double d0[M], d1[M];
#pragma unroll
    for (int q = 0; q < M; ++q) {
      d0[q] = r0 + q < nz ? -(double)nxt[q].x : 0.0;
      d1[q] = r0 + q < nz ? -(double)nxt[q].y : 0.0;
    }
    const double lam0 = sxn + syn;
    const bool zero_col = lam0 == 0.0;  // Poisson's (0,0) only
    const unsigned tn = tile_of(++it);
    const bool more = tn < ntiles;  // uniform
    // the rows are taken over before their registers are loaded again (left
    // to itself the compiler converts them later, from copies whose making
    // waits for the loads)
#pragma unroll
    for (int q = 0; q < M; ++q) asm volatile("" : "+v"(d0[q]), "+v"(d1[q]));
    load(more ? tn : t);  // the last turn's values are not used
    sep_solve<M, TP, 1, true, true, PS>(d0, d1, zero_col ? 1.0 : lam0, tag, tag + ch, tex + ch, X1, P, ch, pc);
    // a first pass stores both columns, except column 1 of the slots 0 and 1
    // (with x walls of every pair), which a second pass stores
    V *cp = fresh(reinterpret_cast<V *>(data + (size_t)p.j * nx + p.i + (size_t)r0 * sp));
    const bool own = xr || p.i == 0;
    if (p.pass == 0 && !own) {
#pragma unroll
      for (int q = 0; q < M; ++q)
        if (r0 + q < nz) cp[(size_t)q * vplane] = V{(TS)d0[q], (TS)d1[q]};
    } else if (own) {
      TS *e = reinterpret_cast<TS *>(cp) + p.pass;
#pragma unroll
      for (int q = 0; q < M; ++q)
        if (r0 + q < nz) e[(size_t)q * sp] = (TS)(p.pass ? d1[q] : zero_col ? 0.0 : d0[q]);
    }
    if (!more) break;
    t = tn;
  }
}

// waves per SIMD the registers leave room for
template <typename TS>
constexpr int z4_waves() { return sizeof(TS) == 4 ? 4 : 3; }
template <typename TS, int M, int TP, int PS>
__global__ __launch_bounds__(PS *TP, z4_waves<TS>()) void k_zsolve4(TS *data, int nx, int ny, int nz, int P,
                                                                    const double *zal, const double *zga,
                                                                    const double *zex, const double *sx,
                                                                    const double *sy, size_t sp, int xr,
                                                                    ZeroJob zj) {
  unsigned bx = blockIdx.x, G = gridDim.x;
  if (zj.m) {  // the first workgroup takes the zero mode
    if (bx == 0) return zero_solve(zj, zga, nz);
    --bx;
    --G;
  }
  zsolve4_body<TS, M, TP, PS>(data, nx, ny, nz, P, zal, zga, zex, sx, sy, sp, xr, bx, G);
}
// Several problems of one chunk count (see GJobs), float32 and periodic x;
// J.nblk is the job's share of the resident workgroups. The grid is the zero
// modes' workgroups, then every job's share, without gaps: a block that only
// exits would still wait for a compute unit of its own, and with it the
// blocks behind it (one workgroup a compute unit at 1024 rows).
template <int M, int TP, int PS>
__global__ __launch_bounds__(PS *TP, z4_waves<float>()) void k_zsolve4_grp(const GJobs g) {
  unsigned b = blockIdx.x;
  for (int k = 0; k < g.count; ++k) {  // uniform
    const GJob &J = g.j[k];
    if (!J.in2) continue;
    if (b == 0)
      return zero_solve(ZeroJob{J.zm, J.aux, const_cast<double *>(static_cast<const double *>(J.in2))}, J.zga,
                        J.nz);
    --b;
  }
  int k = 0;
  while (k < g.count && b >= g.j[k].nblk) b -= g.j[k++].nblk;
  if (k == g.count) return;  // uniform
  const GJob &J = g.j[k];
  zsolve4_body<float, M, TP, PS>(static_cast<float *>(J.out), J.nx, J.ny, J.nz, J.P, J.zal, J.zga, J.zex, J.sx,
                                 J.sy, J.sp, 0, b, J.nblk);
}

// one z-solve shape for several problems with the same chunk count (see
// GJobs): float32 storage, periodic x
template <int M, int TP, int NR, int WAVES, int MAXT, bool TILE, int R, bool DB = false>
__global__ __launch_bounds__(MAXT, WAVES) void k_zsolve3_grp(const GJobs g) {
  const GJob &J = g.j[blockIdx.y];
  unsigned bx = blockIdx.x;
  if (J.in2) {  // the job's first workgroup takes its zero mode
    if (bx == 0)
      return zero_solve(ZeroJob{J.zm, J.aux, const_cast<double *>(static_cast<const double *>(J.in2))}, J.zga,
                        J.nz);
    --bx;
  }
  if (bx >= J.nblk) return;  // uniform per block
  zsolve3_body<float, M, TP, NR, WAVES, MAXT, TILE, R, DB>(static_cast<float *>(J.out), J.nx, J.ny, J.nz,
                                                           J.P, J.zal, J.zga, J.zex, J.sx, J.sy, J.sp, 0,
                                                           bx, J.nblk);
}

// Launch shapes of the z solve: rows per thread M, columns per workgroup
// TI, minimum waves per SIMD (0: none), fast reciprocals.
// Paired variants (two columns per thread sharing their shift) take TI
// columns per workgroup as TI/2 thread pairs; nr is the Newton-step count
// of their reciprocal.
struct ZVariant {
  int M, TI, waves;
  bool fast;
  bool paired;
  int nr;
  bool skew = true;  // paired: gaps between reduced row pairs in LDS
  bool sep = false;  // paired: separator form, P reduced rows
  int maxt = 512;    // threads per workgroup at most
  bool tile = false; // separator form with the column tile staged through LDS
  int rounds = 1;    // tiled: the threads take the TI columns in rounds of TI/rounds
  bool dbl = false;  // separator form: double-buffered reduced rows, one barrier per reduction step
  bool persist = false;  // persistent workgroups that load the next tile ahead (k_zsolve4)
};
static const ZVariant kZVariants[] = {
    {16, 16, 0, false, false, 2}, {16, 16, 4, true, false, 2}, {16, 16, 0, true, false, 2},
    {8, 8, 0, true, false, 2},    {16, 8, 0, true, false, 2},  {8, 16, 0, true, false, 2},
    {16, 32, 0, true, false, 2},  {8, 8, 4, true, false, 2},   {16, 16, 0, true, true, 1},
    {8, 16, 0, true, true, 1},    {16, 32, 0, true, true, 1},  {8, 32, 0, true, true, 1},
    {16, 16, 0, true, true, 2},   {8, 8, 0, true, true, 1},    {8, 8, 4, true, true, 1},
    {8, 16, 4, true, true, 1},    {8, 8, 4, true, true, 1, false}, {8, 16, 4, true, true, 1, false},
    // separator form (k_zsolve3)
    {8, 8, 4, true, true, 1, false, true},   {8, 16, 4, true, true, 1, false, true},
    {16, 16, 0, true, true, 1, false, true}, {16, 32, 0, true, true, 1, false, true},
    {8, 32, 4, true, true, 1, false, true},
    // wide separator shapes for short columns (few chunks per column)
    {8, 64, 4, true, true, 1, false, true},  {8, 128, 4, true, true, 1, false, true},
    {16, 64, 1, true, true, 1, false, true}, {16, 128, 1, true, true, 1, false, true},
    // separator form in 1024-thread workgroups: wider rows for the long
    // columns (8 rows per thread; 16 spilled)
    {8, 32, 1, true, true, 1, false, true, 1024}, {8, 16, 1, true, true, 1, false, true, 1024},
    // separator form with 128-byte row tiles through LDS (32 float32 or 16
    // float64 columns), the 32 float32 columns of 1024-row tiles in two
    // rounds of 16: one workgroup per compute unit at 1024 rows
    {8, 32, 1, true, true, 1, false, true, 1024, true, 2},  {16, 32, 1, true, true, 1, false, true, 512, true, 2},
    {8, 16, 1, true, true, 1, false, true, 1024, true, 1},  {16, 16, 1, true, true, 1, false, true, 512, true, 1},
    {16, 32, 1, true, true, 1, false, true, 512, true, 1},  {8, 32, 1, true, true, 1, false, true, 1024, true, 1},
    {8, 16, 1, true, true, 1, false, true, 512, true, 1},   {8, 32, 1, true, true, 1, false, true, 512, true, 2},
    // 1024-thread separator shapes with double-buffered reduced rows (LDS
    // room for the second set): the 16-column float32 tile and the direct form
    {8, 16, 1, true, true, 1, false, true, 1024, true, 1, true},
    {8, 16, 1, true, true, 1, false, true, 1024, false, 1, true},
    // the 512-thread defaults of 512-row columns with double-buffered reduced rows
    {8, 16, 1, true, true, 1, false, true, 512, true, 1, true},
    {16, 32, 0, true, true, 1, false, true, 512, false, 1, true},
    // persistent: 16 columns a tile, and 32 for columns of up to 128 rows
    {8, 16, 4, true, true, 1, false, true, 1024, false, 1, true, true},
    {8, 32, 4, true, true, 1, false, true, 256, false, 1, true, true},
};
constexpr int kZVariantCount = sizeof(kZVariants) / sizeof(kZVariants[0]);

// the zero mode's rows fit the lanes of a workgroup of `threads`
static bool zero_fits(int nz, int threads) {
  int lanes = 64;
  while (lanes > threads) lanes >>= 1;
  return lanes > 0 && nz <= lanes * kZeroRows;
}

int zsolve_variant_count() { return kZVariantCount; }

// LDS bytes of a launch: paired variants hold the column's z tables and
// three double2 arrays of the reduced rows, unpaired ones four double arrays;
// tiled ones the tables and the larger of the reduced-row arrays and the
// column tile (elements of esize bytes).
static size_t zsolve_lds(const ZVariant &z, int P, int esize) {
  const int tp = z.TI / 2;
  const size_t tables = (size_t)3 * P * z.M * sizeof(double);
  const size_t nxa = z.dbl ? 6 : 3;  // reduced-row arrays
  if (z.tile) {
    const int tpr = tp / z.rounds;  // thread pairs of a round
    return tables + z.rounds * std::max(nxa * P * tpr * 2 * sizeof(double),
                                        (size_t)P * z.M * 2 * tpr * esize);
  }
  if (z.paired && z.sep) return tables + nxa * P * tp * 2 * sizeof(double);
  return z.paired ? (size_t)3 * P * (2 * tp + zskew(tp, z.skew)) * 2 * sizeof(double) + tables
                  : (size_t)4 * 2 * P * z.TI * sizeof(double);
}

bool zsolve_variant_fits(int v, int nx, int nz, int esize) {
  if (v < 0 || v >= kZVariantCount) return false;
  const ZVariant &z = kZVariants[v];
  const int P = (nz + z.M - 1) / z.M;
  const int threads = z.paired ? P * z.TI / 2 / z.rounds : P * z.TI;
  // float64 persistent launches: up to 16 chunks of 16-column tiles
  if (z.persist && esize == 8 && (P > 16 || z.TI != 16)) return false;
  // a tiled launch needs whole 16-byte vectors per round's row segment and
  // at least two chunks
  if (z.tile && (z.TI / z.rounds * esize % 16 != 0 || P < 2)) return false;
  return threads <= z.maxt && nx % z.TI == 0 && P * z.M <= (nz + 15) / 16 * 16 &&
         zsolve_lds(z, P, esize) <= (z.maxt > 512 || z.tile ? 160 * 1024 : 65536);
}

int zsolve_default_variant(int nx, int ny, int nz, bool fp64, bool xr) {
  // Float32 storage: the persistent shapes, 32-column tiles while a column has
  // at most 16 chunks (3456 x 3072 x 30 0.53 against 0.80 ms with 16 columns;
  // 256 x 256 x 192 0.039 against 0.033).
  // Float64 at 1024x512x512: 40 (1.037 ms: separator form, 16 rows, 32
  // columns, double-buffered reduced rows), 21 (1.050, the same with one set),
  // 10 (1.11); at 1024 rows 38 (11.06 ms at 2048x1024x1024: 28 with
  // double-buffered reduced rows; 28 11.30, 20 11.52, the tiled 31 12.8, 4
  // 22.2). Planes of up to 131072 columns do not fill the chip with those
  // shapes: 18 (8 rows, 8 columns: 256x256x384 0.078 against 0.106 ms,
  // 512x256x193 0.071 against 0.078), as long as the field stays in the 256 MB
  // last-level cache, which is where its 64-byte row segments cost nothing
  // (2^25 points and more lose: 384x256x300 0.084 against 0.124 ms, but
  // 384x256x384 0.197 against 0.165, 256x128x1024 0.154 against 0.138). Up to
  // 65536 columns of 16 chunks the persistent 41 (64x64x64 8.1 against 10.5 us,
  // 256x256x128 31 against 35). Other short columns (few chunks) would leave
  // the first shapes with tiny workgroups, so the first fitting shape with at
  // least 128 threads wins, widened by the 64- and 128-column shapes; the
  // unpaired 4 and 3 are fall-backs where the LDS or thread budget excludes the
  // paired shapes.
  // x walls (xr): a persistent workgroup reads every tile once for each of its
  // two passes, which the direct shapes do not. Float64 takes 41 up to 8192
  // columns only (64x64x64 9.2 against 11.5 us; 128x128x64 19.0 against 16.3,
  // 256x256x16 24 against 13). Float32 storage takes the 128-column 24 for
  // planes of 65536 columns and more of at most 16 rows (512x512x16 20 against
  // 24 us; 128x128x16 11 against 8, 512x512x24 28 against 26), and the tiled 39
  // for 161-256 rows of a cached field of 131072 columns and more (512x512x256
  // 0.241 against 0.280 ms, 512x256x192 0.094 against 0.102; 512x512x160 0.172
  // against 0.171, 1024x512x192 beyond the cache 0.475 against 0.439).
  static const int f64[] = {40, 21, 10, 19, 38, 26, 25, 24, 23, 20, 8, 4, 3}, f32[] = {42, 41};
  const long cols = (long)nx * ny, cached = (1l << 28) / (fp64 ? 8 : 4);
  auto fits = [&](int v) { return zsolve_variant_fits(v, nx, nz, fp64 ? 8 : 4); };
  if (!fp64) {
    if (xr && cols >= 65536 && nz <= 16 && fits(24)) return 24;
    if (xr && cols >= 131072 && nz > 160 && nz <= 256 && cols * nz <= cached && fits(39)) return 39;
    for (int v : f32)
      if (fits(v)) return v;
    return -1;
  }
  if (cols <= (xr ? 8192 : 65536) && fits(41)) return 41;
  if (cols <= 131072 && nz > 64 && cols * nz < cached && fits(18)) return 18;
  auto threads = [&](int v) {
    const ZVariant &z = kZVariants[v];
    const int P = (nz + z.M - 1) / z.M;
    return z.paired ? P * z.TI / 2 / z.rounds : P * z.TI;
  };
  for (int v : f64)
    if (fits(v) && threads(v) >= 128) return v;
  for (int v : f64)
    if (fits(v)) return v;
  return -1;
}

// LDS of a persistent workgroup, and how many of them the device holds: 4 or
// 3 waves a SIMD (the kernel's registers) and 160 KB a compute unit.
template <int M, int TP, int PS>
constexpr size_t z4_lds() { return (size_t)3 * PS * M * 8 + (size_t)6 * PS * TP * 16; }
template <typename TS, int M, int TP, int PS>
static long z4_resident(int P) {
  const int waves = (P * TP + 63) / 64;
  return std::max<long>(std::min<long>(4 * z4_waves<TS>() / waves, 160 * 1024 / z4_lds<M, TP, PS>()), 1) *
         device_cus();
}
template <typename TS, int M, int TP, int PS>
static hipError_t launch_z4(int nx, int ny, int nz, TS *data, size_t sp, const double *zal, const double *zga,
                            const double *zex, const double *sx, const double *sy, bool xr, const ZeroJob &zj,
                            hipStream_t st) {
  const int P = (nz + M - 1) / M;
  const unsigned n1 = (unsigned)((long)(nx / (2 * TP)) * ny), ntiles = n1 + (xr ? n1 : (unsigned)ny);
  const long res = z4_resident<TS, M, TP, PS>(P);
  if (P > PS || res < 1) return hipErrorInvalidValue;
  const unsigned G = (unsigned)std::min<long>(ntiles, res);
  hipLaunchKernelGGL((k_zsolve4<TS, M, TP, PS>), dim3(G + (zj.m ? 1 : 0)), dim3(P * TP), (z4_lds<M, TP, PS>()),
                     st, data, nx, ny, nz, P, zal, zga, zex, sx, sy, sp, (int)xr, zj);
  return hipGetLastError();
}
// Each job's share of the resident workgroups, by its tiles: rounded down (one
// at least), then one more for whichever job has the most tiles a workgroup. They sum to
// `resident` at most: a workgroup beyond it would start its tiles when a whole
// round of others has ended theirs.
void z_group_shares(long resident, int count, const long *tiles, unsigned *share) {
  long total = 0, used = 0;
  for (int k = 0; k < count; ++k) total += tiles[k];
  for (int k = 0; k < count; ++k) {
    share[k] = (unsigned)(total <= resident ? tiles[k] : std::max(1l, resident * tiles[k] / total));
    used += share[k];
  }
  for (; used < resident; ++used) {
    int most = -1;
    for (int k = 0; k < count; ++k)
      if (share[k] < tiles[k] && (most < 0 || tiles[k] * share[most] > tiles[most] * share[k])) most = k;
    if (most < 0) break;
    ++share[most];
  }
  // one workgroup for each of many tiny jobs comes out of the largest share
  for (; used > resident; --used) {
    unsigned *const big = std::max_element(share, share + count);
    if (*big < 2) break;
    --*big;
  }
}
template <int M, int TP, int PS>
static hipError_t launch_z4_grp(GJobs &g, int P, hipStream_t st) {
  const long res = z4_resident<float, M, TP, PS>(P);
  if (P > PS || res < 1) return hipErrorInvalidValue;
  long tiles[kMaxGroupJobs];
  unsigned share[kMaxGroupJobs], nb = 0;
  for (int k = 0; k < g.count; ++k) tiles[k] = (long)(g.j[k].nx / (2 * TP) + 1) * g.j[k].ny;
  z_group_shares(res, g.count, tiles, share);
  for (int k = 0; k < g.count; ++k) {
    g.j[k].nblk = share[k];
    nb += share[k] + (g.j[k].in2 ? 1 : 0);
  }
  hipLaunchKernelGGL((k_zsolve4_grp<M, TP, PS>), dim3(nb), dim3(P * TP), (z4_lds<M, TP, PS>()), st, g);
  return hipGetLastError();
}
// the smallest layout that holds P chunks: F<M, TP, PS>
#define PF_Z4_PICK(TI_, P_, CALL)   \
  if (TI_ == 32) {                  \
    if (P_ <= 4) CALL(16, 4);       \
    if (P_ <= 8) CALL(16, 8);       \
    CALL(16, 16);                   \
  }                                 \
  if (P_ <= 16) CALL(8, 16);        \
  if (P_ <= 32) CALL(8, 32);        \
  if (P_ <= 64) CALL(8, 64);        \
  CALL(8, 128);

template <typename TS>
hipError_t launch_zsolve(int nx, int ny, int nz, TS *data, size_t sp, const double *zal,
                         const double *zga, const double *zex, const double *sx, const double *sy,
                         int variant, hipStream_t st, bool xr, const ZeroJob &zj) {
  // the z tables hold whole 16-row chunks (identity padding past nz)
  if (!zsolve_variant_fits(variant, nx, nz, (int)sizeof(TS))) return hipErrorInvalidValue;
  const ZVariant &z = kZVariants[variant];
  const int P = (nz + z.M - 1) / z.M;
  if (zj.m && !zero_fits(nz, z.paired ? P * z.TI / 2 / z.rounds : P * z.TI)) return hipErrorInvalidValue;
  if (z.persist) {
#define PF_CALL(TP_, PS_) \
  return launch_z4<TS, 8, TP_, PS_>(nx, ny, nz, data, sp, zal, zga, zex, sx, sy, xr, zj, st)
    if constexpr (sizeof(TS) == 8) {
      PF_CALL(8, 16);
    } else {
      PF_Z4_PICK(z.TI, P, PF_CALL)
    }
#undef PF_CALL
  }
  const size_t shm = zsolve_lds(z, P, (int)sizeof(TS));
  dim3 g((unsigned)((long)(nx / z.TI) * ny) + (zj.m ? 1 : 0)), b(z.paired ? P * z.TI / 2 / z.rounds : P * z.TI);
#define PF_ZV(ID, M_, TI_, W_, F_)                                                                \
  case ID:                                                                                        \
    hipLaunchKernelGGL((k_zsolve<TS, M_, TI_, W_, F_>), g, b, shm, st, data, nx, ny, nz, P, zal, \
                       zga, zex, sx, sy, sp, zj);                                                         \
    break;
  switch (variant) {
    PF_ZV(0, 16, 16, 0, false)
    PF_ZV(1, 16, 16, 4, true)
    PF_ZV(2, 16, 16, 0, true)
    PF_ZV(3, 8, 8, 0, true)
    PF_ZV(4, 16, 8, 0, true)
    PF_ZV(5, 8, 16, 0, true)
    PF_ZV(6, 16, 32, 0, true)
    PF_ZV(7, 8, 8, 4, true)
#define PF_ZP(ID, M_, TI_, NR_, W_, SK_)                                                         \
  case ID:                                                                                       \
    hipLaunchKernelGGL((k_zsolve2<TS, M_, TI_ / 2, NR_, W_, SK_>), g, b, shm, st, data, nx, ny,  \
                       nz, P, zal, zga, zex, sx, sy, sp, (int)xr, zj);                                   \
    break;
    PF_ZP(8, 16, 16, 1, 1, true)
    PF_ZP(9, 8, 16, 1, 1, true)
    PF_ZP(10, 16, 32, 1, 1, true)
    PF_ZP(11, 8, 32, 1, 1, true)
    PF_ZP(12, 16, 16, 2, 1, true)
    PF_ZP(13, 8, 8, 1, 1, true)
    PF_ZP(14, 8, 8, 1, 4, true)
    PF_ZP(15, 8, 16, 1, 4, true)
    PF_ZP(16, 8, 8, 1, 4, false)
    PF_ZP(17, 8, 16, 1, 4, false)
#define PF_ZS(ID, M_, TI_, W_)                                                                   \
  case ID:                                                                                       \
    hipLaunchKernelGGL((k_zsolve3<TS, M_, TI_ / 2, 1, W_>), g, b, shm, st, data, nx, ny, nz, P,  \
                       zal, zga, zex, sx, sy, sp, (int)xr, zj);                                          \
    break;
    PF_ZS(18, 8, 8, 4)
    PF_ZS(19, 8, 16, 4)
    PF_ZS(20, 16, 16, 1)
    PF_ZS(21, 16, 32, 1)
    PF_ZS(22, 8, 32, 4)
    PF_ZS(23, 8, 64, 4)
    PF_ZS(24, 8, 128, 4)
    PF_ZS(25, 16, 64, 1)
    PF_ZS(26, 16, 128, 1)
#define PF_ZW(ID, M_, TI_)                                                                       \
  case ID:                                                                                       \
    hipLaunchKernelGGL((k_zsolve3<TS, M_, TI_ / 2, 1, 1, 1024>), g, b, shm, st, data, nx, ny, nz, \
                       P, zal, zga, zex, sx, sy, sp, (int)xr, zj);                                   \
    break;
    PF_ZW(27, 8, 32)
    PF_ZW(28, 8, 16)
#define PF_ZT(ID, M_, TI_, MAXT_, R_)                                                            \
  case ID:                                                                                       \
    hipLaunchKernelGGL((k_zsolve3<TS, M_, TI_ / 2 / R_, 1, 1, MAXT_, true, R_>), g, b, shm, st,   \
                       data, nx, ny, nz, P, zal, zga, zex, sx, sy, sp, (int)xr, zj);                 \
    break;
    PF_ZT(29, 8, 32, 1024, 2)
    PF_ZT(30, 16, 32, 512, 2)
    PF_ZT(31, 8, 16, 1024, 1)
    PF_ZT(32, 16, 16, 512, 1)
    PF_ZT(33, 16, 32, 512, 1)
    PF_ZT(34, 8, 32, 1024, 1)
    PF_ZT(35, 8, 16, 512, 1)
    PF_ZT(36, 8, 32, 512, 2)
  case 37:
    hipLaunchKernelGGL((k_zsolve3<TS, 8, 8, 1, 1, 1024, true, 1, true>), g, b, shm, st, data, nx, ny, nz, P,
                       zal, zga, zex, sx, sy, sp, (int)xr, zj);
    break;
  case 38:
    hipLaunchKernelGGL((k_zsolve3<TS, 8, 8, 1, 1, 1024, false, 1, true>), g, b, shm, st, data, nx, ny, nz, P,
                       zal, zga, zex, sx, sy, sp, (int)xr, zj);
    break;
  case 39:
    hipLaunchKernelGGL((k_zsolve3<TS, 8, 8, 1, 1, 512, true, 1, true>), g, b, shm, st, data, nx, ny, nz, P,
                       zal, zga, zex, sx, sy, sp, (int)xr, zj);
    break;
  case 40:
    hipLaunchKernelGGL((k_zsolve3<TS, 16, 16, 1, 1, 512, false, 1, true>), g, b, shm, st, data, nx, ny, nz,
                       P, zal, zga, zex, sx, sy, sp, (int)xr, zj);
    break;
#undef PF_ZT
#undef PF_ZW
#undef PF_ZS
#undef PF_ZP
    default:
      return hipErrorInvalidValue;
  }
#undef PF_ZV
  return hipGetLastError();
}
bool zsolve_variant_groups(int variant) { return variant >= 18 && variant < kZVariantCount; }
int zsolve_chunks(int variant, int nz) { return (nz + kZVariants[variant].M - 1) / kZVariants[variant].M; }

hipError_t launch_zsolve_grp(int variant, GJobs &g, hipStream_t st) {
  if (!zsolve_variant_groups(variant) || g.count < 1 || g.count > kMaxGroupJobs) return hipErrorInvalidValue;
  const ZVariant &z = kZVariants[variant];
  const int P = (g.j[0].nz + z.M - 1) / z.M;
  unsigned mb = 1;
  for (int k = 0; k < g.count; ++k) {
    GJob &J = g.j[k];
    if ((J.nz + z.M - 1) / z.M != P || J.P != P || !zsolve_variant_fits(variant, J.nx, J.nz, 4))
      return hipErrorInvalidValue;
    J.nblk = (unsigned)((long)(J.nx / z.TI) * J.ny);
    if (J.in2 && (!J.zm || !J.aux || !zero_fits(J.nz, P * z.TI / 2 / z.rounds))) return hipErrorInvalidValue;
    const unsigned nb = J.nblk + (J.in2 ? 1 : 0);
    mb = nb > mb ? nb : mb;
  }
  if (z.persist) {
#define PF_CALL(TP_, PS_) return launch_z4_grp<8, TP_, PS_>(g, P, st)
    PF_Z4_PICK(z.TI, P, PF_CALL)
#undef PF_CALL
  }
  const size_t shm = zsolve_lds(z, P, 4);
  const dim3 gr(mb, (unsigned)g.count), b(P * z.TI / 2 / z.rounds);
#define PF_G(ID, M_, TI_, W_, MAXT_, TILE_, R_)                                                     \
  case ID:                                                                                         \
    hipLaunchKernelGGL((k_zsolve3_grp<M_, TI_ / 2 / R_, 1, W_, MAXT_, TILE_, R_>), gr, b, shm, st, g); \
    break;
  switch (variant) {
    PF_G(18, 8, 8, 4, 512, false, 1)
    PF_G(19, 8, 16, 4, 512, false, 1)
    PF_G(20, 16, 16, 1, 512, false, 1)
    PF_G(21, 16, 32, 1, 512, false, 1)
    PF_G(22, 8, 32, 4, 512, false, 1)
    PF_G(23, 8, 64, 4, 512, false, 1)
    PF_G(24, 8, 128, 4, 512, false, 1)
    PF_G(25, 16, 64, 1, 512, false, 1)
    PF_G(26, 16, 128, 1, 512, false, 1)
    PF_G(27, 8, 32, 1, 1024, false, 1)
    PF_G(28, 8, 16, 1, 1024, false, 1)
    PF_G(29, 8, 32, 1, 1024, true, 2)
    PF_G(30, 16, 32, 1, 512, true, 2)
    PF_G(31, 8, 16, 1, 1024, true, 1)
    PF_G(32, 16, 16, 1, 512, true, 1)
    PF_G(33, 16, 32, 1, 512, true, 1)
    PF_G(34, 8, 32, 1, 1024, true, 1)
    PF_G(35, 8, 16, 1, 512, true, 1)
    PF_G(36, 8, 32, 1, 512, true, 2)
  case 37:
    hipLaunchKernelGGL((k_zsolve3_grp<8, 8, 1, 1, 1024, true, 1, true>), gr, b, shm, st, g);
    break;
  case 38:
    hipLaunchKernelGGL((k_zsolve3_grp<8, 8, 1, 1, 1024, false, 1, true>), gr, b, shm, st, g);
    break;
  case 39:
    hipLaunchKernelGGL((k_zsolve3_grp<8, 8, 1, 1, 512, true, 1, true>), gr, b, shm, st, g);
    break;
  case 40:
    hipLaunchKernelGGL((k_zsolve3_grp<16, 16, 1, 1, 512, false, 1, true>), gr, b, shm, st, g);
    break;
#undef PF_G
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template hipError_t launch_zsolve<double>(int, int, int, double *, size_t, const double *, const double *,
                                          const double *, const double *, const double *, int,
                                          hipStream_t, bool, const ZeroJob &);
template hipError_t launch_zsolve<float>(int, int, int, float *, size_t, const double *, const double *,
                                         const double *, const double *, const double *, int,
                                         hipStream_t, bool, const ZeroJob &);

// ------------------------------------------------------- Helmholtz apply
// Algorithm 2, Steps 2-4, with the Step 1 coefficients of pcr_prepare. One
// wave (64 consecutive columns) per chunk of M rows, so every coefficient
// address is uniform across the wave. Columns are padded to P*M rows with
// identity rows (see the Poisson z solve). The reduced 2P-row system is the
// same for all columns, so its eliminations are precomputed and only the
// right-hand sides cross LDS.
// Read-only tables through the constant address space: wave-uniform reads of
// them stay scalar loads even after the kernel has stored to LDS.
template <typename T>
using cptr = const T __attribute__((address_space(4))) *;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const void *p) {
  return (cptr<T>)p;
}

// The rows of a Step 1 table that a lane's chunk uses, from row r0 on. With
// 64-column chunks r0 is wave-uniform and the tables are read through the
// constant address space as scalar loads (GRow); narrower chunks put two or
// four chunks in a wave, and their tables are read from a copy in LDS
// (LRow): per-lane vector loads of the tables in global memory spilled the
// 32-row shapes, and wave-uniform loads of every chunk of the wave with a
// per-lane select ran out of scalar registers.
template <typename T>
struct GRow {
  cptr<T> t;
  int r0;
  __device__ __forceinline__ T operator[](int q) const { return t[r0 + q]; }
};
template <typename T>
struct LRow {
  const T *t;
  int r0;
  __device__ __forceinline__ T operator[](int q) const { return t[r0 + q]; }
};

__device__ __forceinline__ double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Steps 2-4 on the M rows d of one chunk. Step 3 is a twisted elimination:
// after one barrier every wave reads the 2P reduced right-hand sides of its
// columns and sweeps from the top down to its first reduced row and from the
// bottom up to its last, with the plan's multipliers; the two sweeps meet at
// the chunk's rows. With NBR it also returns the end values of the
// neighbouring chunks, x[2w-1] and x[2w+2] (0 past the walls), by extending
// its sweeps two rows. Those must equal bitwise what the neighbouring waves
// compute for their own rows (the residual has to see the values that are
// stored), so every sweep step is an explicit fused multiply-add: each
// y[r] and z[r] is then the same chain of roundings in every wave. RD holds
// 2P rows of CW values and is written once per call.
template <typename TC, int M, bool NBR, typename RW, typename CP>
__device__ __forceinline__ void helm_solve_regs(TC (&d)[M], RW fa, RW bg, RW ib, RW ra, RW rc, CP tf,
                                                CP tb, CP ti, int P, TC *RD, int w, int lane,
                                                bool active, int CW, TC &below, TC &above) {
  if (active) {
    // Step 2: forward and backward reduction of d
#pragma unroll
    for (int q = 2; q < M; ++q) {
      d[q] = d[q] + fa[q] * d[q - 1];
      sched_fence(q);
    }
#pragma unroll
    for (int q = M - 3; q >= 0; --q) {
      d[q] = d[q] + bg[q] * d[q + 1];
      sched_fence(q);
    }
    RD[(2 * w) * CW + lane] = d[0];
    RD[(2 * w + 1) * CW + lane] = d[M - 1];
  }
  __syncthreads();
  if (!active) return;
  // Step 3: forward sweep y[r] = D[r] + tf[r] y[r-1] down to row lo, backward
  // sweep z[r] = D[r] + tb[r] z[r+1] up to row hi = lo + 1
  const int nr = 2 * P, lo = 2 * w, hi = lo + 1;
  const TC *col = RD + lane;
  TC y = col[0], y1 = TC(0), y2 = TC(0);
#pragma unroll 8
  for (int r = 1; r <= lo; ++r) {
    y2 = y1;
    y1 = y;
    y = fmad(tf[r], y, col[r * CW]);
  }
  TC z = col[(nr - 1) * CW], z1 = TC(0), z2 = TC(0);
  const int nb = nr - 1 - hi;  // rows nr-2 down to hi
#pragma unroll 8
  for (int k = 0; k < nb; ++k) {
    const int r = nr - 2 - k;
    z2 = z1;
    z1 = z;
    z = fmad(tb[r], z, col[r * CW]);
  }
  // x[lo] = (y[lo] + tb z[hi]) ti[lo], x[hi] = (z[hi] + tf y[lo]) ti[hi]
  const TC x0 = fmad(tb[lo], z, y) * ti[lo];
  const TC xl = fmad(tf[hi], y, z) * ti[hi];
  if constexpr (NBR) {
    below = TC(0);
    above = TC(0);
    if (lo > 0) {  // extend the backward sweep by rows lo and lo-1
      const TC zl = fmad(tb[lo], z, col[lo * CW]);
      const TC zm = fmad(tb[lo - 1], zl, col[(lo - 1) * CW]);
      below = fmad(tf[lo - 1], y2, zm) * ti[lo - 1];
    }
    if (hi < nr - 1) {  // extend the forward sweep by rows hi and hi+1
      const TC yh = fmad(tf[hi], y, col[hi * CW]);
      const TC yp = fmad(tf[hi + 1], yh, col[(hi + 1) * CW]);
      above = fmad(tb[hi + 1], z2, yp) * ti[hi + 1];
    }
  }
  // Step 4: rebuild the interior in place
#pragma unroll
  for (int q = 1; q < M - 1; ++q) {
    d[q] = (d[q] + ra[q] * x0 + rc[q] * xl) * ib[q];
    sched_fence(q);
  }
  d[0] = x0;
  d[M - 1] = xl;
}

struct HelmArgs {
  HelmJob job[kMaxHelmJobs];
  int count;
  unsigned wide;  // k_helm_mixed
};

// Steps 2-4 for the chunk of one lane (see k_helm), with the Step 1 rows
// from RW sources (GRow or LRow), the M-matrix rows of the residual from
// constant memory (refinement only) and the reduced system's multipliers
// from constant memory.
template <typename TS, typename TC, int M, bool REFINE, int CW, typename RW>
__device__ __forceinline__ void helm_column(TS *cp, size_t plane, int r0, int n, RW fa, RW bg,
                                            RW ibv, RW ra, RW rc, GRow<double> mal, GRow<double> mga,
                                            GRow<double> mdg, cptr<TC> tf, cptr<TC> tb, cptr<TC> ti,
                                            int P, TC *RD, int w, int lane, bool active) {
  TC below, above;
  if constexpr (!REFINE) {
    TC d[M];
#pragma unroll
    for (int q = 0; q < M; ++q) {
      d[q] = (active && r0 + q < n) ? (TC)cp[(size_t)q * plane] : TC(0);
      if constexpr (CW < 64) sched_fence(q);
    }
    helm_solve_regs<TC, M, false>(d, fa, bg, ibv, ra, rc, tf, tb, ti, P, RD, w, lane, active, CW,
                                  below, above);
    if constexpr (CW < 64) cp = fresh(cp);
    if (active) {
#pragma unroll
      for (int q = 0; q < M; ++q) {
        if (r0 + q < n) cp[(size_t)q * plane] = (TS)d[q];
        if constexpr (CW < 64) sched_fence(q);
      }
    }
  } else {
    static_assert(CW == 64, "narrower chunks eliminate in float64");
    // the float64 right-hand side is held in registers for the residual
    double r[M];
    TC u[M], dd[M];
#pragma unroll
    for (int q = 0; q < M; ++q) {
      r[q] = (active && r0 + q < n) ? (double)cp[(size_t)q * plane] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < M; ++q) u[q] = (TC)r[q];
    // the first solve also gives the neighbours across the chunk ends
    helm_solve_regs<TC, M, true>(u, fa, bg, ibv, ra, rc, tf, tb, ti, P, RD, w, lane, active, CW,
                                 below, above);
    if (active) {
#pragma unroll
      for (int q = 0; q < M; ++q) {
        const double al = mal[q], ga = mga[q], dg = mdg[q];
        const double um = q == 0 ? (double)below : (double)u[q == 0 ? 0 : q - 1];
        const double up = q == M - 1 ? (double)above : (double)u[q == M - 1 ? q : q + 1];
        dd[q] = (TC)(r[q] - (dg * (double)u[q] - al * um - ga * up));
      }
    }
    helm_solve_regs<TC, M, false>(dd, fa, bg, ibv, ra, rc, tf, tb, ti, P, RD + 2 * P * CW, w, lane,
                                  active, CW, below, above);
    if (active) {
#pragma unroll
      for (int q = 0; q < M; ++q) {
        if (r0 + q < n) cp[(size_t)q * plane] = (TS)((double)u[q] + (double)dd[q]);
      }
    }
  }
}

// TS = TC = double (float64), TS = TC = float (float32 storage), or TS =
// double, TC = float with REFINE: a float32 solve, the float64 residual
// r - (I - s L_z) u in registers, a float32 solve for the correction.
// CW columns per chunk: 64 (one wave per chunk, wave-uniform coefficient
// addresses), 32 or 16 (two or four chunks per wave, so that a column of 32
// chunks fits a workgroup; the Step 1 tables are then copied to LDS after
// the reduced rows: 5 P M values of TC). REFINE has 64 only: a column of more
// than 512 rows is eliminated once in float64 instead, because two float32
// solves and the residual between them do not fit the registers of the 1024
// threads that such a column takes (1024x1024x1024, three components: 14.8 ms
// refined with half the rows parked in LDS, 11.0 ms in float64).
template <typename TS, typename TC, int M, int CW, bool REFINE>
__device__ __forceinline__ void helm_body(const HelmJob &J) {
  extern __shared__ double shd[];
  const HelmCoef &C = J.c;
  const int nib = J.nx / CW;
  const long nblk = (long)nib * J.ny;
  if ((long)blockIdx.x >= nblk) return;  // uniform per block
  // the 2P reduced rows of each solve (two solves with REFINE)
  TC *RD = reinterpret_cast<TC *>(shd);
  const int w = CW == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / 64) : threadIdx.x / CW;
  const int lane = threadIdx.x % CW;
  const bool active = w < C.P;
  // narrow chunks (the long columns): every XCD walks a contiguous range of
  // column blocks (2048x1024x1024, three components: float64 27.4 -> 24.1 ms,
  // the float32 forms likewise; the 64-column shapes lost up to 8 %). Only
  // when the launch has no spare blocks beyond this job's count.
  const unsigned bk = CW < 64 && gridDim.x == nblk ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
  const int ib = bk % nib;
  const int j = bk / nib;
  const int r0 = active ? w * M : 0;
  const size_t plane = (size_t)J.nx * J.ny;
  TS *cp = reinterpret_cast<TS *>(J.field) + (size_t)j * J.nx + ib * CW + lane + (size_t)r0 * plane;
  const cptr<TC> tf = as_const<TC>(C.tf), tb = as_const<TC>(C.tb), ti = as_const<TC>(C.ti);
  const GRow<double> mal{as_const<double>(C.al), r0}, mga{as_const<double>(C.ga), r0},
      mdg{as_const<double>(C.dg), r0};
  if constexpr (CW == 64) {
    using R = GRow<TC>;
    helm_column<TS, TC, M, REFINE, CW>(
        cp, plane, r0, C.n, R{as_const<TC>(C.fa), r0}, R{as_const<TC>(C.bg), r0},
        R{as_const<TC>(C.ib), r0}, R{as_const<TC>(C.ra), r0}, R{as_const<TC>(C.rc), r0}, mal, mga, mdg,
        tf, tb, ti, C.P, RD, w, lane, active);
  } else {
    const int npad = C.P * M;
    TC *T0 = reinterpret_cast<TC *>(shd + 2 * C.P * CW);  // past the reduced rows
    TC *fa = T0, *bg = T0 + npad, *ibv = T0 + 2 * npad, *ra = T0 + 3 * npad, *rc = T0 + 4 * npad;
    {
      const TC *sfa = (const TC *)C.fa, *sbg = (const TC *)C.bg, *sib = (const TC *)C.ib;
      const TC *sra = (const TC *)C.ra, *src = (const TC *)C.rc;
      for (int r = threadIdx.x; r < npad; r += blockDim.x) {
        fa[r] = sfa[r]; bg[r] = sbg[r]; ibv[r] = sib[r]; ra[r] = sra[r]; rc[r] = src[r];
      }
    }
    __syncthreads();
    using R = LRow<TC>;
    helm_column<TS, TC, M, REFINE, CW>(cp, plane, r0, C.n, R{fa, r0}, R{bg, r0}, R{ibv, r0}, R{ra, r0},
                                       R{rc, r0}, mal, mga, mdg, tf, tb, ti, C.P, RD, w, lane, active);
  }
}
template <typename TS, typename TC, int M, int CW, bool REFINE>
__global__ __launch_bounds__(1024) void k_helm(HelmArgs args) {
  helm_body<TS, TC, M, CW, REFINE>(args.job[blockIdx.y]);
}
// Refined plans of 32-row chunks of both kinds in one launch: the jobs of args.wide
// refine in 64-column chunks, the others eliminate in float64 in 32-column ones
// (u, v and w of a channel of 513 rows, 513, 513 and 512 unknowns: two launches
// on a 64 x 8 plane took 28 us, one 16.5).
__global__ __launch_bounds__(1024) void k_helm_mixed(HelmArgs args) {
  if (args.wide >> blockIdx.y & 1u) helm_body<double, float, 32, 64, true>(args.job[blockIdx.y]);
  else helm_body<double, double, 32, 32, false>(args.job[blockIdx.y]);
}

// Same algorithm, coefficient tables staged in LDS. A persistent workgroup
// (CW columns per chunk, any CW) copies its job's Step 1 tables into LDS once
// and then walks column blocks; chunks that share a wave read their
// different coefficient rows from LDS instead of global memory, so CW = 32
// gives 512-thread workgroups that keep more than one resident per compute
// unit and overlap one block's loads with another's elimination.
template <typename TC, int M>
__device__ __forceinline__ void helm_solve_lds(TC (&d)[M], TC &x0, TC &xl, int r0, const TC *fa,
                                               const TC *bg, const TC *ib, const TC *ra,
                                               const TC *rc, const TC *k1, const TC *k2,
                                               const TC *invd, int P, int steps, TC *RD, int w,
                                               int lane, bool active, int CW) {
  if (active) {
#pragma unroll
    for (int q = 2; q < M; ++q) d[q] = d[q] + fa[r0 + q] * d[q - 1];
#pragma unroll
    for (int q = M - 3; q >= 0; --q) d[q] = d[q] + bg[r0 + q] * d[q + 1];
  }
  const int nr = 2 * P;
  x0 = d[0];
  xl = d[M - 1];
  for (int st = 0; st < steps; ++st) {
    const int s = 1 << st;
    if (active) {
      RD[(2 * w) * CW + lane] = x0;
      RD[(2 * w + 1) * CW + lane] = xl;
    }
    __syncthreads();
    if (active) {
      const int ra0 = 2 * w, ra1 = 2 * w + 1;
      TC n0 = x0, n1 = xl;
      if (ra0 - s >= 0) n0 += k1[st * nr + ra0] * RD[(ra0 - s) * CW + lane];
      if (ra0 + s < nr) n0 += k2[st * nr + ra0] * RD[(ra0 + s) * CW + lane];
      if (ra1 - s >= 0) n1 += k1[st * nr + ra1] * RD[(ra1 - s) * CW + lane];
      if (ra1 + s < nr) n1 += k2[st * nr + ra1] * RD[(ra1 + s) * CW + lane];
      x0 = n0;
      xl = n1;
    }
    __syncthreads();
  }
  if (active) {
    x0 = x0 * invd[2 * w];
    xl = xl * invd[2 * w + 1];
#pragma unroll
    for (int q = 1; q < M - 1; ++q) d[q] = (d[q] + ra[r0 + q] * x0 + rc[r0 + q] * xl) * ib[r0 + q];
    d[0] = x0;
    d[M - 1] = xl;
  }
}

template <typename TS, typename TC, int M, int CW, bool REFINE>
__global__ __launch_bounds__(512, 4) void k_helm_lds(HelmArgs args) {
  extern __shared__ double shd[];
  const HelmJob &J = args.job[blockIdx.y];
  const HelmCoef &C = J.c;
  const int P = C.P, steps = C.steps, nr = 2 * P, npad = P * M;
  // LDS layout (in TC units unless noted): fa bg ib ra rc [npad each],
  // k1 k2 [steps*nr], invd [nr], RD [nr*CW]; then float64: al ga ep [npad]
  // (refinement only), NB [nr*CW]
  TC *L = reinterpret_cast<TC *>(shd);
  TC *fa = L, *bg = fa + npad, *ibv = bg + npad, *ra = ibv + npad, *rc = ra + npad;
  TC *k1 = rc + npad, *k2 = k1 + steps * nr, *invd = k2 + steps * nr, *RD = invd + nr;
  double *D = reinterpret_cast<double *>(
      (reinterpret_cast<uintptr_t>(RD + nr * CW) + 7) & ~uintptr_t(7));
  double *mal = D, *mga = D + npad, *mdg = D + 2 * npad, *NB = D + 3 * npad;
  {
    const TC *sfa = (const TC *)C.fa, *sbg = (const TC *)C.bg, *sib = (const TC *)C.ib;
    const TC *sra = (const TC *)C.ra, *src = (const TC *)C.rc;
    for (int r = threadIdx.x; r < npad; r += blockDim.x) {
      fa[r] = sfa[r]; bg[r] = sbg[r]; ibv[r] = sib[r]; ra[r] = sra[r]; rc[r] = src[r];
      if (REFINE) { mal[r] = C.al[r]; mga[r] = C.ga[r]; mdg[r] = C.dg[r]; }
    }
    const TC *sk1 = (const TC *)C.k1, *sk2 = (const TC *)C.k2, *sinv = (const TC *)C.invd;
    for (int r = threadIdx.x; r < steps * nr; r += blockDim.x) { k1[r] = sk1[r]; k2[r] = sk2[r]; }
    for (int r = threadIdx.x; r < nr; r += blockDim.x) invd[r] = sinv[r];
  }
  __syncthreads();
  const int w = threadIdx.x / CW;
  const int lane = threadIdx.x % CW;
  const bool active = w < P;
  const int n = C.n;
  const int r0 = active ? w * M : 0;
  const int nib = J.nx / CW;
  const long nblk = (long)nib * J.ny;
  const size_t plane = (size_t)J.nx * J.ny;
  for (long blk = blockIdx.x; blk < nblk; blk += gridDim.x) {   // uniform per block
    const int ibk = (int)(blk % nib);
    const long j = blk / nib;
    TS *cp = reinterpret_cast<TS *>(J.field) + (size_t)j * J.nx + (size_t)ibk * CW + lane +
             (size_t)r0 * plane;
    TC x0, xl;
    if constexpr (!REFINE) {
      TC d[M];
#pragma unroll
      for (int q = 0; q < M; ++q) d[q] = (active && r0 + q < n) ? (TC)cp[(size_t)q * plane] : TC(0);
      helm_solve_lds<TC, M>(d, x0, xl, r0, fa, bg, ibv, ra, rc, k1, k2, invd, P, steps, RD, w,
                            lane, active, CW);
      if (active) {
#pragma unroll
        for (int q = 0; q < M; ++q)
          if (r0 + q < n) cp[(size_t)q * plane] = (TS)d[q];
      }
    } else {
      double r[M];
      TC u[M], dd[M];
#pragma unroll
      for (int q = 0; q < M; ++q) {
        r[q] = (active && r0 + q < n) ? (double)cp[(size_t)q * plane] : 0.0;
        u[q] = (TC)r[q];
      }
      helm_solve_lds<TC, M>(u, x0, xl, r0, fa, bg, ibv, ra, rc, k1, k2, invd, P, steps, RD, w,
                            lane, active, CW);
      if (active) {
        NB[(2 * w) * CW + lane] = (double)u[0];
        NB[(2 * w + 1) * CW + lane] = (double)u[M - 1];
      }
      __syncthreads();
      double below = 0.0, above = 0.0;
      if (active) {
        if (w > 0) below = NB[(2 * w - 1) * CW + lane];
        if (w < P - 1) above = NB[(2 * w + 2) * CW + lane];
      }
      __syncthreads();
      if (active) {
#pragma unroll
        for (int q = 0; q < M; ++q) {
          const double al = mal[r0 + q], ga = mga[r0 + q], dg = mdg[r0 + q];
          const double um = q == 0 ? below : (double)u[q == 0 ? 0 : q - 1];
          const double up = q == M - 1 ? above : (double)u[q == M - 1 ? q : q + 1];
          dd[q] = (TC)(r[q] - (dg * (double)u[q] - al * um - ga * up));
        }
      }
      helm_solve_lds<TC, M>(dd, x0, xl, r0, fa, bg, ibv, ra, rc, k1, k2, invd, P, steps, RD, w,
                            lane, active, CW);
      if (active) {
#pragma unroll
        for (int q = 0; q < M; ++q)
          if (r0 + q < n) cp[(size_t)q * plane] = (TS)((double)u[q] + (double)dd[q]);
      }
    }
  }
}

size_t helm_lds_bytes(int precision, int M, int P, int steps, int CW) {
  const size_t tc = precision == 0 ? 8 : 4;
  const size_t npad = (size_t)P * M, nr = 2 * (size_t)P;
  size_t b = tc * (5 * npad + 2 * steps * nr + nr + nr * CW);
  b = (b + 7) & ~size_t(7);
  b += 8 * (3 * npad + nr * CW);
  return b;
}

int helm_default_cw(int P) { return P <= 16 ? 64 : 32; }

hipError_t launch_helm_mixed(int count, const HelmJob *jobs, unsigned wide, hipStream_t st) {
  if (count < 1 || count > kMaxHelmJobs) return hipErrorInvalidValue;
  HelmArgs a;
  a.count = count;
  a.wide = wide;
  long blocks = 0;
  int threads = 0;
  size_t shm = 0;
  for (int t = 0; t < count; ++t) {
    a.job[t] = jobs[t];
    const int cw = wide >> t & 1u ? 64 : 32, P = jobs[t].c.P;
    if (P < 1 || P * cw > 1024 || jobs[t].nx % cw) return hipErrorInvalidValue;
    blocks = std::max(blocks, (long)(jobs[t].nx / cw) * jobs[t].ny);
    threads = std::max(threads, P * cw);
    // reduced rows; narrow chunks add the float64 Step 1 tables (see k_helm)
    shm = std::max(shm, (size_t)2 * P * cw * sizeof(double) + (cw < 64 ? (size_t)P * 32 * 5 * 8 : 0));
  }
  hipLaunchKernelGGL(k_helm_mixed, dim3((unsigned)blocks, (unsigned)count), dim3(threads), shm, st, a);
  return hipGetLastError();
}

hipError_t launch_helm(int precision, int chunk_rows, int cw, bool staged, int count,
                       const HelmJob *jobs, hipStream_t st) {
  if (count < 1 || count > kMaxHelmJobs) return hipErrorInvalidValue;
  HelmArgs a;
  a.count = count;
  int maxP = 0;
  for (int t = 0; t < count; ++t) maxP = jobs[t].c.P > maxP ? jobs[t].c.P : maxP;
  const int CW = cw;
  if (maxP < 1 || maxP * CW > 1024 || (CW != 16 && CW != 32 && CW != 64)) return hipErrorInvalidValue;
  long maxblk = 0;
  for (int t = 0; t < count; ++t) {
    a.job[t] = jobs[t];
    if (jobs[t].nx % CW) return hipErrorInvalidValue;
    const long nb = (long)(jobs[t].nx / CW) * jobs[t].ny;
    if (nb > maxblk) maxblk = nb;
  }
  if (staged) {
    if (maxP * CW > 512) return hipErrorInvalidValue;
    int maxsteps = 0;
    for (int t = 0; t < count; ++t) maxsteps = jobs[t].c.steps > maxsteps ? jobs[t].c.steps : maxsteps;
    const size_t shm = helm_lds_bytes(precision, chunk_rows, maxP, maxsteps, CW);
    if (shm > 160 * 1024) return hipErrorInvalidValue;
    // persistent: a few workgroups per compute unit walk the column blocks
    const long gx = maxblk < 2048 ? maxblk : 2048;
    dim3 g((unsigned)gx, (unsigned)count), b(CW * maxP);
#define PF_HELMS_CW(M, CWV)                                                                      \
  if (precision == 0)                                                                            \
    hipLaunchKernelGGL((k_helm_lds<double, double, M, CWV, false>), g, b, shm, st, a);           \
  else if (precision == 1)                                                                       \
    hipLaunchKernelGGL((k_helm_lds<float, float, M, CWV, false>), g, b, shm, st, a);             \
  else                                                                                           \
    hipLaunchKernelGGL((k_helm_lds<double, float, M, CWV, true>), g, b, shm, st, a);
#define PF_HELMS(M)                   \
  case M:                             \
    if (CW == 64) {                   \
      PF_HELMS_CW(M, 64)              \
    } else if (CW == 32) {            \
      PF_HELMS_CW(M, 32)              \
    } else {                          \
      PF_HELMS_CW(M, 16)              \
    }                                 \
    break;
    switch (chunk_rows) {
      PF_HELMS(8)
      PF_HELMS(16)
      PF_HELMS(32)
      default:
        return hipErrorInvalidValue;
    }
#undef PF_HELMS
#undef PF_HELMS_CW
    return hipGetLastError();
  }
  dim3 g((unsigned)maxblk, (unsigned)count), b(CW * maxP);
  // the reduced rows: one float64 array, or two float32 arrays (refinement);
  // chunks narrower than a wave add the Step 1 tables (see k_helm)
  if (precision == 2 && CW < 64) return hipErrorInvalidValue;
  size_t shm = (size_t)2 * maxP * CW * sizeof(double);
  if (CW < 64) shm += (size_t)maxP * chunk_rows * 5 * (precision == 0 ? 8 : 4);
  if (shm > 160 * 1024) return hipErrorInvalidValue;
#define PF_HELM_CW(M, CWV)                                                                      \
  if (precision == 0)                                                                           \
    hipLaunchKernelGGL((k_helm<double, double, M, CWV, false>), g, b, shm, st, a);              \
  else if (precision == 1)                                                                      \
    hipLaunchKernelGGL((k_helm<float, float, M, CWV, false>), g, b, shm, st, a);                \
  else if constexpr (CWV == 64)                                                                 \
    hipLaunchKernelGGL((k_helm<double, float, M, CWV, true>), g, b, shm, st, a);
#define PF_HELM(M)                    \
  case M:                             \
    if (CW == 64) {                   \
      PF_HELM_CW(M, 64)               \
    } else if (CW == 32) {            \
      PF_HELM_CW(M, 32)               \
    } else {                          \
      PF_HELM_CW(M, 16)               \
    }                                 \
    break;
  switch (chunk_rows) {
    PF_HELM(8)
    PF_HELM(16)
    PF_HELM(32)
    default:
      return hipErrorInvalidValue;
  }
#undef PF_HELM
#undef PF_HELM_CW
  return hipGetLastError();
}

// ------------------------------------------- Algorithm 2, Step 1 on the device
// The Step 1 coefficients of (I - s L_z) for every chunk, the reduced
// system's twisted-elimination multipliers and its cyclic-reduction
// multipliers, recomputed from the rows of -L_z and s by one workgroup, so
// that a new s (one per Runge-Kutta substep) needs no host work, no copy and
// no synchronisation. Rows in sign-normalised form: row r of I - s L_z is
// -A x[r-1] + (A + G + E) x[r] - G x[r+1] with A = s alpha, G = s gamma,
// E = 1 + s excess; the padding rows (alpha = gamma = excess = 0) are
// identity rows.
//
// Per chunk of m rows (one thread each), eliminating the interior onto the
// two end rows keeps every pivot as a sum of non-negative parts: the forward
// elimination's pivot b = G + a + ef (a the coupling to the chunk's first
// row, ef the carried excess), the backward pass's couplings a, c and excess
// eta. The reduced 2P rows couple chunk ends; they are factored from both
// ends (twisted elimination) and by cyclic reduction, each with the excess
// carried instead of a diagonal formed by subtraction.
constexpr int kPrepRows = 32 * 32;  // P * M at most
__global__ __launch_bounds__(64) void k_pcr_prepare(PcrPrep t, double s) {
  __shared__ double sb[kPrepRows], sa[kPrepRows], sc[kPrepRows], sef[kPrepRows], seta[kPrepRows];
  __shared__ double RA[64], RG[64], RE[64], fe[64], be[64];
  const int tid = threadIdx.x, P = t.P, m = t.M, nr = 2 * P, np = P * m;
  double *T0 = t.d[0], *T1 = t.d[1], *T2 = t.d[2], *T3 = t.d[3], *T4 = t.d[4];
  if (tid < P) {
    const int r0 = tid * m;
    double *b = sb + r0, *a = sa + r0, *c = sc + r0, *ef = sef + r0, *eta = seta + r0;
    auto A = [&](int i) { return s * t.al[r0 + i]; };
    auto G = [&](int i) { return s * t.ga[r0 + i]; };
    auto E = [&](int i) { return 1.0 + s * t.ex[r0 + i]; };
    a[1] = A(1);
    ef[1] = E(1);
    b[1] = G(1) + A(1) + E(1);
    for (int i = 2; i < m; ++i) {
      const double q = A(i) / b[i - 1];
      a[i] = q * a[i - 1];
      ef[i] = E(i) + q * ef[i - 1];
      b[i] = G(i) + a[i] + ef[i];
    }
    c[m - 2] = G(m - 2);
    eta[m - 2] = ef[m - 2];
    for (int i = m - 3; i >= 1; --i) {
      const double q = G(i) / b[i + 1];
      a[i] = a[i] + q * a[i + 1];
      c[i] = q * c[i + 1];
      eta[i] = ef[i] + q * eta[i + 1];
    }
    const double q0 = G(0) / b[1];
    RA[2 * tid] = A(0);
    RG[2 * tid] = q0 * c[1];
    RE[2 * tid] = E(0) + q0 * eta[1];
    RA[2 * tid + 1] = a[m - 1];
    RG[2 * tid + 1] = G(m - 1);
    RE[2 * tid + 1] = ef[m - 1];
    for (int i = 0; i < m; ++i) {
      T0[r0 + i] = i >= 2 ? A(i) / b[i - 1] : 0.0;
      T1[r0 + i] = i <= m - 3 ? G(i) / b[i + 1] : 0.0;
      const bool in = i >= 1 && i <= m - 2;
      T2[r0 + i] = in ? 1.0 / b[i] : 0.0;
      T3[r0 + i] = in ? a[i] : 0.0;
      T4[r0 + i] = in ? c[i] : 0.0;
    }
  }
  __syncthreads();
  // twisted elimination of the reduced rows: forward pivots G + fe,
  // backward pivots A + be, both sums of non-negative parts
  if (tid == 0) {
    fe[0] = RA[0] + RE[0];
    for (int r = 1; r < nr; ++r) fe[r] = RE[r] + RA[r] * fe[r - 1] / (RG[r - 1] + fe[r - 1]);
    be[nr - 1] = RG[nr - 1] + RE[nr - 1];
    for (int r = nr - 2; r >= 0; --r) be[r] = RE[r] + RG[r] * be[r + 1] / (RA[r + 1] + be[r + 1]);
  }
  __syncthreads();
  if (tid < nr) {
    const int r = tid;
    const double fp = r > 0 ? RG[r - 1] + fe[r - 1] : 1.0;
    const double bp = r < nr - 1 ? RA[r + 1] + be[r + 1] : 1.0;
    const double lo = r > 0 ? RA[r] * fe[r - 1] / fp : RA[r];
    const double hi = r < nr - 1 ? RG[r] * be[r + 1] / bp : RG[r];
    t.d[8][r] = r > 0 ? RA[r] / fp : 0.0;
    t.d[9][r] = r < nr - 1 ? RG[r] / bp : 0.0;
    t.d[10][r] = 1.0 / (RE[r] + lo + hi);
  }
  // cyclic reduction of the reduced rows: step st couples rows 2^st apart;
  // the new excess is the old one plus the eliminated neighbours' excesses
  for (int st = 0; st < t.steps; ++st) {
    const int h = 1 << st;
    double nA = 0.0, nG = 0.0, nE = 0.0;
    if (tid < nr) {
      const int r = tid;
      double k1 = 0.0, k2 = 0.0, em = 0.0, ep2 = 0.0, am = 0.0, gp = 0.0;
      if (r - h >= 0) {
        k1 = RA[r] / (RA[r - h] + RG[r - h] + RE[r - h]);
        am = RA[r - h];
        em = RE[r - h];
      }
      if (r + h < nr) {
        k2 = RG[r] / (RA[r + h] + RG[r + h] + RE[r + h]);
        gp = RG[r + h];
        ep2 = RE[r + h];
      }
      t.d[5][st * nr + r] = k1;
      t.d[6][st * nr + r] = k2;
      nA = k1 * am;
      nG = k2 * gp;
      nE = RE[r] + k1 * em + k2 * ep2;
    }
    __syncthreads();
    if (tid < nr) {
      RA[tid] = nA;
      RG[tid] = nG;
      RE[tid] = nE;
    }
    __syncthreads();
  }
  if (tid < nr) t.d[7][tid] = 1.0 / (RA[tid] + RG[tid] + RE[tid]);
  // the float32 copies and the M-matrix rows of the refinement's residual
  __syncthreads();
  const int len[11] = {np, np, np, np, np, t.steps * nr, t.steps * nr, nr, nr, nr, nr};
  for (int k = 0; k < 11; ++k)
    for (int i = tid; i < len[k]; i += 64) t.f[k][i] = (float)t.d[k][i];
  for (int r = tid; r < np; r += 64) {
    const double a = s * t.al[r], g = s * t.ga[r], e = 1.0 + s * t.ex[r];
    t.mA[r] = a;
    t.mG[r] = g;
    t.mE[r] = e;
    t.mD[r] = a + g + e;
  }
}

hipError_t launch_pcr_prepare(const PcrPrep &p, double s, hipStream_t st) {
  if (p.P < 1 || p.P > 32 || p.P * p.M > kPrepRows || p.M < 3) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pcr_prepare, dim3(1), dim3(64), 0, st, p, s);
  return hipGetLastError();
}

// dst[i] = src[i] + kappa: the x-slot shifts of a 3-D Helmholtz plan for a
// new s (kappa = 1/s)
__global__ __launch_bounds__(256) void k_shift_add(const double *__restrict__ src, double *__restrict__ dst,
                                                   int n, double kappa) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src[i] + kappa;
}

hipError_t launch_shift_add(const double *src, double *dst, int n, double kappa, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_shift_add, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, n, kappa);
  return hipGetLastError();
}

// ------------------------------------------------------------ plain copy
// The fastest copy measured on MI355X (4 GiB: 5.6 TB/s, against 4.9 TB/s for
// one 16-byte element per thread and grid stride): four 16-byte nontemporal
// loads in flight per thread over a 16 KiB block tile, 16384 workgroups
// striding over the tiles, then the tail one element per thread.
typedef unsigned int pf_v4u __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_copy(const pf_v4u *__restrict__ src, pf_v4u *__restrict__ dst,
                                              size_t n) {
  constexpr int U = 4;
  constexpr size_t kTile = (size_t)256 * U;
  const size_t full = n / kTile * kTile;
  for (size_t b = (size_t)blockIdx.x * kTile; b < full; b += (size_t)gridDim.x * kTile) {
    pf_v4u v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(src + b + u * 256 + threadIdx.x);
#pragma unroll
    for (int u = 0; u < U; ++u) __builtin_nontemporal_store(v[u], dst + b + u * 256 + threadIdx.x);
  }
  for (size_t i = full + (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
    dst[i] = src[i];
}

hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 16;
  size_t blocks = (n + 1023) / 1024;
  if (blocks > 16384) blocks = 16384;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)blocks), dim3(256), 0, st, (const pf_v4u *)src,
                     (pf_v4u *)dst, n);
  return hipGetLastError();
}

}  // namespace pf
