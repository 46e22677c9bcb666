// Complex FFT engine that keeps its lines in registers.
//
// fft_lds.hpp holds a line as N complex float64 values in LDS, 16 bytes a
// point, which for long lines is the whole of what a compute unit can hold:
// one workgroup, whose loads, passes and stores then run back to back. Here
// every thread holds its N / TPL points of a line in registers from the
// first pass to the last, and the LDS only carries the exchange between two
// passes, the real parts first and the imaginary parts after them through the
// same array: 8 bytes a point, so that twice the lines, or two workgroups
// where one fitted, share a compute unit. The passes are the same Stockham
// passes (radix 16 and less, composite radices by the prime-factor mapping),
// in an order per length whose butterflies fill the threads of a line.
#pragma once
#include "fft_lds.hpp"

namespace pf {

// R = R1 R2 with coprime factors, without twiddles (Good's mapping): input
// n = (R2 n1 + R1 n2) mod R, output k = k1 mod R1 = k2 mod R2.
__host__ __device__ constexpr int pfa_out(int r1, int r2, int k1, int k2) {
  for (int k = 0; k < r1 * r2; ++k)
    if (k % r1 == k1 && k % r2 == k2) return k;
  return 0;
}
template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_any(cplx<T> *v);
template <typename T, int R1, int R2, bool INV>
__device__ __forceinline__ void dft_pfa(cplx<T> *v) {
  cplx<T> y[R2][R1];
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) y[n2][n1] = v[(R2 * n1 + R1 * n2) % (R1 * R2)];
    dft_any<T, R1, INV>(y[n2]);
  }
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) {
    cplx<T> b[R2];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) b[n2] = y[n2][k1];
    dft_any<T, R2, INV>(b);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) v[pfa_out(R1, R2, k1, k2)] = b[k2];
  }
}
template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_any(cplx<T> *v) {
  if constexpr (R == 6) dft_pfa<T, 2, 3, INV>(v);
  else if constexpr (R == 10) dft_pfa<T, 2, 5, INV>(v);
  else if constexpr (R == 12) dft_pfa<T, 4, 3, INV>(v);
  else if constexpr (R == 18) dft_pfa<T, 2, 9, INV>(v);
  else if constexpr (R == 20) dft_pfa<T, 4, 5, INV>(v);
  else dft_r<T, R, INV>(v);
}

// The passes of a length and the threads of a line.
template <int N> struct LinePlan;
#define PF_LINE_PLAN(N, TPL_, ...) PF_PLAN(LinePlan, N, TPL_, __VA_ARGS__)
#define PF_PLAN(NAME, N, TPL_, ...)                             \
  template <> struct NAME<N> {                                  \
    static constexpr int n = N;                                 \
    static constexpr int radix[] = {__VA_ARGS__};               \
    static constexpr int passes = sizeof(radix) / sizeof(int);  \
    static constexpr int tpl = TPL_;                            \
    static constexpr int ns(int i) {                            \
      int s = 1;                                                \
      for (int k = 0; k < i; ++k) s *= radix[k];                \
      return s;                                                 \
    }                                                           \
    static_assert(N % TPL_ == 0, "whole points per thread");    \
  };
PF_LINE_PLAN(192, 12, 16, 12)
PF_LINE_PLAN(256, 16, 16, 16)
PF_LINE_PLAN(384, 24, 16, 4, 6)
PF_LINE_PLAN(512, 32, 16, 8, 4)
PF_LINE_PLAN(768, 48, 16, 8, 6)
PF_LINE_PLAN(1024, 64, 16, 8, 8)
PF_LINE_PLAN(1536, 96, 16, 16, 6)
PF_LINE_PLAN(2048, 128, 16, 16, 8)
PF_LINE_PLAN(3072, 192, 16, 16, 12)
PF_LINE_PLAN(3200, 200, 16, 20, 10)
PF_LINE_PLAN(3456, 216, 16, 18, 12)
#undef PF_LINE_PLAN
// The same lengths and threads with a last pass of radix 8 and two butterflies
// a thread, j and N/8 - j: a thread then ends with positions q and N - q in
// its own registers, for the transforms that fold a spectrum with its mirror
// image.
template <int N> struct PairPlan;
PF_PLAN(PairPlan, 192, 12, 8, 3, 8)
PF_PLAN(PairPlan, 256, 16, 8, 4, 8)
PF_PLAN(PairPlan, 384, 24, 16, 3, 8)
PF_PLAN(PairPlan, 512, 32, 16, 4, 8)
PF_PLAN(PairPlan, 768, 48, 16, 6, 8)
PF_PLAN(PairPlan, 1024, 64, 16, 8, 8)
PF_PLAN(PairPlan, 1536, 96, 16, 12, 8)
PF_PLAN(PairPlan, 2048, 128, 16, 16, 8)
PF_PLAN(PairPlan, 3072, 192, 16, 4, 6, 8)
PF_PLAN(PairPlan, 3200, 200, 16, 5, 5, 8)
PF_PLAN(PairPlan, 3456, 216, 16, 9, 3, 8)
// The reverse: a first pass of radix 8 on the butterflies j and N/8 - j, for
// inverses that unfold such a spectrum as they read it.
template <int N> struct UnpairPlan;
PF_PLAN(UnpairPlan, 192, 12, 8, 3, 8)
PF_PLAN(UnpairPlan, 256, 16, 8, 4, 8)
PF_PLAN(UnpairPlan, 384, 24, 8, 3, 16)
PF_PLAN(UnpairPlan, 512, 32, 8, 4, 16)
PF_PLAN(UnpairPlan, 768, 48, 8, 6, 16)
PF_PLAN(UnpairPlan, 1024, 64, 8, 8, 16)
PF_PLAN(UnpairPlan, 1536, 96, 8, 12, 16)
PF_PLAN(UnpairPlan, 2048, 128, 8, 16, 16)
PF_PLAN(UnpairPlan, 3072, 192, 8, 6, 4, 16)
PF_PLAN(UnpairPlan, 3200, 200, 8, 5, 5, 16)
PF_PLAN(UnpairPlan, 3456, 216, 8, 3, 9, 16)
#undef PF_PLAN
#define PF_FOR_LINE_PLANS(X) X(192) X(256) X(384) X(512) X(768) X(1024) X(1536) X(2048) X(3072) X(3200) X(3456)

// threads of a line, 0 for a length without a plan
constexpr int rx_tpl(int n) {
  switch (n) {
#define PF_CASE(N) \
  case N:          \
    return LinePlan<N>::tpl;
    PF_FOR_LINE_PLANS(PF_CASE)
#undef PF_CASE
    default:
      return 0;
  }
}

// v[r] times W^(e r), from one table read W^e (two, W^(4e) too, from radix 8
// on): the powers r = 4 m + d as products of W^(4 m) and W^d, made where they
// are used. The scheduling barriers keep the compiler from making them all
// first, which took 40 registers more and a third of the waves.
template <typename T, int R>
__device__ __forceinline__ void apply_twiddles(cplx<T> (&v)[R], cplx<T> w1, cplx<T> w4, bool inv) {
  const cplx<T> w2 = cmul<T>(w1, w1), w3 = R > 3 ? cmul<T>(w2, w1) : w2;
  if (R < 8 && R > 4) w4 = cmul<T>(w2, w2);
  auto mul = [&](cplx<T> &x, cplx<T> w) { x = inv ? cmulc<T>(x, w) : cmul<T>(x, w); };
  cplx<T> hi = w4;
#pragma unroll
  for (int m = 0; 4 * m < R; ++m) {
    if (m >= 2) hi = cmul<T>(hi, w4);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if (4 * m + d == 0 || 4 * m + d >= R) continue;
      const cplx<T> lo = d == 1 ? w1 : d == 2 ? w2 : w3;
      mul(v[4 * m + d], m == 0 ? lo : d == 0 ? hi : cmul<T>(hi, lo));
    }
    if (R >= 8) __builtin_amdgcn_sched_barrier(0);
  }
}

// One padding value per 16, and the stride between the lines of a workgroup
// whose lanes run over the LPW lines first: 32 / LPW mod 32, so that the 32
// lanes of one 64-bit LDS access hit different bank pairs in the strided
// writes of the first exchange and in the contiguous ones after it.
__host__ __device__ constexpr int rx_idx(int i) { return i + (i >> 4); }
// the slot of position i + c for c a multiple of 16: a constant away from i's
__host__ __device__ constexpr int rx_off(int c) { return c + c / 16; }
__host__ __device__ constexpr int rx_stride(int n, int lpw) {
  int s = rx_idx(n);
  while (s % 32 != (32 / lpw) % 32) ++s;
  return s;
}

// Butterfly `it` of thread t in pass I: t + it TPL, or in the last pass of a
// kPair transform (the first of a kUnpair one) the butterflies t and NB - t
// (0 and NB/2 for t = 0).
enum : int { kPlain = 0, kPair = 1, kUnpair = 2 };
template <class P, int I, int PAIR>
__device__ __forceinline__ int rx_butterfly(int t, int it) {
  constexpr int NB = P::n / P::radix[I];
  if constexpr ((PAIR == kPair && I + 1 == P::passes) || (PAIR == kUnpair && I == 0)) {
    static_assert(NB == 2 * P::tpl, "two butterflies a thread");
    return it == 0 ? t : (t == 0 ? NB / 2 : NB - t);
  }
  return t + it * P::tpl;
}

// Pass I of a line on the thread's butterflies v[it][r] (inputs j + r N/R, j
// = rx_butterfly), then the passes after it. The last pass hands its
// outputs to dst(j, c, value, it, r), for position j + c, c the same in every
// thread; a kPair transform hands dst(j, c, value, mirror, it, r), mirror the
// value at position N - (j + c) (mod N). sync_last (uniform): dst writes the
// LDS, so the last exchange ends with a barrier.
template <class P, int I, bool INV, int PAIR = kPlain, class V, int IT, int R, class Dst>
__device__ __forceinline__ void rx_passes(double *buf, const cplx<double> *__restrict__ tw, int t, V (&v)[IT][R],
                                          bool sync_last, Dst dst) {
  constexpr int N = P::n, TPL = P::tpl, NS = P::ns(I), NB = N / R;
  static_assert(R == P::radix[I] && IT == (NB + TPL - 1) / TPL, "butterflies of a pass");
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int j = rx_butterfly<P, I, PAIR>(t, it);
    if (NB % TPL == 0 || j < NB) {
      if constexpr (NS > 1) {
        const int e = (j % NS) * (N / (NS * R));
        const cplx<double> w1 = tw[e], w4 = R >= 8 ? tw[4 * e] : w1;
        apply_twiddles<double, R>(v[it], w1, w4, INV);
      }
      dft_any<double, R, INV>(v[it]);
      if (IT > 1) __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (I + 1 == P::passes) {
    static_assert(NS * R == N, "the radices multiply to the length");
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int j = rx_butterfly<P, I, PAIR>(t, it);
      if (NB % TPL == 0 || j < NB) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if constexpr (PAIR == kPair) {
            const V o = v[1 - it][R - 1 - r], s = it == 0 ? v[0][(R - r) % R] : v[1][R - 1 - r];
            dst(j, r * NS, v[it][r], mkc<double>(t ? o.x : s.x, t ? o.y : s.y), it, r);
          } else {
            dst(j, r * NS, v[it][r], it, r);
          }
        }
      }
    }
  } else {
    constexpr int R2 = P::radix[I + 1], NB2 = N / R2, IT2 = (NB2 + TPL - 1) / TPL;
    V w[IT2][R2];
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int j = rx_butterfly<P, I, PAIR>(t, it);
        if (NB % TPL == 0 || j < NB) {
          // constant offsets from one slot of a butterfly where the padding
          // allows them
          constexpr bool kConst = NS % 16 == 0 || (NS == 1 && (R == 16 || R == 8));
          const int p0 = (j / NS) * NS * R + (j % NS);
          double *b = buf + rx_idx(p0);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double x = part ? v[it][r].y : v[it][r].x;
            if constexpr (kConst) b[NS == 1 ? r : rx_off(r * NS)] = x;
            else buf[rx_idx(p0 + r * NS)] = x;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < IT2; ++it) {
        const int j = rx_butterfly<P, I + 1, PAIR>(t, it);
        if (NB2 % TPL == 0 || j < NB2) {
          const double *b = buf + rx_idx(j);
#pragma unroll
          for (int r = 0; r < R2; ++r) {
            const double x = NB2 % 16 == 0 ? b[rx_off(r * NB2)] : buf[rx_idx(j + r * NB2)];
            if (part) w[it][r].y = x;
            else w[it][r].x = x;
          }
        }
      }
      if (part == 0 || I + 2 < P::passes || sync_last) __syncthreads();
    }
    rx_passes<P, I + 1, INV, PAIR>(buf, tw, t, w, sync_last, dst);
  }
}

// The thread's first-pass butterflies and their inputs through src(j, c), for
// position j + c.
template <class P> struct RxFirst {
  static constexpr int R = P::radix[0], NB = P::n / R, IT = (NB + P::tpl - 1) / P::tpl;
  using Regs = cplx<double>[IT][R];
};
template <class P, class V, int IT, int R, class Src>
__device__ __forceinline__ void rx_load(V (&v)[IT][R], int t, Src src) {
  using F = RxFirst<P>;
  static_assert(IT == F::IT && R == F::R, "registers of the first pass");
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int j = t + it * P::tpl;
    if (F::NB % P::tpl == 0 || j < F::NB) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[it][r] = src(j, r * F::NB);
    }
  }
}

}  // namespace pf
