// Length-N transforms of even N = 2M held whole in registers, two lanes to a line.
//
// Every y and z transform of the plane kernels has at most K + 1 + K frequencies that a
// sphere function reaches, n in [-K, K] with K = (N - 1) / 4 (the grid holds products of
// two of them), and all N points on the other side. Lane p of a pair takes the points
// p + 2 k, k < M:
//   X[p + 2 k] = sum_n x[n] e^{+- 2 pi i n p / N} e^{+- 2 pi i n k / M},
// and as n and n - M never both are reached, that is one twiddle per frequency and one
// M-point DFT in registers: the half of the first radix-2 stage that would only add zeros
// is not there, and no value is exchanged. Back from points to frequencies it is the
// transpose: an M-point DFT of the lane's own points, one twiddle per frequency, and the
// sum of the two lanes' parts, which is one exchange with the neighbouring lane (DPP); the
// even lane ends up with n >= 0, the odd one with n < 0.
#pragma once
#include "fft_dev.hpp"

namespace stern {

template <>
struct Split<18> { static constexpr int A = 9, B = 2; };
template <>
struct Split<24> { static constexpr int A = 8, B = 3; };
template <>
struct Split<27> { static constexpr int A = 9, B = 3; };
template <>
struct Split<32> { static constexpr int A = 8, B = 4; };
template <>
struct Split<36> { static constexpr int A = 9, B = 4; };
template <>
struct Split<48> { static constexpr int A = 16, B = 3; };
template <>
struct Split<54> { static constexpr int A = 27, B = 2; };
template <>
struct Split<64> { static constexpr int A = 8, B = 8; };

constexpr int pfa_gcd(int a, int b) { return b == 0 ? a : pfa_gcd(b, a % b); }
// Good and Thomas: for coprime A and B the DFT of A B values is A x B with no twiddles between, input
// (a, b) at (B a + A b) mod A B, output (k, l) where it is k mod A and l mod B (the index maps are
// compile-time constants of the unrolled code)
template <int A, int B>
__device__ constexpr int pfa_in(int a, int b) {
  return (B * a + A * b) % (A * B);
}
template <int A, int B>
__device__ constexpr int pfa_out(int k, int l) {
  int n = k;
  while (n % B != l) n += A;
  return n;
}

// DFT of M = A B values in registers, one sub-transform after the other: the barriers keep the
// scheduler from running several at once, whose extra live values would not fit.
template <int A, int B, int DIR, class T, int... N2>
__device__ __forceinline__ void dft_steps_first(const Z<T>* v, Z<T>* y, std::integer_sequence<int, N2...>) {
  ((composite_first<A, B, DIR, T, N2>(v, y), __builtin_amdgcn_sched_barrier(0)), ...);
}
template <int A, int B, int DIR, int K1, class T, int... L>
__device__ __forceinline__ void pfa_last(const Z<T>* y, Z<T>* v, std::integer_sequence<int, L...>) {
  Z<T> s[B];
  ((s[L] = y[L * A + K1]), ...);
  dft<B, DIR>(s);
  ((v[std::integral_constant<int, pfa_out<A, B>(K1, L)>::value] = s[L]), ...);
  __builtin_amdgcn_sched_barrier(0);
}
template <int A, int B, int DIR, class T, int... K1>
__device__ __forceinline__ void pfa_all_last(const Z<T>* y, Z<T>* v, std::integer_sequence<int, K1...>) {
  (pfa_last<A, B, DIR, K1>(y, v, std::make_integer_sequence<int, B>{}), ...);
}
template <int M, int DIR, class T>
__device__ __forceinline__ void dft_steps(Z<T>* v) {
  if constexpr (M <= 9 && M != 6) {
    dft<M, DIR>(v);
  } else {
    constexpr int A = Split<M>::A, B = Split<M>::B;
    Z<T> y[M];
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (pfa_gcd(A, B) == 1) {
#pragma unroll
      for (int b = 0; b < B; ++b) {
        Z<T> s[A];
#pragma unroll
        for (int a = 0; a < A; ++a) s[a] = v[pfa_in<A, B>(a, b)];
        dft<A, DIR>(s);
#pragma unroll
        for (int k = 0; k < A; ++k) y[b * A + k] = s[k];
        __builtin_amdgcn_sched_barrier(0);
      }
      pfa_all_last<A, B, DIR>(y, v, std::make_integer_sequence<int, A>{});
    } else {
      dft_steps_first<A, B, DIR, T>(v, y, std::make_integer_sequence<int, B>{});
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) {
        Z<T> s[B];
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) s[n2] = y[n2 * A + k1];
        dft<B, DIR>(s);
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = s[k2];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// the value of the other lane of the pair
__device__ __forceinline__ float pair_swap(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ double pair_swap(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0xB1, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0xB1, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

template <int N, class T>
struct HalfFft {
  static constexpr int M = N / 2, K = (N - 1) / 4;
  // twiddles e^{2 pi i n p / N}, n = 0..K, of one lane parity; an odd stride keeps the two parities' tables
  // on different banks
  static constexpr int TW = (K + 1) | 1;

  // table of both parities in LDS from the global one, exp(-2 pi i m / N); zero beyond nm, the
  // largest frequency that is reached, so that what is loaded there does not matter
  static __device__ __forceinline__ void twiddles(Z<T>* t, const Z<T>* __restrict__ tw, int nm, int tid, int nt) {
    for (int i = tid; i < 2 * TW; i += nt) {
      const int n = i % TW;
      t[i] = n > nm ? zmk(T(0), T(0)) : i < TW ? zmk(T(1), T(0)) : zconj(tw[n]);  // n <= K + 1 < N
    }
  }

  // v[k] = X[p + 2 k] for frequencies x(n) = ld(n), n in [-K, K]; t: this lane's twiddles
  template <class Ld>
  static __device__ __forceinline__ void to_points(Z<T> (&v)[M], const Z<T>* t, Ld ld) {
    v[0] = ld(0);
#pragma unroll
    for (int n = K + 1; n < M - K; ++n) v[n] = zmk(T(0), T(0));
#pragma unroll
    for (int n = 1; n <= K; ++n) {
      v[n] = ld(n);
      v[M - n] = ld(-n);
    }
    __builtin_amdgcn_sched_barrier(0);  // all loads issued; the twiddles come in small groups
#pragma unroll
    for (int n = 1; n <= K; ++n) {
      const Z<T> a = v[n], b = v[M - n], w = t[n];
      v[n] = zmk(a.re * w.re - a.im * w.im, a.im * w.re + a.re * w.im);
      v[M - n] = zmk(b.re * w.re + b.im * w.im, b.im * w.re - b.re * w.im);
      if (n % 6 == 0) __builtin_amdgcn_sched_barrier(0);
    }
    dft_steps<M, +1>(v);
  }

  // frequencies of the points v[k] at p + 2 k (destroyed): calls st(n, x) for n = K, ..., 1 with the
  // frequency n in the even lane and -n in the odd one, last st(0, x) in both. Both lanes of a pair
  // take part.
  template <class St>
  static __device__ __forceinline__ void to_freqs(Z<T> (&v)[M], const Z<T>* t, bool odd, St st) {
    dft_steps<M, -1>(v);
#pragma unroll
    for (int n = K; n >= 1; --n) {
      const Z<T> a = v[n], b = v[M - n], w = t[n];
      const Z<T> ua = zmk(a.re * w.re + a.im * w.im, a.im * w.re - a.re * w.im);
      const Z<T> ub = zmk(b.re * w.re - b.im * w.im, b.im * w.re + b.re * w.im);
      const Z<T> keep = odd ? ub : ua, send = odd ? ua : ub;
      st(n, zmk(keep.re + pair_swap(send.re), keep.im + pair_swap(send.im)));
      if (n % 4 == 0) __builtin_amdgcn_sched_barrier(0);
    }
    st(0, zmk(v[0].re + pair_swap(v[0].re), v[0].im + pair_swap(v[0].im)));
  }
};

// The same from frequencies to points with four lanes to a line, N = 4 M: lane p takes the points p + 4 k,
// k < M, with both of a residue's frequencies n and n - M folded into its input. A third more arithmetic than
// two lanes, for half the registers: for kernels that keep sums of the points beside them.
template <int N, class T>
struct QuarterFft {
  static constexpr int M = N / 4, K = (N - 1) / 4;  // K = M - 1
  static constexpr int TW = M | 1;                  // twiddles e^{2 pi i n p / N}, n = 0..K, of one lane

  static __device__ __forceinline__ void twiddles(Z<T>* t, const Z<T>* __restrict__ tw, int nm, int tid, int nt) {
    for (int i = tid; i < 4 * TW; i += nt) {
      const int n = i % TW, p = i / TW;
      t[i] = n > nm ? zmk(T(0), T(0)) : zconj(tw[n * p % N]);
    }
  }

  template <class Ld>
  static __device__ __forceinline__ void to_points(Z<T> (&v)[M], const Z<T>* t, Ld ld) {
    v[0] = ld(0);
#pragma unroll
    for (int n = 1; n < M; ++n) v[n] = ld(n);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 1; n < M; ++n) {
      const Z<T> a = v[n], b = ld(n - M), w = t[n], u = t[M - n];
      v[n] = zmk(a.re * w.re - a.im * w.im + b.re * u.re + b.im * u.im,
                 a.im * w.re + a.re * w.im + b.im * u.re - b.re * u.im);
      if (n % 6 == 0) __builtin_amdgcn_sched_barrier(0);
    }
    dft_steps<M, +1>(v);
  }
};

}  // namespace stern
