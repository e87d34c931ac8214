// Small forward DFTs in registers for the stages of the general kernels:
// radices 2..16 without twiddle tables (2, 3, 4, 5, 8, 16: hp_device.hpp).
#pragma once

#include "hp_device.hpp"

namespace hp {

// cos and sin of 2 pi j / R, 1 <= j <= (R - 1) / 2, of the odd primes 7, 11, 13.
template <int R>
struct OddTrig;
template <>
struct OddTrig<7> {
  static constexpr double c[3] = {0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624};
  static constexpr double s[3] = {0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048};
};
template <>
struct OddTrig<11> {
  static constexpr double c[5] = {0.84125353283118116886, 0.41541501300188642553, -0.14231483827328514044,
                                  -0.65486073394528506406, -0.95949297361449738989};
  static constexpr double s[5] = {0.54064081745559758211, 0.90963199535451837141, 0.98982144188093273238,
                                  0.75574957435425828377, 0.28173255684142969771};
};
template <>
struct OddTrig<13> {
  static constexpr double c[6] = {0.88545602565320989590,  0.56806474673115580251,  0.12053668025532305335,
                                  -0.35460488704253562597, -0.74851074817110109863, -0.97094181742605202716};
  static constexpr double s[6] = {0.46472317204376854566, 0.82298386589365639458, 0.99270887409805399280,
                                  0.93501624268541482344, 0.66312265824079520238, 0.23931566428755776715};
};

// Odd prime R by the even / odd parts of the input: with s_t = v_t + v_{R-t}
// and d_t = v_t - v_{R-t}, X_u, X_{R-u} = v_0 + sum_t s_t cos(2 pi t u / R)
// -+ i sum_t d_t sin(2 pi t u / R): a quarter of the direct sum's products.
template <typename T, int R>
__device__ __forceinline__ void dft_odd(C2<T>* v) {
  constexpr int H = (R - 1) / 2;
  C2<T> s[H], d[H];
  C2<T> sum = v[0];
#pragma unroll
  for (int t = 0; t < H; ++t) {
    s[t] = cadd(v[t + 1], v[R - 1 - t]);
    d[t] = csub(v[t + 1], v[R - 1 - t]);
    sum = cadd(sum, s[t]);
  }
  C2<T> out[R];
#pragma unroll
  for (int u = 1; u <= H; ++u) {
    C2<T> C = v[0], S = {(T)0, (T)0};
#pragma unroll
    for (int t = 1; t <= H; ++t) {
      const int m = (t * u) % R;
      const T c = (T)OddTrig<R>::c[(m <= H ? m : R - m) - 1];
      const T sn = (T)(m <= H ? OddTrig<R>::s[m - 1] : -OddTrig<R>::s[R - m - 1]);
      C = cadd(C, cscale(s[t - 1], c));
      S = cadd(S, cscale(d[t - 1], sn));
    }
    out[u] = {C.re + S.im, C.im - S.re};      // C - i S
    out[R - u] = {C.re - S.im, C.im + S.re};  // C + i S
  }
  v[0] = sum;
#pragma unroll
  for (int u = 1; u < R; ++u) v[u] = out[u];
}

template <typename T, int R>
__device__ __forceinline__ void dft_any(C2<T>* v);

// N1 and N2 coprime: inputs n = N2 n1 + N1 n2, outputs k with k mod N1 = k1
// and k mod N2 = k2 (mod N1 N2); the two index maps leave no twiddles.
template <typename T, int N1, int N2>
__device__ __forceinline__ void dft_coprime(C2<T>* v) {
  constexpr int N = N1 * N2;
  C2<T> a[N2][N1];
#pragma unroll
  for (int n2 = 0; n2 < N2; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < N1; ++n1) a[n2][n1] = v[(N2 * n1 + N1 * n2) % N];
    dft_any<T, N1>(a[n2]);
  }
  auto inv = [](int x, int m) constexpr {
    int i = 1;
    while ((x * i) % m != 1) ++i;
    return i;
  };
  constexpr int e1 = N2 * inv(N2 % N1, N1), e2 = N1 * inv(N1 % N2, N2);
#pragma unroll
  for (int k1 = 0; k1 < N1; ++k1) {
    C2<T> b[N2];
#pragma unroll
    for (int n2 = 0; n2 < N2; ++n2) b[n2] = a[n2][k1];
    dft_any<T, N2>(b);
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) v[(e1 * k1 + e2 * k2) % N] = b[k2];
  }
}

template <typename T>
__device__ __forceinline__ void dft9(C2<T>* v) {
  // 3 x 3 with the twiddles W_9^(n2 k1)
  const C2<T> w1 = {(T)0.76604444311897803520, (T)-0.64278760968653932632};
  const C2<T> w2 = {(T)0.17364817766693034885, (T)-0.98480775301220805937};
  const C2<T> w4 = {(T)-0.93969262078590838405, (T)-0.34202014332566873304};
  C2<T> a[3][3];
#pragma unroll
  for (int n2 = 0; n2 < 3; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < 3; ++n1) a[n2][n1] = v[3 * n1 + n2];
    dft3<T, false>(a[n2]);
  }
  a[1][1] = cmul(a[1][1], w1);
  a[1][2] = cmul(a[1][2], w2);
  a[2][1] = cmul(a[2][1], w2);
  a[2][2] = cmul(a[2][2], w4);
#pragma unroll
  for (int k1 = 0; k1 < 3; ++k1) {
    C2<T> b[3] = {a[0][k1], a[1][k1], a[2][k1]};
    dft3<T, false>(b);
#pragma unroll
    for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = b[k2];
  }
}

template <typename T, int R>
__device__ __forceinline__ void dft_any(C2<T>* v) {
  if constexpr (R == 7 || R == 11 || R == 13) dft_odd<T, R>(v);
  else if constexpr (R == 6) dft_coprime<T, 2, 3>(v);
  else if constexpr (R == 9) dft9<T>(v);
  else if constexpr (R == 10) dft_coprime<T, 2, 5>(v);
  else if constexpr (R == 12) dft_coprime<T, 4, 3>(v);
  else if constexpr (R == 14) dft_coprime<T, 2, 7>(v);
  else if constexpr (R == 15) dft_coprime<T, 3, 5>(v);
  else dftN<T, R, false>(v);
}

}  // namespace hp
