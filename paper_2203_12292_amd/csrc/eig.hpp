// The 1D eigenbasis of the operator on axis-aligned cubes (host tables).
#pragma once

#include <cmath>
#include <utility>
#include <vector>

#include "device.hpp"

namespace mfmg {

// The 1D matrices of a cube of side 1 share a basis: K = W L W^T, M = W W^T
// (L diagonal, the generalised eigenvalues of K v = l M v), so the cell matrix
// K(x)M(x)M + M(x)K(x)M + M(x)M(x)K is (W(x)W(x)W) (L_i + L_j + L_m) (W(x)W(x)W)^T
// (the fast diagonalisation of Lynch, Rice and Thomas, 1964): one sweep of
// W^T and one of W per axis.  M and K are centrosymmetric, so every column of
// W is even or odd; a sweep multiplies the even and the odd half of a line
// separately.  Modes are numbered even ones first.
// Arithmetic of the operator inside a cell, whatever the vectors' type: FP64
// and FP32 instructions issue at the same rate here, and the basis change in
// FP32 would leave the result up to 1.7 times further off than the sweeps of M
// and K it replaces (a Q3 smoothing step 1.7e-7 against 1.0e-7; in FP64
// 6e-8).  FP64 costs the Q6 operator on 8 FP32 vectors 7 %, Q3 20 %.
using CellReal = double;

template <typename T, int N>
struct EigTab {
  static constexpr int NE = (N + 1) / 2, NO = N / 2;
  T we[NE * NE];                    // [j][m], nodes j < NE, even modes
  T wo[NO * NO];                    // [j][m], nodes j < NO, odd modes
  T lam[N];
  T H[N * N];                       // hanging interpolation, lower half; row 0 is e_0
};

// W (n x n, row-major) and L of an SPD pair: M = C C^T (Cholesky), C^-1 K C^-T
// = Q L Q^T (Jacobi rotations), W = C Q; in long double.
inline void eig_block(int n, std::vector<long double> M, std::vector<long double> K, std::vector<long double>& W,
                      std::vector<long double>& L) {
  std::vector<long double> C(n * n, 0.0L), Q(n * n, 0.0L);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j <= i; ++j) {
      long double s = M[i * n + j];
      for (int q = 0; q < j; ++q) s -= C[i * n + q] * C[j * n + q];
      C[i * n + j] = i == j ? std::sqrt(s) : s / C[j * n + j];
    }
  for (int pass = 0; pass < 2; ++pass) {  // K <- C^-1 K, then its transpose
    for (int c = 0; c < n; ++c)
      for (int i = 0; i < n; ++i) {
        long double s = K[i * n + c];
        for (int q = 0; q < i; ++q) s -= C[i * n + q] * K[q * n + c];
        K[i * n + c] = s / C[i * n + i];
      }
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < i; ++j) std::swap(K[i * n + j], K[j * n + i]);
  }
  for (int i = 0; i < n; ++i) Q[i * n + i] = 1.0L;
  for (int sweep = 0; sweep < 60; ++sweep)
    for (int p = 0; p < n; ++p)
      for (int q = p + 1; q < n; ++q) {
        const long double apq = 0.5L * (K[p * n + q] + K[q * n + p]);
        if (std::fabs(apq) < 1e-40L) continue;
        const long double th = (K[q * n + q] - K[p * n + p]) / (2.0L * apq);
        const long double t = (th >= 0 ? 1.0L : -1.0L) / (std::fabs(th) + std::sqrt(th * th + 1.0L));
        const long double c = 1.0L / std::sqrt(t * t + 1.0L), s = t * c;
        for (int r = 0; r < n; ++r) {
          const long double a = K[r * n + p], b = K[r * n + q];
          K[r * n + p] = c * a - s * b;
          K[r * n + q] = s * a + c * b;
        }
        for (int r = 0; r < n; ++r) {
          const long double a = K[p * n + r], b = K[q * n + r];
          K[p * n + r] = c * a - s * b;
          K[q * n + r] = s * a + c * b;
        }
        for (int r = 0; r < n; ++r) {
          const long double a = Q[r * n + p], b = Q[r * n + q];
          Q[r * n + p] = c * a - s * b;
          Q[r * n + q] = s * a + c * b;
        }
      }
  W.assign(n * n, 0.0L);
  L.assign(n, 0.0L);
  for (int m = 0; m < n; ++m) {
    L[m] = K[m * n + m];
    for (int i = 0; i < n; ++i)
      for (int q = 0; q <= i; ++q) W[i * n + m] += C[i * n + q] * Q[q * n + m];
  }
}

template <typename T, int N>
EigTab<T, N> make_eigtab() {
  using E = EigTab<T, N>;
  const Tables1D& t = tables(N - 1);
  E o{};
  long double lam[N];
  for (int odd = 0; odd < 2; ++odd) {
    // the even (odd) block in the orthonormal basis (e_j +- e_{n-1-j})/sqrt 2, e_mid
    const int n = odd ? E::NO : E::NE;
    const long double sg = odd ? -1.0L : 1.0L;
    auto block = [&](const std::vector<double>& A) {
      std::vector<long double> B(n * n);
      for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) {
          const bool mi = 2 * i == N - 1, mj = 2 * j == N - 1;
          const long double a = A[i * N + j], b = A[i * N + (N - 1 - j)];
          B[i * n + j] = mi && mj ? a : mi || mj ? std::sqrt(2.0L) * a : a + sg * b;
        }
      return B;
    };
    std::vector<long double> W, L;
    eig_block(n, block(t.M), block(t.K), W, L);
    for (int m = 0; m < n; ++m) {
      lam[odd * E::NE + m] = std::fabs(L[m]) < 1e-12L ? 0.0L : L[m];  // (constants: exactly in the null space)
      for (int j = 0; j < n; ++j) {
        const long double w = W[j * n + m] * (2 * j == N - 1 ? 1.0L : std::sqrt(0.5L));
        (odd ? o.wo : o.we)[j * n + m] = static_cast<T>(w);
      }
    }
  }
  for (int i = 0; i < N; ++i) o.lam[i] = static_cast<T>(lam[i]);
  for (int i = 0; i < N * N; ++i) o.H[i] = static_cast<T>(t.H[0][i]);
  return o;
}

// the table of degree k as bytes
inline std::vector<char> eig_table(int k) {
  std::vector<char> out;
  auto put = [&](auto tab) {
    const char* p = reinterpret_cast<const char*>(&tab);
    out.assign(p, p + sizeof(tab));
  };
  switch (k) {
    case 1: put(make_eigtab<CellReal, 2>()); break;
    case 2: put(make_eigtab<CellReal, 3>()); break;
    case 3: put(make_eigtab<CellReal, 4>()); break;
    case 4: put(make_eigtab<CellReal, 5>()); break;
    case 5: put(make_eigtab<CellReal, 6>()); break;
    case 6: put(make_eigtab<CellReal, 7>()); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "degree");
  }
  return out;
}

}  // namespace mfmg
