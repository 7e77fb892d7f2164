// The cell operator on mapped cells (Eq. impl:mf with the general Q_e), shared
// by the operator and the diagonal.
#pragma once

#include "device.hpp"
#include "geometry.hpp"
#include "slots.hpp"

namespace mfmg {

// The hanging interpolation matrices of both halves, copied to LDS.
template <typename T, int N>
struct HangTab {
  T v[2 * N * N];  // [s][i][j] = l_j((s + xi_i)/2)
};

template <typename T, int N>
HangTab<T, N> make_hangtab() {
  const Tables1D& t = tables(N - 1);
  HangTab<T, N> o;
  for (int i = 0; i < N * N; ++i) {
    o.v[i] = static_cast<T>(t.H[0][i]);
    o.v[N * N + i] = static_cast<T>(t.H[1][i]);
  }
  return o;
}

// In-place hanging interpolation of a line from the LDS table Hg (both
// halves, [s][i][j]): u <- H_s u (H_s^T u if TRANS).
template <int N, typename T, bool TRANS>
__device__ __forceinline__ void interp_lds(const T* __restrict__ Hg, int s, T (&u)[N]) {
  const T* Hs = Hg + s * N * N;
  T out[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T acc = T(0);
#pragma unroll
    for (int j = 0; j < N; ++j) acc += Hs[TRANS ? j * N + i : i * N + j] * u[j];
    out[i] = acc;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) u[i] = out[i];
}

// Gauss-point tables of the operator on mapped cells: S[q][i] = l_i(g_q)
// (Gauss-Lobatto basis at the Gauss points), D[q][p] = L_p'(g_q) (derivative
// of the Lagrange basis on the Gauss points: gradients from point values),
// the Gauss points g and weights w on [0, 1].
template <typename T, int N>
struct MapTab {
  T S[N * N];
  T D[N * N];
  T g[N];
  T w[N];
};

template <typename T, int N>
MapTab<T, N> make_maptab() {
  const Tables1D& t = tables(N - 1);
  MapTab<T, N> m;
  for (int q = 0; q < N; ++q) {
    m.g[q] = static_cast<T>(t.qp[q]);
    m.w[q] = static_cast<T>(t.qw[q]);
    for (int i = 0; i < N; ++i) {
      m.S[q * N + i] = static_cast<T>(t.S[q * N + i]);
      m.D[q * N + i] = static_cast<T>(lagrange_deriv(t.qp, i, t.qp[q]));
    }
  }
  return m;
}

// y = A x (TRANS: y = A^T x) for an n x n table A
template <int N, typename T, bool TRANS>
__device__ __forceinline__ void mat_mv(const T* __restrict__ A, const T (&x)[N], T (&y)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T acc = (TRANS ? A[i] : A[i * N]) * x[0];
#pragma unroll
    for (int j = 1; j < N; ++j) acc += (TRANS ? A[j * N + i] : A[i * N + j]) * x[j];
    y[i] = acc;
  }
}

// Geometry of one cell of a mapped level: the coarse cell's map coefficients
// (monomial form, see geometry.hpp) and the cell's box inside it,
// t = (r + xi) * scale.
template <typename T>
struct CellGeo {
  const T* A;
  T r[3];
  T scale;
};

// The cell pipeline C^T S^T Q S C on a mapped cell (Eq. impl:mf with the
// general Q_e): values at the Gauss points by three sweeps of S, reference
// gradients at the points by sweeps of D, the metric term
// c_e w_q |det J| J^{-1} J^{-T} at every point (J from the cell's trilinear
// map), the transposed sweeps D^T and S^T.  The one n^3 buffer B of the cell
// re-distributes the values between the line directions.  Input: this lane's
// z-line (x = ta, y = tb) of gathered slot values; output: the same z-line
// of the result (the gather layout).  Hanging lines are interpolated as in
// the axis-aligned pipeline (before: z in registers, y and x in LDS; after:
// the transposes, z in registers, y and x in LDS).  Must be called by all
// lanes of the wavefront.
template <int K, typename T, typename Sync>
__device__ __forceinline__ void cell_pipeline_mapped(T* __restrict__ B, uint32_t m, int any_hang, T coef,
                                                     const MapTab<T, K + 1>& mt, const CellGeo<T>& geo,
                                                     const T* __restrict__ Hg, int ta, int tb, T (&u)[K + 1]) {
  constexpr int N = K + 1, N2 = N * N;
  const Sync sync{};
  const bool hang = mask_hanging(m);
  auto zl = [&](int c) { return c * N2 + tb * N + ta; };  // z-line (x = ta, y = tb)
  auto yl = [&](int r) { return tb * N2 + r * N + ta; };  // y-line (x = ta, z = tb)
  auto xl = [&](int r) { return tb * N2 + ta * N + r; };  // x-line (y = ta, z = tb)
  if (any_hang) {
    if (hang && hanging_line(m, 2, ta, tb, K)) interp_lds<N, T, false>(Hg, mask_sub(m, 2), u);
#pragma unroll
    for (int c = 0; c < N; ++c) B[zl(c)] = u[c];
    sync();
    if (hang && hanging_line(m, 1, ta, tb, K)) {
#pragma unroll
      for (int r = 0; r < N; ++r) u[r] = B[yl(r)];
      interp_lds<N, T, false>(Hg, mask_sub(m, 1), u);
#pragma unroll
      for (int r = 0; r < N; ++r) B[yl(r)] = u[r];
    }
    sync();
    if (hang && hanging_line(m, 0, ta, tb, K)) {
#pragma unroll
      for (int r = 0; r < N; ++r) u[r] = B[xl(r)];
      interp_lds<N, T, false>(Hg, mask_sub(m, 0), u);
#pragma unroll
      for (int r = 0; r < N; ++r) B[xl(r)] = u[r];
    }
    sync();
#pragma unroll
    for (int c = 0; c < N; ++c) u[c] = B[zl(c)];
    sync();
  }
  T v[N], w[N], gx[N], gy[N], gz[N];
  // values at the Gauss points: z, y, x
  mat_mv<N, T, false>(mt.S, u, v);
#pragma unroll
  for (int c = 0; c < N; ++c) B[zl(c)] = v[c];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) w[r] = B[yl(r)];
  mat_mv<N, T, false>(mt.S, w, v);
#pragma unroll
  for (int r = 0; r < N; ++r) B[yl(r)] = v[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) w[r] = B[xl(r)];
  mat_mv<N, T, false>(mt.S, w, v);
  mat_mv<N, T, false>(mt.D, v, gx);  // d/dxi_1 along this x-line
#pragma unroll
  for (int r = 0; r < N; ++r) B[xl(r)] = v[r];
  sync();
  // d/dxi_2 (y-lines) and d/dxi_3 (z-lines), brought to this lane's x-line
#pragma unroll
  for (int r = 0; r < N; ++r) w[r] = B[yl(r)];
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] = B[zl(r)];
  mat_mv<N, T, false>(mt.D, w, gy);
  mat_mv<N, T, false>(mt.D, v, gz);
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) B[yl(r)] = gy[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) gy[r] = B[xl(r)];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) B[zl(r)] = gz[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) gz[r] = B[xl(r)];
  // quadrature points (x = r, y = ta, z = tb): flux G grad u
  {
    const T t2 = (geo.r[1] + mt.g[ta]) * geo.scale, t3 = (geo.r[2] + mt.g[tb]) * geo.scale;
    const T wyz = mt.w[ta] * mt.w[tb] * coef;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const T t1 = (geo.r[0] + mt.g[r]) * geo.scale;
      T J[3][3];
      geo_jacobian<T>(geo.A, t1, t2, t3, J);
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int e = 0; e < 3; ++e) J[d][e] *= geo.scale;
      T G[6];
      geo_metric<T>(J, wyz * mt.w[r], G);
      const T a = gx[r], b = gy[r], c = gz[r];
      gx[r] = G[0] * a + G[1] * b + G[2] * c;
      gy[r] = G[1] * a + G[3] * b + G[4] * c;
      gz[r] = G[2] * a + G[4] * b + G[5] * c;
    }
  }
  // transposed gradient sweeps, summed along this lane's x-line
  mat_mv<N, T, true>(mt.D, gx, v);
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) B[xl(r)] = gy[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) w[r] = B[yl(r)];
  mat_mv<N, T, true>(mt.D, w, gy);
#pragma unroll
  for (int r = 0; r < N; ++r) B[yl(r)] = gy[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] += B[xl(r)];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) B[xl(r)] = gz[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) w[r] = B[zl(r)];
  mat_mv<N, T, true>(mt.D, w, gz);
#pragma unroll
  for (int r = 0; r < N; ++r) B[zl(r)] = gz[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] += B[xl(r)];
  // back to the nodes: S^T along x, y, z
  mat_mv<N, T, true>(mt.S, v, w);
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) B[xl(r)] = w[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] = B[yl(r)];
  mat_mv<N, T, true>(mt.S, v, w);
#pragma unroll
  for (int r = 0; r < N; ++r) B[yl(r)] = w[r];
  sync();
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] = B[zl(r)];
  mat_mv<N, T, true>(mt.S, v, u);
  if (!any_hang) return;
  if (hang && hanging_line(m, 2, ta, tb, K)) interp_lds<N, T, true>(Hg, mask_sub(m, 2), u);
  sync();
#pragma unroll
  for (int c = 0; c < N; ++c) B[zl(c)] = u[c];
  sync();
  if (hang && hanging_line(m, 1, ta, tb, K)) {
#pragma unroll
    for (int r = 0; r < N; ++r) w[r] = B[yl(r)];
    interp_lds<N, T, true>(Hg, mask_sub(m, 1), w);
#pragma unroll
    for (int r = 0; r < N; ++r) B[yl(r)] = w[r];
  }
  sync();
  if (hang && hanging_line(m, 0, ta, tb, K)) {
#pragma unroll
    for (int r = 0; r < N; ++r) w[r] = B[xl(r)];
    interp_lds<N, T, true>(Hg, mask_sub(m, 0), w);
#pragma unroll
    for (int r = 0; r < N; ++r) B[xl(r)] = w[r];
  }
  sync();
#pragma unroll
  for (int c = 0; c < N; ++c) u[c] = B[zl(c)];
}

// geometry of cell `cell` of a mapped level (its lattice position ijk and
// level l; the coarse grid has n0 cells per axis)
template <typename T>
__device__ __forceinline__ CellGeo<T> cell_geo(const T* __restrict__ table, const int32_t* __restrict__ ijk,
                                               int64_t cell, int l, int n0) {
  CellGeo<T> g;
  const int i = ijk[3 * cell], j = ijk[3 * cell + 1], k = ijk[3 * cell + 2];
  const int I = i >> l, J = j >> l, Kc = k >> l;
  g.A = table + (static_cast<int64_t>(I) + n0 * (J + static_cast<int64_t>(n0) * Kc)) * 24;
  g.r[0] = static_cast<T>(i - (I << l));
  g.r[1] = static_cast<T>(j - (J << l));
  g.r[2] = static_cast<T>(k - (Kc << l));
  g.scale = static_cast<T>(ldexp(1.0, -l));
  return g;
}

}  // namespace mfmg
