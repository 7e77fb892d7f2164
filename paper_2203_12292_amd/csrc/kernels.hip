// Set-up kernels (diagonal, load vector, constraint distribution, coefficient),
// vector kernels and the pieces of the outer CG (CDNA4 / gfx950).
//
// The cell kernels here take n^2 threads per cell (n = k+1), each owning one
// line of n nodes: a phase works on lines along one axis in registers; LDS
// re-distributes the cell's n^3 values between phases.  Hanging-node
// constraints (Section 3.2, the in-place interpolation variant) are 1D
// interpolations along the lines of the hanging faces/edges, applied in the
// phase whose lines run along that axis.
#include <algorithm>

#include "device.hpp"
#include "kernels.hpp"
#include "mapped.hpp"
#include "slots.hpp"

namespace mfmg {

// ---------------------------------------------------------------------------
// tables passed by value as kernel arguments (scalar-loaded)
template <typename T, int N>
struct OpTab {
  T M[N * N];
  T K[N * N];
  T H[2][N * N];
};

template <typename T, int N>
OpTab<T, N> make_optab() {
  const Tables1D& t = tables(N - 1);
  OpTab<T, N> o;
  for (int i = 0; i < N * N; ++i) {
    o.M[i] = static_cast<T>(t.M[i]);
    o.K[i] = static_cast<T>(t.K[i]);
    o.H[0][i] = static_cast<T>(t.H[0][i]);
    o.H[1][i] = static_cast<T>(t.H[1][i]);
  }
  return o;
}

template <int N>
struct Gauss1D {
  double x[N];      // Gauss points on [0, 1]
  double w[N];      // weights
  double S[N * N];  // S[q*N + i] = l_i(x_q)
};

template <int N>
Gauss1D<N> make_gauss() {
  const Tables1D& t = tables(N - 1);
  Gauss1D<N> g;
  for (int i = 0; i < N; ++i) {
    g.x[i] = t.qp[i];
    g.w[i] = t.qw[i];
  }
  for (int i = 0; i < N * N; ++i) g.S[i] = t.S[i];
  return g;
}

// ---------------------------------------------------------------------------
// small dense 1D contractions on register arrays
template <int N, typename T>
__device__ __forceinline__ void mv(const T* __restrict__ A, const T (&x)[N], T (&y)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T s = A[i * N] * x[0];
#pragma unroll
    for (int j = 1; j < N; ++j) s += A[i * N + j] * x[j];
    y[i] = s;
  }
}

// y = A x + B z (A, B symmetric use)
template <int N, typename T>
__device__ __forceinline__ void mv2(const T* __restrict__ A, const T (&x)[N], const T* __restrict__ B,
                                    const T (&z)[N], T (&y)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T s = A[i * N] * x[0];
#pragma unroll
    for (int j = 1; j < N; ++j) s += A[i * N + j] * x[j];
#pragma unroll
    for (int j = 0; j < N; ++j) s += B[i * N + j] * z[j];
    y[i] = s;
  }
}

// in-place hanging interpolation u <- H_s u (transpose: u <- H_s^T u)
template <int N, typename T, bool TRANS>
__device__ __forceinline__ void interp(const T (&H)[2][N * N], int s, T (&u)[N]) {
  T out[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T acc = T(0);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int idx = TRANS ? j * N + i : i * N + j;
      const T h = s ? H[1][idx] : H[0][idx];
      acc += h * u[j];
    }
    out[i] = acc;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) u[i] = out[i];
}

// scatter-add of the line of nodes (a, 0..k, c) (along y); cell interiors are
// owned by the cell (plain store), shared entities use atomics.
// `plain`: no other cell writes the same entities concurrently (deterministic
// mode, colour by colour), a plain read-modify-write.
template <typename T>
__device__ __forceinline__ void scatter_add(T* p, T v, bool plain) {
  if (plain) *p += v;
  else atomic_add(p, v);
}

template <int K, typename T>
__device__ __forceinline__ void scatter_yline(const int32_t* __restrict__ ent, int64_t nc, int64_t cell,
                                              int a, int c, const T (&w)[K + 1], T* __restrict__ dst, int nv,
                                              int v, bool plain = false) {
  const int s0 = node_slot(a, 0, c, K), s1 = node_slot(a, K, c, K);
  const int o0 = node_offset(a, 0, c, K);
  const int32_t e0 = ent[s0 * nc + cell], e1 = ent[s1 * nc + cell];
  if (e0 >= 0) scatter_add(&dst[static_cast<int64_t>(e0 + o0) * nv + v], w[0], plain);
  if (e1 >= 0) scatter_add(&dst[static_cast<int64_t>(e1 + o0) * nv + v], w[K], plain);
  if constexpr (K > 1) {
    const int sm = node_slot(a, 1, c, K);
    const int om = node_offset(a, 1, c, K);
    const int st = K > 2 ? node_offset(a, 2, c, K) - om : 0;
    const int32_t em = ent[sm * nc + cell];
    if (em >= 0) {
      if (sm == 26) {
#pragma unroll
        for (int b = 1; b < K; ++b) dst[static_cast<int64_t>(em + om + (b - 1) * st) * nv + v] = w[b];
      } else {
#pragma unroll
        for (int b = 1; b < K; ++b)
          scatter_add(&dst[static_cast<int64_t>(em + om + (b - 1) * st) * nv + v], w[b], plain);
      }
    }
  }
}

// The cell pipeline C^T S^T Q S C on the block's LDS.  Input: this thread's
// z-line (x = ta, y = tb) of gathered slot values.  Output: this thread's
// y-line (x = ta, z = tb) of the result, before the scatter.  Must be called
// by all threads of the block (contains barriers).
template <int K, typename T, typename Sync>
__device__ __forceinline__ void cell_pipeline(T* __restrict__ B0, T* __restrict__ B1, bool active, uint32_t m,
                                              int block_hang, T h, const OpTab<T, K + 1>& tab, int ta, int tb,
                                              T (&u)[K + 1]) {
  const Sync sync{};
  constexpr int N = K + 1, N2 = N * N;
  const bool hang = mask_hanging(m);
  // phase 1: z-lines (x = ta, y = tb): hanging z-interpolation, store
  if (active) {
    if (hang && hanging_line(m, 2, ta, tb, K)) interp<N, T, false>(tab.H, mask_sub(m, 2), u);
#pragma unroll
    for (int c = 0; c < N; ++c) B0[c * N2 + tb * N + ta] = u[c];
  }
  sync();
  // phase 2: y-lines (x = ta, z = tb): hanging y-interpolation
  if (block_hang) {
    if (active && hang && hanging_line(m, 1, ta, tb, K)) {
#pragma unroll
      for (int r = 0; r < N; ++r) u[r] = B0[tb * N2 + r * N + ta];
      interp<N, T, false>(tab.H, mask_sub(m, 1), u);
#pragma unroll
      for (int r = 0; r < N; ++r) B0[tb * N2 + r * N + ta] = u[r];
    }
    sync();
  }
  // phase 3: x-lines (y = ta, z = tb): hanging x-interpolation, M_x, K_x
  T a[N], b[N];
  if (active) {
#pragma unroll
    for (int r = 0; r < N; ++r) u[r] = B0[tb * N2 + ta * N + r];
    if (hang && hanging_line(m, 0, ta, tb, K)) interp<N, T, false>(tab.H, mask_sub(m, 0), u);
    mv<N>(tab.M, u, a);
    mv<N>(tab.K, u, b);
#pragma unroll
    for (int r = 0; r < N; ++r) {
      B0[tb * N2 + ta * N + r] = a[r];
      B1[tb * N2 + ta * N + r] = b[r];
    }
  }
  sync();
  // phase 4: y-lines (x = ta, z = tb): M_y a ; K_y a + M_y b
  if (active) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      a[r] = B0[tb * N2 + r * N + ta];
      b[r] = B1[tb * N2 + r * N + ta];
    }
    T c1[N], f[N];
    mv<N>(tab.M, a, c1);
    mv2<N>(tab.K, a, tab.M, b, f);
#pragma unroll
    for (int r = 0; r < N; ++r) {
      B0[tb * N2 + r * N + ta] = c1[r];
      B1[tb * N2 + r * N + ta] = f[r];
    }
  }
  sync();
  // phase 5: z-lines (x = ta, y = tb): h (K_z c + M_z f), transposed z-interpolation
  if (active) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      a[r] = B0[r * N2 + tb * N + ta];
      b[r] = B1[r * N2 + tb * N + ta];
    }
    mv2<N>(tab.K, a, tab.M, b, u);
#pragma unroll
    for (int r = 0; r < N; ++r) u[r] *= h;
    if (hang && hanging_line(m, 2, ta, tb, K)) interp<N, T, true>(tab.H, mask_sub(m, 2), u);
#pragma unroll
    for (int r = 0; r < N; ++r) B0[r * N2 + tb * N + ta] = u[r];
  }
  sync();
  // phase 6: x-lines (y = ta, z = tb): transposed x-interpolation
  if (block_hang) {
    if (active && hang && hanging_line(m, 0, ta, tb, K)) {
#pragma unroll
      for (int r = 0; r < N; ++r) u[r] = B0[tb * N2 + ta * N + r];
      interp<N, T, true>(tab.H, mask_sub(m, 0), u);
#pragma unroll
      for (int r = 0; r < N; ++r) B0[tb * N2 + ta * N + r] = u[r];
    }
    sync();
  }
  // phase 7: y-lines (x = ta, z = tb): transposed y-interpolation
  if (active) {
#pragma unroll
    for (int r = 0; r < N; ++r) u[r] = B0[tb * N2 + r * N + ta];
    if (hang && hanging_line(m, 1, ta, tb, K)) interp<N, T, true>(tab.H, mask_sub(m, 1), u);
  }
}

// Does the hanging-node interpolation C_e touch node (a, b, c)?  Only if one
// of the three lines through the node is interpolated: otherwise C_e e_s =
// e_s for its slot s (the in-place line interpolations mix values along
// their own lines only), and (C_e^T A_e C_e)_ss = A_e(s, s).
__device__ __forceinline__ bool node_constrained(uint32_t m, int a, int b, int c, int k) {
  return hanging_line(m, 0, b, c, k) || hanging_line(m, 1, a, c, k) || hanging_line(m, 2, a, b, k);
}

// Diagonal (Eq. impl:mf:diagonal).  d_e(i) = A_e(i,i) = h (K_aa M_bb M_cc +
// M_aa K_bb M_cc + M_aa M_bb K_cc) for every node that the cell's hanging-node
// interpolation leaves alone; for the others (the nodes of hanging faces and
// edges) apply C_e^T A_e C_e to the unit slot vector e_s and keep entry s.
// One cell per block, n^2 threads.
template <int K>
__global__ void __launch_bounds__((K + 1) * (K + 1))
    diag_kernel(const int32_t* __restrict__ ent, const uint32_t* __restrict__ mask, int64_t nc, double h0,
                OpTab<double, K + 1> tab, double* __restrict__ diag, const int32_t* __restrict__ cells) {
  constexpr int N = K + 1, N2 = N * N, N3 = N2 * N;
  __shared__ double B0[N3];
  __shared__ double B1[N3];
  const int64_t cell = cells ? cells[blockIdx.x] : blockIdx.x;  // cells: one colour (deterministic mode)
  const int ta = threadIdx.x % N, tb = threadIdx.x / N;
  const uint32_t m = mask[cell];
  const double h = ldexp(h0, -mask_level(m)) * static_cast<double>(mask_coef(m));
  double d[N];  // y-line (x = ta, z = tb)
#pragma unroll
  for (int r = 0; r < N; ++r)
    d[r] = h * (tab.K[ta * N + ta] * tab.M[r * N + r] * tab.M[tb * N + tb] +
                tab.M[ta * N + ta] * tab.K[r * N + r] * tab.M[tb * N + tb] +
                tab.M[ta * N + ta] * tab.M[r * N + r] * tab.K[tb * N + tb]);
  if (mask_hanging(m)) {
    for (int s = 0; s < N3; ++s) {
      const int sa = s % N, sb = (s / N) % N, sc = s / N2;
      if (!node_constrained(m, sa, sb, sc, K)) continue;  // uniform over the block
      double u[N];
#pragma unroll
      for (int c = 0; c < N; ++c) u[c] = (ta == sa && tb == sb && c == sc) ? 1.0 : 0.0;
      cell_pipeline<K, double, WaveSync>(B0, B1, true, m, 1, h, tab, ta, tb, u);
      if (ta == sa && tb == sc) {
#pragma unroll
        for (int r = 0; r < N; ++r)
          if (r == sb) d[r] = u[r];
      }
      WaveSync{}();
    }
  }
  scatter_yline<K>(ent, nc, cell, ta, tb, d, diag, 1, 0, cells != nullptr);
}

// scatter-add of the line of nodes (a, b, 0..k) (along z), as scatter_yline
template <int K, typename T, bool INTERIOR = true>
__device__ __forceinline__ void scatter_zline(const int32_t* __restrict__ ent, int64_t nc, int64_t cell, int a,
                                              int b, const T (&w)[K + 1], T* __restrict__ dst, bool plain = false) {
  const int s0 = node_slot(a, b, 0, K), s1 = node_slot(a, b, K, K);
  const int o0 = node_offset(a, b, 0, K);
  const int32_t e0 = ent[s0 * nc + cell], e1 = ent[s1 * nc + cell];
  if (e0 >= 0) scatter_add(&dst[e0 + o0], w[0], plain);
  if (e1 >= 0) scatter_add(&dst[e1 + o0], w[K], plain);
  if constexpr (K > 1) {
    const int sm = node_slot(a, b, 1, K);
    const int om = node_offset(a, b, 1, K);
    const int st = K > 2 ? node_offset(a, b, 2, K) - om : 0;
    const int32_t em = ent[sm * nc + cell];
    if (em >= 0 && (INTERIOR || sm != 26)) {
#pragma unroll
      for (int c = 1; c < K; ++c) {
        if (sm == 26) dst[em + om + (c - 1) * st] = w[c];
        else scatter_add(&dst[em + om + (c - 1) * st], w[c], plain);
      }
    }
  }
}

// Diagonal of a mapped cell without constraints, A_e(i,i) =
// sum_q grad phi_i(q)^T G_q grad phi_i(q), G_q = c_e w_q |det J| J^-1 J^-T:
// with phi_i = l_a l_b l_c, d_xi1 phi_i = l'_a l_b l_c etc., every product of
// two gradient components is a product of 1D factors, so the six symmetric
// components of G contract with squared 1D tables (E = S.S, F = S'.S',
// X = S'.S elementwise; S' = l'(g_q)) axis by axis: 6 x 3 sweeps.  One cell
// per block of n^2 threads.  In cells with hanging nodes the nodes that the
// interpolation touches are left to diag_mapped_kernel (written as 0 here).
template <typename T, int N>
struct DiagTab {
  T E[N * N], F[N * N], X[N * N];  // [q][a]
};

template <int K>
__global__ void __launch_bounds__((K + 1) * (K + 1))
    diag_mapped_direct_kernel(const int32_t* __restrict__ ent, const uint32_t* __restrict__ mask, int64_t nc,
                              const double* __restrict__ geo, const int32_t* __restrict__ ijk, int n0,
                              MapTab<double, K + 1> mt, DiagTab<double, K + 1> dt, double* __restrict__ diag,
                              const int32_t* __restrict__ cells) {
  constexpr int N = K + 1, N2 = N * N, N3 = N2 * N;
  __shared__ double B[N3];
  const int64_t cell = cells ? cells[blockIdx.x] : blockIdx.x;
  const uint32_t m = mask[cell];
  const int ta = threadIdx.x % N, tb = threadIdx.x / N;
  const CellGeo<double> g = cell_geo<double>(geo, ijk, cell, mask_level(m), n0);
  const double coef = static_cast<double>(mask_coef(m));
  double G[6][N];  // this lane's x-line of quadrature points (x = r, y = ta, z = tb)
  {
    const double t2 = (g.r[1] + mt.g[ta]) * g.scale, t3 = (g.r[2] + mt.g[tb]) * g.scale;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      double J[3][3], Gq[6];
      geo_jacobian<double>(g.A, (g.r[0] + mt.g[r]) * g.scale, t2, t3, J);
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int e = 0; e < 3; ++e) J[d][e] *= g.scale;
      geo_metric<double>(J, coef * mt.w[r] * mt.w[ta] * mt.w[tb], Gq);
#pragma unroll
      for (int q = 0; q < 6; ++q) G[q][r] = Gq[q];
    }
  }
  // (component of G, factor, x table, y table, z table): g00 F E E, g11 E F E,
  // g22 E E F, 2 g01 X X E, 2 g02 X E X, 2 g12 E X X
  const double* tabs[6][3] = {{dt.F, dt.E, dt.E}, {dt.X, dt.X, dt.E}, {dt.X, dt.E, dt.X},
                              {dt.E, dt.F, dt.E}, {dt.E, dt.X, dt.X}, {dt.E, dt.E, dt.F}};
  const double fac[6] = {1.0, 2.0, 2.0, 1.0, 2.0, 1.0};
  double d[N];
#pragma unroll
  for (int c = 0; c < N; ++c) d[c] = 0.0;
  for (int q = 0; q < 6; ++q) {
    double v[N], w[N];
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = fac[q] * G[q][r];
    mat_mv<N, double, true>(tabs[q][0], v, w);  // x: node a <- point
    WaveSync{}();
#pragma unroll
    for (int r = 0; r < N; ++r) B[tb * N2 + ta * N + r] = w[r];
    WaveSync{}();
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = B[tb * N2 + r * N + ta];
    mat_mv<N, double, true>(tabs[q][1], v, w);  // y
#pragma unroll
    for (int r = 0; r < N; ++r) B[tb * N2 + r * N + ta] = w[r];
    WaveSync{}();
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = B[r * N2 + tb * N + ta];
    mat_mv<N, double, true>(tabs[q][2], v, w);  // z
#pragma unroll
    for (int c = 0; c < N; ++c) d[c] += w[c];
  }
  if (mask_hanging(m)) {
#pragma unroll
    for (int c = 0; c < N; ++c)
      if (node_constrained(m, ta, tb, c, K)) d[c] = 0.0;
  }
  scatter_zline<K>(ent, nc, cell, ta, tb, d, diag, cells != nullptr);
}

// Diagonal of a mapped cell with hanging nodes (Eq. impl:mf:diagonal), the
// nodes that the interpolation touches: the cell operator C_e^T A_e C_e
// applied to the unit slot vector e_s, entry s kept (the other nodes come
// from diag_mapped_direct_kernel; the cell interior is never touched and not
// written here).  One cell per block of n^2 threads (one wavefront).
template <int K>
__global__ void __launch_bounds__((K + 1) * (K + 1))
    diag_mapped_kernel(const int32_t* __restrict__ ent, const uint32_t* __restrict__ mask, int64_t nc,
                       const double* __restrict__ geo, const int32_t* __restrict__ ijk, int n0,
                       MapTab<double, K + 1> mt, HangTab<double, K + 1> tab, double* __restrict__ diag,
                       const int32_t* __restrict__ cells) {
  constexpr int N = K + 1, N2 = N * N, N3 = N2 * N;
  __shared__ double B[N3];
  __shared__ double Hg[2 * N2];
  for (int i = threadIdx.x; i < 2 * N2; i += blockDim.x) Hg[i] = tab.v[i];
  __syncthreads();
  const int64_t cell = cells ? cells[blockIdx.x] : blockIdx.x;
  const int ta = threadIdx.x % N, tb = threadIdx.x / N;
  const uint32_t m = mask[cell];
  if (!mask_hanging(m)) return;  // (diag_mapped_direct_kernel)
  const CellGeo<double> g = cell_geo<double>(geo, ijk, cell, mask_level(m), n0);
  const double coef = static_cast<double>(mask_coef(m));
  const int any_hang = 1;
  double d[N];
#pragma unroll
  for (int c = 0; c < N; ++c) d[c] = 0.0;
  for (int sc = 0; sc < N; ++sc)
    for (int sb = 0; sb < N; ++sb)
      for (int sa = 0; sa < N; ++sa) {
        if (!node_constrained(m, sa, sb, sc, K)) continue;  // uniform over the block
        double u[N];
#pragma unroll
        for (int c = 0; c < N; ++c) u[c] = (ta == sa && tb == sb && c == sc) ? 1.0 : 0.0;
        cell_pipeline_mapped<K, double, WaveSync>(B, m, any_hang, coef, mt, g, Hg, ta, tb, u);
        if (ta == sa && tb == sb) {
#pragma unroll
          for (int c = 0; c < N; ++c)
            if (c == sc) d[c] += u[c];
        }
        WaveSync{}();
      }
  scatter_zline<K, double, false>(ent, nc, cell, ta, tb, d, diag, cells != nullptr);
}

// Constraint distribution: gather G_e and hanging-node interpolation C_e of
// one cell, written out node by node.  One cell per block, n^2 threads.
template <int K>
__global__ void __launch_bounds__((K + 1) * (K + 1))
    distribute_kernel(const int32_t* __restrict__ ent, const uint32_t* __restrict__ mask, int64_t nc,
                      OpTab<double, K + 1> tab, const double* __restrict__ x, double* __restrict__ out) {
  constexpr int N = K + 1, N2 = N * N, N3 = N2 * N;
  __shared__ double B[N3];
  const int64_t cell = blockIdx.x;
  const int ta = threadIdx.x % N, tb = threadIdx.x / N;
  const uint32_t m = mask[cell];
  double u[N];
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const int s = node_slot(ta, tb, c, K);
    const int32_t e = ent[s * nc + cell];
    u[c] = e < 0 ? 0.0 : x[e + node_offset(ta, tb, c, K)];
  }
  const bool hang = mask_hanging(m);
  if (hang && hanging_line(m, 2, ta, tb, K)) interp<N, double, false>(tab.H, mask_sub(m, 2), u);
#pragma unroll
  for (int c = 0; c < N; ++c) B[c * N2 + tb * N + ta] = u[c];
  __syncthreads();
  // y-lines (x = ta, z = tb)
#pragma unroll
  for (int r = 0; r < N; ++r) u[r] = B[tb * N2 + r * N + ta];
  if (hang && hanging_line(m, 1, ta, tb, K)) interp<N, double, false>(tab.H, mask_sub(m, 1), u);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < N; ++r) B[tb * N2 + r * N + ta] = u[r];
  __syncthreads();
  // x-lines (y = ta, z = tb)
#pragma unroll
  for (int r = 0; r < N; ++r) u[r] = B[tb * N2 + ta * N + r];
  if (hang && hanging_line(m, 0, ta, tb, K)) interp<N, double, false>(tab.H, mask_sub(m, 0), u);
#pragma unroll
  for (int r = 0; r < N; ++r) out[cell * N3 + tb * N2 + ta * N + r] = u[r];
}

// Load vector b_e = int_e f phi (Gauss (k+1)^3), then C_e^T and scatter.
// One cell per block, n^2 threads; f = const or a sum of Gaussians.
template <int K>
__global__ void __launch_bounds__((K + 1) * (K + 1))
    rhs_kernel(const int32_t* __restrict__ ent, const uint32_t* __restrict__ mask,
               const int32_t* __restrict__ cell_ijk, int64_t nc, double h0, double lo, OpTab<double, K + 1> tab,
               Gauss1D<K + 1> g, int kind, const double* __restrict__ params, int n_terms, double* __restrict__ b,
               int nv, const double* __restrict__ geo, int n0, const int32_t* __restrict__ cells) {
  constexpr int N = K + 1, N2 = N * N, N3 = N2 * N;
  __shared__ double B0[N3];
  const int64_t cell = cells ? cells[blockIdx.x] : blockIdx.x;  // cells: one colour (deterministic mode)
  const int v = blockIdx.y;
  const int ta = threadIdx.x % N, tb = threadIdx.x / N;
  const uint32_t m = mask[cell];
  const int lev = mask_level(m);
  const double h = ldexp(h0, -lev);
  const double x0 = lo + h * cell_ijk[3 * cell + 0];
  const double y0 = lo + h * cell_ijk[3 * cell + 1];
  const double z0 = lo + h * cell_ijk[3 * cell + 2];
  // z-line of quadrature points (qx = ta, qy = tb): weighted f values
  double gz[N];
  CellGeo<double> cg{};
  if (geo) cg = cell_geo<double>(geo, cell_ijk, cell, lev, n0);
#pragma unroll
  for (int q = 0; q < N; ++q) {
    double x = x0 + h * g.x[ta], y = y0 + h * g.x[tb], z = z0 + h * g.x[q];
    double vol = h * h * h;  // |det J| of the cell map
    if (geo) {  // mapped cell: physical point and |det J| from its map
      const double t1 = (cg.r[0] + g.x[ta]) * cg.scale, t2 = (cg.r[1] + g.x[tb]) * cg.scale,
                   t3 = (cg.r[2] + g.x[q]) * cg.scale;
      double X[3], J[3][3];
      geo_point<double>(cg.A, t1, t2, t3, X);
      geo_jacobian<double>(cg.A, t1, t2, t3, J);
      x = X[0];
      y = X[1];
      z = X[2];
      vol = (J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
             J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0])) *
            cg.scale * cg.scale * cg.scale;
      vol = vol < 0 ? -vol : vol;
    }
    double f = 0.0;
    if (kind == 0) {
      f = params[0];
    } else if (kind == 2) {
      f = params[0] * sin(params[1] * x) * sin(params[1] * y) * sin(params[1] * z);
    } else {
      const double* p = params + static_cast<int64_t>(v) * n_terms * 5;
      for (int t = 0; t < n_terms; ++t) {
        double dx = x - p[5 * t], dy = y - p[5 * t + 1], dz = z - p[5 * t + 2], w = p[5 * t + 3];
        f += p[5 * t + 4] * exp(-(dx * dx + dy * dy + dz * dz) / (2.0 * w * w));
      }
    }
    gz[q] = f * g.w[ta] * g.w[tb] * g.w[q] * vol;
  }
  // S^T along z: out[c] = sum_q S[q][c] gz[q]
  double u[N];
#pragma unroll
  for (int c = 0; c < N; ++c) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < N; ++q) s += g.S[q * N + c] * gz[q];
    u[c] = s;
  }
#pragma unroll
  for (int c = 0; c < N; ++c) B0[c * N2 + tb * N + ta] = u[c];  // (qx, qy, c)
  __syncthreads();
  // along y at (qx = ta, c = tb)
#pragma unroll
  for (int r = 0; r < N; ++r) gz[r] = B0[tb * N2 + r * N + ta];
#pragma unroll
  for (int bb = 0; bb < N; ++bb) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < N; ++q) s += g.S[q * N + bb] * gz[q];
    u[bb] = s;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < N; ++r) B0[tb * N2 + r * N + ta] = u[r];  // (qx, b, c)
  __syncthreads();
  // along x at (b = ta, c = tb)
#pragma unroll
  for (int r = 0; r < N; ++r) gz[r] = B0[tb * N2 + ta * N + r];
#pragma unroll
  for (int aa = 0; aa < N; ++aa) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < N; ++q) s += g.S[q * N + aa] * gz[q];
    u[aa] = s;
  }
  const bool hang = mask_hanging(m);
  if (hang && hanging_line(m, 0, ta, tb, K)) interp<N, double, true>(tab.H, mask_sub(m, 0), u);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < N; ++r) B0[tb * N2 + ta * N + r] = u[r];  // (a, b, c)
  __syncthreads();
  // z-lines (x = ta, y = tb): transposed z
#pragma unroll
  for (int r = 0; r < N; ++r) u[r] = B0[r * N2 + tb * N + ta];
  if (hang && hanging_line(m, 2, ta, tb, K)) interp<N, double, true>(tab.H, mask_sub(m, 2), u);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < N; ++r) B0[r * N2 + tb * N + ta] = u[r];
  __syncthreads();
  // y-lines (x = ta, z = tb): transposed y, scatter
#pragma unroll
  for (int r = 0; r < N; ++r) u[r] = B0[tb * N2 + r * N + ta];
  if (hang && hanging_line(m, 1, ta, tb, K)) interp<N, double, true>(tab.H, mask_sub(m, 1), u);
  scatter_yline<K>(ent, nc, cell, ta, tb, u, b, nv, v, cells != nullptr);
}

// ---------------------------------------------------------------------------
// vector kernels
__global__ void fill_zero_kernel(uint32_t* __restrict__ x, int64_t nwords) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < nwords;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    x[i] = 0u;
}

__global__ void fill_zero_bytes_kernel(uint8_t* __restrict__ x, int64_t n) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    x[i] = 0;
}

template <typename S>
__global__ void cheb_kernel(int64_t n_dofs, int nv, int first, typename Acc<S>::type c_dd,
                            typename Acc<S>::type c_r, const typename Acc<S>::type* __restrict__ t,
                            const S* __restrict__ b, const typename Acc<S>::type* __restrict__ dinv,
                            S* __restrict__ d, S* __restrict__ x) {
  using A = typename Acc<S>::type;
  const int64_t n = n_dofs * nv;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const A di = dinv[i / nv];
    A dn;
    if (first) {
      dn = c_r * di * load_as<A>(b[i]);
      x[i] = store_as<S>(dn);
    } else {
      dn = (c_dd != A(0) ? c_dd * load_as<A>(d[i]) : A(0)) + c_r * di * (load_as<A>(b[i]) - t[i]);
      x[i] = store_as<S>(load_as<A>(x[i]) + dn);
    }
    d[i] = store_as<S>(dn);
  }
}

template <typename S>
__global__ void residual_kernel(int64_t n, const S* __restrict__ b, const typename Acc<S>::type* __restrict__ t,
                                S* __restrict__ r) {
  using A = typename Acc<S>::type;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    r[i] = store_as<S>(load_as<A>(b[i]) - t[i]);
}

template <typename S>
__global__ void cast_from_f64_kernel(int64_t n, const double* __restrict__ src, S* __restrict__ dst) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    dst[i] = store_as<S>(src[i]);
}

template <typename S>
__global__ void cast_to_f64_kernel(int64_t n, const S* __restrict__ src, double* __restrict__ dst) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    dst[i] = load_as<double>(src[i]);
}

template <typename A, typename B>
__global__ void cast_kernel(int64_t n, const A* __restrict__ src, B* __restrict__ dst) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    dst[i] = store_as<B>(load_as<float>(src[i]));
}

// copy between the active mesh and a local-smoothing level (Algorithm 1):
// dst[di[q]] = src[si[q]], n_vec interleaved values per DoF
template <typename A, typename B>
__global__ void copy_map_kernel(int64_t n, int nv, const int32_t* __restrict__ si, const int32_t* __restrict__ di,
                                const A* __restrict__ src, B* __restrict__ dst) {
  for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < n * nv;
       t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t q = t / nv;
    const int64_t v = t - q * nv;
    dst[static_cast<int64_t>(di[q]) * nv + v] = store_as<B>(load_as<double>(src[static_cast<int64_t>(si[q]) * nv + v]));
  }
}

// refinement-edge DoFs of a local-smoothing level: zero inverse diagonal
__global__ void zero_entries_kernel(int64_t n, const int32_t* __restrict__ idx, double* __restrict__ a64,
                                    float* __restrict__ a32) {
  for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < n;
       t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    a64[idx[t]] = 0.0;
    a32[idx[t]] = 0.0f;
  }
}

template <typename S>
__global__ void acc_to_storage_kernel(int64_t n, const typename Acc<S>::type* __restrict__ src,
                                      S* __restrict__ dst) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    dst[i] = store_as<S>(src[i]);
}

template <typename A>
__global__ void inverse_diag_kernel(int64_t n, const double* __restrict__ diag, A* __restrict__ dinv) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    dinv[i] = diag[i] != 0.0 ? static_cast<A>(1.0 / diag[i]) : A(0);
}

// one wavefront per row: acc[row] = sum_j Ainv[row, j] b[j]
template <typename S>
__global__ void __launch_bounds__(256)
    dense_matvec_kernel(int64_t n0, int nv, const typename Acc<S>::type* __restrict__ Ainv,
                        const S* __restrict__ b, S* __restrict__ x) {
  using A = typename Acc<S>::type;
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * (blockDim.x / 64) + threadIdx.x / 64;
  const int v = blockIdx.y;
  if (row >= n0) return;
  A s = A(0);
  for (int64_t j = lane; j < n0; j += 64) s += Ainv[row * n0 + j] * load_as<A>(b[j * nv + v]);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) x[row * nv + v] = store_as<S>(s);
}

// ---- FP64 reductions and CG updates ----------------------------------------
constexpr int DOT_BLOCKS = 2048, DOT_THREADS = 256;

// Block sums of dot products of nv interleaved vectors ([n][nv], nv <= 8), ND
// per vector: partial[(d * 8 + v) * DOT_BLOCKS + block]; dot_sum_kernel adds the
// blocks.  f(i, v, s) adds entry i (vector v) to the thread's sums s[ND].  The
// threads used per block are a multiple of nv, so a thread stays with one
// vector.  (One launch instead of two, with the last block adding, is slower:
// the fence before its counter writes back the L2 of every XCD; octant solve
// of 2.2M DoFs 7.5 -> 8.2 ms.)
template <int ND, typename F>
__device__ __forceinline__ void dot_block(int64_t n, int nv, double* __restrict__ partial, F f) {
  __shared__ double red[ND][DOT_THREADS];
  const int used = DOT_THREADS / nv * nv, t = threadIdx.x, v = t % nv;
  double s[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) s[d] = 0.0;
  if (t < used)
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * used + t; i < n; i += static_cast<int64_t>(gridDim.x) * used)
      f(i, v, s);
#pragma unroll
  for (int d = 0; d < ND; ++d) red[d][t] = s[d];
  const int groups = used / nv;  // threads of one vector
  for (int w = 128; w > 0; w >>= 1) {
    __syncthreads();
    if (t < used && t / nv < w && t / nv + w < groups) {
#pragma unroll
      for (int d = 0; d < ND; ++d) red[d][t] += red[d][t + w * nv];
    }
  }
  __syncthreads();
  if (t < nv) {
#pragma unroll
    for (int d = 0; d < ND; ++d) partial[(d * 8 + t) * DOT_BLOCKS + blockIdx.x] = red[d][t];
  }
}

// results[d][v] = sum of the blocks' sums in a fixed order, one block per (d, v)
__global__ void __launch_bounds__(DOT_THREADS)
    dot_sum_kernel(int blocks, int nv, const double* __restrict__ partial, double* res0, double* res1) {
  __shared__ double red[DOT_THREADS];
  const int d = blockIdx.x / nv, v = blockIdx.x - d * nv;
  double s = 0.0;
  for (int i = threadIdx.x; i < blocks; i += DOT_THREADS) s += partial[(d * 8 + v) * DOT_BLOCKS + i];
  red[threadIdx.x] = s;
  for (int w = DOT_THREADS / 2; w > 0; w >>= 1) {
    __syncthreads();
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
  }
  if (threadIdx.x == 0) (d ? res1 : res0)[v] = red[0];
}

__global__ void __launch_bounds__(DOT_THREADS)
    dot_kernel(int64_t n, int nv, const double* __restrict__ a, const double* __restrict__ b,
               double* __restrict__ partial) {
  dot_block<1>(n, nv, partial, [&](int64_t i, int, double(&s)[1]) { s[0] += a[i] * b[i]; });
}

// a . b and a . c, reading a once
__global__ void __launch_bounds__(DOT_THREADS)
    dot2_kernel(int64_t n, int nv, const double* __restrict__ a, const double* __restrict__ b,
                const double* __restrict__ c, double* __restrict__ partial) {
  dot_block<2>(n, nv, partial, [&](int64_t i, int, double(&s)[2]) {
    s[0] += a[i] * b[i];
    s[1] += a[i] * c[i];
  });
}

// x += alpha p, r -= alpha q (alpha = num / den per vector), and r . r
__global__ void __launch_bounds__(DOT_THREADS)
    cg_xr_dot_kernel(int64_t n, int nv, const double* __restrict__ num, const double* __restrict__ den,
                     const double* __restrict__ p, const double* __restrict__ q, double* __restrict__ x,
                     double* __restrict__ r, double* __restrict__ partial) {
  const int mine = threadIdx.x % nv;
  const double alpha = den[mine] != 0.0 ? num[mine] / den[mine] : 0.0;
  dot_block<1>(n, nv, partial, [&](int64_t i, int, double(&s)[1]) {
    x[i] += alpha * p[i];
    const double t = r[i] - alpha * q[i];
    r[i] = t;
    s[0] += t * t;
  });
}

__global__ void cg_p_kernel(int64_t n_dofs, int nv, const double* __restrict__ num, const double* __restrict__ sub,
                            const double* __restrict__ den, const double* __restrict__ z, double* __restrict__ p) {
  const int64_t n = n_dofs * nv;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int v = static_cast<int>(i % nv);
    const double beta = den[v] != 0.0 ? (num[v] - (sub ? sub[v] : 0.0)) / den[v] : 0.0;
    p[i] = z[i] + beta * p[i];
  }
}

// ===========================================================================
// host launchers
namespace {

void zero_bytes(void* p, int64_t bytes, hipStream_t s) {
  if (bytes <= 0) return;
  if (bytes % 4 == 0 && reinterpret_cast<uintptr_t>(p) % 4 == 0) {
    fill_zero_kernel<<<grid_for(bytes / 4, 4), VEC_THREADS, 0, s>>>(static_cast<uint32_t*>(p), bytes / 4);
  } else {
    fill_zero_bytes_kernel<<<grid_for(bytes, 4), VEC_THREADS, 0, s>>>(static_cast<uint8_t*>(p), bytes);
  }
  check_launch();
}

// One launch over all cells (cells = NULL: block i is cell i), or in the
// deterministic mode one launch per colour over that colour's cell list.
template <typename F>
void for_colours(const CellView& c, F launch) {
  if (!c.deterministic) {
    launch(static_cast<unsigned>(c.n_cells), static_cast<const int32_t*>(nullptr));
    return;
  }
  for (int k = 0; k < c.n_colors; ++k) {
    const int64_t n = c.color_off[k + 1] - c.color_off[k];
    if (n > 0) launch(static_cast<unsigned>(n), c.color_cells + c.color_off[k]);
  }
}

template <int K>
void diag_k(const CellView& c, double* diag, hipStream_t s) {
  constexpr int N = K + 1;
  zero_bytes(diag, c.n_dofs * 8, s);
  if (c.n_cells == 0) return;
  if (c.geo64) {
    static const MapTab<double, N> mt = make_maptab<double, N>();
    static const HangTab<double, N> tab2 = make_hangtab<double, N>();
    static const DiagTab<double, N> dt = [] {
      const Tables1D& t = tables(N - 1);
      DiagTab<double, N> r;
      for (int q = 0; q < N; ++q)
        for (int a = 0; a < N; ++a) {
          const double sv = t.S[q * N + a], dv = lagrange_deriv(t.nodes, a, t.qp[q]);
          r.E[q * N + a] = sv * sv;
          r.F[q * N + a] = dv * dv;
          r.X[q * N + a] = dv * sv;
        }
      return r;
    }();
    const double* geo = static_cast<const double*>(c.geo64);
    for_colours(c, [&](unsigned n, const int32_t* cells) {
      diag_mapped_direct_kernel<K><<<n, N * N, 0, s>>>(c.ent, c.mask, c.n_cells, geo, c.ijk, c.geo_n0, mt, dt, diag,
                                                       cells);
      check_launch();
      diag_mapped_kernel<K><<<n, N * N, 0, s>>>(c.ent, c.mask, c.n_cells, geo, c.ijk, c.geo_n0, mt, tab2, diag,
                                                cells);
      check_launch();
    });
    return;
  }
  static const OpTab<double, N> tab = make_optab<double, N>();
  for_colours(c, [&](unsigned n, const int32_t* cells) {
    diag_kernel<K><<<n, N * N, 0, s>>>(c.ent, c.mask, c.n_cells, c.h0, tab, diag, cells);
    check_launch();
  });
}

template <int K>
void rhs_k(const CellView& c, int kind, const double* params, int n_terms, int nv, double* b, hipStream_t s) {
  constexpr int N = K + 1;
  zero_bytes(b, c.n_dofs * nv * 8, s);
  if (c.n_cells == 0) return;
  static const OpTab<double, N> tab = make_optab<double, N>();
  static const Gauss1D<N> g = make_gauss<N>();
  for_colours(c, [&](unsigned n, const int32_t* cells) {
    dim3 grid(n, nv);
    rhs_kernel<K><<<grid, N * N, 0, s>>>(c.ent, c.mask, c.ijk, c.n_cells, c.h0, c.lo, tab, g, kind, params,
                                         n_terms, b, nv, static_cast<const double*>(c.geo64), c.geo_n0, cells);
    check_launch();
  });
}

}  // namespace

void launch_vmult_fused(const CellView& c, int dtype, int nv, void* dst, const void* src, const FusedStep& f,
                        hipStream_t s) {
  switch (dtype) {
    case MFMG_F64: vmult_f64(c, nv, dst, src, f, s); break;
    case MFMG_F32: vmult_f32(c, nv, dst, src, f, s); break;
    case MFMG_BF16: vmult_bf16(c, nv, dst, src, f, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
}

void launch_vmult(const CellView& c, int dtype, int nv, void* dst, const void* src, hipStream_t s) {
  launch_vmult_fused(c, dtype, nv, dst, src, FusedStep{}, s);
}

void launch_diagonal(const CellView& c, double* diag, hipStream_t s) {
  switch (c.k) {
    case 1: diag_k<1>(c, diag, s); break;
    case 2: diag_k<2>(c, diag, s); break;
    case 3: diag_k<3>(c, diag, s); break;
    case 4: diag_k<4>(c, diag, s); break;
    case 5: diag_k<5>(c, diag, s); break;
    case 6: diag_k<6>(c, diag, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "degree");
  }
}

template <int K>
void distribute_k(const CellView& c, const double* x, double* out, hipStream_t s) {
  constexpr int N = K + 1;
  if (c.n_cells == 0) return;
  static const OpTab<double, N> tab = make_optab<double, N>();
  distribute_kernel<K><<<static_cast<unsigned>(c.n_cells), N * N, 0, s>>>(c.ent, c.mask, c.n_cells, tab, x, out);
  check_launch();
}

void launch_distribute(const CellView& c, const double* x, double* out, hipStream_t s) {
  switch (c.k) {
    case 1: distribute_k<1>(c, x, out, s); break;
    case 2: distribute_k<2>(c, x, out, s); break;
    case 3: distribute_k<3>(c, x, out, s); break;
    case 4: distribute_k<4>(c, x, out, s); break;
    case 5: distribute_k<5>(c, x, out, s); break;
    case 6: distribute_k<6>(c, x, out, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "degree");
  }
}

void launch_rhs(const CellView& c, int kind, const double* params, int n_terms, int nv, double* b,
                hipStream_t s) {
  switch (c.k) {
    case 1: rhs_k<1>(c, kind, params, n_terms, nv, b, s); break;
    case 2: rhs_k<2>(c, kind, params, n_terms, nv, b, s); break;
    case 3: rhs_k<3>(c, kind, params, n_terms, nv, b, s); break;
    case 4: rhs_k<4>(c, kind, params, n_terms, nv, b, s); break;
    case 5: rhs_k<5>(c, kind, params, n_terms, nv, b, s); break;
    case 6: rhs_k<6>(c, kind, params, n_terms, nv, b, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "degree");
  }
}

void launch_fill(int, void* x, int64_t n_bytes, hipStream_t s) { zero_bytes(x, n_bytes, s); }

void launch_cheb_step(int dtype, int64_t n_dofs, int nv, bool first, double c_dd, double c_r, const void* t,
                      const void* b, const void* dinv, void* d, void* x, hipStream_t s) {
  const unsigned g = grid_for(n_dofs * nv);
  switch (dtype) {
    case MFMG_F64:
      cheb_kernel<double><<<g, VEC_THREADS, 0, s>>>(n_dofs, nv, first, c_dd, c_r, static_cast<const double*>(t),
                                                    static_cast<const double*>(b), static_cast<const double*>(dinv),
                                                    static_cast<double*>(d), static_cast<double*>(x));
      break;
    case MFMG_F32:
      cheb_kernel<float><<<g, VEC_THREADS, 0, s>>>(n_dofs, nv, first, static_cast<float>(c_dd),
                                                   static_cast<float>(c_r), static_cast<const float*>(t),
                                                   static_cast<const float*>(b), static_cast<const float*>(dinv),
                                                   static_cast<float*>(d), static_cast<float*>(x));
      break;
    case MFMG_BF16:
      cheb_kernel<bf16><<<g, VEC_THREADS, 0, s>>>(n_dofs, nv, first, static_cast<float>(c_dd),
                                                  static_cast<float>(c_r), static_cast<const float*>(t),
                                                  static_cast<const bf16*>(b), static_cast<const float*>(dinv),
                                                  static_cast<bf16*>(d), static_cast<bf16*>(x));
      break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
  check_launch();
}

void launch_residual_update(int dtype, int64_t n, const void* b, const void* t, void* r, hipStream_t s) {
  const unsigned g = grid_for(n);
  switch (dtype) {
    case MFMG_F64:
      residual_kernel<double><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const double*>(b),
                                                        static_cast<const double*>(t), static_cast<double*>(r));
      break;
    case MFMG_F32:
      residual_kernel<float><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const float*>(b),
                                                       static_cast<const float*>(t), static_cast<float*>(r));
      break;
    case MFMG_BF16:
      residual_kernel<bf16><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const bf16*>(b), static_cast<const float*>(t),
                                                      static_cast<bf16*>(r));
      break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
  check_launch();
}

void launch_cast_from_f64(int dtype, int64_t n, const double* src, void* dst, hipStream_t s) {
  const unsigned g = grid_for(n);
  switch (dtype) {
    case MFMG_F64: cast_from_f64_kernel<double><<<g, VEC_THREADS, 0, s>>>(n, src, static_cast<double*>(dst)); break;
    case MFMG_F32: cast_from_f64_kernel<float><<<g, VEC_THREADS, 0, s>>>(n, src, static_cast<float*>(dst)); break;
    case MFMG_BF16: cast_from_f64_kernel<bf16><<<g, VEC_THREADS, 0, s>>>(n, src, static_cast<bf16*>(dst)); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
  check_launch();
}

void launch_cast_to_f64(int dtype, int64_t n, const void* src, double* dst, hipStream_t s) {
  const unsigned g = grid_for(n);
  switch (dtype) {
    case MFMG_F64: cast_to_f64_kernel<double><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const double*>(src), dst); break;
    case MFMG_F32: cast_to_f64_kernel<float><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const float*>(src), dst); break;
    case MFMG_BF16: cast_to_f64_kernel<bf16><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const bf16*>(src), dst); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
  check_launch();
}

void launch_cast(int dtype_src, int dtype_dst, int64_t n, const void* src, void* dst, hipStream_t s) {
  if (dtype_src == MFMG_F64) { launch_cast_from_f64(dtype_dst, n, static_cast<const double*>(src), dst, s); return; }
  if (dtype_dst == MFMG_F64) { launch_cast_to_f64(dtype_src, n, src, static_cast<double*>(dst), s); return; }
  const unsigned g = grid_for(n);
  if (dtype_src == MFMG_F32 && dtype_dst == MFMG_BF16)
    cast_kernel<float, bf16><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const float*>(src), static_cast<bf16*>(dst));
  else if (dtype_src == MFMG_BF16 && dtype_dst == MFMG_F32)
    cast_kernel<bf16, float><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const bf16*>(src), static_cast<float*>(dst));
  else if (dtype_src == dtype_dst)
    (void)hipMemcpyAsync(dst, src, n * dtype_size(dtype_src), hipMemcpyDeviceToDevice, s);
  else
    throw Error(MFMG_ERR_UNSUPPORTED, "cast");
  check_launch();
}

namespace {
template <typename A>
void copy_map_to(int dtype_dst, int64_t n, int nv, const int32_t* si, const int32_t* di, const A* src, void* dst,
                 hipStream_t s) {
  const unsigned g = grid_for(n * nv);
  switch (dtype_dst) {
    case MFMG_F64: copy_map_kernel<A, double><<<g, VEC_THREADS, 0, s>>>(n, nv, si, di, src, static_cast<double*>(dst)); break;
    case MFMG_F32: copy_map_kernel<A, float><<<g, VEC_THREADS, 0, s>>>(n, nv, si, di, src, static_cast<float*>(dst)); break;
    case MFMG_BF16: copy_map_kernel<A, bf16><<<g, VEC_THREADS, 0, s>>>(n, nv, si, di, src, static_cast<bf16*>(dst)); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
}
}  // namespace

void launch_copy_map(int dtype_src, int dtype_dst, int64_t n, int nv, const int32_t* src_idx, const int32_t* dst_idx,
                     const void* src, void* dst, hipStream_t s) {
  if (n == 0) return;
  switch (dtype_src) {
    case MFMG_F64: copy_map_to(dtype_dst, n, nv, src_idx, dst_idx, static_cast<const double*>(src), dst, s); break;
    case MFMG_F32: copy_map_to(dtype_dst, n, nv, src_idx, dst_idx, static_cast<const float*>(src), dst, s); break;
    case MFMG_BF16: copy_map_to(dtype_dst, n, nv, src_idx, dst_idx, static_cast<const bf16*>(src), dst, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
  check_launch();
}

void launch_zero_entries(int64_t n, const int32_t* idx, double* a64, float* a32, hipStream_t s) {
  if (n == 0) return;
  zero_entries_kernel<<<grid_for(n), VEC_THREADS, 0, s>>>(n, idx, a64, a32);
  check_launch();
}

void launch_acc_to_storage(int dtype, int64_t n, const void* acc, void* dst, hipStream_t s) {
  const unsigned g = grid_for(n);
  switch (dtype) {
    case MFMG_F64:
      acc_to_storage_kernel<double><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const double*>(acc),
                                                              static_cast<double*>(dst));
      break;
    case MFMG_F32:
      acc_to_storage_kernel<float><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const float*>(acc),
                                                             static_cast<float*>(dst));
      break;
    case MFMG_BF16:
      acc_to_storage_kernel<bf16><<<g, VEC_THREADS, 0, s>>>(n, static_cast<const float*>(acc),
                                                            static_cast<bf16*>(dst));
      break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
  check_launch();
}

namespace {
__global__ void coef_check_kernel(int64_t n, const double* __restrict__ c, int* __restrict__ flag) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    if (!(c[i] >= 1e-30 && c[i] <= 1e30)) flag[0] = 1;
}

__global__ void coef_restrict_kernel(int64_t n_ident, const int32_t* __restrict__ ident_c,
                                     const int32_t* __restrict__ ident_f, int64_t n_ref,
                                     const int32_t* __restrict__ ref_c, const int32_t* __restrict__ ref_f,
                                     const double* __restrict__ cf, double* __restrict__ cc) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n_ident + n_ref;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    if (i < n_ident) {
      cc[ident_c[i]] = cf[ident_f[i]];
    } else {
      const int64_t r = i - n_ident;
      double sum = 0.0;
      for (int ch = 0; ch < 8; ++ch) sum += cf[ref_f[ch * n_ref + r]];
      cc[ref_c[r]] = sum / 8.0;
    }
  }
}

__global__ void coef_apply_kernel(int64_t n, const double* __restrict__ c, uint32_t* __restrict__ mask,
                                  CellMeta* __restrict__ meta) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const uint32_t m = (mask[i] & ~MASK_COEF_BITS) | coef_bits(c[i]);
    mask[i] = m;
    meta[i].mask = (meta[i].mask & ~MASK_COEF_BITS) | (m & MASK_COEF_BITS);  // (it has its own orientation bits)
  }
}
}  // namespace

void launch_coef_check(int64_t n, const double* c, int* flag, hipStream_t s) {
  if (n == 0) return;
  coef_check_kernel<<<grid_for(n), VEC_THREADS, 0, s>>>(n, c, flag);
  check_launch();
}

void launch_coef_restrict(const TransferView& t, const double* c_fine, double* c_coarse, hipStream_t s) {
  const int64_t n = t.n_ident + t.n_refined;
  if (n == 0) return;
  coef_restrict_kernel<<<grid_for(n), VEC_THREADS, 0, s>>>(t.n_ident, t.ident_coarse, t.ident_fine, t.n_refined,
                                                         t.refined_coarse, t.refined_fine, c_fine, c_coarse);
  check_launch();
}

void launch_coef_apply(int64_t n_cells, const double* c, uint32_t* mask, CellMeta* meta, hipStream_t s) {
  if (n_cells == 0) return;
  coef_apply_kernel<<<grid_for(n_cells), VEC_THREADS, 0, s>>>(n_cells, c, mask, meta);
  check_launch();
}

void launch_inverse_diag(int dtype, int64_t n, const double* diag, void* dinv, hipStream_t s) {
  const unsigned g = grid_for(n);
  if (dtype == MFMG_F64)
    inverse_diag_kernel<double><<<g, VEC_THREADS, 0, s>>>(n, diag, static_cast<double*>(dinv));
  else
    inverse_diag_kernel<float><<<g, VEC_THREADS, 0, s>>>(n, diag, static_cast<float*>(dinv));
  check_launch();
}

void launch_dense_matvec(int dtype, int64_t n0, int nv, const void* Ainv, const void* b, void* x, void*,
                         hipStream_t s) {
  if (n0 == 0) return;
  dim3 grid(static_cast<unsigned>((n0 + 3) / 4), nv);
  switch (dtype) {
    case MFMG_F64:
      dense_matvec_kernel<double><<<grid, 256, 0, s>>>(n0, nv, static_cast<const double*>(Ainv),
                                                       static_cast<const double*>(b), static_cast<double*>(x));
      break;
    case MFMG_F32:
      dense_matvec_kernel<float><<<grid, 256, 0, s>>>(n0, nv, static_cast<const float*>(Ainv),
                                                      static_cast<const float*>(b), static_cast<float*>(x));
      break;
    case MFMG_BF16:
      dense_matvec_kernel<bf16><<<grid, 256, 0, s>>>(n0, nv, static_cast<const float*>(Ainv),
                                                     static_cast<const bf16*>(b), static_cast<bf16*>(x));
      break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
  check_launch();
}

int dot_partials_needed() { return 16 * DOT_BLOCKS; }

namespace {
// blocks of a dot product over n entries: about four entries a thread
unsigned dot_grid(int64_t n, int nv) {
  if (nv < 1 || nv > 8) throw Error(MFMG_ERR_INVALID_ARG, "dot: n_vec must be in [1, 8]");
  return static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(DOT_BLOCKS, (n + 4 * DOT_THREADS - 1) / (4 * DOT_THREADS))));
}
}  // namespace

void launch_dot(int64_t n_dofs, int nv, const double* a, const double* b, double* partial, double* result,
                hipStream_t s) {
  const int64_t n = n_dofs * nv;
  const unsigned g = dot_grid(n, nv);
  dot_kernel<<<g, DOT_THREADS, 0, s>>>(n, nv, a, b, partial);
  check_launch();
  dot_sum_kernel<<<nv, DOT_THREADS, 0, s>>>(g, nv, partial, result, nullptr);
  check_launch();
}

void launch_dot2(int64_t n_dofs, int nv, const double* a, const double* b, const double* c, double* partial,
                 double* result_b, double* result_c, hipStream_t s) {
  const int64_t n = n_dofs * nv;
  const unsigned g = dot_grid(n, nv);
  dot2_kernel<<<g, DOT_THREADS, 0, s>>>(n, nv, a, b, c, partial);
  check_launch();
  dot_sum_kernel<<<2 * nv, DOT_THREADS, 0, s>>>(g, nv, partial, result_b, result_c);
  check_launch();
}

void launch_cg_update_xr(int64_t n_dofs, int nv, const double* num, const double* den, const double* p,
                         const double* q, double* x, double* r, double* partial, double* rr, hipStream_t s) {
  const int64_t n = n_dofs * nv;
  const unsigned g = dot_grid(n, nv);
  cg_xr_dot_kernel<<<g, DOT_THREADS, 0, s>>>(n, nv, num, den, p, q, x, r, partial);
  check_launch();
  dot_sum_kernel<<<nv, DOT_THREADS, 0, s>>>(g, nv, partial, rr, nullptr);
  check_launch();
}

void launch_cg_update_p(int64_t n_dofs, int nv, const double* num, const double* sub, const double* den,
                        const double* z, double* p, hipStream_t s) {
  cg_p_kernel<<<grid_for(n_dofs * nv), VEC_THREADS, 0, s>>>(n_dofs, nv, num, sub, den, z, p);
  check_launch();
}

}  // namespace mfmg
