// Intergrid transfer (Section 3.5, Eq. eq:impl:loop:categorized): one coarse
// cell (transfer group) at a time.  Prolongation:
//   coarse gather G_c with constraints C_c (in-place interpolation),
//   category prolongation P (three 1D sweeps; identity category: none),
//   weights W, scatter S_f.
// Restriction is the transpose of every step.  The weights: the paper's W
// divides each fine value by the number of groups that reach it, so that the
// groups' equal contributions sum to it once.  Here W is 1 on one owner
// (group, lattice entity) pair per fine entity and 0 elsewhere (and on
// constrained fine DoFs): the same operator, and the prolongation writes each
// fine DoF from one block with a plain read-modify-write instead of atomics.
//
// Lattice of a group: NF nodes per axis.  Refinement category: NF = 2k+1
// nodes covering the 8 children; polynomial category: NF = k_f+1; identity:
// NF = NC, no sweeps.
#include "device.hpp"
#include "kernels.hpp"
#include "slots.hpp"

namespace mfmg {

namespace {

template <typename T, int NF, int NC>
struct TrTab {
  T P[NF * NC];  // 1D prolongation, row-major NF x NC
  T H[NC * NC];  // hanging interpolation of the coarse cell, lower half
};

// Lattice of n nodes per axis over cells of degree K: n = K + 1 (one cell) or
// 2 K + 1 (two cells per axis).  Along an axis the nodes fall into 3 or 5
// classes (end points of the cells, and the interiors between them, which
// have odd class numbers); a lattice entity is a triple of classes and its
// DoFs are numbered x fastest.
template <int K, int N>
__device__ __forceinline__ int axis_class(int I) {
  if constexpr (N == 2 * K + 1) return I == 0 ? 0 : I < K ? 1 : I == K ? 2 : I < 2 * K ? 3 : 4;
  else return I == 0 ? 0 : I < K ? 1 : 2;
}

// Nodes of a lattice seen by the owner of its x index I: the owner's row
// (J, 0..N-1) of nodes along z lies in NCLS entities; f(L, DoF), DoF < 0:
// skipped node.  `ents`: the group's record.
template <int K, int N>
struct LatticeRows {
  static constexpr int NCLS = N == 2 * K + 1 ? 5 : 3, KM = K > 1 ? K - 1 : 1;
  int ci, off, sx;
  __device__ __forceinline__ explicit LatticeRows(int I) {
    ci = axis_class<K, N>(I);
    off = (ci & 1) ? (ci == 3 ? I - K : I) - 1 : 0;
    sx = (ci & 1) ? KM : 1;
  }
  template <typename F>
  __device__ __forceinline__ void row(int J, const int32_t* ents, F f) const {
    const int cj = axis_class<K, N>(J);
    const int o = off + ((cj & 1) ? ((cj == 3 ? J - K : J) - 1) * sx : 0);
    const int sz = (cj & 1) ? sx * KM : sx;
#pragma unroll
    for (int q = 0; q < NCLS; ++q) {
      const int lo = q == 0 ? 0 : q == 1 ? 1 : q == 2 ? K : q == 3 ? K + 1 : 2 * K;
      const int cnt = (q & 1) ? K - 1 : 1;
      if (cnt == 0) continue;
      const int32_t e = ents[ci + NCLS * (cj + NCLS * q)];
#pragma unroll
      for (int r = 0; r < cnt; ++r) f(lo + r, e < 0 ? -1 : e + o + ((q & 1) ? r * sz : 0));
    }
  }
};

// u <- H_s u (H_s^T u if TRANS): the halves are mirror images, H_1 = J H_0 J
template <int N, typename T, bool TRANS>
__device__ __forceinline__ void half_interp(const T (&H)[N * N], int s, T (&u)[N]) {
  T w[N];
#pragma unroll
  for (int j = 0; j < N; ++j) w[j] = s ? u[N - 1 - j] : u[j];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T acc = T(0);
#pragma unroll
    for (int j = 0; j < N; ++j) acc += H[TRANS ? j * N + i : i * N + j] * w[j];
    if (s) u[N - 1 - i] = acc;
    else u[i] = acc;
  }
}

// y = P x (TRANS: P^T x) for the NF x NC matrix P
template <int NI, int NO, typename T, bool TRANS>
__device__ __forceinline__ void sweep(const T* __restrict__ P, const T (&x)[NI], T (&y)[NO]) {
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    T acc = T(0);
#pragma unroll
    for (int j = 0; j < NI; ++j) acc += (TRANS ? P[j * NO + i] : P[i * NI + j]) * x[j];
    y[i] = acc;
  }
}

constexpr int TR_WAVES = 2;  // independent wavefronts per block
enum { PLANES, LINES_ONE, LINES_EACH };  // how the lanes split a group: planes, or lines of one or of each vector

// How a launch splits the work: `groups` transfer groups per wavefront, 2^lv
// interleaved vectors at a time.
struct TrShape {
  int groups, lv;
};

// Values of one group and vector in LDS, nodes x fastest in rows of odd length
// (neighbouring rows fall on different banks): the coarse cell's NC^3 nodes,
// widened in place to NF along x; behind them (LINES) the nodes after the
// y-sweep.
template <int NF, int NC, bool LINES>
struct TrLds {
  static constexpr int RS = NF | 1;
  static constexpr int Y = NC * NC * RS;
  static constexpr int N = Y + (LINES ? NC * NF * NF : 0);
};

// What bounds it: HBM traffic (Q3 -> Q6, 8 FP32 vectors: 4.5 GB in 1.00 ms;
// the restriction's 2.8 GB in 1.11 ms, beside 1.4e8 atomic adds; 4.3 and 4.2 ms
// with one 256-thread block per group and its nodes looked up one by one).  On
// one vector latency (Q4 prolongation onto 17M FP64 DoFs 110 us, 326 before).
// A wavefront works on its own groups without
// block barriers.  All index data of a group is one contiguous record (the
// first DoF of each lattice entity, -1 where another group owns it or it is
// constrained).  A lane owns one x index of the fine lattice and one vector,
// so the y- and z-sweeps of its plane run in registers between LDS and global
// memory; only the x-sweep goes through LDS.  The fine values of the next row
// are loaded while one is worked on; the vector index is the fastest one of
// the lanes (adjacent lanes touch adjacent memory).
//
// LINES (one vector per wavefront): the lanes go over the z-lines of the fine lattice
// instead, x fastest, with the y-sweep through LDS.  A load then covers the
// runs of whole faces and interiors ((k-1)^2 adjacent values) where the
// planes' load covers one row of each of several groups, k-1 values apiece
// (the same prolongation 110 us by lines, 156 us by planes at its best).
template <int KF, int KC, int NF, typename S, typename T, bool PROLONG, int HOW>
__global__ void __launch_bounds__(64 * TR_WAVES)
    transfer_kernel(const int32_t* __restrict__ fdesc, const int32_t* __restrict__ cdesc, int64_t n_groups,
                    int64_t n_blocks, int groups, int lv, TrTab<T, NF, KC + 1> tab, const S* __restrict__ src,
                    S* __restrict__ dst, int nv, bool plain) {
  constexpr int NC = KC + 1, FS = transfer_record(LatticeRows<KF, NF>::NCLS), CS = transfer_record(3);
  constexpr bool IDENT = NF == NC && KF == KC, LINES = HOW != PLANES;
  if constexpr (HOW == LINES_ONE) nv = 1;  // (the index arithmetic folds: 3 to 15 % of the time)
  using L = TrLds<NF, NC, LINES>;
  constexpr int RS = L::RS, LN = L::N;
  extern __shared__ __align__(16) char lds_raw[];
  // blocks of an XCD (block i runs on XCD i mod 8) take one contiguous range
  // of groups: the neighbours' partially used lines meet in its L2
  const int64_t per = gridDim.x / 8;
  const int64_t blk = static_cast<int64_t>(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (blk >= n_blocks) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  // (lines: the vectors of a group are neighbouring wavefronts)
  const int64_t unit = blk * TR_WAVES + wave;
  const int only = LINES ? static_cast<int>(unit % nv) : 0;
  const int64_t g0 = (LINES ? unit / nv : unit) * groups;
  if (g0 >= n_groups) return;  // (no block barriers below)
  const int ng = n_groups - g0 < groups ? static_cast<int>(n_groups - g0) : groups;
  const WaveSync sync{};
  const int vb = 1 << lv;
  const int wave_values = (groups * LN) << lv, wave_ints = groups * (FS + CS);
  T* X = reinterpret_cast<T*>(lds_raw) + wave * wave_values;
  int32_t* Ef = reinterpret_cast<int32_t*>(reinterpret_cast<T*>(lds_raw) + TR_WAVES * wave_values) + wave * wave_ints;
  int32_t* Ec = Ef + groups * FS;
  int hang = 0;
  for (int i = lane; i < ng * CS; i += 64) {
    const int32_t e = cdesc[g0 * CS + i];
    Ec[i] = e;
    if (i % CS == 27 && mask_hanging(static_cast<uint32_t>(e))) hang = 1;
  }
  for (int i = lane; i < ng * FS; i += 64) Ef[i] = fdesc[g0 * FS + i];
  const bool any_hang = __any(hang) != 0;
  sync();

  auto at = [&](int g, int a, int b, int c, int v) { return ((g * LN + (c * NC + b) * RS + a) << lv) + v; };
  auto y_at = [&](int g, int i, int j, int c) { return g * LN + L::Y + (c * NF + j) * NF + i; };  // (LINES)
  // f(group, p, q, vector inside the chunk) for the NC^2 lines of every group
  auto for_lines = [&](int nb, auto f) {
    const int n = (ng * NC * NC) << lv;
    for (int t = lane; t < n; t += 64) {
      const int q = t >> lv, g = q / (NC * NC), line = q - g * NC * NC, v = t & (vb - 1);
      if (v < nb) f(g, line % NC, line / NC, v);
    }
  };
  // this lane's plane of the fine lattice
  const int q0 = lane >> lv, pg = q0 / NF, pi = q0 - pg * NF, pv = lane & (vb - 1);
  const LatticeRows<KF, NF> rows(pi);
  const int32_t* ef = Ef + pg * FS;

  for (int v0 = only; v0 < (LINES ? only + 1 : nv); v0 += vb) {
    const int nb = nv - v0 < vb ? nv - v0 : vb;
    const bool mine = pg < ng && pv < nb;
    auto fine_at = [&](int32_t e) {
      if constexpr (HOW == LINES_ONE) return static_cast<int64_t>(e);
      return static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(e)) * nv + (LINES ? v0 : v0 + pv));
    };
    auto load_row = [&](const S* p, int J, T (&w)[NF]) {
      if (mine)
        rows.row(J, ef, [&](int l, int32_t e) { w[l] = e < 0 ? T(0) : load_as<T>(p[fine_at(e)]); });
    };
    T w[NF], next[NF];
#pragma unroll
    for (int l = 0; l < NF; ++l) w[l] = next[l] = T(0);
    auto load_line = [&](const S* p, int t, T (&w)[NF]) {  // z-line t of the wavefront's groups
      if (t >= ng * NF * NF) return;
      const int g = t / (NF * NF), r0 = t - g * NF * NF;
      LatticeRows<KF, NF>(r0 % NF).row(r0 / NF, Ef + g * FS,
                                       [&](int l, int32_t e) { w[l] = e < 0 ? T(0) : load_as<T>(p[fine_at(e)]); });
    };
    if constexpr (LINES) load_line(PROLONG ? dst : src, lane, next);
    else load_row(PROLONG ? dst : src, 0, next);
    auto coarse_line = [&](int g, int a, int b, int v, auto f) {  // f(c, value index) along z
      LatticeRows<KC, NC>(a).row(b, Ec + g * CS, [&](int c, int32_t e) {
        f(c, e, static_cast<uint64_t>(static_cast<uint32_t>(e)) * nv + (v0 + v));
      });
    };
    auto mask_of = [&](int g) { return static_cast<uint32_t>(Ec[g * CS + 27]); };
    auto interp_y = [&]() {
      for_lines(nb, [&](int g, int a, int c, int v) {
        const uint32_t m = mask_of(g);
        if (!hanging_line(m, 1, a, c, KC)) return;
        T u[NC];
#pragma unroll
        for (int r = 0; r < NC; ++r) u[r] = X[at(g, a, r, c, v)];
        half_interp<NC, T, !PROLONG>(tab.H, mask_sub(m, 1), u);
#pragma unroll
        for (int r = 0; r < NC; ++r) X[at(g, a, r, c, v)] = u[r];
      });
      sync();
    };
    if constexpr (PROLONG) {
      // z-lines of coarse nodes from global memory, hanging z-interpolation
      for_lines(nb, [&](int g, int a, int b, int v) {
        T u[NC];
        coarse_line(g, a, b, v, [&](int c, int32_t e, uint64_t i) { u[c] = e < 0 ? T(0) : load_as<T>(src[i]); });
        if (any_hang) {
          const uint32_t m = mask_of(g);
          if (hanging_line(m, 2, a, b, KC)) half_interp<NC, T, false>(tab.H, mask_sub(m, 2), u);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) X[at(g, a, b, c, v)] = u[c];
      });
      sync();
      if (any_hang) interp_y();
      if (!IDENT || any_hang) {  // x-lines: hanging interpolation, x-sweep in place
        for_lines(nb, [&](int g, int b, int c, int v) {
          const uint32_t m = mask_of(g);
          const bool h = any_hang && hanging_line(m, 0, b, c, KC);
          if (IDENT && !h) return;
          T u[NC];
#pragma unroll
          for (int r = 0; r < NC; ++r) u[r] = X[at(g, r, b, c, v)];
          if (h) half_interp<NC, T, false>(tab.H, mask_sub(m, 0), u);
          T y[NF];
          if constexpr (IDENT) {
#pragma unroll
            for (int r = 0; r < NF; ++r) y[r] = u[r];
          } else {
            sweep<NC, NF, T, false>(tab.P, u, y);
          }
#pragma unroll
          for (int r = 0; r < NF; ++r) X[at(g, r, b, c, v)] = y[r];
        });
        sync();
      }
      if constexpr (LINES) {
        if constexpr (!IDENT) {  // y-lines (x = i)
          for (int t = lane; t < ng * NF * NC; t += 64) {
            const int g = t / (NF * NC), r0 = t - g * NF * NC, i = r0 % NF, c = r0 / NF;
            T u[NC], y[NF];
#pragma unroll
            for (int b = 0; b < NC; ++b) u[b] = X[at(g, i, b, c, 0)];
            sweep<NC, NF, T, false>(tab.P, u, y);
#pragma unroll
            for (int j = 0; j < NF; ++j) X[y_at(g, i, j, c)] = y[j];
          }
          sync();
        }
        for (int t = lane; t < ng * NF * NF; t += 64) {
          T old[NF];
#pragma unroll
          for (int l = 0; l < NF; ++l) old[l] = next[l];
          load_line(dst, t + 64, next);
          const int g = t / (NF * NF), r0 = t - g * NF * NF, i = r0 % NF, j = r0 / NF;
          if constexpr (IDENT) {
#pragma unroll
            for (int l = 0; l < NF; ++l) w[l] = X[at(g, i, j, l, 0)];
          } else {
            T u[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) u[c] = X[y_at(g, i, j, c)];
            sweep<NC, NF, T, false>(tab.P, u, w);
          }
          LatticeRows<KF, NF>(i).row(j, Ef + g * FS, [&](int l, int32_t e) {
            if (e >= 0) dst[fine_at(e)] = store_as<S>(old[l] + w[l]);
          });
        }
      } else {
        // this lane's plane: y- and z-sweeps, rows added to the owned DoFs
        T plane[IDENT ? 1 : NC * NC];
        if constexpr (!IDENT) {
          if (mine) {
#pragma unroll
            for (int r = 0; r < NC * NC; ++r) plane[r] = X[at(pg, pi, r % NC, r / NC, pv)];
          }
        }
#pragma unroll 1
        for (int J = 0; J < NF; ++J) {
          T old[NF];
#pragma unroll
          for (int l = 0; l < NF; ++l) old[l] = next[l];
          if (J + 1 < NF) load_row(dst, J + 1, next);
          if (!mine) continue;
          if constexpr (IDENT) {
#pragma unroll
            for (int l = 0; l < NF; ++l) w[l] = X[at(pg, pi, J, l, pv)];
          } else {
            T u[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
              T acc = T(0);
#pragma unroll
              for (int b = 0; b < NC; ++b) acc += tab.P[J * NC + b] * plane[c * NC + b];
              u[c] = acc;
            }
            sweep<NC, NF, T, false>(tab.P, u, w);
          }
          rows.row(J, ef, [&](int l, int32_t e) {
            if (e >= 0) dst[fine_at(e)] = store_as<S>(old[l] + w[l]);
          });
        }
      }
      sync();
    } else {
      if constexpr (LINES) {
        // z-lines of fine values (each owned one enters once), transposed z-sweep
        for (int t = lane; t < ng * NF * NF; t += 64) {
#pragma unroll
          for (int l = 0; l < NF; ++l) w[l] = next[l];
          load_line(src, t + 64, next);
          const int g = t / (NF * NF), r0 = t - g * NF * NF, i = r0 % NF, j = r0 / NF;
          if constexpr (IDENT) {
#pragma unroll
            for (int l = 0; l < NF; ++l) X[at(g, i, j, l, 0)] = w[l];
          } else {
            T u[NC];
            sweep<NF, NC, T, true>(tab.P, w, u);
#pragma unroll
            for (int c = 0; c < NC; ++c) X[y_at(g, i, j, c)] = u[c];
          }
        }
        if constexpr (!IDENT) {
          sync();
          for (int t = lane; t < ng * NF * NC; t += 64) {  // y-lines (x = i)
            const int g = t / (NF * NC), r0 = t - g * NF * NC, i = r0 % NF, c = r0 / NF;
            T u[NC], y[NF];
#pragma unroll
            for (int j = 0; j < NF; ++j) y[j] = X[y_at(g, i, j, c)];
            sweep<NF, NC, T, true>(tab.P, y, u);
#pragma unroll
            for (int b = 0; b < NC; ++b) X[at(g, i, b, c, 0)] = u[b];
          }
        }
      } else {
        // this lane's plane: rows of fine values (each owned one enters once),
        // transposed z- and y-sweeps
        T plane[IDENT ? 1 : NC * NC];
        if constexpr (!IDENT) {
#pragma unroll
          for (int r = 0; r < NC * NC; ++r) plane[r] = T(0);
        }
#pragma unroll 1
        for (int J = 0; J < NF; ++J) {
#pragma unroll
          for (int l = 0; l < NF; ++l) w[l] = next[l];
          if (J + 1 < NF) load_row(src, J + 1, next);
          if constexpr (IDENT) {
            if (mine) {
#pragma unroll
              for (int l = 0; l < NF; ++l) X[at(pg, pi, J, l, pv)] = w[l];
            }
          } else {
            T u[NC];
            sweep<NF, NC, T, true>(tab.P, w, u);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
              for (int b = 0; b < NC; ++b) plane[c * NC + b] += tab.P[J * NC + b] * u[c];
          }
        }
        if constexpr (!IDENT) {
          if (mine) {
#pragma unroll
            for (int r = 0; r < NC * NC; ++r) X[at(pg, pi, r % NC, r / NC, pv)] = plane[r];
          }
        }
      }
      sync();
      if (!IDENT || any_hang) {  // x-lines: transposed x-sweep and interpolation, in place
        for_lines(nb, [&](int g, int b, int c, int v) {
          const uint32_t m = mask_of(g);
          const bool h = any_hang && hanging_line(m, 0, b, c, KC);
          if (IDENT && !h) return;
          T y[NF], u[NC];
#pragma unroll
          for (int r = 0; r < NF; ++r) y[r] = X[at(g, r, b, c, v)];
          if constexpr (IDENT) {
#pragma unroll
            for (int r = 0; r < NC; ++r) u[r] = y[r];
          } else {
            sweep<NF, NC, T, true>(tab.P, y, u);
          }
          if (h) half_interp<NC, T, true>(tab.H, mask_sub(m, 0), u);
#pragma unroll
          for (int r = 0; r < NC; ++r) X[at(g, r, b, c, v)] = u[r];
        });
        sync();
      }
      if (any_hang) interp_y();
      // z-lines of coarse nodes: transposed z-interpolation, scatter-add
      for_lines(nb, [&](int g, int a, int b, int v) {
        T u[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) u[c] = X[at(g, a, b, c, v)];
        if (any_hang) {
          const uint32_t m = mask_of(g);
          if (hanging_line(m, 2, a, b, KC)) half_interp<NC, T, true>(tab.H, mask_sub(m, 2), u);
        }
        const bool inner = a > 0 && a < KC && b > 0 && b < KC;  // the cell interior is this group's alone
        coarse_line(g, a, b, v, [&](int c, int32_t e, uint64_t i) {
          if (e >= 0) add_to<S, T>(&dst[i], u[c], plain || (inner && c > 0 && c < KC));
        });
      });
      sync();
    }
  }
}

template <typename T, int NF, int NC>
TrTab<T, NF, NC> make_trtab(int kf, int kc) {
  TrTab<T, NF, NC> t;
  const Tables1D& tc = tables(kc);
  for (int i = 0; i < NC * NC; ++i) t.H[i] = static_cast<T>(tc.H[0][i]);
  if (kf == kc && NF == 2 * kc + 1) {
    for (int i = 0; i < NF * NC; ++i) t.P[i] = static_cast<T>(tc.T[i]);
  } else if (kf != kc && NF == 2 * kf + 1) {
    std::vector<double> P = hp_transfer_matrix(kf, kc);
    for (int i = 0; i < NF * NC; ++i) t.P[i] = static_cast<T>(P[i]);
  } else if (kf != kc) {
    std::vector<double> P = p_transfer_matrix(kf, kc);
    for (int i = 0; i < NF * NC; ++i) t.P[i] = static_cast<T>(P[i]);
  } else {
    for (int i = 0; i < NF * NC; ++i) t.P[i] = static_cast<T>((i / NC) == (i % NC) ? 1.0 : 0.0);
  }
  return t;
}

// Vectors at a time and groups per wavefront.  Planes: NF x 2^lv lanes work on
// a group, and as many groups as fit fill the wavefront; 2^lv is the smallest
// that takes all vectors in one pass, or the largest that fits (a pass more
// costs more than idle lanes: 3 FP32 vectors, Q3, 270,000 cells, prolongation
// 237 us in three full passes, 60 us in one with a quarter of the lanes idle;
// 8 vectors, Q4, 37,000 cells 153 us in four, 86 us in two).  Lines: the fewest groups
// whose NF^2 lines use 75 % of the lanes of their rounds, within LDS for 14
// wavefronts per CU (Q4, 30,000 refinement groups: FP32 88 us with one group
// of 2.5 KB per wavefront, 104 us with three).  Levels with fewer groups than would give every SIMD
// (1024) a wavefront spread them out.
template <int NF, int NC, bool LINES>
TrShape transfer_shape(int nv, int64_t n_groups, int bytes) {
  TrShape s{1, 0};
  const int64_t spread = std::max<int64_t>(1, n_groups / 1024);
  if constexpr (LINES) {
    double best = 0.0;
    for (int g = 1; g <= 8 && best < 0.75; ++g) {
      if (g > 1 && g * TrLds<NF, NC, true>::N * bytes > 11 * 1024) break;
      const int lines = g * NF * NF;
      const double used = lines / static_cast<double>((lines + 63) / 64 * 64);
      if (used > best) {
        best = used;
        s.groups = g;
      }
    }
  } else {
    while ((1 << s.lv) < nv && (NF << (s.lv + 1)) <= 64) ++s.lv;
    s.groups = 64 / (NF << s.lv);
  }
  s.groups = static_cast<int>(std::min<int64_t>(s.groups, spread));
  return s;
}

template <int KF, int KC, int NF, typename S, bool PROLONG, int HOW>
void transfer_run(const int32_t* fdesc, const int32_t* cdesc, int64_t n, int nv, void* dst, const void* src,
                  bool plain, hipStream_t s) {
  using T = typename Acc<S>::type;
  constexpr bool LINES = HOW != PLANES;
  if (n == 0) return;
  static const TrTab<T, NF, KC + 1> tab = make_trtab<T, NF, KC + 1>(KF, KC);
  const TrShape sh = transfer_shape<NF, KC + 1, LINES>(nv, n, sizeof(T));
  const int64_t units = (n + sh.groups - 1) / sh.groups * (LINES ? nv : 1);  // wavefronts
  const int64_t per_block = static_cast<int64_t>(sh.groups) * TR_WAVES;
  const int64_t blocks = (units + TR_WAVES - 1) / TR_WAVES, grid = (blocks + 7) / 8 * 8;
  constexpr int ints = transfer_record(LatticeRows<KF, NF>::NCLS) + transfer_record(3);
  const size_t lds = per_block * (ints * 4 + (TrLds<NF, KC + 1, LINES>::N << sh.lv) * sizeof(T));
  transfer_kernel<KF, KC, NF, S, T, PROLONG, HOW><<<static_cast<unsigned>(grid), 64 * TR_WAVES, lds, s>>>(
      fdesc, cdesc, n, blocks, sh.groups, sh.lv, tab, static_cast<const S*>(src), static_cast<S*>(dst), nv, plain);
  check_launch();
}

// Lines for one vector, and for several on levels with few groups, where a
// plane's chain of NF rows per lane takes longer than all the rest (64 cells,
// FP64, 3 vectors, Q6: restriction 93 us by planes, 37 us by lines; Q4 26 and
// 17 us; prolongation 61 and 27 us, 27 and 16 us).  With more groups the
// lines' wavefronts, one vector each, touch every line of memory (and the
// restriction's atomics every line of the coarse vector) n_vec times (8 FP32
// vectors, Q4, 37,000 cells: restriction 313 us against 79 us).  The two
// meet at 6,000 (FP64) and 8,000 (FP32) groups x vectors for the prolongation;
// for the restriction at 5 NF^3, at most 11,000 and 6,000: measured at every
// degree, 2 to 8 vectors, 64 to 270,000 cells.
template <int KF, int KC, int NF, typename S, bool PROLONG>
void transfer_split(const int32_t* fdesc, const int32_t* cdesc, int64_t n, int nv, void* dst, const void* src,
                    bool plain, hipStream_t s) {
  constexpr bool wide = sizeof(typename Acc<S>::type) == 8;
  constexpr int64_t most = PROLONG ? (wide ? 6000 : 8000) : std::min(5 * NF * NF * NF, wide ? 11000 : 6000);
  if (nv == 1) transfer_run<KF, KC, NF, S, PROLONG, LINES_ONE>(fdesc, cdesc, n, nv, dst, src, plain, s);
  else if (n * nv <= most) transfer_run<KF, KC, NF, S, PROLONG, LINES_EACH>(fdesc, cdesc, n, nv, dst, src, plain, s);
  else transfer_run<KF, KC, NF, S, PROLONG, PLANES>(fdesc, cdesc, n, nv, dst, src, plain, s);
}

template <int KF, int KC, int NF, typename S>
void transfer_launch(bool prolong, const TransferView& t, bool refined, int nv, void* dst, const void* src,
                     hipStream_t s) {
  constexpr int FS = transfer_record(LatticeRows<KF, NF>::NCLS), CS = transfer_record(3);
  const int32_t* fd = refined ? t.refined_fdesc : t.ident_fdesc;
  const int32_t* cd = refined ? t.refined_cdesc : t.ident_cdesc;
  const int64_t n = refined ? t.n_refined : t.n_ident;
  if (prolong) {  // each fine DoF has one writer: no colouring needed
    transfer_split<KF, KC, NF, S, true>(fd, cd, n, nv, dst, src, true, s);
    return;
  }
  // restriction: one launch, or in the deterministic mode one per colour of
  // the group list (plain adds into the coarse DoFs)
  const int64_t* off = refined ? t.refined_off : t.ident_off;
  if (!t.deterministic || !off) {
    transfer_split<KF, KC, NF, S, false>(fd, cd, n, nv, dst, src, false, s);
    return;
  }
  const int n_col = refined ? t.n_refined_colors : t.n_ident_colors;
  for (int k = 0; k < n_col; ++k)
    transfer_split<KF, KC, NF, S, false>(fd + off[k] * FS, cd + off[k] * CS, off[k + 1] - off[k], nv, dst, src, true,
                                       s);
}

template <int K, typename S>
void transfer_h(bool prolong, const TransferView& t, int nv, void* dst, const void* src, hipStream_t s) {
  transfer_launch<K, K, K + 1, S>(prolong, t, false, nv, dst, src, s);
  transfer_launch<K, K, 2 * K + 1, S>(prolong, t, true, nv, dst, src, s);
}

// geometric and polynomial coarsening in one step: identity pairs change the
// degree only, refined groups change both
template <int KF, int KC, typename S>
void transfer_hp(bool prolong, const TransferView& t, int nv, void* dst, const void* src, hipStream_t s) {
  transfer_launch<KF, KC, KF + 1, S>(prolong, t, false, nv, dst, src, s);
  transfer_launch<KF, KC, 2 * KF + 1, S>(prolong, t, true, nv, dst, src, s);
}

template <typename S>
void transfer_s(bool prolong, int kf, int kc, const TransferView& t, int nv, void* dst, const void* src,
                hipStream_t s) {
  if (!t.polynomial && kf != kc) {
    switch (kf * 10 + kc) {
      case 21: transfer_hp<2, 1, S>(prolong, t, nv, dst, src, s); break;
      case 31: transfer_hp<3, 1, S>(prolong, t, nv, dst, src, s); break;
      case 42: transfer_hp<4, 2, S>(prolong, t, nv, dst, src, s); break;
      case 52: transfer_hp<5, 2, S>(prolong, t, nv, dst, src, s); break;
      case 63: transfer_hp<6, 3, S>(prolong, t, nv, dst, src, s); break;
      default: throw Error(MFMG_ERR_UNSUPPORTED, "combined h and p transfer pair");
    }
    return;
  }
  if (!t.polynomial) {
    switch (kf) {
      case 1: transfer_h<1, S>(prolong, t, nv, dst, src, s); break;
      case 2: transfer_h<2, S>(prolong, t, nv, dst, src, s); break;
      case 3: transfer_h<3, S>(prolong, t, nv, dst, src, s); break;
      case 4: transfer_h<4, S>(prolong, t, nv, dst, src, s); break;
      case 5: transfer_h<5, S>(prolong, t, nv, dst, src, s); break;
      case 6: transfer_h<6, S>(prolong, t, nv, dst, src, s); break;
      default: throw Error(MFMG_ERR_UNSUPPORTED, "degree");
    }
    return;
  }
  switch (kf * 10 + kc) {
    case 21: transfer_launch<2, 1, 3, S>(prolong, t, false, nv, dst, src, s); break;
    case 31: transfer_launch<3, 1, 4, S>(prolong, t, false, nv, dst, src, s); break;
    case 42: transfer_launch<4, 2, 5, S>(prolong, t, false, nv, dst, src, s); break;
    case 52: transfer_launch<5, 2, 6, S>(prolong, t, false, nv, dst, src, s); break;
    case 63: transfer_launch<6, 3, 7, S>(prolong, t, false, nv, dst, src, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "polynomial transfer pair");
  }
}

void transfer(bool prolong, const CellView& f, const CellView& c, const TransferView& t, int dtype, int nv, void* dst,
              const void* src, hipStream_t s) {
  switch (dtype) {
    case MFMG_F64: transfer_s<double>(prolong, f.k, c.k, t, nv, dst, src, s); break;
    case MFMG_F32: transfer_s<float>(prolong, f.k, c.k, t, nv, dst, src, s); break;
    case MFMG_BF16: transfer_s<bf16>(prolong, f.k, c.k, t, nv, dst, src, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "dtype");
  }
}

}  // namespace

void launch_prolongate(const CellView& f, const CellView& c, const TransferView& t, int dtype, int nv, void* dst,
                       const void* src, hipStream_t s) {
  transfer(true, f, c, t, dtype, nv, dst, src, s);
}

void launch_restrict(const CellView& f, const CellView& c, const TransferView& t, int dtype, int nv, void* dst,
                     const void* src, hipStream_t s) {
  transfer(false, f, c, t, dtype, nv, dst, src, s);
}

}  // namespace mfmg
