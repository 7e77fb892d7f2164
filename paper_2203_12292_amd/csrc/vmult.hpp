// The matrix-free operator: batch kernels, the reduction over shared DoFs and
// their launchers, instantiated once per storage type (vmult_*.hip).
//
// Cell operator (Eq. impl:mf): v = sum_e G_e^T C_e^T S_e^T Q_e S_e C_e G_e x.
// On an axis-aligned cube of side h the quadrature-point operation reduces to
// the scalar h * w_q and the cell matrix has the tensor form
// h (K (x) M (x) M + M (x) K (x) M + M (x) M (x) K) with the 1D mass M and
// stiffness K integrated exactly by the (k+1)-point Gauss rule.
#pragma once

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device.hpp"
#include "eig.hpp"
#include "kernels.hpp"
#include "mapped.hpp"
#include "slots.hpp"

namespace mfmg {

namespace {

// Per-lane constants of the operator kernel, for lane t = ta + n tb of a
// cell: entity slot and in-entity offsets (first node, first interior node,
// stride between interior nodes) of the lane's z-line (x = ta, y = tb).  Built at compile time, read once per wavefront.
struct LaneLines {
  uint8_t zs0, zs1, zsm, zo0, zom, zst;
};
template <int K>
struct LaneLineTable {
  LaneLines t[(K + 1) * (K + 1)];
};
template <int K>
constexpr LaneLineTable<K> make_lane_lines() {
  LaneLineTable<K> r{};
  for (int tb = 0; tb <= K; ++tb)
    for (int ta = 0; ta <= K; ++ta) {
      LaneLines& l = r.t[ta + (K + 1) * tb];
      l.zs0 = static_cast<uint8_t>(node_slot(ta, tb, 0, K));
      l.zs1 = static_cast<uint8_t>(node_slot(ta, tb, K, K));
      l.zsm = static_cast<uint8_t>(K > 1 ? node_slot(ta, tb, 1, K) : 26);
      l.zo0 = static_cast<uint8_t>(node_offset(ta, tb, 0, K));
      l.zom = static_cast<uint8_t>(K > 1 ? node_offset(ta, tb, 1, K) : 0);
      l.zst = static_cast<uint8_t>(K > 2 ? node_offset(ta, tb, 2, K) - node_offset(ta, tb, 1, K) : 0);
    }
  return r;
}
template <int K>
__constant__ LaneLineTable<K> kLaneLines = make_lane_lines<K>();

// Shared-DoF route of the batch kernel, or-ed into the fused kind by the
// launcher: the shared DoFs' sums are added with global atomics (into dst for
// the plain operator, else into an accumulator that finish_shared_kernel
// completes) instead of being written as partial sums
constexpr int FUSE_ATOMIC = 4;
constexpr int base_kind(int fk) { return fk & 3; }

// The fused step's operands at entry e (DoF g), loaded ahead of its output
template <typename S, typename T, int FK>
struct FinishIn {
  T b = T(0), dinv = T(0), d = T(0), x = T(0);
  __device__ __forceinline__ void load(const FusedStep& f, int64_t g, int64_t e) {
    if constexpr (base_kind(FK) != FUSE_NONE) b = load_as<T>(static_cast<const S*>(f.b)[e]);
    if constexpr (base_kind(FK) == FUSE_CHEB) {
      dinv = static_cast<const T*>(f.dinv)[g];
      if (f.c_dd != 0.0) d = load_as<T>(static_cast<const S*>(f.d)[e]);
      x = load_as<T>(static_cast<const S*>(f.x)[e]);
    }
  }
  // final value t = (A x) of entry e, and the fused step applied to it
  __device__ __forceinline__ void store(const FusedStep& f, int64_t e, T t, T* __restrict__ dst) const {
    if constexpr (base_kind(FK) == FUSE_NONE) {
      dst[e] = t;
    } else if constexpr (base_kind(FK) == FUSE_RESIDUAL) {
      static_cast<S*>(f.r)[e] = store_as<S>(b - t);
    } else {
      const T dd = f.c_dd != 0.0 ? static_cast<T>(f.c_dd) * d : T(0);
      const T dn = dd + static_cast<T>(f.c_r) * dinv * (b - t);
      static_cast<S*>(f.x)[e] = store_as<S>(x + dn);
      static_cast<S*>(f.d)[e] = store_as<S>(dn);
    }
  }
};

// Final value t = (A x) of DoF g, vector v, and the fused step applied to it
template <typename S, typename T, int FK>
__device__ __forceinline__ void finish_dof(const FusedStep& f, int64_t g, int nv, int v, T t, T* __restrict__ dst) {
  FinishIn<S, T, FK> in;
  in.load(f, g, g * nv + v);
  in.store(f, g * nv + v, t, dst);
}

// Operator evaluation on mapped cells by cell batches: n^2 lanes per cell,
// several rounds of cells per block.  The blocks are persistent: the
// batches are split into 8 contiguous ranges, one per XCD (block i runs on XCD
// i mod 8), and the blocks of an XCD take the batches of its range in turn,
// so neighbouring batches share that XCD's L2.  Per batch, the batch's DoFs
// are loaded into LDS (shared DoFs through their index list, exclusive DoFs as
// one contiguous range), the cells are evaluated group by group from LDS and
// their contributions accumulated in LDS, then the exclusive DoFs are stored
// contiguously and the shared DoFs either added with global atomics
// (FUSE_ATOMIC route, one vector: into dst, or into the level's accumulator
// when a step is fused; either clear before) or written as
// this batch's partial sums (reduced afterwards).  gridDim.x is a multiple
// of 8.
// register budget: the three gradient components and the metric terms of a
// line of points take the registers of 2 wavefronts per SIMD
template <int K, typename S, typename T, int FK, bool DET>
__global__ void __launch_bounds__(BATCH_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2)))
    vmult_mapped_kernel(const CellMeta* __restrict__ meta, const int32_t* __restrict__ bcell,
                       const int32_t* __restrict__ bsh, const int32_t* __restrict__ bex,
                       const int32_t* __restrict__ sh_idx, int64_t nb,
                       int64_t n_shared, HangTab<T, K + 1> tab, const S* __restrict__ src,
                       T* __restrict__ partial, T* __restrict__ dst, int nv, FusedStep fs,
                       const T* __restrict__ geo, const int32_t* __restrict__ ijk, int n0, MapTab<T, K + 1> mt) {
  constexpr int N = K + 1, N2 = N * N, N3 = N2 * N, CPW = cells_per_wave(N), MCAP = batch_mcap(K);
  constexpr int NZ = batch_zero_entries(K), ZB = MCAP;  // zero block behind the batch's DoFs
  constexpr int BT = BATCH_WAVES * 64, PER = (MCAP + BT - 1) / BT;
  __shared__ T in_[MCAP + NZ];
  __shared__ double out_[MCAP + NZ];  // contributions accumulate in FP64 (also for FP32 arithmetic)
  __shared__ T Hg[2 * N2];
  constexpr bool META_LDS = batch_meta_in_lds(K);
  __shared__ CellMeta metaL[META_LDS ? batch_max_cells(K) : 1];
  __shared__ T buf0[(BATCH_WAVES * CPW + 1) * N3];
  for (int i = threadIdx.x; i < NZ; i += BT) in_[ZB + i] = T(0);
  for (int i = threadIdx.x; i < 2 * N2; i += BT) Hg[i] = tab.v[i];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int lc = lane / N2;
  const int t = lane - lc * N2;
  const bool lane_used = lc < CPW;
  const int ta = t % N, tb = t / N;
  // lanes without a cell work on the block's spare buffers (results unused)
  T* B0 = buf0 + (lane_used ? wave * CPW + lc : BATCH_WAVES * CPW) * N3;
  const LaneLines ll = kLaneLines<K>.t[t];
  const int gsm = ll.zsm, go0 = ll.zo0, gom = ll.zom, gst = ll.zst;
  // the three slots of the lane's z-line (each < 27), five bits apiece: the
  // metadata fetch unpacks them each time instead of holding 64-bit offsets
  // through the batch loop
  const uint32_t slots = ll.zs0 | (ll.zs1 << 5) | (ll.zsm << 10);
  struct Pre {
    int g0, g1, gm;
    uint32_t mask;
    int lev;  // of the record read (its cell's own, also on lanes without a cell: it indexes the geometry table)
  };

  if constexpr ((FK & FUSE_ATOMIC) != 0) nv = 1;  // (one vector: the index arithmetic folds)
  const int64_t per = (nb + 7) / 8;
  const int64_t lo = (blockIdx.x % 8) * per;
  const int64_t hi = lo + per < nb ? lo + per : nb;
  // several interleaved vectors: nv blocks of one XCD (consecutive block
  // indices there) take the same batch at the same time, one vector each,
  // so that the nv values of a DoF, adjacent in memory, are read once into
  // that XCD's L2 and their partial-line writes meet there.  (Vectors one
  // after the other in one block left a whole pass of the other blocks'
  // traffic between two passes over a line, so that it was fetched and
  // written back up to nv times.)  The launch gives every XCD at least nv
  // blocks.
  const int groups = static_cast<int>(gridDim.x / 8) / nv;
  const int j = static_cast<int>(blockIdx.x / 8);
  if (j >= groups * nv) return;  // (whole block: no barrier passed yet)
  const int v = j % nv;
  const int64_t b0 = lo + j / nv;
  for (int64_t w = 0;; ++w) {
    const int64_t b = b0 + w * groups;
    if (b >= hi) break;
    const int c0 = bcell[b], c1 = bcell[b + 1];
    const int sh0 = bsh[b], nsh = bsh[b + 1] - sh0;
    const int64_t ex0 = n_shared + bex[b];
    const int m = nsh + (bex[b + 1] - bex[b]);
    // stage the batch's DoFs: all index loads of a thread, then all value
    // loads, then the LDS stores, so that the loads of a thread overlap
    {
      int32_t gi[PER];  // DoF indices (a level has fewer than 2^31 DoFs)
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int i = threadIdx.x + q * BT;
        gi[q] = i < nsh ? sh_idx[sh0 + i] : static_cast<int32_t>(ex0 + (i - nsh));
      }
      T val[PER];
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int i = threadIdx.x + q * BT;
        val[q] = i < m ? load_as<T>(src[static_cast<int64_t>(gi[q]) * nv + v]) : T(0);
      }
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int i = threadIdx.x + q * BT;
        if (i < m) {
          in_[i] = val[q];
          out_[i] = 0.0;
        }
      }
    }
    // metadata of this lane's cell, fetched one cell group ahead: the three
    // local entity starts of its z-line and the mask (the loads are
    // unconditional, from the batch's first cell for lanes without a cell, so
    // that the wait for them can be counted exactly; such lanes then point at
    // the zero block)
    if constexpr (META_LDS) {  // the batch's cell records, 16 bytes per thread
      const uint4* gsrc = reinterpret_cast<const uint4*>(meta + c0);
      uint4* ldst = reinterpret_cast<uint4*>(metaL);
      for (int i = threadIdx.x; i < (c1 - c0) * 4; i += BT) ldst[i] = gsrc[i];
    }
    auto fetch = [&](int64_t cell) {
      const bool ok = lane_used && cell < c1;
      const CellMeta* M = META_LDS ? metaL + (ok ? cell - c0 : 0) : meta + (ok ? cell : c0);
      const uint16_t* L = M->loc;
      uint32_t sl = slots;
      asm volatile("" : "+v"(sl));  // (keeps the unpacking here, not hoisted out of the loops)
      Pre p{L[sl & 31u], L[(sl >> 5) & 31u], L[sl >> 10], M->mask, 0};
      p.lev = mask_level(p.mask);
      p.g0 = ok ? p.g0 : ZB;
      p.g1 = ok ? p.g1 : ZB;
      p.gm = ok ? p.gm : ZB;
      p.mask = ok ? p.mask : 0u;
      return p;
    };
    int cw = c0 + wave * CPW;
    if constexpr (META_LDS) __syncthreads();
    Pre nx = fetch(cw + lc);
    if constexpr (!META_LDS) __syncthreads();
    // deterministic mode: every wavefront runs the same number of rounds (the
    // last one partly without cells), and the scatter below goes one cell at
    // a time in cell order
    const int rounds = DET ? (c1 - c0 + BATCH_WAVES * CPW - 1) / (BATCH_WAVES * CPW) : 0;
    for (int round = 0;; ++round, cw += BATCH_WAVES * CPW) {
      if constexpr (DET) {
        if (round >= rounds) break;
      } else {
        if (cw >= c1) break;
      }
      const Pre cur = nx;
      nx = fetch(cw + BATCH_WAVES * CPW + lc);
      const uint32_t mk = cur.mask;
      const int wave_hang = __any(mask_hanging(mk) ? 1 : 0);
      T u[N];
      u[0] = in_[cur.g0 + go0];
      u[K] = in_[cur.g1 + go0];
      if constexpr (K > 1) {
#pragma unroll
        for (int c = 1; c < K; ++c) u[c] = in_[cur.gm + gom + (c - 1) * gst];
      }
      const int64_t cell = (lane_used && cw + lc < c1) ? cw + lc : c0;
      const CellGeo<T> g = cell_geo<T>(geo, ijk, cell, cur.lev, n0);
      cell_pipeline_mapped<K, T, WaveSync>(B0, mk, wave_hang, static_cast<T>(mask_coef(mk)), mt, g, Hg, ta, tb, u);
      // scatter-add along the z-line, skipping absent entities and
      // lanes without a cell (they point at the zero block); a line through
      // the cell interior (slot 26) holds DoFs of this cell only
      const int s0 = cur.g0, s1 = cur.g1, sm = cur.gm;
      auto add = [&](int i, T v) {
        if constexpr (DET) out_[i] += static_cast<double>(v);  // the only writer at this moment
        else atomicAdd(&out_[i], static_cast<double>(v));
      };
      auto scatter = [&]() {
        if (s0 < ZB) add(s0 + go0, u[0]);
        if (s1 < ZB) add(s1 + go0, u[K]);
        if constexpr (K > 1) {
          if (sm < ZB) {
            if (gsm == 26) {
#pragma unroll
              for (int r = 1; r < K; ++r) out_[sm + gom + (r - 1) * gst] = static_cast<double>(u[r]);
            } else {
#pragma unroll
              for (int r = 1; r < K; ++r) add(sm + gom + (r - 1) * gst, u[r]);
            }
          }
        }
      };
      if constexpr (DET) {
        for (int q = 0; q < BATCH_WAVES * CPW; ++q) {  // cell c0 + round * (block's cells) + q
          if (lane_used && wave * CPW + lc == q) scatter();
          __syncthreads();
        }
      } else {
        scatter();
      }
      WaveSync{}();  // the next cell group reuses this wavefront's buffers
    }
    // write back: the shared DoFs' sums atomically into dst or the
    // accumulator (their indices read again: keeping them in registers
    // through the evaluation would spill) or as one contiguous range of
    // partial sums (the batch's part of the partial buffer); exclusive DoFs
    // in place, with the fused step
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int i = threadIdx.x + q * BT;
      if (i < nsh) {
        if constexpr ((FK & FUSE_ATOMIC) != 0)
          unsafeAtomicAdd(&(base_kind(FK) == FUSE_NONE ? dst : partial)[sh_idx[sh0 + i]], static_cast<T>(out_[i]));
        else partial[static_cast<int64_t>(sh0 + i) * nv + v] = static_cast<T>(out_[i]);
      } else if (i < m) finish_dof<S, T, FK>(fs, ex0 + (i - nsh), nv, v, static_cast<T>(out_[i]), dst);
    }
    __syncthreads();  // the next batch or vector overwrites in_ and out_
  }
}


// ---------------------------------------------------------------------------
// Operator evaluation on axis-aligned cubes.

// u <- W^T u, in place (u: nodes, then modes)
template <int N, typename T, typename Tab>
__device__ __forceinline__ void to_modes(const Tab* tab, T (&u)[N]) {
  constexpr int NE = (N + 1) / 2, NO = N / 2;
  T e[NE], o[NO];
#pragma unroll
  for (int j = 0; j < NO; ++j) {
    e[j] = u[j] + u[N - 1 - j];
    o[j] = u[j] - u[N - 1 - j];
  }
  if constexpr (N % 2) e[NO] = u[NO];
#pragma unroll
  for (int m = 0; m < NE; ++m) {
    T s = tab->we[m] * e[0];
#pragma unroll
    for (int j = 1; j < NE; ++j) s += tab->we[j * NE + m] * e[j];
    u[m] = s;
  }
#pragma unroll
  for (int m = 0; m < NO; ++m) {
    T s = tab->wo[m] * o[0];
#pragma unroll
    for (int j = 1; j < NO; ++j) s += tab->wo[j * NO + m] * o[j];
    u[NE + m] = s;
  }
}

// u <- W u, in place (u: modes, then nodes)
template <int N, typename T, typename Tab>
__device__ __forceinline__ void from_modes(const Tab* tab, T (&u)[N]) {
  constexpr int NE = (N + 1) / 2, NO = N / 2;
  T e[NE], o[NO];
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    T s = tab->we[j * NE] * u[0];
#pragma unroll
    for (int m = 1; m < NE; ++m) s += tab->we[j * NE + m] * u[m];
    e[j] = s;
  }
#pragma unroll
  for (int j = 0; j < NO; ++j) {
    T s = tab->wo[j * NO] * u[NE];
#pragma unroll
    for (int m = 1; m < NO; ++m) s += tab->wo[j * NO + m] * u[NE + m];
    o[j] = s;
  }
#pragma unroll
  for (int j = 0; j < NO; ++j) {
    u[j] = e[j] + o[j];
    u[N - 1 - j] = e[j] - o[j];
  }
  if constexpr (N % 2) u[NO] = e[NO];
}

// u <- H u (H^T u if TRANS) where `on`; H (tab) is the lower half's interpolation,
// whose row 0 is e_0
template <int N, typename T, bool TRANS, typename H>
__device__ __forceinline__ void half_line(H tab, bool on, T (&u)[N]) {
  T v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T s = i == 0 ? u[0] : T(0);
    if (TRANS || i > 0) {
#pragma unroll
      for (int j = TRANS ? 1 : 0; j < N; ++j) s += tab[TRANS ? j * N + i : i * N + j] * u[j];
    }
    v[i] = s;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) u[i] = on ? v[i] : u[i];
}

// Hanging faces and edges of a cell whose parent's corner is node (0,0,0):
// lines along d at indices p, q
// of the other axes (in axis order) are interpolated where p = 0 on a hanging
// face normal to the first, q = 0 on one normal to the second, or both on a
// hanging edge.
struct HangBits {
  bool face[3], edge[3];
  __device__ __forceinline__ explicit HangBits(uint32_t m) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      face[d] = mask_face(m, d);
      edge[d] = mask_edge(m, d);
    }
  }
  __device__ __forceinline__ bool line(int d, bool p0, bool q0) const {
    const int e = d == 0 ? 1 : 0, f = d == 2 ? 1 : 2;
    return (face[e] && p0) || (face[f] && q0) || (edge[d] && p0 && q0);
  }
};

// One block per batch (and vector).  The batch's DoFs are staged in LDS
// (shared DoFs through their index list, exclusive ones as one contiguous
// range), every cell of the batch is gathered into registers at once, worked on,
// and accumulated in LDS (FP64) in the place of the staged input; exclusive
// DoFs are stored contiguously and the shared ones either added with global
// atomics (FUSE_ATOMIC route, one vector: into dst, or into the level's
// accumulator when a step is fused; either clear before) or written as this
// batch's partial sums (reduced afterwards).
//
// A cell takes n lanes, one per plane (x, y) of its nodes: the x- and y-sweeps
// run in registers, and one exchange each way between the cell's lanes through
// LDS turns the planes for the z-sweeps (up to degree 2 one lane holds the
// whole cell, no exchange).  Against one lane per line of nodes (n^2 lanes per
// cell) that is 60 instead of 50 busy lanes per wavefront at degree 4, 6
// instead of 10 passes of the cell's values through LDS, and one set of
// addresses per plane instead of two per line.
//
// What bounds it (Q4, 67.8M FP64 DoFs, 0.42 to 0.50 ms on the cards measured,
// against 0.78 ms by lines): HBM.  Its traffic, 2.05 GB with the clearing
// (vectors, repeated reads of the shared DoFs, their index list and atomic
// adds), goes by at 4.1 to 4.9 TB/s, where a plain copy of 4 GiB reaches
// 4.7 TB/s; runs of 16 to 512 batches an XCD instead of 4 change nothing.  Q6 on 8
// FP32 vectors (3.4 ms against 6.15 ms): VALU 58 % busy, two wavefronts
// per SIMD.
//
// Cells with hanging nodes come with their axes reflected and permuted (the
// cell operator of a cube commutes with both): their parent's corner is node
// (0,0,0), so only lines at index 0 are interpolated, with one matrix, and
// hanging faces are normal to x first, then y, so that all but the cells with
// three of them interpolate one line along x and one along y per plane in
// registers and one or two along z through the exchange buffer.  The record
// holds the starts of the entities in that order; the strides between an
// entity's nodes follow from the orientation in the mask and are used by
// wavefronts with such cells only.
template <int K>
struct CellLayout {
  static constexpr int N = K + 1;
  static constexpr int LPC = K <= 2 ? 1 : N;                 // lanes per cell
  static constexpr int CPW = 64 / LPC;                       // cells per wavefront
  static constexpr int SLOTS = (64 + LPC - 1) / LPC;         // exchange slots (the spare lanes' too)
  static constexpr int RS = N | 1;                           // exchange rows of odd length
  static constexpr int MAX_THREADS = 64 * ((batch_max_cells_hard(K) + CPW - 1) / CPW);
  // DoFs a thread stages at a time: enough for one or two rounds of loads at
  // the usual batch (Q6, 8 FP32 vectors: 10 at a time 3.48 ms, 20 3.38 ms)
  static constexpr int CHUNK = K <= 4 ? 8 : K == 5 ? 10 : 20;
  // wavefronts per SIMD the registers are cut to: as many as the LDS of the
  // usual batches lets run (Q4 FP64: 4 0.446 ms, 5 0.422 ms), if they spill
  // little.  Q3: 8 leave 39 registers of a fused FP64 step in scratch (a
  // smoothing step on 270,000 cells 500 us, with 6 360 us, with 5 307 us), and
  // 5 is no worse for FP64 vectors and fused FP32 steps anywhere; only the
  // plain operator on FP32 vectors gains from 8 where most cells have hanging
  // nodes (a smoothing step of 8 vectors on 306,536 cells 2.83 ms, with 5 3.01 ms).
  // The deterministic mode: no spills.
  template <typename T, int FK, bool DET, bool SKIP>
  static constexpr int waves_per_eu() {
    if (DET) return K <= 4 ? 4 : 2;
    if (K == 3) return sizeof(T) == 4 && base_kind(FK) == FUSE_NONE ? 8 : 5;
    return K <= 2 ? 4 : K == 4 ? 5 : SKIP ? 3 : 2;
  }
  // Wavefronts past a batch's cells (the block fits the level's largest batch)
  // work on zeros, or with SKIP on nothing.  Q6: two wavefronts for batches of
  // 8 cells, where a few at the boundary have up to 16 (15,163 cells, 3 FP64
  // vectors 114 us, skipping 95 us); where all have cells the branch costs up
  // to 5 %.  Q3: one or two of 8 to 10 (270,000 cells, 3 FP64 vectors 231 us,
  // skipping 194 us).
  template <typename T, int FK>
  static constexpr bool skip(int waves) {
    return (K == 6 && waves > 1) || (K == 3 && !(sizeof(T) == 4 && base_kind(FK) == FUSE_NONE));
  }
};

// Stage a batch's DoFs in LDS, CH at a time per thread so that their loads
// overlap; threads past the end repeat the last entry instead of branching.
// Behind them the zero block.
template <int K, int CH, typename S, typename T>
__device__ __forceinline__ void stage_batch(const int32_t* __restrict__ sh, int nsh, int nex, const S* __restrict__ src,
                                            int64_t ex0, int nv, int v, int zb, T* in_) {
  const int bt = blockDim.x, tid = threadIdx.x;
  for (int i0 = tid; i0 < nsh; i0 += bt * CH) {
    int at[CH];
    int32_t gi[CH];
    T val[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) at[q] = min(i0 + q * bt, nsh - 1);
#pragma unroll
    for (int q = 0; q < CH; ++q) gi[q] = sh[at[q]];
#pragma unroll
    for (int q = 0; q < CH; ++q)
      val[q] = load_as<T>(src[static_cast<uint64_t>(static_cast<uint32_t>(gi[q])) * nv + v]);
#pragma unroll
    for (int q = 0; q < CH; ++q) in_[at[q]] = val[q];
  }
  const S* ex = src + ex0 * nv + v;
  for (int i0 = tid; i0 < nex; i0 += bt * CH) {
    int at[CH];
    T val[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) at[q] = min(i0 + q * bt, nex - 1);
#pragma unroll
    for (int q = 0; q < CH; ++q) val[q] = load_as<T>(ex[at[q] * nv]);
#pragma unroll
    for (int q = 0; q < CH; ++q) in_[nsh + at[q]] = val[q];
  }
  for (int i = tid; i < batch_zero_entries(K); i += bt) in_[zb + i] = T(0);
}

// Write back: the shared DoFs' sums atomically into dst or the accumulator,
// or as one contiguous range of partial sums (the batch's part of the
// partial buffer); exclusive DoFs in place, with the fused step (its operands
// loaded before the first of them is stored)
template <typename S, typename T, int FK>
__device__ __forceinline__ void write_batch(const int32_t* __restrict__ sh, int sh0, int nsh, int nex, int64_t ex0,
                                            int nv, int v, const double* out_, T* __restrict__ partial,
                                            T* __restrict__ dst, const FusedStep& fs) {
  const int bt = blockDim.x, tid = threadIdx.x;
  constexpr int WB = base_kind(FK) == FUSE_NONE ? 4 : 2;
  auto put_shared = [&](int i, int32_t g, double t) {
    if constexpr ((FK & FUSE_ATOMIC) != 0)
      unsafeAtomicAdd(&(base_kind(FK) == FUSE_NONE ? dst : partial)[g], static_cast<T>(t));
    else partial[static_cast<int64_t>(sh0 + i) * nv + v] = static_cast<T>(t);
  };
  auto index_of = [&](int i) { return (FK & FUSE_ATOMIC) != 0 ? sh[i] : 0; };
  int i0 = tid;
  for (; i0 + bt * (WB - 1) < nsh; i0 += bt * WB) {
    int32_t gi[WB];
    double t[WB];
#pragma unroll
    for (int q = 0; q < WB; ++q) {
      gi[q] = index_of(i0 + q * bt);
      t[q] = out_[i0 + q * bt];
    }
#pragma unroll
    for (int q = 0; q < WB; ++q) put_shared(i0 + q * bt, gi[q], t[q]);
  }
  for (; i0 < nsh; i0 += bt) put_shared(i0, index_of(i0), out_[i0]);
  const double* oex = out_ + nsh;
  for (i0 = tid; i0 + bt * (WB - 1) < nex; i0 += bt * WB) {
    FinishIn<S, T, FK> in[WB];
    double t[WB];
#pragma unroll
    for (int q = 0; q < WB; ++q) {
      in[q].load(fs, ex0 + i0 + q * bt, (ex0 + i0 + q * bt) * nv + v);
      t[q] = oex[i0 + q * bt];
    }
#pragma unroll
    for (int q = 0; q < WB; ++q) in[q].store(fs, (ex0 + i0 + q * bt) * nv + v, static_cast<T>(t[q]), dst);
  }
  for (; i0 < nex; i0 += bt) finish_dof<S, T, FK>(fs, ex0 + i0, nv, v, static_cast<T>(oex[i0]), dst);
}

// An opaque copy of the tables' address: their scalar loads stay in the phase
// that uses them (all tables at once do not fit the scalar registers)
template <typename P>
__device__ __forceinline__ const __attribute__((address_space(4))) P* here(const P* p) {
  using CP = const __attribute__((address_space(4))) P*;
  CP c = reinterpret_cast<CP>(reinterpret_cast<uintptr_t>(p));
  asm volatile("" : "+s"(c));
  return c;
}

template <int K, typename S, typename T, int FK, bool DET, bool SKIP>
__global__ void __launch_bounds__(CellLayout<K>::MAX_THREADS) __attribute__((amdgpu_waves_per_eu(CellLayout<K>::template waves_per_eu<T, FK, DET, SKIP>())))
    vmult_batch_kernel(const CellMeta* __restrict__ meta, const int32_t* __restrict__ bcell,
                      const int32_t* __restrict__ bsh, const int32_t* __restrict__ bex,
                      const int32_t* __restrict__ sh_idx, int nb, int run, int64_t n_shared, int zb, double h0,
                      const EigTab<CellReal, K + 1>* __restrict__ tab, const S* __restrict__ src, T* __restrict__ partial, T* __restrict__ dst,
                      int nv, FusedStep fs) {
  using Y = CellLayout<K>;
  using C = CellReal;
  using Tab = EigTab<C, K + 1>;
  constexpr int N = Y::N, KM = K > 1 ? K - 1 : 1, LPC = Y::LPC, RS = Y::RS, CH = Y::CHUNK;
  constexpr bool PLANE = LPC > 1;
  constexpr int NZ = PLANE ? 1 : N;  // planes per lane
  constexpr int NB = PLANE ? 9 : 27;
  extern __shared__ __align__(16) char lds_raw[];
  T* in_ = reinterpret_cast<T*>(lds_raw);
  double* out_ = reinterpret_cast<double*>(lds_raw);
  if constexpr ((FK & FUSE_ATOMIC) != 0) nv = 1;  // (one vector: the index arithmetic folds)
  // runs of `run` neighbouring batches go to the XCDs in turn (block i runs on
  // XCD i mod 8): neighbours share an L2, and batches that take longer (hanging
  // nodes come in clusters) are spread; the nv vectors of a batch are
  // consecutive blocks of one XCD, so that the nv values of a DoF, adjacent in
  // memory, meet there
  const int jb = static_cast<int>(blockIdx.x / 8), bj = jb / nv, v = jb - bj * nv;
  const int b = (bj / run * 8 + static_cast<int>(blockIdx.x % 8)) * run + bj % run;
  if (b >= nb) return;  // (whole block)
  const int c0 = bcell[b], c1 = bcell[b + 1];
  const int sh0 = bsh[b], nsh = bsh[b + 1] - sh0;
  const int64_t ex0 = n_shared + bex[b];
  const int m = nsh + (bex[b + 1] - bex[b]);
  const int bt = blockDim.x, tid = threadIdx.x;
  const int wave = tid / 64, lane = tid % 64;
  const int lc = lane / LPC, zl = lane - lc * LPC;
  const int cell = c0 + wave * Y::CPW + lc;
  const bool ok = lc < Y::CPW && cell < c1;
  // SKIP: a wavefront past the batch's cells only stages and writes back
  const bool busy = !SKIP || c0 + __builtin_amdgcn_readfirstlane(wave) * Y::CPW < c1;
  // the cell's record: its mask and the local entity starts of this lane's
  // plane (or of the cell), absent ones at the zero block
  const CellMeta* M = meta + (ok ? cell : c0);
  const uint32_t mk = ok ? M->mask : 0u;
  const bool any_hang = __any(mask_hanging(mk) ? 1 : 0) != 0;
  const int zc = zl == 0 ? 0 : zl == K ? 2 : 1;
  uint32_t rec[PLANE ? 5 : 15];
  {
    const uint32_t* r = reinterpret_cast<const uint32_t*>(M->loc) + (PLANE ? 5 * zc : 0);
#pragma unroll
    for (int i = 0; i < (PLANE ? 5 : 15); ++i) rec[i] = r[i];
  }
  // stage the batch's DoFs, CH at a time per thread so that their loads
  // overlap; threads past the end repeat the last entry instead of branching
  const int nex = m - nsh;
  for (int i0 = tid; i0 < nsh; i0 += bt * CH) {
    int at[CH];
    int32_t gi[CH];
    T val[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) at[q] = min(i0 + q * bt, nsh - 1);
#pragma unroll
    for (int q = 0; q < CH; ++q) gi[q] = sh_idx[sh0 + at[q]];
#pragma unroll
    for (int q = 0; q < CH; ++q)
      val[q] = load_as<T>(src[static_cast<uint64_t>(static_cast<uint32_t>(gi[q])) * nv + v]);
#pragma unroll
    for (int q = 0; q < CH; ++q) in_[at[q]] = val[q];
  }
  {
    const S* ex = src + ex0 * nv + v;
    for (int i0 = tid; i0 < nex; i0 += bt * CH) {
      int at[CH];
      T val[CH];
#pragma unroll
      for (int q = 0; q < CH; ++q) at[q] = min(i0 + q * bt, nex - 1);
#pragma unroll
      for (int q = 0; q < CH; ++q) val[q] = load_as<T>(ex[at[q] * nv]);
#pragma unroll
      for (int q = 0; q < CH; ++q) in_[nsh + at[q]] = val[q];
    }
  }
  for (int i = tid; i < batch_zero_entries(K); i += bt) in_[zb + i] = T(0);
  if (!ok) {  // lanes without a cell work on the zero block
#pragma unroll
    for (int i = 0; i < (PLANE ? 5 : 15); ++i) rec[i] = static_cast<uint32_t>(zb) * 0x10001u;
  }
  // strides along x and y between the nodes of an entity of this lane's plane
  // that extends along one of them (sx1, sy1) or both (sx2, sy2)
  int base[PLANE ? 9 : 1], sx1 = 1, sy1 = 1, sx2 = 1, sy2 = KM;
  if constexpr (PLANE) {
    const int zi = zc == 1 ? zl - 1 : 0;
    int sz[3] = {1, KM, KM * KM};  // along z: entities extending along z alone, z and x (or y), all
    int szy = KM;
    if (any_hang) {
      int r[3], sg[3];  // the cell's own axis and the direction of each axis
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        r[d] = op_axis(mk, d);
        sg[d] = mask_sub(mk, d) ? -1 : 1;
      }
      auto s2 = [&](int d, int e) { return sg[d] * (r[d] < r[e] ? 1 : KM); };
      auto s3 = [&](int d) { return sg[d] * (r[d] == 0 ? 1 : r[d] == 1 ? KM : KM * KM); };
      const bool in = zc == 1;
      sx1 = in ? s2(0, 2) : sg[0];
      sy1 = in ? s2(1, 2) : sg[1];
      sx2 = in ? s3(0) : s2(0, 1);
      sy2 = in ? s3(1) : s2(1, 0);
      sz[0] = sg[2];
      sz[1] = s2(2, 0);
      szy = s2(2, 1);
      sz[2] = s3(2);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const bool ex = i % 3 == 1, ey = i / 3 == 1;
      base[i] = static_cast<int>((rec[i / 2] >> (16 * (i % 2))) & 0xffffu) +
                zi * (ex && ey ? sz[2] : ex ? sz[1] : ey ? szy : sz[0]);
    }
  }
  // local start of entity i (whole cells: unpacked at each use, 15 registers
  // instead of 27)
  auto start = [&](int i) {
    if constexpr (PLANE) return base[i];
    const int w = (i / 9) * 10 + i % 9;  // rows of ten 16-bit entries
    return static_cast<int>((rec[w / 2] >> (16 * (w % 2))) & 0xffffu);
  };
  // LDS position of node (x, y) of plane z; gen: with the lane's strides
  auto cls = [](int a) { return a == 0 ? 0 : a == K ? 2 : 1; };
  auto pos = [&](auto gen, int z, int y, int x) {
    const int cx = cls(x), cy = cls(y), cz = PLANE ? 0 : cls(z);
    const int p = start(9 * cz + 3 * cy + cx);
    if constexpr (!PLANE) return p;  // (degree <= 2: an entity has one DoF)
    if constexpr (decltype(gen)::value)
      return p + (cx == 1 ? (x - 1) * (cy == 1 ? sx2 : sx1) : 0) + (cy == 1 ? (y - 1) * (cx == 1 ? sy2 : sy1) : 0);
    return p + (cx == 1 ? x - 1 : 0) + (cy == 1 ? (y - 1) * (cx == 1 ? KM : 1) : 0);
  };
  C u[NZ][N][N];  // [z][y][x]
  auto gather = [&](auto gen) {
#pragma unroll
    for (int z = 0; z < NZ; ++z)
#pragma unroll
      for (int y = 0; y < N; ++y)
#pragma unroll
        for (int x = 0; x < N; ++x) u[z][y][x] = static_cast<C>(in_[pos(gen, z, y, x)]);
  };
  __syncthreads();
  if (busy) {
    if (PLANE && any_hang) gather(std::true_type{});
    else gather(std::false_type{});
  }
  __syncthreads();  // the staged input is no longer needed

  // exchange buffer of this lane's cell, in the place of the input
  C* X = reinterpret_cast<C*>(lds_raw) + (wave * Y::SLOTS + lc) * N * RS;
  const WaveSync sync{};
  const HangBits hb(mk);
  // the interpolation of the hanging lines, axis by axis (the axes commute);
  // trans: transposed
  auto interpolate = [&](auto trans) {
    constexpr bool TR = decltype(trans)::value;
    const auto H = &here(tab)->H[0];
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
      const bool z0 = PLANE ? zl == 0 : z == 0;
      const bool all = z0 && hb.face[2];  // on a hanging face normal to z
      const bool any_all = (PLANE || z == 0) && __any(all ? 1 : 0);
      half_line<N, C, TR>(H, hb.line(0, true, z0), u[z][0]);
      if (any_all) {
#pragma unroll
        for (int y = 1; y < N; ++y) half_line<N, C, TR>(H, all, u[z][y]);
      }
      auto y_line = [&](int x, bool on) {
        C w[N];
#pragma unroll
        for (int y = 0; y < N; ++y) w[y] = u[z][y][x];
        half_line<N, C, TR>(H, on, w);
#pragma unroll
        for (int y = 0; y < N; ++y) u[z][y][x] = w[y];
      };
      y_line(0, hb.line(1, true, z0));
      if (any_all) {
#pragma unroll
        for (int x = 1; x < N; ++x) y_line(x, all);
      }
    }
    // lines along z at (0, y) and at (x, 0)
    if constexpr (PLANE) {
      const bool line0 = zl == 0 ? hb.line(2, true, true) : hb.face[0];
      if (__any(line0 ? 1 : 0)) {
        C w[N];
#pragma unroll
        for (int y = 0; y < N; ++y) X[zl * RS + y] = u[0][y][0];
        sync();
#pragma unroll
        for (int z = 0; z < N; ++z) w[z] = X[z * RS + zl];
        half_line<N, C, TR>(H, line0, w);
        sync();
#pragma unroll
        for (int z = 0; z < N; ++z) X[z * RS + zl] = w[z];
        sync();
#pragma unroll
        for (int y = 0; y < N; ++y) u[0][y][0] = X[zl * RS + y];
        sync();
      }
      const bool line1 = zl > 0 && hb.face[1];
      if (__any(line1 ? 1 : 0)) {
        C w[N];
#pragma unroll
        for (int x = 0; x < N; ++x) X[zl * RS + x] = u[0][0][x];
        sync();
#pragma unroll
        for (int z = 0; z < N; ++z) w[z] = X[z * RS + zl];
        half_line<N, C, TR>(H, line1, w);
        sync();
#pragma unroll
        for (int z = 0; z < N; ++z) X[z * RS + zl] = w[z];
        sync();
#pragma unroll
        for (int x = 0; x < N; ++x) u[0][0][x] = X[zl * RS + x];
        sync();
      }
    } else {
#pragma unroll
      for (int q = 0; q < 2 * N - 1; ++q) {
        const int x = q < N ? 0 : q - N + 1, y = q < N ? q : 0;
        C w[N];
#pragma unroll
        for (int z = 0; z < N; ++z) w[z] = u[z][y][x];
        half_line<N, C, TR>(H, hb.line(2, x == 0, y == 0), w);
#pragma unroll
        for (int z = 0; z < N; ++z) u[z][y][x] = w[z];
      }
    }
  };

  if (busy) {
    if (any_hang) interpolate(std::false_type{});
    // to modes along x and y
    const auto* tp = here(tab);
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
#pragma unroll
      for (int y = 0; y < N; ++y) to_modes<N, C>(tp, u[z][y]);
#pragma unroll
      for (int x = 0; x < N; ++x) {
        C w[N];
#pragma unroll
        for (int y = 0; y < N; ++y) w[y] = u[z][y][x];
        to_modes<N, C>(tp, w);
#pragma unroll
        for (int y = 0; y < N; ++y) u[z][y][x] = w[y];
      }
    }
    const C h = static_cast<C>(ldexp(h0, -op_level(mk)) * static_cast<double>(mask_coef(mk)));
    if constexpr (PLANE) {
      // lane z holds modes (x, y) of its plane; lane j takes the z-lines of y-mode j
#pragma unroll
      for (int x = 0; x < N; ++x) {
#pragma unroll
        for (int y = 0; y < N; ++y) X[zl * RS + y] = u[0][y][x];
        sync();
#pragma unroll
        for (int z = 0; z < N; ++z) u[0][z][x] = X[z * RS + zl];
        sync();
      }
      const auto* tz = here(tab);
      C lj = tz->lam[0];
#pragma unroll
      for (int j = 1; j < N; ++j) lj = zl == j ? tz->lam[j] : lj;
      C a[N];  // h (L_j + L_z)
#pragma unroll
      for (int z = 0; z < N; ++z) a[z] = h * tz->lam[z] + h * lj;
#pragma unroll
      for (int x = 0; x < N; ++x) {
        const C hx = h * tz->lam[x];
        C w[N];
#pragma unroll
        for (int z = 0; z < N; ++z) w[z] = u[0][z][x];
        to_modes<N, C>(tz, w);
#pragma unroll
        for (int z = 0; z < N; ++z) w[z] *= a[z] + hx;
        from_modes<N, C>(tz, w);
#pragma unroll
        for (int z = 0; z < N; ++z) u[0][z][x] = w[z];
      }
#pragma unroll
      for (int x = 0; x < N; ++x) {
#pragma unroll
        for (int z = 0; z < N; ++z) X[z * RS + zl] = u[0][z][x];
        sync();
#pragma unroll
        for (int y = 0; y < N; ++y) u[0][y][x] = X[zl * RS + y];
        sync();
      }
    } else {
      C a[N];
#pragma unroll
      for (int z = 0; z < N; ++z) a[z] = h * tp->lam[z];
#pragma unroll
      for (int y = 0; y < N; ++y)
#pragma unroll
        for (int x = 0; x < N; ++x) {
          C w[N];
#pragma unroll
          for (int z = 0; z < N; ++z) w[z] = u[z][y][x];
          to_modes<N, C>(tp, w);
#pragma unroll
          for (int z = 0; z < N; ++z) w[z] *= a[z] + h * (tp->lam[x] + tp->lam[y]);
          from_modes<N, C>(tp, w);
#pragma unroll
          for (int z = 0; z < N; ++z) u[z][y][x] = w[z];
        }
    }
    tp = here(tab);
    // back to nodes along y and x
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
#pragma unroll
      for (int x = 0; x < N; ++x) {
        C w[N];
#pragma unroll
        for (int y = 0; y < N; ++y) w[y] = u[z][y][x];
        from_modes<N, C>(tp, w);
#pragma unroll
        for (int y = 0; y < N; ++y) u[z][y][x] = w[y];
      }
#pragma unroll
      for (int y = 0; y < N; ++y) from_modes<N, C>(tp, u[z][y]);
    }
    if (any_hang) interpolate(std::true_type{});
  }

  if constexpr (!PLANE) {
#pragma unroll
    for (int i = 0; i < 15; ++i) asm volatile("" : "+v"(rec[i]));  // (unpack again, instead of keeping 27 values)
  }
  // accumulate in LDS, absent entities skipped
  __syncthreads();
  for (int i = tid; i < (m + 1) / 2; i += bt) reinterpret_cast<double2*>(out_)[i] = double2{0.0, 0.0};
  __syncthreads();
  auto scatter_with = [&](auto gen) {
    if constexpr (DET) {
      // plain adds of one phase's cells, which share no DoF; the loads of two
      // rows of nodes (or of a plane of a whole cell) go out together, absent
      // entities add to the entry behind the batch's DoFs instead of branching
#pragma unroll
      for (int i = 0; i < (PLANE ? 9 : 1); ++i) asm volatile("" : "+v"(base[i]));  // (addresses made in each phase)
#pragma unroll
      for (int z = 0; z < NZ; ++z) {
        constexpr int ROWS = PLANE ? 2 : N;
#pragma unroll
        for (int y0 = 0; y0 < N; y0 += ROWS) {
          const int n = (N - y0 < ROWS ? N - y0 : ROWS) * N;
          int at[ROWS * N];
          double old[ROWS * N];
#pragma unroll
          for (int i = 0; i < n; ++i) at[i] = min(pos(gen, z, y0 + i / N, i % N), zb);
#pragma unroll
          for (int i = 0; i < n; ++i) old[i] = out_[at[i]];
#pragma unroll
          for (int i = 0; i < n; ++i) out_[at[i]] = old[i] + static_cast<double>(u[z][y0 + i / N][i % N]);
        }
      }
      return;
    }
#pragma unroll
    for (int e = 0; e < NB; ++e) {
      if (start(e) >= zb) continue;
#pragma unroll
      for (int z = 0; z < NZ; ++z)
#pragma unroll
        for (int y = 0; y < N; ++y)
#pragma unroll
          for (int x = 0; x < N; ++x) {
            if (9 * (PLANE ? 0 : cls(z)) + 3 * cls(y) + cls(x) != e) continue;
            atomicAdd(out_ + pos(gen, z, y, x), static_cast<double>(u[z][y][x]));
          }
    }
  };
  auto scatter = [&]() {
    if (PLANE && any_hang) scatter_with(std::true_type{});
    else scatter_with(std::false_type{});
  };
  if constexpr (DET) {  // phase by phase: every DoF's sum in one order
    const int phases = meta[c0].loc[META_PHASES], mine = M->loc[META_PHASE];
    for (int p = 0; p < phases; ++p) {
      if (ok && mine == p) scatter();
      __syncthreads();
    }
  } else {
    if (busy) scatter();
    __syncthreads();
  }
  // write back: the shared DoFs' sums atomically into dst or the accumulator,
  // or as one contiguous range of partial sums (the batch's part of the
  // partial buffer); exclusive DoFs in place, with the fused step (its operands
  // loaded before the first of them is stored)
  constexpr int WB = base_kind(FK) == FUSE_NONE ? 8 : 4;
  auto put_shared = [&](int i, int32_t g, double t) {
    if constexpr ((FK & FUSE_ATOMIC) != 0)
      unsafeAtomicAdd(&(base_kind(FK) == FUSE_NONE ? dst : partial)[g], static_cast<T>(t));
    else partial[static_cast<int64_t>(sh0 + i) * nv + v] = static_cast<T>(t);
  };
  auto index_of = [&](int i) { return (FK & FUSE_ATOMIC) != 0 ? sh_idx[sh0 + i] : 0; };
  int i0 = tid;
  for (; i0 + bt * (WB - 1) < nsh; i0 += bt * WB) {
    int32_t gi[WB];
    double t[WB];
#pragma unroll
    for (int q = 0; q < WB; ++q) {
      gi[q] = index_of(i0 + q * bt);
      t[q] = out_[i0 + q * bt];
    }
#pragma unroll
    for (int q = 0; q < WB; ++q) put_shared(i0 + q * bt, gi[q], t[q]);
  }
  for (; i0 < nsh; i0 += bt) put_shared(i0, index_of(i0), out_[i0]);
  const double* oex = out_ + nsh;
  for (i0 = tid; i0 + bt * (WB - 1) < nex; i0 += bt * WB) {
    FinishIn<S, T, FK> in[WB];
    double t[WB];
#pragma unroll
    for (int q = 0; q < WB; ++q) {
      in[q].load(fs, ex0 + i0 + q * bt, (ex0 + i0 + q * bt) * nv + v);
      t[q] = oex[i0 + q * bt];
    }
#pragma unroll
    for (int q = 0; q < WB; ++q) in[q].store(fs, (ex0 + i0 + q * bt) * nv + v, static_cast<T>(t[q]), dst);
  }
  for (; i0 < nex; i0 += bt) finish_dof<S, T, FK>(fs, ex0 + i0, nv, v, static_cast<T>(oex[i0]), dst);
}

// The same with one lane per line of nodes and a wavefront per cell, for levels
// of degree 5 and 6 with few batches, where a batch's latency is all that
// counts: a lane of the plane kernel works through 36 or 49 values, and a batch
// is staged by the 64 or 128 threads that its 8 to 16 cells take; a lane here
// works through 6 or 7 values, turned between the axes through LDS (4 times,
// with hanging nodes 8 times).  Registers for two blocks of 16 wavefronts per
// CU.  One FP64 vector, lines against planes (and one lane per line in the
// Gauss-Lobatto basis): Q6, 104 batches 13.3 us, 21.1 us (13.8 us), 589 batches
// 19.2, 22.5 (22.5); Q5, about 140 batches 13.5, 15.1 (15.7).
template <int K>
struct LineLayout {
  static constexpr int N = K + 1, RS = N | 1, CELL = N * N * RS;  // exchange rows of odd length
  static constexpr int MAX_CELLS = batch_max_cells_hard(K), MAX_THREADS = 64 * MAX_CELLS;
  // batches x vectors up to which lines are the better ones: Q5 480 (one FP32
  // vector) 18.9 us by lines, 20.2 us by planes, 592 (8 vectors) 30.6, 25.7; Q6
  // 589 see above, 704 (8 FP32 vectors) 26.7, 24.2
  static constexpr int MOST_BLOCKS = K == 5 ? 512 : 640;
};

template <int K, typename S, typename T, int FK, bool DET>
__global__ void __launch_bounds__(LineLayout<K>::MAX_THREADS) __attribute__((amdgpu_waves_per_eu(8)))
    vmult_line_kernel(const CellMeta* __restrict__ meta, const int32_t* __restrict__ bcell,
                      const int32_t* __restrict__ bsh, const int32_t* __restrict__ bex,
                      const int32_t* __restrict__ sh_idx, int nb, int run, int64_t n_shared, int zb, double h0,
                      const EigTab<CellReal, K + 1>* __restrict__ tab, const S* __restrict__ src, T* __restrict__ partial, T* __restrict__ dst,
                      int nv, FusedStep fs) {
  using Y = LineLayout<K>;
  using C = CellReal;
  constexpr int N = Y::N, KM = K - 1, RS = Y::RS;
  extern __shared__ __align__(16) char lds_raw[];
  T* in_ = reinterpret_cast<T*>(lds_raw);
  double* out_ = reinterpret_cast<double*>(lds_raw);
  if constexpr ((FK & FUSE_ATOMIC) != 0) nv = 1;
  const int jb = static_cast<int>(blockIdx.x / 8), bj = jb / nv, v = jb - bj * nv;  // (as in the plane kernel)
  const int b = (bj / run * 8 + static_cast<int>(blockIdx.x % 8)) * run + bj % run;
  if (b >= nb) return;  // (whole block)
  const int c0 = bcell[b], c1 = bcell[b + 1];
  const int sh0 = bsh[b], nsh = bsh[b + 1] - sh0, nex = bex[b + 1] - bex[b];
  const int64_t ex0 = n_shared + bex[b];
  const int bt = blockDim.x, tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const bool busy = c0 + wave < c1;  // (one cell per wavefront)
  const CellMeta* M = meta + (busy ? c0 + wave : c0);
  const uint32_t mk = M->mask;
  const bool hang = mask_hanging(mk);
  // lane (a, b): z-line x = a, y = b; y-line x = a, z = b; x-line y = a, z = b
  // (the spare lanes repeat the last one)
  const bool on = lane < N * N;
  const int t = on ? lane : N * N - 1, la = t % N, lb = t / N;
  const C lab = tab->lam[la] + tab->lam[lb];
  // positions of the z-line's nodes: first, inner ones (start and stride), last
  int p0, p1, pm, sz;
  {
    const int cx = la == 0 ? 0 : la == K ? 2 : 1, cy = lb == 0 ? 0 : lb == K ? 2 : 1;
    const bool ex = cx == 1, ey = cy == 1;
    int r[3] = {0, 1, 2}, sg[3] = {1, 1, 1};
    if (hang) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        r[d] = op_axis(mk, d);
        sg[d] = mask_sub(mk, d) ? -1 : 1;
      }
    }
    auto over = [&](bool e, int a, int d) { return e && r[a] < r[d] ? KM : 1; };  // axis a runs faster than d
    const int sx = sg[0] * over(ey, 1, 0), sy = sg[1] * over(ex, 0, 1);
    const int oe = (ex ? (la - 1) * sx : 0) + (ey ? (lb - 1) * sy : 0);
    const int om = (ex ? (la - 1) * sx * over(true, 2, 0) : 0) + (ey ? (lb - 1) * sy * over(true, 2, 1) : 0);
    const uint16_t* L = M->loc + 3 * cy + cx;
    p0 = L[0] + oe;
    pm = L[10] + om;
    p1 = L[20] + oe;
    sz = sg[2] * over(ex, 0, 2) * over(ey, 1, 2);
  }
  auto pos = [&](int z) { return z == 0 ? p0 : z == K ? p1 : pm + (z - 1) * sz; };
  stage_batch<K, 8>(sh_idx + sh0, nsh, nex, src, ex0, nv, v, zb, in_);
  __syncthreads();
  C u[N];
  if (busy) {
#pragma unroll
    for (int z = 0; z < N; ++z) u[z] = static_cast<C>(in_[pos(z)]);
  }
  __syncthreads();  // the staged input is no longer needed
  if (busy) {
    C* X = out_ + wave * Y::CELL;
    const WaveSync sync{};
    const auto* tp = here(tab);
    using X_ = std::integral_constant<int, 0>;
    using Y_ = std::integral_constant<int, 1>;
    using Z_ = std::integral_constant<int, 2>;
    auto at = [&](auto d, int r) {
      return decltype(d)::value == 0 ? (lb * N + la) * RS + r
             : decltype(d)::value == 1 ? (lb * N + r) * RS + la : (r * N + lb) * RS + la;
    };
    auto turn = [&](auto from, auto to) {
#pragma unroll
      for (int r = 0; r < N; ++r) X[at(from, r)] = u[r];
      sync();
#pragma unroll
      for (int r = 0; r < N; ++r) u[r] = X[at(to, r)];
      sync();
    };
    const C h = static_cast<C>(ldexp(h0, -op_level(mk)) * static_cast<double>(mask_coef(mk)));
    auto scale = [&]() {
#pragma unroll
      for (int r = 0; r < N; ++r) u[r] *= h * (tp->lam[r] + lab);
    };
    if (!hang) {
      to_modes<N, C>(tp, u);
      turn(Z_{}, Y_{});
      to_modes<N, C>(tp, u);
      turn(Y_{}, X_{});
      to_modes<N, C>(tp, u);
      scale();
      from_modes<N, C>(tp, u);
      turn(X_{}, Y_{});
      from_modes<N, C>(tp, u);
      turn(Y_{}, Z_{});
      from_modes<N, C>(tp, u);
    } else {
      const HangBits hb(mk);
      auto half = [&](auto d, auto trans) {  // (half_line, its table loaded row by row)
        constexpr bool TR = decltype(trans)::value;
        const bool set = hb.line(decltype(d)::value, la == 0, lb == 0);
        C w[N];
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = i == 0 ? u[0] : C(0);
#pragma unroll
        for (int i = 1; i < N; ++i) {
          const auto* H = &here(tab)->H[i * N];
#pragma unroll
          for (int j = 0; j < N; ++j) {
            if constexpr (TR) w[j] += H[j] * u[i];
            else w[i] += H[j] * u[j];
          }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) u[i] = set ? w[i] : u[i];
      };
      half(Z_{}, std::false_type{});
      turn(Z_{}, Y_{});
      half(Y_{}, std::false_type{});
      turn(Y_{}, X_{});
      half(X_{}, std::false_type{});
      to_modes<N, C>(tp, u);
      turn(X_{}, Y_{});
      to_modes<N, C>(tp, u);
      turn(Y_{}, Z_{});
      to_modes<N, C>(tp, u);
      scale();
      from_modes<N, C>(tp, u);
      turn(Z_{}, Y_{});
      from_modes<N, C>(tp, u);
      turn(Y_{}, X_{});
      from_modes<N, C>(tp, u);
      half(X_{}, std::true_type{});
      turn(X_{}, Y_{});
      half(Y_{}, std::true_type{});
      turn(Y_{}, Z_{});
      half(Z_{}, std::true_type{});
    }
  }
  __syncthreads();
  for (int i = tid; i < (nsh + nex + 1) / 2; i += bt) reinterpret_cast<double2*>(out_)[i] = double2{0.0, 0.0};
  __syncthreads();
  if constexpr (DET) {  // phase by phase (as in the plane kernel)
    const int phases = meta[c0].loc[META_PHASES], mine = M->loc[META_PHASE];
    for (int p = 0; p < phases; ++p) {
      if (busy && on && mine == p) {
        double old[N];
#pragma unroll
        for (int z = 0; z < N; ++z) old[z] = out_[min(pos(z), zb)];
#pragma unroll
        for (int z = 0; z < N; ++z) out_[min(pos(z), zb)] = old[z] + static_cast<double>(u[z]);
      }
      __syncthreads();
    }
  } else {
    if (busy && on) {
      if (p0 < zb) atomicAdd(out_ + p0, static_cast<double>(u[0]));
      if (p1 < zb) atomicAdd(out_ + p1, static_cast<double>(u[K]));
      if (pm < zb) {
#pragma unroll
        for (int z = 1; z < K; ++z) atomicAdd(out_ + pos(z), static_cast<double>(u[z]));
      }
    }
    __syncthreads();
  }
  write_batch<S, T, FK>(sh_idx + sh0, sh0, nsh, nex, ex0, nv, v, out_, partial, dst, fs);
}

template <typename T>
__global__ void clear_shared_kernel(int64_t n, T* __restrict__ dst) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    dst[i] = T(0);
}

// the fused step on the shared DoFs of one vector, from their sums (A x)_s
// accumulated atomically in acc, which is left cleared for the next operator
// application (a clearing launch of its own costs a small level as much as the
// operator: Q2 solve of 2,808 cells 3.59 -> 3.32 ms without it)
template <typename S, typename T, int FK>
__global__ void finish_shared_kernel(int64_t n_shared, T* __restrict__ acc, T* __restrict__ dst, FusedStep fs) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n_shared;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const T t = acc[i];
    acc[i] = T(0);
    finish_dof<S, T, FK>(fs, i, 1, 0, t, dst);
  }
}

// (A x)_s = sum of the partial sums of shared DoF s, in the fixed order of its
// batches (red_idx holds their positions in the batch-ordered partial
// buffer), then the fused step
template <typename S, typename T, int FK>
__global__ void reduce_shared_kernel(int64_t n_shared, int nv, const int32_t* __restrict__ red_off,
                                     const int32_t* __restrict__ red_idx, const T* __restrict__ partial,
                                     T* __restrict__ dst, FusedStep fs) {
  const int64_t n = n_shared * nv;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t sd = i / nv;
    const int v = static_cast<int>(i - sd * nv);
    T acc = T(0);
    for (int j = red_off[sd]; j < red_off[sd + 1]; ++j)
      acc += partial[static_cast<int64_t>(red_idx[j]) * nv + v];
    finish_dof<S, T, FK>(fs, sd, nv, v, acc, dst);
  }
}

// The same for NV interleaved vectors, one thread per shared DoF: the NV
// values of a partial sum are one aligned vector load, its index is read once
// for all of them, and every value is summed in the same order as above
template <typename S, typename T, int FK, int NV>
__global__ void reduce_shared_vec_kernel(int64_t n_shared, const int32_t* __restrict__ red_off,
                                         const int32_t* __restrict__ red_idx, const T* __restrict__ partial,
                                         T* __restrict__ dst, FusedStep fs) {
  typedef T VecT __attribute__((ext_vector_type(NV)));
  for (int64_t sd = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; sd < n_shared;
       sd += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    VecT acc = T(0);
    for (int j = red_off[sd]; j < red_off[sd + 1]; ++j)
      acc += *reinterpret_cast<const VecT*>(partial + static_cast<int64_t>(red_idx[j]) * NV);
#pragma unroll
    for (int v = 0; v < NV; ++v) finish_dof<S, T, FK>(fs, sd, NV, v, acc[v], dst);
  }
}

template <int K, typename S, int FK, int GEO, bool DET>
void vmult_run(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  using T = typename Acc<S>::type;
  constexpr int N = K + 1;
  if (c.n_cells == 0) return;
  constexpr bool atom = (FK & FUSE_ATOMIC) != 0;
  constexpr bool into_dst = base_kind(FK) == FUSE_NONE;
  // shared sums: added atomically into dst, cleared first (the shared DoFs are
  // the first n_shared), or for a fused step into the level's accumulator,
  // which every finish leaves cleared; else partial sums
  T* sums = static_cast<T*>(atom && !into_dst ? c.acc : c.partial);
  // a call that throws between the batches and the finish (check_launch also
  // reports errors that the caller's own HIP calls left behind) leaves the
  // accumulator marked; the next fused step clears it first
  const bool unclean = atom && !into_dst && *c.acc_unclean;
  if (((atom && into_dst) || unclean) && c.n_shared > 0) {
    clear_shared_kernel<T><<<grid_for(c.n_shared), VEC_THREADS, 0, s>>>(c.n_shared, into_dst ? static_cast<T*>(dst) : sums);
    check_launch();
  }
  if constexpr (atom && !into_dst) *c.acc_unclean = true;
  const int64_t nb = c.n_batches;
  if constexpr (GEO != 0) {
    static const HangTab<T, N> tab = make_hangtab<T, N>();
    static const MapTab<T, N> mt = make_maptab<T, N>();
    const T* geo = static_cast<const T*>(sizeof(T) == 8 ? c.geo64 : c.geo32);
    // persistent blocks: as many as are resident on the device at once (a
    // multiple of 8, one share per XCD), at most one per batch
    static const int64_t resident = [] {
      int dev = 0, cus = 0, per_cu = 0;
      if (hipGetDevice(&dev) != hipSuccess ||
          hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
          hipOccupancyMaxActiveBlocksPerMultiprocessor(
              &per_cu, reinterpret_cast<const void*>(&vmult_mapped_kernel<K, S, T, FK, DET>), BATCH_WAVES * 64, 0) !=
              hipSuccess) {
        (void)hipGetLastError();
        return int64_t(0);
      }
      return static_cast<int64_t>(cus) * per_cu * BATCH_GRID_FACTOR;
    }();
    int64_t blocks = 8 * ((nb * nv + 7) / 8);  // (several vectors: one block per (batch, vector) at most)
    if (resident >= 8 && blocks > resident / 8 * 8) blocks = resident / 8 * 8;
    if (blocks < 8 * nv) blocks = 8 * nv;  // every XCD runs all vectors of a batch together
    vmult_mapped_kernel<K, S, T, FK, DET><<<static_cast<unsigned>(blocks), BATCH_WAVES * 64, 0, s>>>(
        c.meta, c.batch_cell, c.batch_sh, c.batch_ex, c.sh_idx, nb, c.n_shared, tab, static_cast<const S*>(src),
        sums, static_cast<T*>(dst), nv, f, geo, c.ijk, c.geo_n0, mt);
  } else {
    using Y = CellLayout<K>;
    using C = CellReal;
    const EigTab<C, N>* tab = static_cast<const EigTab<C, N>*>(c.eig);
    const int waves = (c.max_batch_cells + Y::CPW - 1) / Y::CPW;
    MFMG_REQUIRE(waves * 64 <= Y::MAX_THREADS, MFMG_ERR_INVALID_ARG, "batch exceeds the operator's block");
    // LDS: the batch's DoFs as FP64 sums, cleared in pairs (as T the input and
    // the zero block behind it), or the exchange buffers
    size_t lds = std::max(static_cast<size_t>(c.max_batch_dofs + 1) * 8,
                          static_cast<size_t>(c.max_batch_dofs + batch_zero_entries(K)) * sizeof(T));
    if (Y::LPC > 1) lds = std::max(lds, static_cast<size_t>(waves) * Y::SLOTS * N * Y::RS * sizeof(C));
    // (runs of 4 batches: one range of batches per XCD costs the Q3 smoothing
    // step of 8 vectors 5 %, the others nothing)
    const int64_t run = std::max<int64_t>(1, std::min<int64_t>(4, nb / 64));
    const int64_t blocks = 8 * run * ((nb + 8 * run - 1) / (8 * run)) * nv;
    auto launch = [&](auto kernel, int wavefronts, size_t bytes) {
      kernel<<<static_cast<unsigned>(blocks), 64 * wavefronts, bytes, s>>>(
          c.meta, c.batch_cell, c.batch_sh, c.batch_ex, c.sh_idx, static_cast<int>(nb), static_cast<int>(run), c.n_shared,
          c.max_batch_dofs, c.h0, tab, static_cast<const S*>(src), sums, static_cast<T*>(dst), nv, f);
    };
    // levels with few batches take a line per lane (see vmult_line_kernel)
    bool lines = false;
    if constexpr (K >= 5) lines = nb * nv <= LineLayout<K>::MOST_BLOCKS;
    if constexpr (K >= 5) {
      using Z = LineLayout<K>;
      MFMG_REQUIRE(c.max_batch_cells <= Z::MAX_CELLS, MFMG_ERR_INVALID_ARG, "batch exceeds the operator's block");
      if (lines)
        launch(&vmult_line_kernel<K, S, T, FK, DET>, c.max_batch_cells,
               std::max(lds, static_cast<size_t>(c.max_batch_cells) * Z::CELL * sizeof(C)));
    }
    if (!lines) {  // (degree 6: instantiated with and without SKIP)
      if (K == 6 && waves > 1) launch(&vmult_batch_kernel<K, S, T, FK, DET, Y::template skip<T, FK>(2)>, waves, lds);
      else launch(&vmult_batch_kernel<K, S, T, FK, DET, Y::template skip<T, FK>(1)>, waves, lds);
    }
  }
  check_launch();
  if constexpr (atom && !into_dst) {
    if (c.n_shared > 0) {
      finish_shared_kernel<S, T, base_kind(FK)><<<grid_for(c.n_shared), VEC_THREADS, 0, s>>>(
          c.n_shared, sums, static_cast<T*>(dst), f);
      check_launch();
    }
    // (a clearing that was only captured has not run yet: it stays marked)
    *c.acc_unclean = unclean && capturing(s);
  }
  if constexpr (!atom) {
    if (c.n_shared > 0) {
      const T* part = static_cast<const T*>(c.partial);  // (256-byte aligned: vector loads of NV values)
      T* out = static_cast<T*>(dst);
      const unsigned g = grid_for(c.n_shared);
      if (nv == 8) {
        reduce_shared_vec_kernel<S, T, FK, 8><<<g, VEC_THREADS, 0, s>>>(c.n_shared, c.red_off, c.red_idx, part, out, f);
      } else if (nv == 4) {
        reduce_shared_vec_kernel<S, T, FK, 4><<<g, VEC_THREADS, 0, s>>>(c.n_shared, c.red_off, c.red_idx, part, out, f);
      } else if (nv == 2) {
        reduce_shared_vec_kernel<S, T, FK, 2><<<g, VEC_THREADS, 0, s>>>(c.n_shared, c.red_off, c.red_idx, part, out, f);
      } else {
        reduce_shared_kernel<S, T, FK><<<grid_for(c.n_shared * nv), VEC_THREADS, 0, s>>>(
            c.n_shared, nv, c.red_off, c.red_idx, part, out, f);
      }
      check_launch();
    }
  }
}

// One vector: the shared DoFs' sums go out with global atomics, which run
// alongside the evaluation and replace the partial sums' write and the
// reduction's gathers.  Interleaved vectors keep the partial sums (their
// atomics would meet in one line, which measured slower), and so does the
// deterministic mode (their fixed order).
template <int K, typename S, int FK, int GEO, bool DET>
void vmult_kgd(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  if constexpr (!DET) {
    if (nv == 1) {
      vmult_run<K, S, FK | FUSE_ATOMIC, GEO, false>(c, nv, dst, src, f, s);
      return;
    }
  }
  vmult_run<K, S, FK, GEO, DET>(c, nv, dst, src, f, s);
}

template <int K, typename S, int FK, int GEO>
void vmult_kg(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  if (c.deterministic) vmult_kgd<K, S, FK, GEO, true>(c, nv, dst, src, f, s);
  else vmult_kgd<K, S, FK, GEO, false>(c, nv, dst, src, f, s);
}

template <int K, typename S, int FK>
void vmult_k(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  if (c.geo64) vmult_kg<K, S, FK, 1>(c, nv, dst, src, f, s);
  else vmult_kg<K, S, FK, 0>(c, nv, dst, src, f, s);
}

template <int K, typename S>
void vmult_kf(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  switch (f.kind) {
    case FUSE_NONE: vmult_k<K, S, FUSE_NONE>(c, nv, dst, src, f, s); break;
    case FUSE_CHEB: vmult_k<K, S, FUSE_CHEB>(c, nv, dst, src, f, s); break;
    case FUSE_RESIDUAL: vmult_k<K, S, FUSE_RESIDUAL>(c, nv, dst, src, f, s); break;
    default: throw Error(MFMG_ERR_INVALID_ARG, "fused step");
  }
}

template <typename S>
void vmult_s(const CellView& c, int nv, void* dst, const void* src, const FusedStep& f, hipStream_t s) {
  switch (c.k) {
    case 1: vmult_kf<1, S>(c, nv, dst, src, f, s); break;
    case 2: vmult_kf<2, S>(c, nv, dst, src, f, s); break;
    case 3: vmult_kf<3, S>(c, nv, dst, src, f, s); break;
    case 4: vmult_kf<4, S>(c, nv, dst, src, f, s); break;
    case 5: vmult_kf<5, S>(c, nv, dst, src, f, s); break;
    case 6: vmult_kf<6, S>(c, nv, dst, src, f, s); break;
    default: throw Error(MFMG_ERR_UNSUPPORTED, "degree");
  }
}


}  // namespace
}  // namespace mfmg
