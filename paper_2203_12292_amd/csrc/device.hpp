// Small pieces shared by the HIP translation units.
#pragma once

#include "common.hpp"
#include "fe1d.hpp"

namespace mfmg {

inline const Tables1D& tables(int k) {
  static Tables1D t[7] = {Tables1D(1), Tables1D(1), Tables1D(2), Tables1D(3),
                          Tables1D(4), Tables1D(5), Tables1D(6)};
  return t[k];
}

inline void check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) throw Error(MFMG_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
}

inline bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  MFMG_HIP(hipStreamIsCapturing(s, &st));
  return st != hipStreamCaptureStatusNone;
}

template <typename T> __device__ __forceinline__ void atomic_add(T* p, T v) { unsafeAtomicAdd(p, v); }

// bfloat16 add through a compare-and-swap on the enclosing 32-bit word
// (used only on the small levels stored in bfloat16)
__device__ __forceinline__ void atomic_add_bf16(bf16* p, float v) {
  uintptr_t addr = reinterpret_cast<uintptr_t>(p);
  unsigned int* word = reinterpret_cast<unsigned int*>(addr & ~uintptr_t(3));
  const unsigned int shift = (addr & 2) ? 16u : 0u;
  unsigned int old = *word, assumed;
  do {
    assumed = old;
    bf16 cur;
    cur.bits = static_cast<uint16_t>((assumed >> shift) & 0xffffu);
    bf16 nv = float_to_bf16(bf16_to_float(cur) + v);
    unsigned int repl = (assumed & ~(0xffffu << shift)) | (static_cast<unsigned int>(nv.bits) << shift);
    old = atomicCAS(word, assumed, repl);
  } while (old != assumed);
}

// dst += v for a storage-typed vector entry; `exclusive` entries have no
// concurrent writer and use a plain read-modify-write.
template <typename S, typename T>
__device__ __forceinline__ void add_to(S* p, T v, bool exclusive) {
  if (exclusive) {
    *p = store_as<S>(load_as<T>(*p) + v);
  } else {
    if constexpr (sizeof(S) == 2) atomic_add_bf16(reinterpret_cast<bf16*>(p), static_cast<float>(v));
    else atomic_add(p, static_cast<S>(v));
  }
}

// Barrier between phases of a wavefront on its own LDS buffers.  All lanes
// belong to one wavefront and LDS operations of a wavefront execute in order, so a compiler
// code-motion barrier with wavefront-scope fences is enough.
struct WaveSync {
  __device__ __forceinline__ void operator()() const {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
};

constexpr int VEC_THREADS = 256;

inline unsigned grid_for(int64_t n, int per_thread = 1) {
  int64_t b = (n + static_cast<int64_t>(VEC_THREADS) * per_thread - 1) / (static_cast<int64_t>(VEC_THREADS) * per_thread);
  if (b < 1) b = 1;
  if (b > 1 << 20) b = 1 << 20;
  return static_cast<unsigned>(b);
}

}  // namespace mfmg
