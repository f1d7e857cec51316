// Device-side helpers shared by the gfx950 kernels of the FP-Sketch verifier: vector types,
// half-precision element access, loads with a zero buffer in place of branches, and the
// launcher that lets dispatch packets time-stamp events.
#pragma once

#include "fpsk_internal.h"

#include <hip/hip_ext.h>

namespace fpsk {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// ----------------------------------------------------------------------------------------
// Element helpers.  DT: 0 = FP16, 1 = BF16.

template <int DT>
__device__ __forceinline__ float lo_half(uint32_t w) {
  if constexpr (DT == 1) {
    return __uint_as_float(w << 16);
  } else {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w & 0xffffu)));
  }
}

template <int DT>
__device__ __forceinline__ float hi_half(uint32_t w) {
  if constexpr (DT == 1) {
    return __uint_as_float(w & 0xffff0000u);
  } else {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w >> 16)));
  }
}

template <int DT>
__device__ __forceinline__ float half_bits_to_float(uint32_t h) {
  return lo_half<DT>(h);
}

// Running max of |x| over both halves of a word, on the bit patterns (|x| is monotone in the
// low 15 bits for non-negative patterns).
__device__ __forceinline__ uint32_t absmax2(uint32_t mx, uint32_t w) {
  const u16x2 a = __builtin_bit_cast(u16x2, mx);
  const u16x2 b = __builtin_bit_cast(u16x2, w & 0x7fff7fffu);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, b));
}

// Branch-free 16-byte loads for the vector path: an invalid row or lane reads the zero buffer
// instead of branching, so a group of loads issues back to back.
__device__ __forceinline__ u32x4 load8h_sel(const uint16_t* p, bool ok, const void* zero) {
  const u32x4* q = ok ? reinterpret_cast<const u32x4*>(p) : static_cast<const u32x4*>(zero);
  return __builtin_nontemporal_load(q);
}

__device__ __forceinline__ void load8f_sel(const float* p, bool ok, const void* zero, f32x4& v0,
                                           f32x4& v1) {
  const f32x4* q = ok ? reinterpret_cast<const f32x4*>(p) : static_cast<const f32x4*>(zero);
  v0 = __builtin_nontemporal_load(q);
  v1 = __builtin_nontemporal_load(q + 1);
}

// Ragged rows: a row length that is no multiple of 8 or a base off a 16-byte boundary.  gfx950
// takes 16-byte global loads at any element alignment, so ragged rows keep the vector path's
// loads (8 elements a lane, all issued back to back) instead of 8 element loads under branches:
// 2047 x 8191 x 8191 BF16 at m = 64, stream kernel 152.5 -> 50.9 us (3947 GB/s of A, B and C; the
// aligned 2048 x 8192 x 8192 takes 43 us); 1531 x 4096 x 32003 FP16 at m = 279, call 493 -> 231
// us.  Three things keep them right:
//   - `last` is the matrix's element count less 8.  A lane whose 8 elements would pass the end of
//     the matrix (in its last row or rows) loads the final 8 instead and rag_shift moves them
//     down.  (A matrix of fewer than 8 elements comes in a copy padded to 8, with last = 0.)
//   - elements past the row's end are the next row's and are masked off (rag_keep).
//   - rag_near says, uniformly for a wave, whether any lane of a row needs the shift.
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));

__device__ __forceinline__ int64_t rag_last(int64_t rows, int64_t n) {
  const int64_t l = rows * n - 8;
  return l > 0 ? l : 0;
}

// Element offset, from the tile's first element `base` in the matrix, that a lane at offset
// `off` loads from.
__device__ __forceinline__ int rag_off(int64_t base, int off, int64_t last) {
  const int64_t rem = last - base;
  const int lim = rem < -(1 << 30) ? -(1 << 30) : (rem > (1 << 30) ? (1 << 30) : static_cast<int>(rem));
  return off < lim ? off : lim;
}

__device__ __forceinline__ bool rag_near(int64_t base, int max_off, int64_t last) {
  return base + max_off > last;
}

__device__ __forceinline__ u32x4 load8h_rag(const uint16_t* X, int64_t base, int off,
                                            int64_t last, bool ok, const void* zero) {
  const uint16_t* p = X + base + rag_off(base, off, last);
  const u32x4_a2* q = ok ? reinterpret_cast<const u32x4_a2*>(p)
                                      : static_cast<const u32x4_a2*>(zero);
  return __builtin_nontemporal_load(q);
}

__device__ __forceinline__ void load8f_rag(const float* X, int64_t base, int off, int64_t last,
                                           bool ok, const void* zero, f32x4& v0, f32x4& v1) {
  const float* p = X + base + rag_off(base, off, last);
  const f32x4_a4* q = ok ? reinterpret_cast<const f32x4_a4*>(p)
                                      : static_cast<const f32x4_a4*>(zero);
  v0 = __builtin_nontemporal_load(q);
  v1 = __builtin_nontemporal_load(q + 1);
}

// The rows rag_near picks: the final 8 elements of the matrix moved down to the lane's own
// (zeros beyond the end).
__device__ __forceinline__ void rag_shift(u32x4& v, int64_t base, int off, int64_t last, bool ok) {
  const int s = ok ? off - rag_off(base, off, last) : 0;    // 0 .. 7 elements
  if (s & 1) {
    v = u32x4{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16),
              (v[2] >> 16) | (v[3] << 16), v[3] >> 16};
  }
  if (s & 2) v = u32x4{v[1], v[2], v[3], 0u};
  if (s & 4) v = u32x4{v[2], v[3], 0u, 0u};
}

__device__ __forceinline__ void rag_shift(f32x4& v0, f32x4& v1, int64_t base, int off,
                                          int64_t last, bool ok) {
  const int s = ok ? off - rag_off(base, off, last) : 0;    // 0 .. 7 elements
  if (s & 1) {
    v0 = f32x4{v0[1], v0[2], v0[3], v1[0]};
    v1 = f32x4{v1[1], v1[2], v1[3], 0.0f};
  }
  if (s & 2) {
    v0 = f32x4{v0[2], v0[3], v1[0], v1[1]};
    v1 = f32x4{v1[2], v1[3], 0.0f, 0.0f};
  }
  if (s & 4) {
    v0 = v1;
    v1 = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
}

// Masks of the elements col .. col + 7 that lie in a row of n.
__device__ __forceinline__ u32x4 rag_keep(int64_t col, int64_t n) {
  u32x4 k;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    k[h] = (col + 2 * h < n ? 0xffffu : 0u) | (col + 2 * h + 1 < n ? 0xffff0000u : 0u);
  }
  return k;
}

__device__ __forceinline__ void rag_mask(f32x4& v0, f32x4& v1, int64_t col, int64_t n) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (col + e >= n) v0[e] = 0.0f;
    if (col + 4 + e >= n) v1[e] = 0.0f;
  }
}

// Replace loaded C values by the recomputed values of absolute entries in this row (compile-time
// element indices only, so the loaded vectors stay in registers).
__device__ __forceinline__ void apply_patches(const StreamArgs& s, int64_t row, int64_t col,
                                              f32x4& v0, f32x4& v1) {
  const int q0 = s.patch_rowptr[row];
  const int q1 = s.patch_rowptr[row + 1];
  for (int q = q0; q < q1; ++q) {
    const int64_t d = static_cast<int64_t>(s.patch_col[q]) - col;
    const float pv = s.patch_val[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (d == e) v0[e] = pv;
      if (d == e + 4) v1[e] = pv;
    }
  }
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t o = __shfl_xor(v, off, 64);
    v = v > o ? v : o;
  }
  return v;
}

// Block-wide max of the half-bit maxima; thread 0 returns the value as a float.
template <int DT>
__device__ float block_absmax_half(uint32_t mx, uint32_t* ldsu) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t m16 = (mx & 0xffffu) > (mx >> 16) ? (mx & 0xffffu) : (mx >> 16);
  m16 = wave_max_u32(m16);
  if (lane == 0) ldsu[w] = m16;
  __syncthreads();
  float r = 0.0f;
  if (threadIdx.x == 0) {
    uint32_t b = ldsu[0];
    for (int i = 1; i < kThreads / 64; ++i) b = ldsu[i] > b ? ldsu[i] : b;
    r = half_bits_to_float<DT>(b);
  }
  __syncthreads();
  return r;
}

// A launch whose dispatch packet, when e0 / e1 are given, records its own start / end time in
// them (no extra queue packets, so the events bracket exactly the kernel).
template <typename K, typename... Args>
static hipError_t launch_k(K kernel, dim3 grid, dim3 block, size_t shmem, hipStream_t st,
                           hipEvent_t e0, hipEvent_t e1, Args... args) {
  if (e0 != nullptr || e1 != nullptr) {
    hipExtLaunchKernelGGL(kernel, grid, block, static_cast<uint32_t>(shmem), st, e0, e1, 0u,
                          args...);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, shmem, st, args...);
  }
  return hipGetLastError();
}

// One launch of a sequence: the launcher returns at the first that fails, since the kernels after
// it take indices and counts from what it writes.
#define FPSK_LAUNCH(kernel, grid, block, shmem, st, ...)                                        \
  do {                                                                                          \
    const hipError_t e_ = launch_k(kernel, grid, block, shmem, st, nullptr, nullptr, __VA_ARGS__); \
    if (e_ != hipSuccess) return e_;                                                            \
  } while (0)
#define FPSK_LAUNCH_TIMED(kernel, grid, block, shmem, st, e0, e1, ...)                          \
  do {                                                                                          \
    const hipError_t e_ = launch_k(kernel, grid, block, shmem, st, e0, e1, __VA_ARGS__);        \
    if (e_ != hipSuccess) return e_;                                                            \
  } while (0)

// ----------------------------------------------------------------------------------------
// Work-group timeline, compiled only with FPSK_WG_TIMELINE (a diagnostic build of the library;
// the build the binding loads has none of it).  A work-group that holds a WgStamp leaves one
// record of four words at slot `slot` of `base`: its start and end on the 100 MHz constant
// clock, the XCD and the hardware-id word of the CU it ran on, and the launch's work-group
// count with the work-group's type.  Thread 0 stamps the end after the kernel's last block
// reduction, so the record spans the whole work-group.  Each launch overwrites the records of
// the one before.
#ifdef FPSK_WG_TIMELINE
constexpr int kTimelineMax = 1 << 16;

struct WgStamp {
  unsigned long long* rec;
  unsigned long long t0;
  int type;
  __device__ WgStamp(unsigned long long* base, unsigned slot, int ty)
      : rec(slot < static_cast<unsigned>(kTimelineMax) ? base + 4 * slot : nullptr),
        t0(__builtin_amdgcn_s_memrealtime()), type(ty) {}
  __device__ ~WgStamp() {
    if (threadIdx.x == 0 && rec != nullptr) {
      const unsigned long long t1 = __builtin_amdgcn_s_memrealtime();
      const unsigned hw = __builtin_amdgcn_s_getreg((31 << 11) | 4);     // HW_ID, 32 bits
      const unsigned xcc = __builtin_amdgcn_s_getreg((15 << 11) | 20);   // XCC_ID, 16 bits
      rec[0] = t0;
      rec[1] = t1;
      rec[2] = (static_cast<unsigned long long>(xcc & 15u) << 32) | hw;
      rec[3] = (static_cast<unsigned long long>(gridDim.x) << 8) | static_cast<unsigned>(type);
    }
  }
};
#endif

}  // namespace fpsk
