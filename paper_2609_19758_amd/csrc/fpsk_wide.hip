// The C and B sides of the stream pass for more than 1024 buckets a side, as launches of their own
// (the A side, and W = B^T, take the stream kernel's row-bucket work-groups at every m).
//
// With thousands of buckets a 512-column tile holds none or one of most buckets' columns, and the
// fold's cost is its segment starts, barriers and half-empty steps rather than its columns.  A
// work-group of 1024 threads takes 8192 columns at a time instead (16 tiles, one per wave) and a
// thread folds at most 4 buckets: at 16384^3, m = 4096, the moment pass folds a row bucket of C in 2
// steps of 2 columns a bucket where 256 threads took 32 steps of 16 buckets a thread, and B goes 4
// rows at a time, whose 16-byte pieces of the transposed Q need no transpose afterwards (it went 1
// row at a time, k-major).  Bound by the reads of C and B: one work-group per CU, its loads and its
// fold alternating: the fold, bound by its FP64 adds over the longest of 64 lanes' segments, is about
// half of it (two entries a step was slower: C 480 -> 523 us).  16384^3 FP16, m = 4096, moment pass:
// 2400 us and two transposes of 146 us -> C 480 us, B 490 us (1.1 and 0.55 GB read), A 242 us; and
// localization 20.8 -> 15.8 ms.
#include "fpsk_device.h"

namespace fpsk {

constexpr int kWideThreads = 1024;
constexpr int kWideGroups = (kMaxM + kWideThreads - 1) / kWideThreads;    // buckets per thread

// Staged slot of column c of a chunk: the 8 consecutive columns of a thread go to 8 planes, so the
// lanes of a wave write consecutive slots.
__device__ __forceinline__ int wide_slot(int c) { return (c & 7) * (kWideCols / 8) + (c >> 3); }

// Block max of half-bit maxima over 16 waves; thread 0 returns it as a float.
template <int DT>
__device__ float wide_absmax(uint32_t mx, uint32_t* lds) {
  uint32_t m16 = (mx & 0xffffu) > (mx >> 16) ? (mx & 0xffffu) : (mx >> 16);
  m16 = wave_max_u32(m16);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = m16;
  __syncthreads();
  uint32_t b = 0;
  if (threadIdx.x == 0) {
    for (int i = 0; i < kWideThreads / 64; ++i) b = lds[i] > b ? lds[i] : b;
  }
  return half_bits_to_float<DT>(b);
}

// Row bucket a of C: per chunk of 8192 columns each wave sums the bucket's rows (times v1, and with
// moments w_i) over its 512-column tile in FP64, and thread b, b + 1024, ... folds the columns of
// those buckets from the chunk's bucket-sorted list.  In a chunk of at most 8 tiles and with
// buckets of many rows the waves without a tile share the rows: wave w takes tile w mod T (T tiles,
// a power of two) and every (16 / T)-th group of rows, and the 16 / T sums of a column are added in
// wave order before the fold
// (65536 x 1024 x 512 BF16, m = 1030: one wave of 16 read C, 71.5 us; now 42.2 us for its 134 MB).
template <bool MOM, bool VEC>
__global__ __launch_bounds__(kWideThreads) void wide_c_kernel(StreamArgs s) {
  constexpr int U = 4;                       // rows in flight per wave
  extern __shared__ double wide_lds[];
  double* cs = wide_lds;                     // column sums, and the row-weighted ones
  double* csw = wide_lds + kWideCols;
  uint16_t* list = reinterpret_cast<uint16_t*>(wide_lds + (MOM ? 2 : 1) * kWideCols);
  const int m = s.m, a = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int32_t* prow = s.perm + static_cast<int64_t>(a) * s.cap;
  const int64_t last = rag_last(s.n1, s.n3);
  const bool patched = s.patch_rowptr != nullptr;
  double fS[kWideGroups], fR[kWideGroups], fT[kWideGroups];
#pragma unroll
  for (int g = 0; g < kWideGroups; ++g) {
    fS[g] = 0.0;
    fR[g] = 0.0;
    fT[g] = 0.0;
  }
  for (int ch = 0; ch < s.TC; ++ch) {
    // 16 >> sh tiles in this chunk (rounded up), 1 << sh waves to each: at most what leaves a wave
    // two groups of rows in the largest bucket (one group each costs more in the extra sums and
    // barrier than it saves: 4096^3, m = 1030, up to 13 rows, 27.8 -> 31.2 us)
    const int64_t cols = s.n3 - static_cast<int64_t>(ch) * kWideCols;
    int sh = 0;
    while (sh < 4 && cols <= (kWideCols >> (sh + 1)) && (U << (sh + 2)) <= s.cap) ++sh;
    const int T = 16 >> sh, share = 1 << sh, part = w >> (4 - sh);
    const int64_t tcol = static_cast<int64_t>(ch) * kWideCols + (w & (T - 1)) * kColTile;
    const int64_t col = tcol + lane * 8;
    const bool lane_ok = col < s.n3;
    const u32x4 tv = reinterpret_cast<const u32x4*>(s.ctab + static_cast<int64_t>(ch) * s.ctab_stride)[t];
    const int32_t* coff = s.coff + static_cast<int64_t>(ch) * (m + 1);
    int qb[kWideGroups], qe[kWideGroups];
#pragma unroll
    for (int g = 0; g < kWideGroups; ++g) {
      const int b = t + kWideThreads * g;
      qb[g] = b < m ? coff[b] : 0;
      qe[g] = b < m ? coff[b + 1] : 0;
    }
    double acc[8], accw[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      acc[k] = 0.0;
      accw[k] = 0.0;
    }
    if (tcol < s.n3) {
      for (int base = 0; base < s.cap; base += 64) {
        const int32_t pe = base + lane < s.cap ? prow[base + lane] : -1;
        const int nr = __popcll(__ballot(pe != -1));   // valid entries are a prefix of the lanes
        if (nr == 0) break;
        for (int r0 = part * U; r0 < nr; r0 += share * U) {
          f32x4 v0[U], v1[U];
          double sg[U], sw[U];
          int64_t rows[U];
          bool near = false;
#pragma unroll
          for (int q = 0; q < U; ++q) {
            const bool ok = r0 + q < nr;
            const int32_t e = __builtin_amdgcn_readlane(pe, ok ? r0 + q : 0);
            const int64_t row = e & 0x7fffffff;
            rows[q] = row;
            sg[q] = ok ? (e < 0 ? -1.0 : 1.0) : 0.0;
            sw[q] = MOM ? sg[q] * static_cast<double>(row + 1) * s.inv_l1 : 0.0;
            if (VEC) {
              load8f_sel(s.C + row * s.n3 + col, ok && lane_ok, s.zero, v0[q], v1[q]);
            } else {
              load8f_rag(s.C, row * s.n3 + tcol, lane * 8, last, ok && lane_ok, s.zero, v0[q], v1[q]);
              near |= rag_near(row * s.n3 + tcol, kColTile - 8, last);
            }
          }
          if (!VEC) {
            if (near) {
#pragma unroll
              for (int q = 0; q < U; ++q) {
                rag_shift(v0[q], v1[q], rows[q] * s.n3 + tcol, lane * 8, last,
                          r0 + q < nr && lane_ok);
              }
            }
            if (tcol + kColTile > s.n3) {
#pragma unroll
              for (int q = 0; q < U; ++q) rag_mask(v0[q], v1[q], col, s.n3);
            }
          }
          if (patched) {
#pragma unroll
            for (int q = 0; q < U; ++q) {
              if (r0 + q < nr && lane_ok) apply_patches(s, rows[q], col, v0[q], v1[q]);
            }
          }
#pragma unroll
          for (int q = 0; q < U; ++q) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const double x = static_cast<double>(e < 4 ? v0[q][e] : v1[q][e - 4]);
              acc[e] = fma(x, sg[q], acc[e]);
              if (MOM) accw[e] = fma(x, sw[q], accw[e]);
            }
          }
        }
      }
    }
    // column w 512 + lane 8 + e of the chunk is slot e 1024 + w 64 + lane = e 1024 + t; the sums of
    // row group g stand T tiles further on for each
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      cs[e * (kWideCols / 8) + t] = acc[e];
      if (MOM) csw[e * (kWideCols / 8) + t] = accw[e];
    }
    reinterpret_cast<u32x4*>(list)[t] = tv;
    __syncthreads();
    if (share > 1) {
      // thread t has slot i = t mod 64 T of planes e = t / 64 T, ... (share of them at a time)
      const int i = t & (64 * T - 1);
      for (int e = t >> (10 - sh); e < 8; e += share) {
        double x = 0.0, y = 0.0;
        for (int g = 0; g < share; ++g) {
          x += cs[e * (kWideCols / 8) + g * 64 * T + i];
          if (MOM) y += csw[e * (kWideCols / 8) + g * 64 * T + i];
        }
        cs[e * (kWideCols / 8) + i] = x;
        if (MOM) csw[e * (kWideCols / 8) + i] = y;
      }
      __syncthreads();
    }
    const double cbase = static_cast<double>(static_cast<int64_t>(ch) * kWideCols + 1);
#pragma unroll
    for (int g = 0; g < kWideGroups; ++g) {
      for (int q = qb[g]; q < qe[g]; ++q) {
        const uint32_t e = list[q];
        const int c = e & 0x7fff;
        const double sgd = (e & 0x8000u) ? -1.0 : 1.0;
        const double x = sgd * cs[wide_slot(c)];
        fS[g] += x;
        if (MOM) {
          const double wj = (cbase + static_cast<double>(c)) * s.inv_l3;
          fT[g] = fma(x, wj, fT[g]);
          fR[g] += sgd * csw[wide_slot(c)];
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int g = 0; g < kWideGroups; ++g) {
    const int b = t + kWideThreads * g;
    if (b < m) {
      const int64_t o = static_cast<int64_t>(a) * m + b;
      s.partS[o] = fS[g];
      if (MOM) {
        s.partR[o] = fR[g];
        s.partT[o] = fT[g];
      }
    }
  }
}

// Four consecutive rows of B, 8192 columns at a time: thread t loads its 8 columns of the four rows
// (the next chunk's while it folds this one), stages them column-major with the signs v2 applied, and
// folds buckets t, t + 1024, ... in FP64.  Row blocks go to the XCDs in runs of 8 whose 16-byte pieces
// fill one 128-byte line of every Q row (launch index i runs on XCD i mod 8).
template <int DT, bool MOM, bool VEC>
__global__ __launch_bounds__(kWideThreads) void wide_b_kernel(StreamArgs s) {
  constexpr int RB = 4;
  extern __shared__ double wide_lds[];
  __shared__ uint32_t red[kWideThreads / 64];
  uint16_t* L = reinterpret_cast<uint16_t*>(wide_lds);          // [slot][4 rows]
  uint16_t* list = L + kWideCols * RB;
  const int m = s.m, t = threadIdx.x;
  int u = blockIdx.x;
  if (u < s.nB / 64 * 64) u = (u & ~63) | ((u & 7) << 3) | ((u >> 3) & 7);
  const int64_t k0 = static_cast<int64_t>(u) * RB;
  const int64_t last = rag_last(s.n2, s.n3);
  double acc[kWideGroups][RB], accw[kWideGroups][RB];
#pragma unroll
  for (int g = 0; g < kWideGroups; ++g)
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      acc[g][r] = 0.0;
      accw[g][r] = 0.0;
    }
  uint32_t mx = 0;
  u32x4 v[RB], tv;
  uint32_t sb;
  auto issue = [&](int ch) {
    const int64_t cbase = static_cast<int64_t>(ch) * kWideCols;
    const int64_t col = cbase + t * 8;
    const bool live = ch < s.TB;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const bool ok = live && k0 + r < s.n2 && col < s.n3;
      if (VEC) {
        v[r] = load8h_sel(s.B + (k0 + r) * s.n3 + col, ok, s.zero);
      } else {
        v[r] = load8h_rag(s.B, (k0 + r) * s.n3 + cbase, t * 8, last, ok, s.zero);
      }
    }
    const uint16_t* btab = s.btab + static_cast<int64_t>(live ? ch : 0) * s.btab_stride;
    tv = reinterpret_cast<const u32x4*>(btab)[t];
    sb = s.bsign[(live ? cbase : 0) / 8 + t];
  };
  issue(0);
  for (int ch = 0; ch < s.TB; ++ch) {
    const int64_t cbase = static_cast<int64_t>(ch) * kWideCols;
    if (!VEC) {
      if (rag_near((k0 + RB - 1) * s.n3 + cbase, kWideCols - 8, last)) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const bool ok = k0 + r < s.n2 && cbase + t * 8 < s.n3;
          rag_shift(v[r], (k0 + r) * s.n3 + cbase, t * 8, last, ok);
        }
      }
      if (cbase + kWideCols > s.n3) {
        const u32x4 keep = rag_keep(cbase + t * 8, s.n3);
#pragma unroll
        for (int r = 0; r < RB; ++r) v[r] &= keep;
      }
    }
    u32x4 smask;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      smask[h] = (((sb >> (2 * h)) & 1u) << 15) | (((sb >> (2 * h + 1)) & 1u) << 31);
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
#pragma unroll
      for (int h = 0; h < 4; ++h) mx = absmax2(mx, v[r][h]);
      v[r] ^= smask;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int h = e >> 1, sh = 16 * (e & 1);
      u32x2 o;
      o[0] = ((v[0][h] >> sh) & 0xffffu) | ((v[1][h] >> sh) & 0xffffu) << 16;
      o[1] = ((v[2][h] >> sh) & 0xffffu) | ((v[3][h] >> sh) & 0xffffu) << 16;
      *reinterpret_cast<u32x2*>(L + (e * (kWideCols / 8) + t) * RB) = o;
    }
    reinterpret_cast<u32x4*>(list)[t] = tv;
    const int32_t* boff = s.boff + static_cast<int64_t>(ch) * (m + 1);
    int qb[kWideGroups], qe[kWideGroups];
#pragma unroll
    for (int g = 0; g < kWideGroups; ++g) {
      const int b = t + kWideThreads * g;
      qb[g] = b < m ? boff[b] : 0;
      qe[g] = b < m ? boff[b + 1] : 0;
    }
    __syncthreads();
    issue(ch + 1);
    const double cb1 = static_cast<double>(cbase + 1);
#pragma unroll
    for (int g = 0; g < kWideGroups; ++g) {
      for (int q = qb[g]; q < qe[g]; ++q) {
        const int c = list[q];               // moments: the column offset, else its slot
        const u32x2 x = *reinterpret_cast<const u32x2*>(L + (MOM ? wide_slot(c) : c) * RB);
        const double wj = MOM ? (cb1 + static_cast<double>(c)) * s.inv_l3 : 0.0;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const double d = static_cast<double>((r & 1) ? hi_half<DT>(x[r >> 1]) : lo_half<DT>(x[r >> 1]));
          acc[g][r] += d;
          if (MOM) accw[g][r] = fma(d, wj, accw[g][r]);
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int g = 0; g < kWideGroups; ++g) {
    const int b = t + kWideThreads * g;
    if (b >= m) continue;
    float* qo = s.Q + static_cast<int64_t>(b) * s.ldp + k0;
    float* qw = MOM ? s.Qw + static_cast<int64_t>(b) * s.ldp + k0 : nullptr;
    if (k0 + RB <= s.n2) {
      // k0 is a multiple of 4 and the rows start on 256-byte boundaries
      *reinterpret_cast<f32x4*>(qo) =
          f32x4{static_cast<float>(acc[g][0]), static_cast<float>(acc[g][1]),
                static_cast<float>(acc[g][2]), static_cast<float>(acc[g][3])};
      if (MOM) {
        *reinterpret_cast<f32x4*>(qw) =
            f32x4{static_cast<float>(accw[g][0]), static_cast<float>(accw[g][1]),
                  static_cast<float>(accw[g][2]), static_cast<float>(accw[g][3])};
      }
    } else {
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        if (k0 + r < s.n2) {
          qo[r] = static_cast<float>(acc[g][r]);
          if (MOM) qw[r] = static_cast<float>(accw[g][r]);
        }
      }
    }
  }
  const float bmax = wide_absmax<DT>(mx, red);
  if (t == 0) s.maxpart[s.nA + blockIdx.x] = bmax;
}

// Dynamic LDS above 64 KB has to be asked for; the attribute is set with every launch, since it is
// the current device's (a host call without device work, taken under capture too).
template <typename K>
static hipError_t wide_launch(K kernel, int grid, size_t lds, hipStream_t st, hipEvent_t e0,
                              hipEvent_t e1, const StreamArgs& s) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           static_cast<int>(lds));
  if (e != hipSuccess) return e;
  return launch_k(kernel, dim3(grid), dim3(kWideThreads), lds, st, e0, e1, s);
}

hipError_t launch_wide_c(const StreamArgs& s, bool mom, hipStream_t st, hipEvent_t e0,
                         hipEvent_t e1) {
  const bool vec = s.vec_a && s.vec_b && s.vec_c;
  const size_t lds = (mom ? 2 : 1) * kWideCols * sizeof(double) + kWideCols * sizeof(uint16_t);
  if (mom) {
    return vec ? wide_launch(wide_c_kernel<true, true>, s.nC, lds, st, e0, e1, s)
               : wide_launch(wide_c_kernel<true, false>, s.nC, lds, st, e0, e1, s);
  }
  return vec ? wide_launch(wide_c_kernel<false, true>, s.nC, lds, st, e0, e1, s)
             : wide_launch(wide_c_kernel<false, false>, s.nC, lds, st, e0, e1, s);
}

template <int DT>
static hipError_t wide_b(const StreamArgs& s, bool mom, hipStream_t st, hipEvent_t e0,
                         hipEvent_t e1) {
  const bool vec = s.vec_a && s.vec_b && s.vec_c;
  const size_t lds = kWideCols * (4 + 1) * sizeof(uint16_t);
  if (mom) {
    return vec ? wide_launch(wide_b_kernel<DT, true, true>, s.nB, lds, st, e0, e1, s)
               : wide_launch(wide_b_kernel<DT, true, false>, s.nB, lds, st, e0, e1, s);
  }
  return vec ? wide_launch(wide_b_kernel<DT, false, true>, s.nB, lds, st, e0, e1, s)
             : wide_launch(wide_b_kernel<DT, false, false>, s.nB, lds, st, e0, e1, s);
}

hipError_t launch_wide_b(const StreamArgs& s, int dt, bool mom, hipStream_t st, hipEvent_t e0,
                         hipEvent_t e1) {
  return dt == 1 ? wide_b<1>(s, mom, st, e0, e1) : wide_b<0>(s, mom, st, e0, e1);
}

}  // namespace fpsk
