// Tables of one hash round, built on the device (Sec. III-B): the row lists of each bucket and
// the bucket-sorted column lists that the stream pass reads.  Built on the host and copied they
// took six copies and about 80 us of every re-probe and localization round with the device idle
// (2048 x 5120 x 5120: the re-probe 158 -> 84 us); three launches on the caller's stream replace
// that.
//   hash_kernel    bucket and sign of every row and column, the column signs as bits;
//   order_kernel   (probe) the buckets' places by size, largest first;
//   tables_kernel  one wave per bucket compacts its rows in ascending order; one work-group per
//                  column tile or chunk counts, places and orders that tile's columns by bucket.
// Every list is in ascending index order, so the sums over it have one fixed order.  Bound by
// launches and their chains of dependent steps: the three take 19 us at 2048 x 5120, m = 48.
#include "fpsk_device.h"

namespace fpsk {

// splitmix64 (Steele, Lea and Flood 2014): output idx of the stream at `key`.
__device__ __forceinline__ uint64_t mix_output(uint64_t key, uint64_t idx) {
  uint64_t z = key + (idx + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Bucket (12 bits: m <= 4096) | negative sign << 15 of one index.
__device__ __forceinline__ uint32_t hash_word(uint64_t key, int64_t idx, int m) {
  const uint64_t x = mix_output(key, static_cast<uint64_t>(idx));
  const uint32_t b = static_cast<uint32_t>(((x >> 32) * static_cast<uint64_t>(m)) >> 32);
  return b | static_cast<uint32_t>(x & 1ull) << 15;
}

// Thread t takes 8 indices of a side: their words as one 16-byte store (0x7fff past the end: no
// bucket), and for the columns their sign byte (zero past n3).  The first nb1 work-groups take
// the rows.
__global__ __launch_bounds__(kThreads) void hash_kernel(TableArgs a, int nb1) {
  const bool side2 = static_cast<int>(blockIdx.x) >= nb1;
  const int64_t g = (static_cast<int64_t>(blockIdx.x) - (side2 ? nb1 : 0)) * kThreads + threadIdx.x;
  const int64_t n = side2 ? a.n3 : a.n1;
  const int64_t groups = side2 ? a.pad3 / 8 : a.pad1 / 8;
  if (g >= groups) return;
  const uint64_t key = side2 ? a.key2 : a.key1;
  u32x4 w;
  uint32_t signs = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t i = 8 * g + e;
    const uint32_t h = i < n ? hash_word(key, i, a.m) : 0x7fffu;
    if (i < n) signs |= (h >> 15) << e;
    if (e & 1) w[e >> 1] |= h << 16;
    else w[e >> 1] = h;
  }
  reinterpret_cast<u32x4*>(side2 ? a.hb2 : a.hb1)[g] = w;
  if (side2 && 8 * g < a.nsign) a.bsign[g] = static_cast<uint8_t>(signs);
}

// slot[b]: the place of bucket b among the buckets by row count, largest first, ties in bucket
// order.  Every work-group counts the rows for itself and places 1024 buckets.
__global__ __launch_bounds__(1024) void order_kernel(TableArgs a) {
  __shared__ uint32_t cnt[kMaxM];
  for (int b = threadIdx.x; b < a.m; b += 1024) cnt[b] = 0;
  __syncthreads();
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < a.n1; i += 1024) atomicAdd(&cnt[a.hb1[i] & 0x7fffu], 1u);
  __syncthreads();
  const int b = blockIdx.x * 1024 + threadIdx.x;
  if (b >= a.m) return;
  const uint32_t mine = cnt[b];
  int r = 0;
#pragma unroll 16
  for (int x = 0; x < a.m; ++x) r += cnt[x] > mine || (cnt[x] == mine && x < b);
  a.slot[b] = r;
}

// One wave: the rows of bucket b in ascending order as row | negative sign << 31, then -1 up to
// cap.  A wave reads 8 words a lane from each of kListLoads 512-word groups at once (a load per
// group waits for memory once per 512 rows).
constexpr int kListLoads = 8;

__device__ void bucket_list(const uint16_t* hb, int64_t pad, int b, int32_t* out, int cap) {
  const int lane = threadIdx.x & 63;
  const u32x4 none = {0x7fff7fffu, 0x7fff7fffu, 0x7fff7fffu, 0x7fff7fffu};
  int pos = 0;
  for (int64_t base = 0; base < pad; base += 512 * kListLoads) {
    u32x4 w[kListLoads];
#pragma unroll
    for (int g = 0; g < kListLoads; ++g) {
      const int64_t i0 = base + 512 * g + 8 * lane;
      w[g] = i0 < pad ? *reinterpret_cast<const u32x4*>(hb + i0) : none;
    }
#pragma unroll
    for (int g = 0; g < kListLoads; ++g) {
      uint32_t h[8];
      int c = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        h[e] = (w[g][e >> 1] >> (16 * (e & 1))) & 0xffffu;
        c += static_cast<int>(h[e] & 0x7fffu) == b;
      }
      if (__ballot(c != 0) == 0) continue;
      int incl = c;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
      }
      int p = pos + incl - c;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (static_cast<int>(h[e] & 0x7fffu) == b) {
          const uint32_t row = static_cast<uint32_t>(base + 512 * g + 8 * lane + e);
          if (p < cap) out[p] = static_cast<int32_t>(row | (h[e] >> 15) << 31);
          ++p;
        }
      }
      pos += __shfl(incl, 63, 64);
    }
  }
  for (int p = pos + lane; p < cap; p += 64) out[p] = -1;
}

// One work-group: the columns of one tile sorted by bucket, segments padded to multiples of
// t.pad with the sentinel offset W.  Columns go to their segment in any order first (LDS), then
// each finds its rank among its segment's smaller column offsets: W^2 / m comparisons in all, 8
// to an LDS read where segments are whole groups of 8.  1024 threads, so that a thread's chain of
// LDS steps covers 4 columns of a 4096-column chunk (256 threads, 16 columns each: 26 us against
// 9.5 at 4096 x 4096, m = 432; 86 against 25 at 16384 x 16384, m = 4096).
constexpr int kTableThreads = 1024;

__device__ void column_tile(const TableArgs& a, const ColTable& t, int tile, char* lds) {
  constexpr int NT = kTableThreads;
  const int m = a.m;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(lds);                       // m
  uint16_t* off = reinterpret_cast<uint16_t*>(cnt + (m + 3) / 4 * 4);     // m + 1
  uint16_t* list = off + (m + 1 + 7) / 8 * 8;                             // stride
  __shared__ uint32_t wsum[NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t j0 = static_cast<int64_t>(tile) * t.W;
  const int nc = static_cast<int>(a.n3 - j0 < t.W ? a.n3 - j0 : t.W);
  const uint16_t* hb = a.hb2 + j0;
  const int pm = t.pad - 1;           // t.pad is 1 or 8
  for (int b = tid; b < m; b += NT) cnt[b] = 0;
  for (int e = tid; e < t.stride; e += NT) list[e] = 0xffffu;
  __syncthreads();
#pragma unroll 4
  for (int c = tid; c < nc; c += NT) atomicAdd(&cnt[hb[c] & 0x7fffu], 1u);
  __syncthreads();
  // segment starts: thread tid takes buckets tid per .. (tid + 1) per
  const int per = (m + NT - 1) / NT;
  const int b0 = tid * per < m ? tid * per : m, b1 = b0 + per < m ? b0 + per : m;
  uint32_t sum = 0;
  for (int b = b0; b < b1; ++b) sum += (cnt[b] + pm) & ~pm;
  uint32_t incl = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t s = incl - sum;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) s += i < w ? wsum[i] : 0u;
  int32_t* offg = t.off + static_cast<int64_t>(tile) * (m + 1);
  for (int b = b0; b < b1; ++b) {
    off[b] = static_cast<uint16_t>(s);
    offg[b] = static_cast<int32_t>(s);
    s += (cnt[b] + pm) & ~pm;
    cnt[b] = 0;
  }
  if (b1 == m && b0 < m) {
    off[m] = static_cast<uint16_t>(s);
    offg[m] = static_cast<int32_t>(s);
  }
  __syncthreads();
#pragma unroll 4
  for (int c = tid; c < nc; c += NT) {
    const int b = hb[c] & 0x7fffu;
    list[off[b] + atomicAdd(&cnt[b], 1u)] = static_cast<uint16_t>(c);
  }
  __syncthreads();
  uint16_t* __restrict__ tab = t.tab + static_cast<int64_t>(tile) * t.stride;
  for (int c = tid; c < nc; c += NT) {
    const uint32_t h = hb[c];
    const int b = h & 0x7fffu;
    const int q0 = off[b], q1 = off[b + 1];
    int rank = 0;
    if (t.pad == 8) {
#pragma unroll 2
      for (int q = q0; q < q1; q += 8) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(list + q);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          rank += static_cast<int>((v[e >> 1] >> (16 * (e & 1))) & 0xffffu) < c;
        }
      }
    } else {
      for (int q = q0; q < q1; ++q) rank += static_cast<int>(list[q]) < c;
    }
    uint32_t e = static_cast<uint32_t>(c);
    if (t.format == 0) e |= h & 0x8000u;
    if (t.format == 2) e = static_cast<uint32_t>((c & 7) * (t.W / 8) + (c >> 3));   // staged slot
    tab[q0 + rank] = static_cast<uint16_t>(e);
  }
  // the padding of every segment, and the table past the last one
  if (pm != 0) {
    for (int b = tid; b < m; b += NT) {
      for (int q = off[b] + static_cast<int>(cnt[b]); q < off[b + 1]; ++q) tab[q] = static_cast<uint16_t>(t.W);
    }
  }
  for (int q = off[m] + tid; q < t.stride; q += NT) tab[q] = static_cast<uint16_t>(t.W);
}

__global__ __launch_bounds__(kTableThreads) void tables_kernel(TableArgs a, int nperm, int nperm2,
                                                                int first) {
  extern __shared__ char lds_tab[];
  constexpr int kWaves = kTableThreads / 64;
  int u = first + static_cast<int>(blockIdx.x);
  const int nct = a.c.tiles + a.b.tiles;
  if (u < nct) {                    // the longer work first
    if (u < a.b.tiles) column_tile(a, a.b, u, lds_tab);
    else column_tile(a, a.c, u - a.b.tiles, lds_tab);
    return;
  }
  u -= nct;
  const int w = threadIdx.x >> 6;
  if (u < nperm) {
    const int b = kWaves * u + w;
    if (b < a.m) {
      const int slot = a.slot != nullptr ? a.slot[b] : b;
      bucket_list(a.hb1, a.pad1, b, a.perm + static_cast<int64_t>(slot) * a.cap, a.cap);
    }
    return;
  }
  u -= nperm;
  if (u < nperm2) {
    const int b = kWaves * u + w;
    if (b < a.m) {
      bucket_list(a.hb2, a.pad3, b, a.perm2 + static_cast<int64_t>(b) * a.cap2, a.cap2);
    }
  }
}

hipError_t launch_tables(const TableArgs& a, hipStream_t st) {
  const int64_t g1 = a.pad1 / 8, g3 = a.pad3 / 8;
  const int nb1 = static_cast<int>((g1 + kThreads - 1) / kThreads);
  const int nb3 = static_cast<int>((g3 + kThreads - 1) / kThreads);
  FPSK_LAUNCH(hash_kernel, dim3(nb1 + nb3), dim3(kThreads), 0, st, a, nb1);
  if (a.slot != nullptr) {
    FPSK_LAUNCH(order_kernel, dim3((a.m + 1023) / 1024), dim3(1024), 0, st, a);
  }
  const int kWaves = kTableThreads / 64;
  const int np = (a.m + kWaves - 1) / kWaves, np2 = a.perm2 != nullptr ? np : 0;
  const int stride = a.c.stride > a.b.stride ? a.c.stride : a.b.stride;
  const size_t lds = static_cast<size_t>((a.m + 3) / 4 * 4) * 4 +
                     static_cast<size_t>((a.m + 1 + 7) / 8 * 8) * 2 + static_cast<size_t>(stride) * 2;
  // (a launch holds fewer than 2^32 threads: rows of 2^31 columns are more tiles than that)
  const int total = a.c.tiles + a.b.tiles + np + np2;
  constexpr int kMost = 1 << 21;
  for (int first = 0; first < total; first += kMost) {
    const int n = total - first < kMost ? total - first : kMost;
    FPSK_LAUNCH(tables_kernel, dim3(n), dim3(kTableThreads), lds, st, a, np, np2, first);
  }
  return hipSuccess;
}

}  // namespace fpsk
