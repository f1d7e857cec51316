// The bucket-space product S = P Q - S_C on the integer matrix cores (S alone, more than 256
// buckets a side, n2 >= 512, m^2 n2 >= 2^28, or 2.75 x 2^28 below n2 = 4096).
//
// A product of floating-point matrices as a sum of exact integer products is the scheme of Ozaki,
// Ogita, Oishi and Rump (2012), here on 8-bit integers as in Ootomo, Ozaki and Yokota (2024).  Each
// row of a factor is scaled by a power of two to 32-bit integers and split into four signed 8-bit
// digits, x 2^e = d0 2^24 + d1 2^16 + d2 2^8 + d3.  All 16 digit products are formed, exact in 32-bit
// sums over at most 16384 k (grouped by i + j into seven accumulators), and joined in 64-bit
// integers, so P Q is exact but for entries with bits below 2^-31 of their row's largest.
//
// What those bits cost depends on both factors: an entry's quantum is its row's, and it is
// multiplied by the other factor's entries at the same k.  Two measures keep it below the rounding
// of the FP32 factors themselves:
//   - channel k of P is multiplied by 2^t and of Q by 2^-t (exact, and nothing in the product), t
//     half the difference of the channel's typical exponents in Q and in P, so that a channel which
//     is small in one factor and large in the other is of middle size in both.  Channels scaled
//     by 1e-6 in A (half of them) and in B (the others) gave S errors of 1855 times the noise without
//     it, 0.0023 times with it, as the FP64 product does (2048 x 4096 x 2048, m = 260, BF16).
//   - a row takes part when its quantum u adds at most about half of the FP32 rounding to S:
//     u^2 / 12 sum_k w_k <= 4/15 2^-50.7 sum_k w_k x_k^2, w_k the channel's typical square in the
//     other factor (equal for both after the scaling) and 2^-50.7 the mean square of FP32 rounding
//     relative to the values; with T = 2^49 u^2, sum_k w_k T <= sum_k w_k x_k^2.  Every x_k^2 counts
//     at most 16 T, so that at least 1/16 of the weight has to lie where the row is above the bound,
//     and not in one entry that most of the other factor's rows may not meet (1e30 in a channel that
//     a single column of B holds: with the uncapped sum the rest of the row was lost).  A Gaussian
//     row has a 200 times smaller left side; rows with 40 channels at 30 times the others' scale
//     still take part (with T four times larger most tiles of 6 such channels were refused: 4096^3,
//     m = 432, 124 -> 147 us a probe).  Rows of one huge entry, or not finite, take no part.
// The typical sizes are means of the exponents over 64 buckets a factor, zeros left out, and the
// weights the share of the buckets that hold the channel: the buckets are random sums of rows, and a
// mean of logarithms is not moved by a few rows of another scale.  Tiles with a row that takes no part
// are left to the FP64 matrix cores, whose kernel runs beside this one and takes only those.
//
// Error of S against 64 bits (rms over the noise), FP64 product and here: 2048 x 4096 x 2048,
// m = 260, BF16 0.002402 both, FP16 0.004215 both; 4096^3 BF16, m = 1000 0.001302 both; channels scaled
// by 1e-2 to 1e-6 as above likewise equal to four digits.
// (13 pairs, i + j <= 4, in 64 x 32 wave tiles of five accumulators were as fast and raised FP16
// errors by 0.1 %.)
//
// Bound by the integer matrix cores: 16 x 2 m^2 n2 operations at 1/64 of the FP64 cores' time each.
// 16384^3 FP16, m = 4096: FP64 8400 us -> 3660 us (product 3340, digits 179, row scales 137, channels
// 7), 2.6 x 10^15 operations a second of the 4.7 x 10^15 that registers alone reach; m = 698: 301 ->
// 190 us; 4096^3, m = 432: 43 us and 15 us of slice sums -> 41 and 8 us.
#include "fpsk_device.h"

namespace fpsk {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

// Channel figures: the power of two t that balances channel k (bal), and the binary logarithm of the
// channel's weight (weight), the product of its typical sizes in both factors times the
// share of the sampled rows that hold it at all; kNoSize where a factor's sample holds only zeros.  A
// work-group takes 128 channels; a thread 4 of them in 8 of the 64 sampled rows of each factor.  A
// channel without a size in one factor is scaled out of the other: a row that has an entry there
// after all is then too far from its typical size to take part.
constexpr int kSampleRows = 64;
constexpr int kNoSize = -32768;

// 2^(lw - top), top the largest of the logarithms: zero below 2^-126.
__device__ __forceinline__ float weight_of(int lw, int top) {
  const int b = 127 + lw - top;
  return lw == kNoSize || b < 0 ? 0.0f : __uint_as_float(static_cast<uint32_t>(b) << 23);
}

__global__ __launch_bounds__(kThreads) void channel_kernel(ProductArgs pa) {
  constexpr int G = kThreads / 32;                   // row groups
  __shared__ uint32_t part[2][G][128];
  __shared__ int stop[2];
  __shared__ float ssum[2];
  const int t = threadIdx.x, g = t >> 5, c0 = 4 * (t & 31);
  const int64_t k = static_cast<int64_t>(blockIdx.x) * 128 + c0;
  f32x4 x[2][kSampleRows / G];
#pragma unroll
  for (int i = 0; i < kSampleRows / G; ++i) {
    const int64_t row = static_cast<int64_t>(g + G * i) * pa.m / kSampleRows;
    x[0][i] = *reinterpret_cast<const f32x4*>(pa.P + row * pa.ldp + k);
    x[1][i] = *reinterpret_cast<const f32x4*>(pa.Q + row * pa.ldp + k);
  }
  // exponents of the normal numbers: their sum and count in one word
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t n = 0;
#pragma unroll
      for (int i = 0; i < kSampleRows / G; ++i) {
        const uint32_t b = (__float_as_uint(x[f][i][e]) >> 23) & 255u;
        n += b != 0 && b != 255 ? (1u << 16) + b : 0u;
      }
      part[f][g][c0 + e] = n;
    }
  __syncthreads();
  int w = kNoSize;
  if (t < 128) {
    int ex[2], held = 0;
    bool none[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      uint32_t n = 0;
#pragma unroll
      for (int i = 0; i < G; ++i) n += part[f][i][t];
      const int cnt = static_cast<int>(n >> 16);
      none[f] = cnt == 0;
      ex[f] = (static_cast<int>(n & 0xffffu) + cnt / 2) / (cnt > 0 ? cnt : 1) - 127;
      held += 31 - __clz(cnt > 0 ? cnt : 1);           // log2 of the rows that hold it
    }
    int bal = (ex[1] - ex[0]) >> 1;
    w = ex[0] + ex[1] + held;
    bal = bal < -100 ? -100 : (bal > 100 ? 100 : bal);
    if (none[0] || none[1]) {
      bal = none[0] == none[1] ? 0 : (none[0] ? 100 : -100);
      w = kNoSize;
    }
    pa.bal[blockIdx.x * 128 + t] = static_cast<int8_t>(bal);
    pa.weight[blockIdx.x * 128 + t] = static_cast<int16_t>(w);
    // the work-group's largest weight, and the sum of its weights relative to that
    const int m64 = static_cast<int>(wave_max_u32(static_cast<uint32_t>(w - kNoSize))) + kNoSize;
    if ((t & 63) == 0) stop[t >> 6] = m64;
  }
  __syncthreads();
  const int top = stop[0] > stop[1] ? stop[0] : stop[1];
  if (t < 128) {
    float sum = weight_of(w, top);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if ((t & 63) == 0) ssum[t >> 6] = sum;
  }
  __syncthreads();
  if (t == 0) {
    pa.wtop[blockIdx.x] = top;
    pa.wsum[blockIdx.x] = ssum[0] + ssum[1];
  }
  if (blockIdx.x == 0 && t == 0) pa.rexp[2 * pa.m] = pa.rexp[2 * pa.m + 1] = 0;
}

// Byte i of a word of four balancing exponents.
__device__ __forceinline__ int bal_of(uint32_t c, int i) {
  return static_cast<int>(c << (24 - 8 * i)) >> 24;
}

// Scale exponent e of each row (2m work-groups: rows of P, then of Q): the balanced row times 2^e
// rounds to integers whose four signed digits exist, |x 2^e| <= 2^31 - 2^24; kNoDigits for a row
// that takes no part.  rexp[2m], rexp[2m + 1]: whether any row of P, of Q does.  The balanced row
// stays in registers between the search for its largest entry and the sum over it (NV 16-byte pieces a
// thread; NV = 0, longer rows, reads it again).  16384^3, m = 698, 92 MB of factors: read twice 28.8 us,
// kept 19.1 us (loads behind branches, one piece at a time: 28 us).
template <int NV>
__global__ __launch_bounds__(kThreads) void row_scale_kernel(ProductArgs pa) {
  __shared__ uint32_t smax[kThreads / 64];
  __shared__ int stop[kThreads / 64];
  __shared__ float sen[kThreads / 64], sws[kThreads / 64];
  const int r = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const bool second = r >= pa.m;
  const float* x = second ? pa.Q + static_cast<int64_t>(r - pa.m) * pa.ldp
                          : pa.P + static_cast<int64_t>(r) * pa.ldp;
  const int sg = second ? -1 : 1;
  // the largest weight of all channels
  const int groups = (pa.n2 + 127) / 128;
  int top = kNoSize;
  for (int i = t; i < groups; i += kThreads) top = pa.wtop[i] > top ? pa.wtop[i] : top;
  uint32_t mx = 0;                          // bits of the largest magnitude (NaN above infinity)
  auto row_at = [&](int k) { return *reinterpret_cast<const f32x4*>(x + k); };
  auto bal_at = [&](int k) { return *reinterpret_cast<const uint32_t*>(pa.bal + k); };
  auto weight_at = [&](int k) { return *reinterpret_cast<const u32x2*>(pa.weight + k); };
  auto balanced = [&](f32x4 v, uint32_t c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = ldexpf(v[e], sg * bal_of(c, e));
    return v;
  };
  auto largest = [&](const f32x4& v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t b = __float_as_uint(v[e]) & 0x7fffffffu;
      mx = b > mx ? b : mx;
    }
  };
  // (pieces past the row read its first ones and count as zeros: loads without branches go out
  // together)
  f32x4 kept[NV > 0 ? NV : 1];
  u32x2 wt[NV > 0 ? NV : 1];
  if constexpr (NV > 0) {
    uint32_t c[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = 4 * t + 4 * kThreads * i, at = k < pa.kact ? k : 0;
      kept[i] = row_at(at);
      c[i] = bal_at(at);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const bool in = 4 * t + 4 * kThreads * i < pa.kact;
      kept[i] = balanced(kept[i], c[i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) kept[i][e] = in ? kept[i][e] : 0.0f;
      largest(kept[i]);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = 4 * t + 4 * kThreads * i;
      wt[i] = weight_at(k < pa.kact ? k : 0);
    }
  } else {
#pragma unroll 4
    for (int k = 4 * t; k < pa.kact; k += 4 * kThreads) largest(balanced(row_at(k), bal_at(k)));
  }
  mx = wave_max_u32(mx);
  top = static_cast<int>(wave_max_u32(static_cast<uint32_t>(top - kNoSize))) + kNoSize;
  if (lane == 0) {
    smax[w] = mx;
    stop[w] = top;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kThreads / 64; ++i) {
    mx = smax[i] > mx ? smax[i] : mx;
    top = stop[i] > top ? stop[i] : top;
  }
  const float big = __uint_as_float(mx);
  int q = 0;                                // quantum 2^-q
  if (mx < 0x7f800000u && big >= 0x1p-120f) {
    int ex;
    const float f = frexpf(big, &ex);       // big = f 2^ex, 0.5 <= f < 1
    q = f <= 1.0f - 0x1p-7f ? 31 - ex : 30 - ex;
  } else if (mx != 0) {
    if (t == 0) pa.rexp[r] = kNoDigits;
    return;
  }
  // sums of the weights times min(2 x^2 / T, 32), and of the weights
  float en = 0.0f, ws = 0.0f;
  for (int i = t; i < groups; i += kThreads) ws += ldexpf(pa.wsum[i], pa.wtop[i] - top);
  auto weigh = [&](const f32x4& v, const u32x2& c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float y = ldexpf(v[e], q - 24);           // at most 2^7
      const int lw = static_cast<int>(c[e >> 1] << (16 - 16 * (e & 1))) >> 16;
      int b = 127 + lw - top;                         // (a channel without a size is far below 0)
      b = b > 0 ? b : 0;
      en = fmaf(fminf(y * y, 32.0f), __uint_as_float(static_cast<uint32_t>(b) << 23), en);
    }
  };
  if constexpr (NV > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) weigh(kept[i], wt[i]);
  } else {
#pragma unroll 4
    for (int k = 4 * t; k < pa.kact; k += 4 * kThreads) {
      weigh(balanced(row_at(k), bal_at(k)), weight_at(k));
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    en += __shfl_xor(en, d, 64);
    ws += __shfl_xor(ws, d, 64);
  }
  if (lane == 0) {
    sen[w] = en;
    sws[w] = ws;
  }
  __syncthreads();
  if (t != 0) return;
  for (int i = 1; i < kThreads / 64; ++i) {
    en += sen[i];
    ws += sws[i];
  }
  const bool takes = mx == 0 || (ws > 0.0f && en >= 2.0f * ws);
  pa.rexp[r] = takes ? q : kNoDigits;
  // (every work-group that does stores the same word: no atomic, which cost 10 ns a row here)
  if (takes) pa.rexp[2 * pa.m + (second ? 1 : 0)] = 1;
}

// Digit fragments.  For a block of 32 rows, 32 k and one digit the matrix instruction's operand
// is 64 lanes of 16 bytes, lane (k / 16 mod 2) 32 + row holding 16 consecutive k: 1 KB in a row,
// [row block][k block][digit].  A work-group converts 32 rows x 128 k, thread (row, k / 16).  Blocks
// that no tile of digits reads (one of their 64 rows takes no part, or none of the other factor's
// does) stay as they are.
__global__ __launch_bounds__(kThreads) void digits_kernel(ProductArgs pa, int nbP) {
  const int t = threadIdx.x, row = t & 31;
  const bool second = static_cast<int>(blockIdx.y) >= nbP;
  const int rb = second ? blockIdx.y - nbP : blockIdx.y;
  const int r = rb * 32 + row;
  const int k = blockIdx.x * 128 + (t >> 5) * 16;
  const int KS = (pa.n2 + 31) / 32;
  const int e = r < pa.m ? pa.rexp[second ? pa.m + r : r] : kNoDigits;
  const int r64 = (rb >> 1) * 64 + (t & 63);
  const bool bad = r64 < pa.m && pa.rexp[second ? pa.m + r64 : r64] == kNoDigits;
  if (__ballot(bad) != 0 || pa.rexp[2 * pa.m + (second ? 0 : 1)] == 0) return;
  if (k >= KS * 32) return;
  const float* x = (second ? pa.Q : pa.P) + static_cast<int64_t>(r < pa.m ? r : 0) * pa.ldp + k;
  const u32x4 ch = *reinterpret_cast<const u32x4*>(pa.bal + k);
  f32x4 v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = reinterpret_cast<const f32x4*>(x)[j];
  u32x4 d[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int bal = bal_of(ch[j], i);
      const int q = e != kNoDigits ? __float2int_rn(ldexpf(v[j][i], second ? e - bal : e + bal)) : 0;
      // signed bytes: each of the lower three hands its carry up
      u[i] = (static_cast<uint32_t>(q) + 0x00808080u) ^ 0x00808080u;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int sh = 24 - 8 * s;
      d[s][j] = ((u[0] >> sh) & 0xffu) | ((u[1] >> sh) & 0xffu) << 8 |
                ((u[2] >> sh) & 0xffu) << 16 | ((u[3] >> sh) & 0xffu) << 24;
    }
  }
  u32x4* out = reinterpret_cast<u32x4*>(second ? pa.digQ : pa.digP) +
               ((static_cast<int64_t>(rb) * KS + (k >> 5)) * 4) * 64 + ((k >> 4) & 1) * 32 + row;
#pragma unroll
  for (int s = 0; s < 4; ++s) out[s * 64] = d[s];
}

// A work-group owns a 128 x 64 tile over one k-slice: four waves of 64 x 32 outputs, one to a SIMD
// (two 32 x 32 blocks of seven accumulators: 224 accumulation registers).  Per 32 k the four digits
// of the tile's 6 row blocks (24 KB) go through LDS, three steps deep: while a wave's 32 matrix
// instructions of step k run on fragments in registers, the fragments of step k + 1 are read from
// LDS and the bytes of steps k + 2 and k + 3 arrive from memory, so that one wave a SIMD keeps its
// matrix core fed.  Launch indices map XCD-locally (index i runs on XCD i mod 8), in groups of 8 row tiles, so
// that an XCD's work-groups share both factors' fragments in its L2.
struct Frags {
  i32x4 a[2][4];
  i32x4 b[4];
};

__global__ __launch_bounds__(kThreads, 1) void digit_product_kernel(ProductArgs pa,
                                                                    const void* zero) {
  __shared__ i32x4 sh[3][6 * 256];
  __shared__ int none[3];
  const int m = pa.m;
  const int64_t mm = static_cast<int64_t>(m) * m;
  const int nta = (m + 127) / 128, ntb = (m + 63) / 64;
  const int ntl = nta * ntb;
  const int per = gridDim.x / 8;
  const int slot = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (slot >= ntl * pa.NS) return;
  const int slice = slot / ntl, pid = slot - slice * ntl;
  const int grp = pid / (8 * ntb), first = 8 * grp;
  const int rows = nta - first < 8 ? nta - first : 8;
  const int within = pid - grp * 8 * ntb;
  const int ta = first + within % rows, tb = within / rows;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (w < 3) {
    // (a half past the last row has nothing to form either)
    const int row0 = w < 2 ? ta * 128 + w * 64 : tb * 64, row = row0 + lane;
    const bool bad = row0 >= m || (row < m && pa.rexp[w < 2 ? row : m + row] == kNoDigits);
    const bool any = __ballot(bad) != 0;
    if (lane == 0) none[w] = any;
  }
  __syncthreads();
  if (none[2] || (none[0] && none[1])) return;
  const int KS = (pa.n2 + 31) / 32;
  const int ks0 = slice * (pa.ksl / 32);
  const int nst = (ks0 + pa.ksl / 32 < KS ? ks0 + pa.ksl / 32 : KS) - ks0;    // at least 1
  // this thread's 16 bytes of each row block's 4 KB per step
  const i32x4* src[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const int64_t rb = c < 4 ? ta * 4 + c : tb * 2 + c - 4;
    src[c] = reinterpret_cast<const i32x4*>(c < 4 ? pa.digP : pa.digQ) + (rb * KS + ks0) * 256 + t;
  }
  const int wr = w >> 1, wc = w & 1;
  i32x16 acc[2][7];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < 7; ++g)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][g][r] = 0;
  // step s of the slice (zeros past the end, which add nothing: the loop takes whole pairs)
  auto fetch = [&](i32x4 (&st)[6], int s) {
    const bool ok = s < nst;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const i32x4* p = ok ? src[c] + s * 256 : reinterpret_cast<const i32x4*>(zero);
      st[c] = *p;
    }
  };
  auto put = [&](const i32x4 (&st)[6], int buf) {
#pragma unroll
    for (int c = 0; c < 6; ++c) sh[buf][c * 256 + t] = st[c];
  };
  auto read = [&](Frags& f, int buf) {
    const i32x4* B = sh[buf] + (4 + wc) * 256 + lane;
    const i32x4* A = sh[buf] + 2 * wr * 256 + lane;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      f.b[s] = B[s * 64];
      f.a[0][s] = A[s * 64];
      f.a[1][s] = A[256 + s * 64];
    }
  };
  auto step = [&](const Frags& f) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[b][i + j] =
              __builtin_amdgcn_mfma_i32_32x32x32_i8(f.a[b][i], f.b[j], acc[b][i + j], 0, 0, 0);
  };
  Frags f0, f1;
  i32x4 st0[6], st1[6];
  fetch(st0, 0);
  fetch(st1, 1);
  put(st0, 0);
  put(st1, 1);
  fetch(st1, 2);
  __syncthreads();
  read(f0, 0);
  int nb = 1;                         // buffer of the next step
  // A step's LDS reads, memory loads and LDS stores are spread between its matrix instructions:
  // a wave issues in order, and the reads of all four waves queued ahead of the matrix
  // instructions, the stores behind them, left the matrix cores idle half of the time (16384^3,
  // 4096 buckets: 3800 us; now 3070).
  auto half = [&](const Frags& cur, Frags& nxt, i32x4 (&ahead)[6], const i32x4 (&due)[6], int s) {
    fetch(ahead, s + 3);
    read(nxt, nb);
    step(cur);
    nb = nb == 2 ? 0 : nb + 1;
    put(due, nb);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // memory load
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // matrix instructions
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // LDS store
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __syncthreads();
  };
  for (int s = 0; s < nst; s += 2) {
    half(f0, f1, st0, st1, s);
    half(f1, f0, st1, st0, s + 1);
  }
  // The sum of the digit pairs i + j = g stands for 2^(8 (6 - g)).  The five upper groups make one
  // 64-bit integer in units of 2^16, the two lower ones another; scaled by the row's and the
  // column's exponents (a power of two, built from its exponent bits).
  auto pow2 = [](int e) {
    return __builtin_bit_cast(double, static_cast<uint64_t>(1023 + e) << 52);
  };
  const int col = tb * 64 + wc * 32 + (lane & 31);
  const int r64 = ta * 2 + wr;                       // 64-row tile of the scratch
  if (none[wr] || r64 >= pa.nt) return;
  const int ec = pa.rexp[m + (col < m ? col : m - 1)];
  int er[2][16];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = r64 * 64 + b * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      er[b][r] = pa.rexp[row < m ? row : m - 1];
    }
  double v[2][16];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t hi = static_cast<int64_t>(acc[b][0][r]) * (int64_t{1} << 32) +
                         static_cast<int64_t>(acc[b][1][r]) * (int64_t{1} << 24) +
                         static_cast<int64_t>(acc[b][2][r]) * (int64_t{1} << 16) +
                         static_cast<int64_t>(acc[b][3][r]) * 256 + acc[b][4][r];
      const int64_t lo = static_cast<int64_t>(acc[b][5][r]) * 256 + acc[b][6][r];
      v[b][r] = (static_cast<double>(hi) * 65536.0 + static_cast<double>(lo)) * pow2(-er[b][r] - ec);
    }
  // this slice's share of the C grid, a group's 32 loads in one round trip
  for (int g = slice; g < pa.npc; g += pa.NS) {
    const double* part = pa.partS + static_cast<int64_t>(g) * mm;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = r64 * 64 + b * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        // (outputs past m subtract some other entry and are dropped)
        v[b][r] -= part[static_cast<int64_t>(row < m ? row : m - 1) * m + (col < m ? col : m - 1)];
      }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rt = b * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);    // row in the tile
      const int row = r64 * 64 + rt;
      if (pa.to_scratch) {
        const int64_t tile = static_cast<int64_t>(slice) * pa.nt * pa.nt + r64 * pa.nt + tb;
        pa.scratch[tile * 4096 + rt * 64 + (col - tb * 64)] = v[b][r];
      } else if (row < m && col < m) {
        pa.S[static_cast<int64_t>(row) * m + col] = v[b][r];
      }
    }
}

hipError_t launch_digit_product(const ProductArgs& a, hipStream_t st, hipEvent_t e0) {
  if (a.ts != 64 || a.ksl % 32 != 0 || a.ksl > kDigitMaxK) return hipErrorInvalidValue;
  const int nbP = (a.m + 127) / 128 * 4, nbQ = (a.m + 63) / 64 * 2;
  const int KS = (a.n2 + 31) / 32;
  FPSK_LAUNCH_TIMED(channel_kernel, dim3((a.n2 + 127) / 128), dim3(kThreads), 0, st, e0, nullptr, a);
  const dim3 rows(2 * a.m), block(kThreads);
  if (a.kact <= 4 * 4 * kThreads) {
    FPSK_LAUNCH(row_scale_kernel<4>, rows, block, 0, st, a);
  } else if (a.kact <= 16 * 4 * kThreads) {
    FPSK_LAUNCH(row_scale_kernel<16>, rows, block, 0, st, a);
  } else {
    FPSK_LAUNCH(row_scale_kernel<0>, rows, block, 0, st, a);
  }
  FPSK_LAUNCH(digits_kernel, dim3((KS + 3) / 4, nbP + nbQ), dim3(kThreads), 0, st, a, nbP);
  const int wgs = (a.m + 127) / 128 * ((a.m + 63) / 64) * a.NS;
  FPSK_LAUNCH(digit_product_kernel, dim3((wgs + 7) / 8 * 8), dim3(kThreads), 0, st, a, a.zero);
  return hipSuccess;
}

}  // namespace fpsk
