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
//   - a row takes part when its quantum u adds at most about a quarter of the FP32 rounding to S:
//     u^2 / 12 sum_k s_k^2 <= 1/15 2^-50.7 sum_k (x_k s_k)^2, s_k the channel's typical size in the
//     other factor (equal for both after the scaling), 2^-50.7 the mean square of FP32 rounding
//     relative to the values.  A Gaussian row has a 50 times smaller left side, one with a channel 30
//     times the others' still a smaller one.  Rows that are not finite do not take part.
// The typical sizes are means of the exponents over 64 buckets a factor, zeros left out: the
// buckets are random sums of rows, and a mean of logarithms is not moved by a few rows of another
// scale.  Tiles with a row that takes no part are left to the FP64 matrix cores, whose kernel runs
// beside this one and takes only those.
//
// Error of S against 64 bits (rms over the noise), FP64 product and here: 2048 x 4096 x 2048,
// m = 260, BF16 0.002402 both, FP16 0.004215 both; 4096^3 BF16, m = 1000 0.001302 both; channels scaled
// by 1e-2 to 1e-6 as above likewise equal to four digits.
// (13 pairs, i + j <= 4, in 64 x 32 wave tiles of five accumulators were as fast and raised FP16
// errors by 0.1 %.)
//
// Bound by the integer matrix cores: 16 x 2 m^2 n2 operations at 1/64 of the FP64 cores' time each.
// 16384^3 FP16, m = 4096: FP64 8400 us -> 3655 us (product 3340, digits 175, row scales 131, channels
// 6), 2.6 x 10^15 operations a second of the 4.7 x 10^15 that registers alone reach; m = 698: 301 ->
// 187 us; 4096^3, m = 432: 43 us and 15 us of slice sums -> 40 and 8 us.
#include "fpsk_device.h"

namespace fpsk {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

// Channel figures: the power of two t that balances channel k (low byte), and the binary logarithm
// v of its typical size in both factors once balanced (high byte; kNoSize where a factor's sample
// holds only zeros).  A work-group takes 128 channels; a thread 4 of them in 8 of the 64 sampled rows
// of each factor.  A channel without a size in one factor is scaled out of the other: a row that
// has an entry there after all is then too far from its typical size to take part.
constexpr int kSampleRows = 64;
constexpr int kNoSize = -128;

__global__ __launch_bounds__(kThreads) void channel_kernel(ProductArgs pa) {
  constexpr int G = kThreads / 32;                   // row groups
  __shared__ uint32_t part[2][G][128];
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
  if (t < 128) {
    int ex[2];
    bool none[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      uint32_t n = 0;
#pragma unroll
      for (int i = 0; i < G; ++i) n += part[f][i][t];
      const int cnt = static_cast<int>(n >> 16);
      none[f] = cnt == 0;
      ex[f] = (static_cast<int>(n & 0xffffu) + cnt / 2) / (cnt > 0 ? cnt : 1) - 127;
    }
    int bal = (ex[1] - ex[0]) >> 1, v = (ex[0] + ex[1]) >> 1;
    bal = bal < -100 ? -100 : (bal > 100 ? 100 : bal);
    v = v < -127 ? -127 : v;
    if (none[0] || none[1]) {
      bal = none[0] == none[1] ? 0 : (none[0] ? 100 : -100);
      v = kNoSize;
    }
    pa.chan[blockIdx.x * 128 + t] =
        static_cast<uint16_t>((bal & 255) | (v & 255) << 8);
  }
  if (blockIdx.x == 0 && t == 0) pa.rexp[2 * pa.m] = pa.rexp[2 * pa.m + 1] = 0;
}

__device__ __forceinline__ int chan_bal(uint32_t c) { return static_cast<int8_t>(c & 255u); }
__device__ __forceinline__ int chan_size(uint32_t c) { return static_cast<int8_t>((c >> 8) & 255u); }

// Scale exponent e of each row (2m work-groups: rows of P, then of Q): the balanced row times 2^e
// rounds to integers whose four signed digits exist, |x 2^e| <= 2^31 - 2^24; kNoDigits for a row
// that takes no part.  rexp[2m], rexp[2m + 1]: whether any row of P, of Q does.
__global__ __launch_bounds__(kThreads) void row_scale_kernel(ProductArgs pa) {
  __shared__ uint32_t smax[kThreads / 64];
  __shared__ double sen[kThreads / 64], sws[kThreads / 64];
  const int r = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const bool second = r >= pa.m;
  const float* x = second ? pa.Q + static_cast<int64_t>(r - pa.m) * pa.ldp
                          : pa.P + static_cast<int64_t>(r) * pa.ldp;
  const int sg = second ? -1 : 1;
  uint32_t mx = 0;                          // bits of the largest magnitude (NaN above infinity)
  double en = 0.0, ws = 0.0;                // sums of (x s)^2 and s^2
#pragma unroll 4
  for (int k = 4 * t; k < pa.kact; k += 4 * kThreads) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(x + k);
    const u32x2 c = *reinterpret_cast<const u32x2*>(pa.chan + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t ce = c[e >> 1] >> (16 * (e & 1));
      const float xs = ldexpf(v[e], sg * chan_bal(ce));
      const uint32_t b = __float_as_uint(xs) & 0x7fffffffu;
      mx = b > mx ? b : mx;
      // s^2 = 2^(2 size), zero for a channel without a size
      const int size = chan_size(ce);
      const uint32_t hi = size == kNoSize ? 0u : static_cast<uint32_t>(1023 + 2 * size) << 20;
      const double s2 = __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32);
      const double xd = static_cast<double>(xs);
      en = fma(xd * xd, s2, en);
      ws += s2;
    }
  }
  mx = wave_max_u32(mx);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    en += __shfl_xor(en, d, 64);
    ws += __shfl_xor(ws, d, 64);
  }
  if (lane == 0) {
    smax[w] = mx;
    sen[w] = en;
    sws[w] = ws;
  }
  __syncthreads();
  if (t != 0) return;
  for (int i = 1; i < kThreads / 64; ++i) {
    mx = smax[i] > mx ? smax[i] : mx;
    en += sen[i];
    ws += sws[i];
  }
  int e = kNoDigits;
  const float big = __uint_as_float(mx);
  if (mx == 0) {
    e = 0;
  } else if (mx < 0x7f800000u && big >= 0x1p-120f && ws > 0.0) {
    int ex;
    const float f = frexpf(big, &ex);              // big = f 2^ex, 0.5 <= f < 1
    const int q = f <= 1.0f - 0x1p-7f ? 31 - ex : 30 - ex;
    // quantum 2^-q: ws 2^(-2q) / 12 <= en 2^-50.7 / 15 (a channel without a size has no part in en,
    // so that a NaN or an infinity there is seen in mx only)
    if (ldexp(en, 2 * q - 51) >= ws) e = q;
  }
  pa.rexp[r] = e;
  // (every work-group that does stores the same word: no atomic, which cost 10 ns a row here)
  if (e != kNoDigits) pa.rexp[2 * pa.m + (second ? 1 : 0)] = 1;
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
  const u32x4* ch = reinterpret_cast<const u32x4*>(pa.chan + k);
  f32x4 v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = reinterpret_cast<const f32x4*>(x)[j];
  const u32x4 c[2] = {ch[0], ch[1]};
  u32x4 d[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int bal = chan_bal(c[j >> 1][2 * (j & 1) + (i >> 1)] >> (16 * (i & 1)));
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
  FPSK_LAUNCH(row_scale_kernel, dim3(2 * a.m), dim3(kThreads), 0, st, a);
  FPSK_LAUNCH(digits_kernel, dim3((KS + 3) / 4, nbP + nbQ), dim3(kThreads), 0, st, a, nbP);
  const int wgs = (a.m + 127) / 128 * ((a.m + 63) / 64) * a.NS;
  FPSK_LAUNCH(digit_product_kernel, dim3((wgs + 7) / 8 * 8), dim3(kThreads), 0, st, a, a.zero);
  return hipSuccess;
}

}  // namespace fpsk
