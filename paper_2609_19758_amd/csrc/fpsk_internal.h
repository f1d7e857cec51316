// Internal interface between the host library and the gfx950 kernels of the FP-Sketch verifier.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace fpsk {

constexpr int kThreads = 256;          // work-group size of every kernel (4 wave64)
constexpr int kColTile = 512;          // columns per A or C tile: 64 lanes x 8 elements
constexpr int kWideCols = 8192;        // columns per step of the C and B sides at m > 1024
constexpr int kBChunkHalfs = 16384;    // halfs of B staged in LDS per chunk (32 KiB)
constexpr int kMaxM = 4096;            // largest bucket count the kernels accept
constexpr double kHugeLimit = 3.4028234663852886e38 / 16.0;   // fp32max / 16
// block product of the probe (m <= 64)
constexpr int kDigitMinK = 512;          // smallest n2, and k per slice, of the digit product
constexpr int kDigitMaxK = 16384;        // k per slice at most: 32-bit sums of 4 products, 4 2^14 k < 2^31
constexpr int32_t kNoDigits = 0x7fffffff;
constexpr int kXSlice = 4096;            // k per block-product work-group
constexpr int kMaxXSlices = 4;           // n2 <= kMaxXSlices * kXSlice

// One pass over A, B and C producing the factors of Eq. 1 (and their weighted forms).
struct StreamArgs {
  const uint16_t* A;          // n1 x n2 half bits
  const uint16_t* B;          // n2 x n3 half bits, or with transb its transpose W (n3 x n2)
  const float* C;             // n1 x n3
  int64_t n1, n2, n3;
  int m;
  // row side: per bucket a, its rows at perm[a * cap + i] (ascending) as row | (v1 < 0) << 31,
  // padded to cap entries with -1
  const int32_t* perm;
  int cap;
  // transb: B is passed as W = B^T (n3 x n2 row-major) and the nB B work-groups are row-bucket
  // work-groups over W's rows (m x TA of them, like A's), with the column lists perm2 / cap2
  // (per bucket b its columns j ascending as j | (v2 < 0) << 31, natural bucket order)
  int transb;
  const int32_t* perm2;
  int cap2;
  // C column tiles of kColTile (kWideCols at m > 1024): per tile (ctab_stride entries), columns sorted by bucket as
  // (offset in tile) | (v2 < 0) << 15, with coff[t * (m + 1) + b] segment starts; for m <= 256
  // each segment is padded to a multiple of 8 with the sentinel offset kColTile (a zero column)
  const uint16_t* ctab;
  const int32_t* coff;
  // B column chunks of cwb columns: sorted lists without signs (the signs v2(j) are applied when
  // a chunk is staged, from the bit mask bsign: bit j % 8 of byte j / 8); entries are the
  // column offset with moments, else the column's staged LDS slot (sentinel cwb)
  const uint8_t* bsign;
  const uint16_t* btab;
  const int32_t* boff;
  int cwb;
  int ctab_stride, btab_stride;
  int tab_off;                // byte offset of the staged column list in dynamic LDS
  // outputs
  // factors, row stride ldp >= n2 (a multiple of 4; entries past n2 are kept at zero)
  float* P;        // m x ldp      H1 A
  float* Pw;       // m x ldp      H1 W1 A            (moments only)
  float* Q;        // m x ldp      (B H2^T)^T: row b holds column b of B H2^T
  float* Qw;       // m x ldp      (B W2 H2^T)^T      (moments only)
  int ldp;
  double* partS;   // npc x m x m  partial H1 C H2^T over column-tile groups
  double* partR;   // npc x m x m  partial H1 W1 C H2^T
  double* partT;   // npc x m x m  partial H1 C W2 H2^T
  float* maxpart;  // nA + nB: max |A| per A work-group, then max |B| per B work-group
  // C entries replaced while sketching (absolute entries): CSR by row, may be null
  const int32_t* patch_rowptr;
  const int32_t* patch_col;
  const float* patch_val;
  // decomposition
  int nA, nB, nC;
  // dispatch order after the C work-groups: A then B when an A work-group reads at least as many
  // bytes as a B work-group (the smaller ones last, where they fill the tail), else B then A
  int a_first;
  int TA, TC, TB;
  int npc, tg;
  // small buckets: row-bucket work-groups of four tiles, one per wave (A side; W side with
  // transb), m x ceil(TA / 4) of them
  int wt_a, wt_w;
  // C work-groups with one column tile per wave, four tiles at a time (256 < m <= 1024, or probes
  // with B as stored at 48 < m <= 192; buckets of at most 32 rows, at least 4 tiles)
  int wt_c;
  // the 4-row probe B work-groups of the one-tile-per-wave instances start at chunk
  // (row block mod TB) and wrap (n3 a whole number of chunks, TB > 1)
  int rot_b;
  double inv_l1, inv_l3;      // 1 / 2^ceil(log2 n1), 1 / 2^ceil(log2 n3)
  int vec_a, vec_b, vec_c;    // rows are whole aligned 16-byte groups
  const void* zero;           // >= 64 bytes of zeros (read in place of invalid rows or lanes)
};

// Bucket-space product S = P Q - S_C (and R = Pw Q - R_C, T = P Qw - T_C), plus the probe
// decision.
struct ProductArgs {
  const float* P;
  const float* Pw;
  const float* Q;
  const float* Qw;
  const double* partS;
  const double* partR;
  const double* partT;
  double* S;
  double* R;
  double* T;
  double* scratch;      // NS x tiles x ts^2 (x 3 with moments) slice partials, row-major tiles
  double* tilestat;     // tiles x 4: sum|S|, max|S|, non-finite count, clipped sum
  int m, n2, nt, NS, ksl, npc;
  int ldp;              // row stride of the factors
  int kact;             // k-range the products cover: n2 rounded up to a multiple of 4
  int mode;             // 0: sketch only; 1: probe decision
  int ts;               // tile edge of the tile path
  int clip_tiles;       // probe, large m: clip_kernel writes each tile's clipped sum to
                        // tilestat[4 tile + 3] and the decision adds those
  const float* maxpart;
  int nA, nB;
  const float* maxpart_b; // max |B| per B work-group when the B side is cached, else null
  double* stats;        // [8] sigma_hat, thr, tau, max|S|, finite, dirty, max|A|, max|B|
  int32_t* d_dirty;     // caller's flag (may be null)
  double* sigma_acc;    // [2] running sum of clean sigma_hat, count
  double mu, c_valid;
  double lim_factor;    // mu sqrt(2 ln m^2): the noise limit in units of sigma_hat
  // probe with m <= 64 (nX > 0): nX = xnb^2 xns block-product work-groups of xb x xb outputs
  // over k-slices of kXSlice, their partials in xpart (xns x m x m, slice 0 minus the C grid)
  int nX, xb, xnb, xns;
  // S alone on 64 x 64 tiles (i8): the factors as 8-bit digits on the integer matrix cores, tiles
  // with a row that does not fit them on the FP64 ones (fpsk_digits.hip)
  int i8;
  // 2 m + 2: scale exponent of every row of P, then of Q (kNoDigits where not), then for
  // either whether any row has one
  int32_t* rexp;
  int8_t* bal;            // per k, padded to 128: balancing exponent and weight (fpsk_digits.hip)
  int16_t* weight;
  int32_t* wtop;          // per 128 k: largest weight, sum relative to it
  float* wsum;
  uint32_t* digP;         // digit fragments of P (rows padded to 128) and Q (to 64)
  uint32_t* digQ;
  const void* zero;       // >= 64 bytes of zeros
  int to_scratch;         // tile partials go to the scratch for reduce_kernel
  // launch index i -> slot (i mod 8) nX / 8 + i / 8; xslots slots per slice, in supertiles of
  // xsr x xsc blocks, xnstc supertiles per row of blocks (slots past the grid are idle)
  int xsr, xsc, xnstc, xslots;
  double* xpart;
};

// Tables of one hash round, built on the device.
struct ColTable {       // column tiles of W columns, their lists sorted by bucket
  uint16_t* tab;        // tiles x stride
  int32_t* off;         // tiles x (m + 1) segment starts
  int tiles, W, stride;
  int pad;              // segments padded to this multiple with the sentinel W
  int format;           // entries: 0 offset | negative sign << 15, 1 offset, 2 staged LDS slot
};
struct TableArgs {
  uint64_t key1, key2;  // streams of the rows' and the columns' hashes
  int64_t n1, n3;
  int64_t pad1, pad3;   // padded to multiples of 8 (pad3 also to whole sign bytes of the chunks)
  int m;
  uint16_t* hb1;        // pad1, pad3 words: bucket | negative sign << 15, 0x7fff past the end
  uint16_t* hb2;
  int32_t* slot;        // null: lists in bucket order; else scratch for the order by size
  int32_t* perm;        // m x cap
  int cap;
  int32_t* perm2;       // m x cap2 (null: none)
  int cap2;
  uint8_t* bsign;       // column signs as bits
  int64_t nsign;        // columns they cover, a multiple of 8 (0: none)
  ColTable c, b;
};
hipError_t launch_tables(const TableArgs& a, hipStream_t st);

// e0 / e1 (may be null): events that the first / last dispatch of the call records its
// start / end time in.
// Pipelined probe launch (m <= 64, block path): the decision of `dec` (if has_dec), the nprod
// block products of `prod` and the stream pass of `s` (which may be empty: nA = nB = nC = 0).
// lds_bytes covers the stream pass and probe_pipe_lds(xb).
size_t probe_pipe_lds(int xb);
// The digit product's launches: row scales, digit fragments, the product of every tile they fit.
hipError_t launch_digit_product(const ProductArgs& a, hipStream_t st, hipEvent_t e0);
hipError_t launch_probe_pipe(const StreamArgs& s, const ProductArgs& prod, const ProductArgs& dec,
                             int nprod, int has_dec, int dt, int xb, size_t lds_bytes,
                             hipStream_t st, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// The C and B sides for m > 1024 (fpsk_wide.hip).
hipError_t launch_wide_c(const StreamArgs& s, bool mom, hipStream_t st, hipEvent_t e0,
                         hipEvent_t e1);
hipError_t launch_wide_b(const StreamArgs& s, int dt, bool mom, hipStream_t st, hipEvent_t e0,
                         hipEvent_t e1);
hipError_t launch_stream(const StreamArgs& s, int dt, bool moments, int rb, int g, int ng,
                         size_t lds_bytes, hipStream_t st, hipEvent_t e0 = nullptr,
                         hipEvent_t e1 = nullptr);
// ts, kw: product tile edge and whether its k-range is split over the 4 waves
hipError_t launch_product(const ProductArgs& a, int ts, bool kw, bool moments, hipStream_t st,
                          hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// Entries of the exact scan as a patch list (at most keep of them), device memory except host_*.
struct AbsArgs {
  int64_t n1;
  int32_t keep;
  const int32_t* counts;   // n1
  int32_t* rowptr;         // n1 + 1
  int32_t* rows;           // keep rows that hold entries, and each one's first entry
  int32_t* base;
  int32_t* nrows;
  int64_t* coords;         // keep pairs
  double* gamma;           // keep
  double* abssum;
  int32_t* col;
  float* val;
  int64_t* host_coords;
  double* host_gamma;
};
hipError_t launch_abs_list(const AbsArgs& g, const uint16_t* A, const uint16_t* B, int64_t bsk,
                           int64_t bsj, const float* C, int64_t n2, int64_t n3, int dt,
                           hipStream_t st);
// B[k][j] is read at B + k * bsk + j * bsj (n3, 1 for B as stored; 1, n2 for W = B^T).
hipError_t launch_recheck(const uint16_t* A, const uint16_t* B, int64_t bsk, int64_t bsj,
                          const float* C, int64_t n2, int64_t n3, int dt, const int64_t* coords,
                          int n, double* gamma, double* abssum, float* cval, hipStream_t st);

// Order statistics on the device (the MAD of a localize round, the median inside rms-hat).  The
// selection state lives in device memory; histograms are zero between selections.
constexpr int kSelSmall = 1 << 14;       // keys that one work-group selects from in one launch
constexpr uint32_t kSelGather = 1 << 16; // keys sharing two digits that are kept
struct SelState {
  uint64_t pref, k;          // first digit, rank within it
  uint64_t pref2, k2, cnt2;  // both digits, rank within them, keys that share them
  uint64_t count;            // keys selected from
  uint64_t next;             // smallest key above those sharing both digits
  uint64_t lo, not_hi;       // range of those when they are too many to keep
  uint32_t ncand;
  uint32_t pad;
  double med, mad;
  double sigma, tau, cut;    // the round's noise, analytic threshold and candidate cut
};
struct SelArgs {
  const double* S;       // the bucket grid (n values) ...
  float* samp;           // ... or the samples C[i stride], i < n
  const float* C;
  int64_t stride, n;
  SelState* st;
  uint32_t* hist;        // 2 x 4096
  uint64_t* cand;        // kSelGather
  int dev;               // 1: |S - state->med| in place of S
  unsigned long long* clear;   // samples: a total that the first pass sets to zero (may be null)
  const double* need;          // samples: none counts when *need is zero (may be null)
};
// Figures of a localize step in host memory (written by a kernel, read after the stream is
// waited for).
struct HostHead {
  double rms;            // rms-hat(C)
  double sigma, extra;   // the round's sigma_MAD; for the setup the words SetupArgs names
  double tau, cut;
  uint32_t found;        // buckets above the cut; for the setup entries of the exact scan
  uint32_t pad;
};
struct PeelEntry {     // S[o] -= ds, R[o] -= dr, T[o] -= dt
  int64_t o;
  double ds, dr, dt;
};
struct Cand {          // a bucket above the cut with its three sketches
  int64_t o;
  double s, r, t;
};
struct RoundArgs {
  const float* maxpart;
  int nA, nB;
  double c_n2;           // c n2 2^-23
  double mx;             // max(n1, n3)
  double radius;         // max(r, 0.5)
  const PeelEntry* peel; // subtracted first (may be null), in host memory; copied to peel_dev
  PeelEntry* peel_dev;
  int npeel;
  Cand* cands;           // buckets above the cut in any order, at most cap of them (at least
  uint32_t cap;          // kSelSmall fit)
  uint32_t* count;       // their number, which may exceed cap
  HostHead* head;        // may be null
};
struct SetupArgs {
  // exact scan of C (n1 x n3): entries of each row, and their total (null: no scan)
  const float* C;
  int64_t n1, n3;
  int32_t* counts;
  unsigned long long* found;
  const double* sigma;   // two doubles to publish (may be null)
  int need;              // 1: rms-hat only where the second of them is not zero
  HostHead* head;
};
// Moment sketches R, T at a list of n buckets o (launch_moments_at): the factors (rows ldp
// apart, zero from n2 to kact), the npc C-grid partials of R and T, the peel list.
struct MomentsAtArgs {
  const float* P;
  const float* Pw;
  const float* Q;
  const float* Qw;
  const double* partR;
  const double* partT;
  const PeelEntry* peel;
  int m, ldp, kact, npc, npeel;
  // either a list of buckets and outputs r, t ...
  const int64_t* o;
  double* r;
  double* t;
  // ... or the *count candidates the device found, written whole to out (host memory) with their
  // number in head->found; nothing is formed when there are more than the launch's n
  const Cand* cands;
  const uint32_t* count;
  Cand* out;
  HostHead* head;
};
hipError_t launch_moments_at(const MomentsAtArgs& g, int n, hipStream_t st);
struct ApplyEntry {    // one record of the apply step: C[o] <- d, or C[o] + d (in host memory)
  int64_t o;
  double d;
  int32_t absolute;
  int32_t pad;
};
// Matrices of fewer than 8 elements, copied into zero-padded slots of 16 halfwords so that the
// stream pass's 8-element loads stay inside: halfwords[b] (0: not copied) of src[b] to slot b.
struct PadTinyArgs {
  const uint16_t* src[3];
  int halfwords[3];
  uint16_t* dst;
};
hipError_t launch_pad_tiny(const PadTinyArgs& a, hipStream_t st);
hipError_t launch_publish_stats(const double* stats, double* out, hipStream_t st);
hipError_t launch_apply(float* C, const ApplyEntry* list, int n, hipStream_t st);
// Zeroes device memory: bytes at p, both multiples of 4.
hipError_t launch_zero(void* p, size_t bytes, hipStream_t st);
// Zeroes columns [c0, c1) of rows x ld FP32 rows (c1 <= ld).
hipError_t launch_zero_cols(float* base, int rows, int ld, int c0, int c1, hipStream_t st);
// A round's decisions on its grid S[0 .. n): the peel, the median and MAD (even counts: the mean
// of the two middle order statistics; NaN orders above +inf), the cut, and the buckets above it.
hipError_t launch_round_cut(const SelArgs& a, const RoundArgs& r, hipStream_t st);
// rms-hat of C from its n samples, the exact scan's counts, and what else the host reads with them.
hipError_t launch_rms(const SelArgs& a, const SetupArgs& u, hipStream_t st);
// The recheck of n search windows of radius r <= kMaxWinR around centers (i, j): outputs
// [center][di][dj], those outside C left alone.  part: window_slices(n2, n) n (2r + 1)^2 pairs.
constexpr int kWinRows = 3;
constexpr int kMaxWinR = 31;
struct WindowArgs {
  const uint16_t* A;
  const uint16_t* B;
  int64_t bsk, bsj;       // B[k][j] at B + k bsk + j bsj
  const float* C;
  int64_t n1, n2, n3;
  const int64_t* centers; // n pairs; these and the outputs may be host memory
  int n, r;
  double* part;
  double* gamma;
  double* abssum;
  float* cval;
  int jl;                 // lanes per row of B and k per slice (set by the launcher)
  int64_t ks;
};
int window_slices(int64_t n2, int n);
hipError_t launch_windows(const WindowArgs& g, int dt, hipStream_t st);
hipError_t launch_read(const void* src, int64_t bytes, uint32_t* out, int grid, hipStream_t st);
hipError_t launch_copy(const void* src, void* dst, int64_t bytes, int grid, hipStream_t st);

}  // namespace fpsk
