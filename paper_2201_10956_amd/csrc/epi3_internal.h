// Internal declarations shared by the HIP translation units of libepi3.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "epi3.h"

namespace epi3 {

constexpr int kWave = 64;        // CDNA wavefront width
constexpr int kSnpPad = 64;      // plane arrays hold roundup(M, 64) + 64 SNP slots
constexpr int kHistBins = 2048;  // radix-select bins per pass
constexpr int kHistPasses = 3;   // 3 x 11 bits >= 32-bit keys
// Sampled first bound: every kSampleStride-th block of kSampleBlock scores.
constexpr int kSampleBlock = 1024;
constexpr int kSampleStride = 32;
// Whether a selection over T scores for k hits starts from the sampled bound
// (the sample must hold comfortably more than k scores).
inline bool sample_select(int64_t T, int64_t k) { return T >= (1ll << 22) && k * 512 <= T; }

// Copies n words of a log-factorial table (16-byte aligned) to LDS with all
// threads of the workgroup, four 16-byte loads in flight per thread (one word
// per step waits for memory once per 256 words: with it a 2048 x 16384 pair
// scan takes 235 us instead of 228).
template <int THREADS>
__device__ __forceinline__ void table_to_lds(uint32_t *dst, const uint32_t *src, int n) {
  const uint4 *s4 = reinterpret_cast<const uint4 *>(src);
  uint4 *d4 = reinterpret_cast<uint4 *>(dst);
  const int n4 = n >> 2;
  int x = threadIdx.x;
  for (; x + 3 * THREADS < n4; x += 4 * THREADS) {
    const uint4 a = s4[x], b = s4[x + THREADS], c = s4[x + 2 * THREADS], d = s4[x + 3 * THREADS];
    d4[x] = a;
    d4[x + THREADS] = b;
    d4[x + 2 * THREADS] = c;
    d4[x + 3 * THREADS] = d;
  }
  for (; x < n4; x += THREADS) d4[x] = s4[x];
  if ((int)threadIdx.x < n - 4 * n4) dst[4 * n4 + threadIdx.x] = src[4 * n4 + threadIdx.x];
}

// Pointer into the constant address space: uniform loads through it become
// scalar (s_load) instructions.  Only used for memory no kernel writes while
// the reading kernel runs.
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;

template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T *p) {
  return (cptr<T>)p;
}

__host__ __device__ __forceinline__ int64_t c2(int64_t x) { return x < 2 ? 0 : x * (x - 1) / 2; }
__host__ __device__ __forceinline__ int64_t c3(int64_t x) {
  return x < 3 ? 0 : x * (x - 1) / 2 * (x - 2) / 3;
}

// Lexicographic rank of the pair (i, j), i < j < M.
__host__ __device__ __forceinline__ int64_t pair_rank(int64_t M, int64_t i, int64_t j) {
  return c2(M) - c2(M - i) + (j - i - 1);
}
// Lexicographic rank of i < j < k < M among all triplets, less k.
__host__ __device__ __forceinline__ int64_t lex_base(int64_t M, int64_t i, int64_t j) {
  return c3(M) - c3(M - i) + c2(M - 1 - i) - c2(M - j) - j - 1;
}

// Order-preserving map of a float to an unsigned key (and back).
__host__ __device__ __forceinline__ uint32_t f2key(float f) {
  uint32_t b;
  __builtin_memcpy(&b, &f, 4);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__host__ __device__ __forceinline__ float key2f(uint32_t k) {
  uint32_t b = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  float f;
  __builtin_memcpy(&f, &b, 4);
  return f;
}

// One scan job as seen by the count kernels: a SPLIT data set, its score
// plane and its share of the global tile queue.
struct Job {
  const uint32_t *planes;  // [W0 + W1][Mp][2]
  const int32_t *pairs;    // [2][Mp][Mp][4]
  float *score;            // [T] FP32 K2 by lexicographic rank
  const int64_t *jprefix;  // [M + 1] job-local tiles before pivot j
  uint32_t *counts;        // optional [T][2][27]
  uint32_t *keyrange;      // [2] atomic min / max of f2key(score)
  int64_t tile_begin;      // first global tile of this job
  int64_t n_tiles;
  int64_t T;
  const uint32_t *lfx;     // fixed-point log factorials (fx_table), lf_len entries
  float scale;             // 2^-fx_shift: fixed-point score to nats
  int32_t lf_len;
  int32_t M, Mp, W0, W1, N0, N1;
  int32_t P;               // pivots i per tile (4 or 8)
  int32_t pad;
};

// Key window of a radix-select pass.
struct SelWindow {
  uint64_t krem;           // 1-based rank of the k-th key inside the window
  uint32_t lo, whi;        // first and last key
  int32_t shift;           // bin width of the pass = 1 << shift
  uint32_t done;           // 1: collapsed to the k-th key; 2: nothing to select; 3: list overflowed
  uint32_t kth;            // done = 1: key of the k-th smallest score
  uint32_t pad;
};

// Per-job radix-select state.
struct SelState {
  uint32_t kmin, kmax;     // key range of the score plane (written by the count kernel)
  uint32_t done;           // 1: candidates collected; 2, 3 as SelWindow
  uint32_t kth;            // key of the k-th smallest score
  float thr;               // candidate threshold (FP32, rounded up)
  uint32_t pending;        // left to the kernels after tail_kernel, from window `rest`
  uint32_t overflow;       // candidates beyond capacity
  unsigned long long ncand;
  int64_t keff;            // min(k, T)
  int64_t T;
  int32_t k;
  float ub;                // compaction bound: last key of the first window + 2 e(N), as float
  uint32_t cmode;          // 1 once the compaction pass ran
  uint32_t pad;
  unsigned long long cn;   // keys <= ub found by the compaction pass
  SelWindow win[kHistPasses], rest;  // windows of the passes over a plane or its sample
};
static_assert(sizeof(SelState) <= 256, "one 256-byte unit of a workspace");

// One scored candidate.
struct CandRec {
  uint64_t key;            // bit pattern of the FP64 K2 (non-negative => ordered)
  int64_t rank;            // lexicographic rank (tie-break)
  uint32_t i, j, k, l;
  float k2f;
  double k2;
  uint32_t counts[162];     // [class][cells]: 27 (triplets), 9 (pairs) or 81 (quads) per class
};

// Phenotype batch for the matrix-core kernel: one MASKED data set and up to
// 64 phenotypes (case masks).
struct PermJob {
  const uint8_t *bytes;       // [Mp][2][S] 0/1 genotype values (bytes, or E2M1 nibbles)
  const uint8_t *ph;          // [64][S] 0/1 case values per phenotype (same format)
  const int32_t *tot_pairs;   // [Mp][Mp][4] pairwise tables over all samples
  const int32_t *case_pairs;  // [Mp][Mp][Qp] uint2 (n00 | n01 << 16, n10 | n11 << 16): pairwise tables
                              // over each phenotype's cases (y >= x)
  const int32_t *n1;          // [Qp] cases per phenotype
  float *score;               // [Q][T]
  const int64_t *jprefix;     // [M + 1]
  uint4 *corners;             // scratch: [pass tile][4 pivots i][16 k][64 q] 8 x uint16 case cells
  uint4 *totals;              // scratch: [pass tile][4 pivots i][16 k] 8 x uint16 all-sample cells
  int64_t n_tiles, T;
  int32_t M, Mp, S, N, Q, Qp;  // S: bytes per staged row (samples for bytes, samples / 2 for nibbles)
};

// Where the phenotype-batch finish kernel puts its FP32 scores.
enum { kPermOutPlane = 0, kPermOutSample = 1, kPermOutBounded = 2 };
struct PermOut {
  int32_t mode;          // kPermOut*
  int32_t pad;
  // sample: the launch's tiles are sample tiles sample_base + n; the score of
  // slot s (= 16 wave + kk) of sample tile m of phenotype q goes to
  // sample[q * sample_T + 64 m + s] (invalid slots keep what the buffer held)
  float *sample;
  int64_t sample_T;
  int64_t sample_base;
  // bounded: phenotype q appends (key, rank) of every score <= st[q].ub to
  // ckey / crank [q * ccap + pos], pos from st[q].cn
  uint32_t *ckey;
  int64_t *crank;
  int64_t ccap;
};

// Where the plain matrix-core finish kernel puts its FP32 scores (modes as
// for PermOut).  The launch's slots q are global tiles tile_begin + q stride.
struct PlainOut {
  int32_t mode;          // kPermOut*
  int32_t pad;
  int64_t stride;
  // sample: the score of triplet x (0 .. 4095, the tile's triplet order) of
  // slot q goes to sample[(sample_base + q) 4096 + x] (slots of no triplet
  // keep what the buffer held); its key range to range[0..1]
  float *sample;
  int64_t sample_base;
  uint32_t *range;
  // bounded: (key, rank) of every score <= st->ub appended to ckey / crank at
  // positions from st->cn (entries past ccap are dropped, st->cn still counts)
  SelState *st;
  uint32_t *ckey;
  int64_t *crank;
  int64_t ccap;
};

// Plain two-class scan on the matrix cores: one SPLIT data set, counted in
// passes of tiles whose corner cells go through a scratch buffer
// ([pass tile][class][16 i][JB j][256 / JB k] 8 x uint16 cells).
struct PlainJob {
  const uint8_t *vals;     // [2][Mp][2][Sb] 0/1 values per class (bytes, or E2M1 nibbles)
  const int32_t *pairs;    // [2][Mp][Mp][4]
  float *score;            // [T] FP32 K2 by lexicographic rank
  uint32_t *counts;        // optional [T][2][27]
  uint32_t *keyrange;      // [2] atomic min / max of f2key(score)
  const int64_t *jprefix;  // [M + 1] tiles before pivot j
  int64_t n_tiles, T;
  const uint32_t *lfx;     // fixed-point log factorials (fx_table), lf_len entries
  float scale;             // 2^-fx_shift: fixed-point score to nats
  int32_t lf_len;
  int32_t M, Mp, Sb, Sb0, Sb1, N0, N1, JB;  // Sb: bytes per row; Sb0 / Sb1: bytes holding each class
};

// Selection job: one score plane plus its candidate buffers.
struct SelJob {
  const float *score;
  int64_t T;
  SelState *st;
  uint32_t *hist;          // [kHistBins] first pass
  uint32_t *hist2;         // [2][kHistBins] second and third; may lie over rec (used before it)
  int64_t *cand;           // [cap] ranks
  uint32_t *candkey;       // [cap] their FP32 score keys
  CandRec *rec;            // [cap]
  epi3_hit *hits;          // [k]
  int64_t cap;
  uint32_t *ckey;          // [ccap] keys of the compacted low end of the plane
  int64_t *crank;          // [ccap] their ranks
  int64_t ccap;
  double err2;             // 2 e(N)
  // data needed to recount a candidate
  const uint32_t *planes;
  const int32_t *pairs;    // [classes][Mp][Mp][4]; MASKED: totals at class 0
  const int32_t *case_pairs; // MASKED: case pairs (uint2, 16-bit counts) of the job's mask (pair (x,y) at
                             // uint2 index (x * Mp + y) * case_stride), else NULL
  const uint32_t *case_mask; // MASKED: [W] mask words, else NULL
  const int32_t *n1_dev;     // MASKED: device count of cases (overrides N1), else NULL
  int64_t case_stride;
  const double *lf64;
  int32_t M, Mp, W0, W1, N0, N1;
  int32_t layout;
  int32_t k;
  int32_t sample;          // 1: the first bound comes from a radix select on a sample (sample_select),
                           // or (score == NULL) from the batch's sample pass with the list already built
  int32_t order;           // 2: pairs (9-row tables, pair_hits); 4: quads (81 rows, quad_hits);
                           // else triplets
  epi3_pair_hit *pair_hits;  // [k] (order 2)
  epi3_quad_hit *quad_hits;  // [k] (order 4)
  // candidate capacities above kRankDirectMax order the candidates by a
  // bitonic sort of (FP64 key, index) pairs in these buffers of sortP entries
  // (a power of two >= cap) instead of counting, for each, the candidates
  // before it; sortP = 0 otherwise
  uint64_t *skey;
  uint32_t *sidx;
  int64_t sortP;
};

constexpr int64_t kRankDirectMax = 16384;
inline int64_t sort_len(int64_t cap) {
  if (cap <= kRankDirectMax) return 0;
  int64_t p = 1;
  while (p < cap) p <<= 1;
  return p;
}

// Two 16-bit counts of one register, added and subtracted as a pair: exact
// modulo 2^16, and every completed count is below that.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_u16x2(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ uint32_t as_u32(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// The 9 cells t[3 a + b] of one class of a pair (a, b in {0, 1, 2}) from the
// counted cells n[2 a + b] (a, b in {0, 1}), the per-SNP counts mi[a], mj[b]
// and the class size: every sample of the class is in exactly one row.
// V: int, or two counts per register (u16x2).
template <typename V>
__device__ __forceinline__ void pair_cells(const V n[4], const V mi[2], const V mj[2], V Nc, V t[9]) {
  t[0] = n[0];
  t[1] = n[1];
  t[3] = n[2];
  t[4] = n[3];
  t[2] = mi[0] - n[0] - n[1];
  t[5] = mi[1] - n[2] - n[3];
  t[6] = mj[0] - n[0] - n[2];
  t[7] = mj[1] - n[1] - n[3];
  t[8] = (Nc - mi[0] - mi[1]) - t[6] - t[7];
}

// The 27 cells of one class from the 8 counted corner cells n[4a + 2b + c]
// (a, b, c in {0, 1}), all nine cells of the pair table (j, k) (fjk[3b + c]),
// the {0, 1}^2 cells of the pair tables (i, j) and (i, k) (pij[2a + b],
// pik[2a + c]) and the two cells pij2[a] = (a, 2) of (i, j).  Every sample of
// the class is in exactly one row, so a cell with genotype 2 at a SNP is the
// lower-order cell without that SNP minus the rows with 0 and 1 there: two
// subtractions for each of the 19.  (j, k) carries the full table because
// callers walk i with j and k held, so its five derived cells leave the loop.
// V: int, or two counts per register (u16x2).
template <typename N, typename V>
__device__ __forceinline__ void complete27(const N n[8], const V fjk[9], const V pij[4],
                                           const V pij2[2], const V pik[4], V t[27]) {
#pragma unroll
  for (int a = 0; a < 2; ++a) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int c = 0; c < 2; ++c) t[9 * a + 3 * b + c] = (V)n[4 * a + 2 * b + c];
#pragma unroll
    for (int b = 0; b < 2; ++b)
      t[9 * a + 3 * b + 2] = pij[2 * a + b] - t[9 * a + 3 * b] - t[9 * a + 3 * b + 1];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      t[9 * a + 6 + c] = pik[2 * a + c] - t[9 * a + c] - t[9 * a + 3 + c];
    t[9 * a + 8] = pij2[a] - t[9 * a + 6] - t[9 * a + 7];
  }
#pragma unroll
  for (int x = 0; x < 9; ++x) t[18 + x] = fjk[x] - t[x] - t[9 + x];
}

// The same from the pair tables' {0, 1}^2 cells, the per-SNP counts mi[a],
// mj[b], mk[c] and the class size.
__device__ __forceinline__ void complete_table(const uint32_t n[8], const int pij[4],
                                               const int pik[4], const int pjk[4], const int mi[2],
                                               const int mj[2], const int mk[2], int Nc, int t[27]) {
  int fjk[9];
  pair_cells(pjk, mj, mk, Nc, fjk);
  const int pij2[2] = {mi[0] - pij[0] - pij[1], mi[1] - pij[2] - pij[3]};
  complete27(n, fjk, pij, pij2, pik, t);
}

// Counts of one class of the quad (i, j, k, l) over words [w0, w1) with
// stride `step` (one thread: 1; the lanes of a wave: 64 from w0 + lane):
// cnt[8 a + 4 b + 2 c + d] = sum popc(X_i[a] & X_j[b] & X_k[c] & X_l[d]),
// then the corner cells of the four sub-triplets, each indexed by its own
// (x, y, z) in {0, 1}^3 as 4 x + 2 y + z: cnt[16 + ...] (i, j, k),
// cnt[24 + ...] (i, j, l), cnt[32 + ...] (i, k, l), cnt[40 + ...] (j, k, l).
__device__ __forceinline__ void quad_counts(const uint32_t *planes, int64_t Mp, int w0, int w1,
                                            int step, int i, int j, int k, int l,
                                            uint32_t cnt[48]) {
#pragma unroll
  for (int x = 0; x < 48; ++x) cnt[x] = 0u;
  const uint2 *pv = reinterpret_cast<const uint2 *>(planes);
  for (int w = w0; w < w1; w += step) {
    const uint2 *row = pv + (int64_t)w * Mp;
    const uint2 xi = row[i], xj = row[j], xk = row[k], xl = row[l];
    const uint32_t X[4][2] = {{xi.x, xi.y}, {xj.x, xj.y}, {xk.x, xk.y}, {xl.x, xl.y}};
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const uint32_t ij = X[0][a] & X[1][b];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const uint32_t ijk = ij & X[2][c];
          cnt[16 + 4 * a + 2 * b + c] += __builtin_popcount(ijk);
#pragma unroll
          for (int d = 0; d < 2; ++d)
            cnt[8 * a + 4 * b + 2 * c + d] += __builtin_popcount(ijk & X[3][d]);
        }
#pragma unroll
        for (int d = 0; d < 2; ++d) cnt[24 + 4 * a + 2 * b + d] += __builtin_popcount(ij & X[3][d]);
      }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const uint32_t kl = X[2][c] & X[3][d];
#pragma unroll
        for (int a = 0; a < 2; ++a) cnt[32 + 4 * a + 2 * c + d] += __builtin_popcount(X[0][a] & kl);
#pragma unroll
        for (int b = 0; b < 2; ++b) cnt[40 + 4 * b + 2 * c + d] += __builtin_popcount(X[1][b] & kl);
      }
  }
}

// Only the 16 quad corner cells of quad_counts (cnt[0..15]).
__device__ __forceinline__ void quad_corner_counts(const uint32_t *planes, int64_t Mp, int w0, int w1,
                                                   int i, int j, int k, int l, uint32_t cnt[16]) {
#pragma unroll
  for (int x = 0; x < 16; ++x) cnt[x] = 0u;
  const uint2 *pv = reinterpret_cast<const uint2 *>(planes);
  for (int w = w0; w < w1; ++w) {
    const uint2 *row = pv + (int64_t)w * Mp;
    const uint2 xi = row[i], xj = row[j], xk = row[k], xl = row[l];
    const uint32_t X[4][2] = {{xi.x, xi.y}, {xj.x, xj.y}, {xk.x, xk.y}, {xl.x, xl.y}};
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const uint32_t ij = X[0][a] & X[1][b];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const uint32_t ijk = ij & X[2][c];
#pragma unroll
          for (int d = 0; d < 2; ++d)
            cnt[8 * a + 4 * b + 2 * c + d] += __builtin_popcount(ijk & X[3][d]);
        }
      }
  }
}

// The 81 cells t[27 a + 9 b + 3 c + d] (a, b, c, d in {0, 1, 2}) of one class
// of the quad (i, j, k, l) from its counts (quad_counts) and the class's
// pairwise tables pairs[x][y] (int4 (n00, n01, n10, n11), per-SNP counts on
// the diagonal) and size.  Each sub-triplet's 27 cells come from its corners
// (complete_table); then the rows with a 2 at SNP i, j, k, l in turn: a count
// with a 2 at one SNP is the sub-triplet table without that SNP minus the
// rows with 0 and 1 there (every sample of the class is in one row).
// SH scales every count by 2^SH (SH = 2: cells as byte offsets into an FP32
// table); cnt and Nc must come scaled alike, the pairwise tables are scaled here.
// ml_in: the per-SNP counts of SNP l already scaled (NULL: read from the
// pairwise table's diagonal).
template <int SH = 0>
__device__ __forceinline__ void quad_cells(const uint32_t cnt[48], const int32_t *pairs, int64_t Mp,
                                           int i, int j, int k, int l, int Nc, int t[81],
                                           const int *ml_in = nullptr) {
  const int4 *pr = reinterpret_cast<const int4 *>(pairs);
  auto pair = [&](int x, int y, int v[4]) {
    const int4 p = pr[(int64_t)x * Mp + y];
    v[0] = p.x << SH; v[1] = p.y << SH; v[2] = p.z << SH; v[3] = p.w << SH;
  };
  auto marg = [&](int x, int v[2]) {
    const int4 p = pr[(int64_t)x * Mp + x];
    v[0] = p.x << SH; v[1] = p.w << SH;
  };
  int pij[4], pik[4], pil[4], pjk[4], pjl[4], pkl[4], mi[2], mj[2], mk[2], ml[2];
  pair(i, j, pij); pair(i, k, pik); pair(i, l, pil);
  pair(j, k, pjk); pair(j, l, pjl); pair(k, l, pkl);
  marg(i, mi); marg(j, mj); marg(k, mk);
  if (ml_in) {
    ml[0] = ml_in[0];
    ml[1] = ml_in[1];
  } else {
    marg(l, ml);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int d = 0; d < 2; ++d) t[27 * a + 9 * b + 3 * c + d] = (int)cnt[8 * a + 4 * b + 2 * c + d];
  int T[27];
  // a = 2 (b, c, d in {0, 1}) from the (j, k, l) table
  complete_table(cnt + 40, pjk, pjl, pkl, mj, mk, ml, Nc, T);
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int d = 0; d < 2; ++d)
        t[54 + 9 * b + 3 * c + d] = T[9 * b + 3 * c + d] - t[9 * b + 3 * c + d] - t[27 + 9 * b + 3 * c + d];
  // b = 2 (c, d in {0, 1}) from the (i, k, l) table
  complete_table(cnt + 32, pik, pil, pkl, mi, mk, ml, Nc, T);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int d = 0; d < 2; ++d)
        t[27 * a + 18 + 3 * c + d] = T[9 * a + 3 * c + d] - t[27 * a + 3 * c + d] - t[27 * a + 9 + 3 * c + d];
  // c = 2 (d in {0, 1}) from the (i, j, l) table
  complete_table(cnt + 24, pij, pil, pjl, mi, mj, ml, Nc, T);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int d = 0; d < 2; ++d)
        t[27 * a + 9 * b + 6 + d] = T[9 * a + 3 * b + d] - t[27 * a + 9 * b + d] - t[27 * a + 9 * b + 3 + d];
  // d = 2 from the (i, j, k) table
  complete_table(cnt + 16, pij, pik, pjk, mi, mj, mk, Nc, T);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        t[27 * a + 9 * b + 3 * c + 2] = T[9 * a + 3 * b + c] - t[27 * a + 9 * b + 3 * c] - t[27 * a + 9 * b + 3 * c + 1];
}

// Lexicographic rank of the quad (i, j, k, l), i < j < k < l < M.
__host__ __device__ __forceinline__ int64_t c4(int64_t x) {
  return x < 4 ? 0 : x * (x - 1) / 2 * (x - 2) / 3 * (x - 3) / 4;
}
__host__ __device__ __forceinline__ int64_t quad_rank(int64_t M, int64_t i, int64_t j, int64_t k,
                                                      int64_t l) {
  return c4(M) - c4(M - i) + c3(M - 1 - i) - c3(M - j) + c2(M - 1 - j) - c2(M - k) + (l - k - 1);
}

// Triplet (i, j, k) of lexicographic rank `rank` among the triplets of M SNPs.
__device__ __forceinline__ void decode_rank(int64_t M, int64_t rank, int &i, int &j, int &k) {
  const int64_t C = c3(M);
  int lo = 0, hi = (int)M - 3;  // last i with first rank <= rank
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (C - c3(M - mid) <= rank) lo = mid; else hi = mid - 1;
  }
  i = lo;
  const int64_t r1 = rank - (C - c3(M - i));
  // within i: pivots j > i, each with M - 1 - j values of k
  int jl = i + 1, jh = (int)M - 2;
  while (jl < jh) {
    const int mid = (jl + jh + 1) >> 1;
    if (c2(M - 1 - i) - c2(M - mid) <= r1) jl = mid; else jh = mid - 1;
  }
  j = jl;
  k = (int)(rank - lex_base(M, i, j));
}

// Quad (i, j, k, l) of lexicographic rank `rank` among the quads of M SNPs.
__device__ __forceinline__ void decode_quad_rank(int64_t M, int64_t rank, int &i, int &j, int &k,
                                                 int &l) {
  const int64_t C = c4(M);
  int lo = 0, hi = (int)M - 4;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (C - c4(M - mid) <= rank) lo = mid; else hi = mid - 1;
  }
  i = lo;
  const int64_t r1 = rank - (C - c4(M - i));
  lo = i + 1;
  hi = (int)M - 3;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (c3(M - 1 - i) - c3(M - mid) <= r1) lo = mid; else hi = mid - 1;
  }
  j = lo;
  const int64_t r2 = r1 - (c3(M - 1 - i) - c3(M - j));
  lo = j + 1;
  hi = (int)M - 2;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (c2(M - 1 - j) - c2(M - mid) <= r2) lo = mid; else hi = mid - 1;
  }
  k = lo;
  l = (int)(r2 - (c2(M - 1 - j) - c2(M - k))) + k + 1;
}

// ---- tile slots of a persistent launch ----
// Slots are cut into 8 contiguous parts, one per XCD (workgroup b runs on XCD
// b mod 8), each with a cleared counter in queue[0..7].
// Workgroup b starts with slot b / 8 of its XCD's part; the counter hands out
// those after the ones started with.  (A workgroup may draw its next tile while
// it works on one: with every slot drawn, and no more tiles than workgroups,
// those launched first took two tiles each and the last ones none: whole scan
// 135 -> 121 us at 157 x 2311, 238 -> 227 at 300 x 3000.)  Once a part is used
// up, the others follow in turn.
// Count: of 32 bits (the low word of each counter) where no part can hold 2^32
// tiles, else of 64.
template <typename Count>
struct TileSlots {
  unsigned long long *queue;
  int64_t n_tiles;
  int part;  // the part being drawn from, counted from the own one
  int xcd;
  __device__ __forceinline__ Count *counter(int y) const { return reinterpret_cast<Count *>(queue + y); }
  __device__ __forceinline__ Count draw() const { return atomicAdd(counter((xcd + part) & 7), (Count)1); }
  // lane's value of c in every lane
  static __device__ __forceinline__ Count from_lane(Count c, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)c, lane);
    if constexpr (sizeof(Count) == 4) return lo;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)c >> 32), lane);
    return (Count)((uint64_t)hi << 32 | lo);
  }
  // First slot that the counter of part y hands out, and their number.
  __device__ __forceinline__ void handed_out(int y, int64_t &begin, Count &size) const {
    const int rem = (int)(n_tiles & 7);
    const int64_t started = (gridDim.x + 7 - y) / 8;
    const int64_t n = n_tiles / 8 + (y < rem ? 1 : 0) - started;  // negative: fewer slots than workgroups
    begin = n_tiles / 8 * y + (y < rem ? y : rem) + started;
    size = n > 0 ? (Count)n : 0;
  }
  // One whole wave: the slot of count c of the current part (lane 0's c) to
  // *slot, or the next one of another part, or n_tiles.  Lane d stands for the
  // d-th part from the own one, so the counters are looked at together: drawing
  // from part after part costs a round trip to memory each, seven at the end of
  // a scan.  (Lanes, not scalars: eight parts' limits in scalar registers
  // spilled 90 of them, 2% of the scan at 512 x 4096.)
  __device__ __forceinline__ void find(Count c, int64_t *slot) {
    int d = threadIdx.x & 63;
    asm volatile("" : "+v"(d));
    const int y = (xcd + d) & 7;
    int64_t begin;
    Count size;
    handed_out(y, begin, size);
    c = from_lane(c, 0);
    for (;;) {
      const bool mine = d == part && c < size;
      if (mine) *slot = begin + (int64_t)c;
      if (__ballot(mine) != 0ull) return;
      Count n = 0;
      if (d < 8) n = __hip_atomic_load(counter(y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned long long m = __ballot(d < 8 && d > part && n < size);
      if (m == 0ull) {
        part = 7;
        if (d == 0) *slot = n_tiles;
        return;
      }
      part = __builtin_ctzll(m);
      if (d == part) n = draw();
      c = from_lane(n, part);
    }
  }
  // One whole wave: the workgroup's first slot.
  __device__ __forceinline__ void first(int64_t *slot) {
    const int rem = (int)(n_tiles & 7);
    const int64_t size = n_tiles / 8 + (xcd < rem ? 1 : 0), lo = n_tiles / 8 * xcd + (xcd < rem ? xcd : rem);
    if ((int64_t)(blockIdx.x >> 3) < size)
      *slot = lo + (blockIdx.x >> 3);
    else
      find(~(Count)0, slot);
  }
};

// ---- fixed-point scoring ----
// K2 is summed in 32-bit fixed point: the table holds round(2^s L[n]) modulo
// 2^32, and the 3 entries of each row are added and subtracted modulo 2^32.
// Entries and partial sums may wrap; the sum itself cannot, because s is the
// largest shift for which every K2 of N samples fits in 32 bits, so the result
// is the exact sum of the rounded entries whatever their order.  Each entry is
// within 2^-(s+1) of L[n] (s = 18 at 16384 samples: 2e-6), where FP32 would
// round an L[n] of 1.4e5 to a step of 0.016, and integer additions have a
// three-operand form (v_add3_u32), so a row costs 1.5 of them instead of
// three FP32 additions.  The score is one conversion to FP32 at the end.
// Measured against FP32 sums in row order (with the shorter completions of
// complete27): 1024 x 8192 x 64 phenotypes 294.0 -> 270.8 ms, 256-SNP quads
// 16.55 -> 15.54 ms, 1003 x 6007 6.44 -> 6.07 ms; relative error of the scores
// against FP64 2e-7 -> 2e-8.
inline int fx_shift(int32_t n_samples) {
  // K2 = sum over rows of log((r + 1) C(r, r_0)) <= N log 2 + sum log(r + 1)
  // <= N log 2 + R log(N / R + 1); R = 81 covers pairs, triplets and quads
  const double n = n_samples > 0 ? (double)n_samples : 1.0;
  const double most = n * 0.69314718055994531 + 81.0 * log(n / 81.0 + 1.0);
  int s = 28;
  while (s > 0 && ldexp(most, s) + 256.0 >= 4294967296.0) --s;  // 256: rounding of 243 entries
  return s;
}
inline float fx_scale(int32_t n_samples) { return (float)ldexp(1.0, -fx_shift(n_samples)); }
// The table's place in an encoded data set's buffer: after lf32, at the next
// 256-byte boundary.
inline const uint32_t *fx_table(const epi3_dataset &d) {
  const uintptr_t end = reinterpret_cast<uintptr_t>(d.lf32) + ((size_t)d.n_samples + 2) * sizeof(float);
  return reinterpret_cast<const uint32_t *>((end + 255) / 256 * 256);
}
// Sum of the table's rows -> FP32 score.
__device__ __forceinline__ float fx_score(uint32_t sum, float scale) { return (float)sum * scale; }

// Table entry at byte offset b >= 0 (b = 4 n for L[n]) of a table in global memory.
// The pointer is cast to that address space: jobs' tables come from records, and
// a lookup through a generic pointer is a flat load with a 64-bit address of its
// own, 81 of them per triplet (vector-ALU scans of 512 x 21000: one wave per SIMD
// at 355 registers 17.4 ms, two at 225 so 9.45 ms).
__device__ __forceinline__ uint32_t fx_at(const uint32_t *L, int b) {
  typedef const __attribute__((address_space(1))) char *gbytes;
  typedef const __attribute__((address_space(1))) uint32_t *gwords;
  return *(gwords)((gbytes)L + (uint32_t)b);
}
// The same for a table at LDS address 0 (the start of the dynamic LDS block
// of a kernel that declares no static LDS): the byte offset is the address,
// so a lookup is a single ds_read.
__device__ __forceinline__ uint32_t fx_at_lds0(int b) {
  return *(const __attribute__((address_space(3))) uint32_t *)(uintptr_t)(uint32_t)b;
}
// 4 x the low half of v (two: a register holding 2).
__device__ __forceinline__ uint32_t lo_x4(uint32_t v, uint32_t two) {
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
      : "=v"(r)
      : "v"(two), "v"(v));
  return r;
}
// 4 x the high half of v.
__device__ __forceinline__ uint32_t hi_x4(uint32_t v, uint32_t two) {
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
      : "=v"(r)
      : "v"(two), "v"(v));
  return r;
}
// K2 of a table of R rows given as byte offsets (4 x count), in fixed point:
// sum over rows of L[r + 1] - L[r_0] - L[r_1].  LDS: table at LDS address 0.
template <int R, bool LDS>
__device__ __forceinline__ uint32_t fx_sum(const int *t0, const int *t1, const uint32_t *L) {
  uint32_t up = 0u, down = 0u;
#pragma unroll
  for (int x = 0; x < R; ++x) {
    const int b0 = t0[x], b1 = t1[x];
    if (LDS) {
      up += fx_at_lds0(b0 + b1 + 4);
      down += fx_at_lds0(b0) + fx_at_lds0(b1);
    } else {
      up += fx_at(L, b0 + b1 + 4);
      down += fx_at(L, b0) + fx_at(L, b1);
      // (quads: the lookups stay near their additions, 202 registers instead of 252:
      // 64 x 140000 9.45 -> 9.29 ms; 27 rows are faster without, 512 x 21000 9.88 / 9.45)
      if (R > 27) asm volatile("" : "+v"(up), "+v"(down));
    }
  }
  return up - down;
}

// The table sits in LDS when it fits in this many bytes (two workgroups per
// CU); larger tables are read from global memory.
constexpr int64_t kLdsTableBytes = 80 * 1024;
inline bool lf_in_lds(int32_t lf_len) { return (int64_t)lf_len * 4 <= kLdsTableBytes; }

// ---- host-side launchers (defined in the .hip files) ----
// bytes, nib: value planes (both or neither)
hipError_t launch_encode(const uint8_t *geno, int64_t ld, const int32_t *sample_list, int32_t M,
                         int32_t Mp, int32_t W0, int32_t W1, int32_t n_classes, int32_t S,
                         uint32_t *planes, uint8_t *bytes, uint8_t *nib, int32_t *status,
                         hipStream_t s);
// The FP4 value planes ([2][Mp][2][S / 2] nibbles) of a SPLIT data set's bit planes.
hipError_t launch_expand_nibbles(const uint32_t *planes, int32_t Mp, int32_t W0, int32_t W1, int32_t S,
                                 uint8_t *nib, hipStream_t s);
hipError_t launch_pairs(const uint32_t *planes, int32_t Mp, int32_t W0, int32_t W1,
                        int32_t n_classes, int32_t *pairs, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s);
constexpr int kStatusWords = 64;  // of an encode buffer's status block
// lf64 and the sample list to the device (src_lf64, src_list: memory the device
// can read, or lf64 and list themselves if they are there already), lf32[x] =
// fl32(lf64[x]), lfx[x] = round(2^shift lf64[x]) mod 2^32, x < n, and a clear
// status block.
hipError_t launch_tables(const double *src_lf64, const int32_t *src_list, int64_t n_list, double *lf64,
                         float *lf32, uint32_t *lfx, int64_t n, int shift, int32_t *list,
                         int32_t *status, hipStream_t s);
int64_t host_tiles(int64_t M, int P);
// Job records, their tile prefixes and a clear tile queue.
constexpr int kJobsPerLaunch = 24;
hipError_t launch_valu_setup(const Job *h, int32_t n, Job *dst_dev, unsigned long long *queue,
                             hipStream_t s);
hipError_t launch_count_valu(const Job *jobs_dev, int32_t n_jobs, int64_t total_tiles,
                             unsigned long long *queue, int32_t lf_len, int32_t P_lo, int32_t P_hi,
                             bool counts, hipStream_t s);
constexpr int kSelJobsPerLaunch = 12;
// Lists and planes up to these lengths are finished by one workgroup: 64 keys
// and 256 scores per thread and pass, about 5 and 15 us.
constexpr int64_t kTailList = 1ll << 16;
constexpr int64_t kTailPlane = 1ll << 18;
// What a launch of selections has to provide for.
struct SelectSizes {
  int64_t max_T;    // scores of the longest plane (no planes: entries of the longest list)
  int64_t max_cap;
  int32_t max_k;
  bool sampled, unsampled;  // some job with a plane has SelJob::sample set / clear
  bool quads;       // jobs of order 4 (all or none)
  bool rest;        // some job may leave its list or plane to the passes after the tail
};
hipError_t launch_select(SelJob *sel_dev, int32_t n_jobs, const SelectSizes &z, hipStream_t s);
// The results of n jobs to memory that the host can read: n states, the n data
// sets' status words (padded to 8 bytes), hit_bytes (a multiple of 8) of hits.
constexpr int64_t result_head_bytes(int64_t n) { return n * (int64_t)sizeof(SelState) + (n + 1) / 2 * 8; }
hipError_t launch_gather_results(const SelState *st, const int32_t *const *status, int32_t n,
                                 const void *hits, int64_t hit_bytes, void *dst, hipStream_t s);
// Adds job J to the sizes of a launch.
inline void add_select_sizes(SelectSizes &z, const SelJob &J) {
  z.max_T = std::max(z.max_T, J.score ? J.T : J.ccap);
  z.max_cap = std::max(z.max_cap, J.cap);
  z.max_k = std::max(z.max_k, J.k);
  z.quads = z.quads || J.order == 4;
  if (J.score) (J.sample ? z.sampled : z.unsampled) = true;
  // a plane's list holds at most ccap >= min(T, ...) entries; past that the plane is read
  z.rest = z.rest || J.ccap > kTailList || (J.score && J.T > J.ccap && J.T > kTailPlane);
}
// The histograms of the three passes that find each job's k-th smallest key
// (jobs with fewer than k keys in their key range end without one).
hipError_t launch_select_kth(SelJob *sel_dev, int32_t n_jobs, int64_t max_T, hipStream_t s);
// After a sample pass: main job x's compacted list bound = the sample's k-th
// score + 2 e(N) (rounded up; +inf if the sample had no k-th score), empty list.
hipError_t launch_sample_bound(const SelJob *main_dev, const SelJob *sample_dev, int32_t n_jobs,
                               hipStream_t s);
// Writes the job records to dst_dev and sets up their states and histograms.
hipError_t launch_init_select(const SelJob *h, int32_t n, SelJob *dst_dev, hipStream_t s);
hipError_t launch_score_triplets(const epi3_dataset &d, const uint32_t *ijk, int64_t n,
                                 uint32_t *counts, float *k2f, double *k2, hipStream_t s);

// One group's record for either scratch buffer; prefix: the tiles' prefix too.
hipError_t launch_perm_setup(const PermJob &pj, const PermJob &alt, PermJob *dst_dev, PermJob *alt_dev,
                             bool prefix, hipStream_t s);
hipError_t launch_mask_bytes(const uint32_t *const *masks_dev, int32_t Q, int32_t Qp, int32_t N,
                             int32_t S, uint8_t *ph, int32_t *n1, bool fp4, hipStream_t s);
// half: only phenotypes 0 .. 31 of the Qp = 64 are read (Q <= 32).
hipError_t launch_case_pairs(const uint32_t *planes, int32_t M, int32_t Mp, int32_t W,
                             const uint32_t *const *masks_dev, int32_t Q, int32_t Qp, bool half,
                             int32_t *out, hipStream_t s);
// Pair scan: FP32 K2 of every pair of a SPLIT data set from its pairwise
// tables, by lexicographic pair rank; key range into keyrange[0..1].
hipError_t launch_pair_scores(const epi3_dataset &d, float *score, uint32_t *keyrange, hipStream_t s);
// Quad scan: FP32 K2 of every quad of a SPLIT data set, by lexicographic quad
// rank; key range into keyrange[0..1].  t3: device buffer of
// quad_triplet_table_bytes for the triplet corner table (classes of at most
// 65535 samples), or NULL to count the sub-triplet corners per quad.
inline int64_t quad_triplet_table_bytes(int64_t M) { return 2 * 16 * (M < 3 ? 0 : M * (M - 1) / 2 * (M - 2) / 3); }
// Corner cells of every triplet per class into t3 (quad_triplet_table_bytes).
hipError_t launch_triplet_corners(const epi3_dataset &d, void *t3, hipStream_t s);
// Quad scan with the counts on the matrix cores (FP4 value planes, classes of
// at most 65535 samples): tiles of 4 i x 1 j x 16 k x 32 l, counted and
// scored pass by pass through a scratch buffer of pass_tiles tiles.
constexpr int64_t kQuadTileScratch = 128 * 1024;  // bytes per tile, both classes
int64_t host_quad_tiles(int32_t M);
hipError_t launch_quad_prefix(int32_t M, int64_t *jprefix, hipStream_t s);
// counts tiles [tile_begin, tile_begin + n_tiles) into scratch slots from 0
hipError_t launch_count_mfma_quad(const epi3_dataset &d, const int64_t *jprefix,
                                  unsigned long long *queue, int64_t tile_begin, int64_t n_tiles,
                                  void *scratch, hipStream_t s);
// Counted and scored in one kernel, where the table leaves room for two
// workgroups per CU (about 12000 samples); stash: kQuadStash bytes per workgroup,
// at most max_blocks of them; queue: one zeroed counter.
constexpr int64_t kQuadStash = 64 * 1024;
bool quad_fused_ok(const epi3_dataset &d);
hipError_t launch_count_score_quad(const epi3_dataset &d, const int64_t *jprefix, const void *t3,
                                   unsigned long long *queue, void *stash, int64_t max_blocks, float *score,
                                   uint32_t *keyrange, hipStream_t s);
// Completes and scores the quads of launch_count_mfma_quad's tiles (t3:
// launch_triplet_corners).
hipError_t launch_finish_quad(const epi3_dataset &d, const void *scratch, const int64_t *jprefix,
                              const void *t3, int64_t tile_begin, int64_t n_tiles, float *score,
                              uint32_t *keyrange, hipStream_t s);
hipError_t launch_quad_scores(const epi3_dataset &d, void *t3, float *score, uint32_t *keyrange,
                              hipStream_t s);
int64_t host_perm_tiles(int64_t M);
// Count / finish the tiles tile_begin + n * stride, n in [0, n_tiles); their
// corner cells go to scratch slot n.
hipError_t launch_count_mfma_perm(const PermJob *pj_dev, int64_t tile_begin, int64_t n_tiles,
                                  int64_t stride, unsigned long long *queue, bool fp4,
                                  hipStream_t s);
hipError_t launch_finish_perm(const PermJob *pj_dev, int64_t tile_begin, int64_t n_tiles,
                              int64_t stride, SelState *st, const uint32_t *lfx, int32_t lf_len,
                              float scale, const PermOut &out, hipStream_t s);
// Count and score in one kernel (FP4 operands, any output mode, the
// log-factorial table of lf_len entries in LDS: perm_fused_ok); no scratch.
bool perm_fused_ok(int32_t lf_len);
hipError_t launch_count_score_perm(const PermJob *pj_dev, int Q, int64_t tile_begin, int64_t n_tiles,
                                   int64_t stride, unsigned long long *queue, SelState *st,
                                   const uint32_t *lfx, int32_t lf_len, float scale,
                                   const PermOut &out, hipStream_t s);
// Triplets (i < j < k < M) in the phenotype-batch tiles 0, stride, 2 stride, ...
int64_t host_perm_sample_valid(int64_t M, int64_t stride);
constexpr int64_t kPermTileScratch = 64 * 64 * 16 + 64 * 16;  // bytes per tile (corners + totals)
hipError_t launch_write_ptrs(const uint32_t *const *h, int32_t n, const uint32_t **dst_dev,
                             hipStream_t s);

int64_t host_plain_tiles(int64_t M, int JB);
constexpr int kPlainI = 16;  // pivots i per plain matrix-core tile (x JB j x 256 / JB k)
constexpr int64_t kPlainTileScratch = 2ll * kPlainI * 256 * 16;  // bytes per tile, both classes
// Job records, their first tiles begin[0 .. n], tile prefixes and 8 clear queue
// counters.
hipError_t launch_plain_setup(const PlainJob *h, const int64_t *begin, int32_t n, PlainJob *dst_dev,
                              int64_t *job_begin_dev, unsigned long long *queue, hipStream_t s);
// Plain matrix-core count / finish of the global tiles tile_begin + q stride,
// q < n_tiles, of n_jobs data sets (same JB and operand type): job x owns
// global tiles job_begin[x] .. job_begin[x + 1] (device int64 [n_jobs + 1]);
// slot q's corner cells sit in scratch slot q of `corners`.
hipError_t launch_count_mfma_plain(const PlainJob *jobs, const int64_t *job_begin, int32_t n_jobs,
                                   int JB, bool fp4, uint4 *corners, int64_t tile_begin,
                                   int64_t n_tiles, int64_t stride, unsigned long long *queue,
                                   hipStream_t s);
// Count and score in one kernel (FP4 operands, no tables out): the tiles as
// above, the first class's corner cells kept in `stash` (kPlainStash bytes per
// workgroup, at most max_blocks of them); lf_len: the longest job's table;
// queue: 8 zeroed 64-bit counters.
constexpr int64_t kPlainStash = kPlainTileScratch / 2;
bool plain_fused_ok(int JB, int32_t lf_len);
hipError_t launch_count_score_plain(const PlainJob *jobs, const int64_t *job_begin, int32_t n_jobs,
                                    int JB, void *stash, int64_t max_blocks, int64_t tile_begin,
                                    int64_t n_tiles, int64_t stride, unsigned long long *queue,
                                    int32_t lf_len, const PlainOut &out, hipStream_t s);
hipError_t launch_finish_plain(const PlainJob *jobs, const int64_t *job_begin, int32_t n_jobs,
                               int JB, const uint4 *corners, int64_t tile_begin, int64_t n_tiles,
                               int32_t lf_len, bool counts, const PlainOut &out, hipStream_t s);
// Triplets (i < j < k < M) in the plain tiles 0, stride, 2 stride, ... of a
// data set of M SNPs (tile JB); the number of such tiles in *n_sample.
int64_t host_plain_sample_valid(int64_t M, int JB, int64_t stride, int64_t *n_sample);

int tile_P_default(int32_t M, int32_t N);

// Device address of the current device's copy of the static scan workspace
// (looked up once per device; out may be NULL to only set it up).
int static_scratch_ptr(void **out);
// epi3_scan; spare: whatever ws_bytes leave past the workspace may be used to
// count on the matrix cores (vector-ALU variant).
int scan_in(const epi3_dataset *d, int32_t k, int32_t variant, int64_t cand_cap, void *ws_dev,
            int64_t ws_bytes, bool spare, void *stream);

}  // namespace epi3
