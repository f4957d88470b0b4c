// Fourth-order scan with the counts on the matrix cores.
//
// Eq. 1 with I = 3^4 rows.  For one class, the 16 cells of quad (i, j, k, l)
// with all four genotypes in {0, 1} are entries of a 0/1 matrix product over
// the class's samples s:
//     C[(i, j, k, a, b, c), (l, d)] = sum_s (X_i[a] X_j[b] X_k[c])[s] X_l[d][s],
// rows = corner rows of the triplet (i, j, k), columns = the value planes of
// SNP l.  The vector-ALU quad kernel fills the same cells with AND + POPCNT
// per 32 samples (the paper's table filling, Alg. 2, with a fourth SNP); here
// they come from FP4 (E2M1) products with exact FP32 accumulation, the other
// 65 cells by inclusion-exclusion (quad_cells) from the sub-triplet corner
// table and the pairwise tables, and K2 in the same fixed point as the
// vector-ALU kernel, so both give the same FP32 score.
//
// Workgroup tile: pivot j, four pivots i (one per wave), 16 consecutive k and
// 32 consecutive l (blocks aligned to their size; combinations outside
// i < j < k < l < M are counted and dropped).  A wave's products: 4 row tiles
// (4 k x 8 corner rows each) x 2 column tiles (16 l x 2 planes each) per 64
// samples.  Per chunk of 128 bytes (256 samples) the 64 l rows, the 32 k rows
// and the 16 pair rows X_i[a] & X_j[b] are staged in LDS; the steps are
// software-pipelined as in the phenotype count kernel.
#include "epi3_internal.h"

namespace epi3 {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

template <typename T>
using gptr = const __attribute__((address_space(1))) T *;

constexpr int kQKB = 16;                             // k per tile
constexpr int kQLB = 32;                             // l per tile
constexpr int kQKC = 128;                            // bytes per staged chunk of a row
constexpr int kQRow = kQKC + 16;                     // padded LDS row
constexpr int kQRowsL = 2 * kQLB;                    // (l, d) rows: B operand
constexpr int kQRowsK = 2 * kQKB;                    // (k, c) rows
constexpr int kQRowsP = 16;                          // pair rows: 4 waves x (a, b)
constexpr int kQRows = kQRowsL + kQRowsK + kQRowsP;  // 112
constexpr int kQStage = kQRows * kQRow;              // one LDS buffer
static_assert(kQuadTileScratch == 2 * 4 * kQKB * 64 * 2 * 8,
              "scratch per tile: 2 classes x 4 waves x 16 k x 64 columns x 2 uint2");

// ---- tile order: pivots j; within j, (k-block, l-block) pairs, then i-blocks ----
__host__ __device__ __forceinline__ int q_kb_lo(int j) { return (j + 1) / kQKB; }
__host__ __device__ __forceinline__ int q_nkb(int M, int j) { return (M - 1) / kQKB - q_kb_lo(j) + 1; }
// first l-block of k-block kb: the block holding (smallest valid k) + 1
__host__ __device__ __forceinline__ int q_lb_lo(int j, int kb) {
  const int kmin = kb * kQKB > j + 1 ? kb * kQKB : j + 1;
  return (kmin + 1) / kQLB;
}
__host__ __device__ __forceinline__ int q_nlb(int M, int j, int kb) {
  const int kmin = kb * kQKB > j + 1 ? kb * kQKB : j + 1;
  if (kmin >= M - 1) return 0;  // no l above the block's smallest k
  return (M - 1) / kQLB - q_lb_lo(j, kb) + 1;
}
__host__ __device__ __forceinline__ int64_t q_pairs_of_j(int M, int j) {
  int64_t n = 0;
  const int nkb = q_nkb(M, j);
  for (int x = 0; x < nkb; ++x) n += q_nlb(M, j, q_kb_lo(j) + x);
  return n;
}
__host__ __device__ __forceinline__ int64_t q_tiles_of_j(int M, int j) {
  if (j < 1 || j > M - 3) return 0;
  return (int64_t)((j + 3) / 4) * q_pairs_of_j(M, j);
}
// (i-block, k-block, l-block) of tile rr of pivot j
__device__ __forceinline__ void q_decode(int M, int j, int64_t rr, int &ib, int &kb, int &lb) {
  const int nib = (j + 3) / 4;
  const int64_t u = rr / nib;
  ib = (int)(rr - u * nib);
  int64_t acc = 0;
  kb = q_kb_lo(j);
  for (;;) {
    const int n = q_nlb(M, j, kb);
    if (u < acc + n) break;
    acc += n;
    ++kb;
  }
  lb = q_lb_lo(j, kb) + (int)(u - acc);
}

__device__ __forceinline__ int64_t rfl64x(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// pre[j] = tiles before pivot j, pre[M] = all tiles (one block).
__global__ void __launch_bounds__(1024) quad_prefix_kernel(int M, int64_t *pre) {
  __shared__ int64_t part[1024];
  const int t = threadIdx.x;
  const int chunk = (M + 1023) / 1024;
  const int a = t * chunk, b = a + chunk < M ? a + chunk : M;
  int64_t sum = 0;
  for (int j = a; j < b; ++j) sum += q_tiles_of_j(M, j);
  part[t] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int64_t v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int64_t run = part[t] - sum;
  for (int j = a; j < b; ++j) {
    pre[j] = run;
    run += q_tiles_of_j(M, j);
  }
  if (t == 1023) pre[M] = part[1023];
}

__device__ __forceinline__ int q_pivot(cptr<int64_t> pre, int M, int64_t t) {
  int lo = 0, hi = M - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// x from quad lane TT in every lane of each quad (DPP quad_perm broadcast).
template <int TT>
__device__ __forceinline__ v4i qbcast(v4i x) {
  constexpr int sel = TT * 0x55;
  v4i y;
  y.x = __builtin_amdgcn_update_dpp(0, x.x, sel, 0xf, 0xf, true);
  y.y = __builtin_amdgcn_update_dpp(0, x.y, sel, 0xf, 0xf, true);
  y.z = __builtin_amdgcn_update_dpp(0, x.z, sel, 0xf, 0xf, true);
  y.w = __builtin_amdgcn_update_dpp(0, x.w, sel, 0xf, 0xf, true);
  return y;
}

__device__ __forceinline__ v16f qmma(v4i a, v4i b, v16f c) {
  const v8i a8 = {a.x, a.y, a.z, a.w, 0, 0, 0, 0};
  const v8i b8 = {b.x, b.y, b.z, b.w, 0, 0, 0, 0};
  // cbsz = blgp = 4: both operands FP4 (E2M1); scale operands of constant 0
  // select the form without the scale prefix (256 x 4096 with the 32-bit fixed
  // point of the scores 15.6 -> 15.5 ms)
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 4, 4, 0, 0, 0, 0);
}

// Counts the 16 corner cells of both classes of every quad of tiles
// [tile_begin, tile_begin + n_tiles) into scratch slot t - tile_begin
// (persistent workgroups, atomic tile queue).  Fragment layout of
// v_mfma_f32_32x32x64_f8f6f4: lane l supplies A row l % 32 and B column
// l % 32 with 32 consecutive samples (16 bytes) starting at 32 (l / 32); the
// result of row r, column c is in lane c + 32 ((r / 4) % 2), register
// 4 (r / 8) + r % 4.
__global__ void __launch_bounds__(256, 2) count_mfma_quad_kernel(
    const uint8_t *__restrict__ nib, const int64_t *__restrict__ pre_p, int M, int Mp, int Sb,
    int Sb0, int Sb1, int64_t tile_begin, int64_t n_tiles, uint2 *__restrict__ corners,
    unsigned long long *__restrict__ queue) {
  __shared__ __attribute__((aligned(16))) unsigned char stage[2 * kQStage];
  __shared__ int64_t sTile[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 31, g = lane >> 5;
  // A row r of a row tile = (triplet ta = r / 8, corner c = (r / 4) % 2,
  // a = (r / 2) % 2, b = r % 2); the four lanes of a quad share (ta, c), each
  // loads the k row of a different row tile and DPP broadcasts it
  const int ta = r >> 3, rc = (r >> 2) & 1, ra = (r >> 1) & 1, rb = r & 1;
  gptr<uint8_t> gv = (gptr<uint8_t>)nib;
  cptr<int64_t> pre = as_const(pre_p);
  const int prow = kQRowsL + kQRowsK + wave * 4 + (ra * 2 + rb);
  const int xrow = kQRowsL + (4 * (r & 3) + ta) * 2 + rc;
  const int o_p = prow * kQRow + 16 * g, o_x = xrow * kQRow + 16 * g;
  const int o_b0 = r * kQRow + 16 * g, o_b1 = (32 + r) * kQRow + 16 * g;
  int j = -1;
  int64_t jlo = 0, jhi = 0;
  for (;;) {
    __syncthreads();  // previous tile's readers of sTile / stage are done
    if (tid == 0) sTile[0] = (int64_t)atomicAdd(queue, 1ull);
    __syncthreads();
    const int64_t slot = rfl64x(sTile[0]);
    if (slot >= n_tiles) break;
    const int64_t t = tile_begin + slot;
    if (j < 0 || t < jlo || t >= jhi) {
      j = q_pivot(pre, M, t);
      jlo = pre[j];
      jhi = pre[j + 1];
    }
    int ib, kb, lb;
    q_decode(M, j, t - jlo, ib, kb, lb);
    const int i = 4 * ib + wave;  // may be >= j: then the wave's results are dropped
    const int kbase = kb * kQKB, lbase = lb * kQLB;
    for (int cls = 0; cls < 2; ++cls) {
      if (cls) __syncthreads();  // class 0's readers of stage are done
      const int nch = ((cls ? Sb1 : Sb0) + kQKC - 1) / kQKC;
      const int64_t crow = (int64_t)cls * Mp * 2;  // first row of the class
      // staging plan: rows [0, 64) (l, d), [64, 96) (k, c), [96, 112) pair
      // rows; main pieces c16 = tid + 256 u; threads tid < 128 also carry one
      // pair piece (both source words, ANDed when stored)
      constexpr int kPc = kQKC / 16;
      constexpr int kMainU = 96 * kPc / 256;
      constexpr int kPairPieces = kQRowsP * kPc;
      static_assert((96 * kPc) % 256 == 0 && kPairPieces <= 256, "staging plan");
      uint32_t off[kMainU], offa = 0, offb = 0;
#pragma unroll
      for (int u = 0; u < kMainU; ++u) {
        const int c16 = tid + 256 * u;
        const int row = c16 / kPc, col = (c16 % kPc) * 16;
        const int snp = row < kQRowsL ? lbase + (row >> 1) : kbase + ((row - kQRowsL) >> 1);
        off[u] = (uint32_t)((crow + (int64_t)snp * 2 + (row & 1)) * Sb + col);
      }
      if (tid < kPairPieces) {
        const int x = tid / kPc, col = (tid % kPc) * 16;  // pair row x: wave x >> 2, (a, b) = x & 3
        const int ii = 4 * ib + (x >> 2);
        offa = (uint32_t)((crow + (int64_t)ii * 2 + ((x >> 1) & 1)) * Sb + col);
        offb = (uint32_t)((crow + (int64_t)j * 2 + (x & 1)) * Sb + col);
      }
      v4i pf[kMainU], pa, pb;
      auto fetch = [&](int ch) {
        const uint32_t c0 = (uint32_t)ch * kQKC;
#pragma unroll
        for (int u = 0; u < kMainU; ++u) pf[u] = *reinterpret_cast<gptr<v4i>>(gv + (off[u] + c0));
        if (tid < kPairPieces) {
          pa = *reinterpret_cast<gptr<v4i>>(gv + (offa + c0));
          pb = *reinterpret_cast<gptr<v4i>>(gv + (offb + c0));
        }
      };
      auto store = [&](int buf) {
        uint8_t *dst = stage + buf * kQStage;
#pragma unroll
        for (int u = 0; u < kMainU; ++u) {
          const int c16 = tid + 256 * u;
          *reinterpret_cast<v4i *>(dst + (c16 / kPc) * kQRow + (c16 % kPc) * 16) = pf[u];
        }
        if (tid < kPairPieces)
          *reinterpret_cast<v4i *>(dst + (kQRowsL + kQRowsK + tid / kPc) * kQRow + (tid % kPc) * 16) = pa & pb;
      };
      v16f acc[4][2];
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[tt][0][v] = acc[tt][1][v] = 0.f;
      fetch(0);
      store(0);
      __syncthreads();
      // Software pipeline over the four steps of a chunk (operand sets X and
      // Y in turn; the next chunk is stored before the chunk's last step)
#define EPI3_QLD(BB, STP, P, X, B0, B1)                                               \
      P = *reinterpret_cast<const v4i *>((BB) + o_p + 32 * (STP));                  \
      X = *reinterpret_cast<const v4i *>((BB) + o_x + 32 * (STP));                  \
      B0 = *reinterpret_cast<const v4i *>((BB) + o_b0 + 32 * (STP));                \
      B1 = *reinterpret_cast<const v4i *>((BB) + o_b1 + 32 * (STP));
#define EPI3_QTILE(TT, P, X, B0, B1)                                                  \
      {                                                                             \
        const v4i a_ = (P) & qbcast<TT>(X);                                         \
        acc[TT][0] = qmma(a_, B0, acc[TT][0]);                                      \
        acc[TT][1] = qmma(a_, B1, acc[TT][1]);                                      \
      }
// a scheduling barrier between steps; the compiler interleaves each row
// tile's A-row ANDs with the products itself
#define EPI3_QSCHED __builtin_amdgcn_sched_barrier(0);
#define EPI3_QSTEP(P, X, B0, B1)                                                      \
      EPI3_QTILE(0, P, X, B0, B1)                                                   \
      EPI3_QTILE(1, P, X, B0, B1)                                                   \
      EPI3_QTILE(2, P, X, B0, B1)                                                   \
      EPI3_QTILE(3, P, X, B0, B1)
      static_assert(kQKC / 32 == 4, "four steps per chunk");
      v4i pX, xX, b0X, b1X, pY, xY, b0Y, b1Y;
      EPI3_QLD(stage, 0, pX, xX, b0X, b1X)
      for (int ch = 0; ch < nch; ++ch) {
        const bool more = ch + 1 < nch;
        if (more) fetch(ch + 1);
        const uint8_t *buf = stage + (ch & 1) * kQStage;
        const uint8_t *nbuf = stage + ((ch + 1) & 1) * kQStage;
        EPI3_QLD(buf, 1, pY, xY, b0Y, b1Y)
        EPI3_QSTEP(pX, xX, b0X, b1X)
        EPI3_QSCHED
        EPI3_QLD(buf, 2, pX, xX, b0X, b1X)
        EPI3_QSTEP(pY, xY, b0Y, b1Y)
        EPI3_QSCHED
        EPI3_QLD(buf, 3, pY, xY, b0Y, b1Y)
        EPI3_QSTEP(pX, xX, b0X, b1X)
        EPI3_QSCHED
        // the products above stay before the branch
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) asm volatile("" : "+v"(acc[tt][0]), "+v"(acc[tt][1]));
        if (more) store((ch + 1) & 1);
        __syncthreads();
        // after the last chunk this reads the other buffer's stale contents,
        // which no product uses
        EPI3_QLD(nbuf, 0, pX, xX, b0X, b1X)
        EPI3_QSTEP(pY, xY, b0Y, b1Y)
        EPI3_QSCHED
      }
#undef EPI3_QLD
#undef EPI3_QTILE
#undef EPI3_QSCHED
#undef EPI3_QSTEP
      if (i >= j) continue;  // padding pivot of the last i-block (wave-uniform)
      // lane (column, c) holds, for the 4 triplets of each row tile, the cells
      // (a, b) at genotype c of SNP k: registers 4 ta + 2 a + b.  Record of
      // (triplet, column) = 2 x uint2 (c = 0, 1), columns 2 l + d adjacent.
      uint2 *cor = corners + ((slot * 2 + cls) * 4 + wave) * (int64_t)(kQKB * 128);
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int t4 = 0; t4 < 4; ++t4) {
            const uint32_t c0 = (uint32_t)acc[tt][cb][4 * t4 + 0], c1 = (uint32_t)acc[tt][cb][4 * t4 + 1];
            const uint32_t c2 = (uint32_t)acc[tt][cb][4 * t4 + 2], c3 = (uint32_t)acc[tt][cb][4 * t4 + 3];
            cor[((4 * tt + t4) * 64 + cb * 32 + r) * 2 + g] = make_uint2(c0 | (c1 << 16), c2 | (c3 << 16));
          }
    }
  }
}

// LDS of the finish kernel past the log-factorial table, per tile: the 27 cells
// of the sub-triplets (i, j, k) (64 of them), cells (a, b, d < 2) of (i, j, l)
// (128), all as two 16-bit counts (class 1 in the high half), and the ranks'
// bases.  Rows of 28 and 20 words: 16-byte reads without bank conflicts.
constexpr int kQTijk = 28, kQTijl = 20;
struct FinishQuadLds {
  uint32_t ijk[4 * kQKB][kQTijk];
  uint32_t ijl[4 * kQLB][kQTijl];
  int64_t ik[4 * kQKB];    // lexicographic rank of triplet (i, k, l) - l
  int64_t quad[4 * kQKB];  // and of the quad (i, j, k, l) - l
  int64_t jk[kQKB];        // and of triplet (j, k, l) - l
};

// Three rows' lookups: L[r + 1], L[r_0], L[r_1].
struct QuadLookups {
  uint32_t u[3], d0[3], d1[3];
};

// Sub-triplet tables of a tile, both classes per register.
struct QuadTables {
  const uint4 *t3;
  const int4 *pr;
  int M, Mp, N0, N1;
  // both classes' entries of a pair
  __device__ __forceinline__ void pair4(int x, int y, u16x2 v[4]) const {
    const int64_t e = (int64_t)x * Mp + y;
    const int4 a = pr[e], b = pr[(int64_t)Mp * Mp + e];
    v[0] = as_u16x2((uint32_t)a.x | ((uint32_t)b.x << 16));
    v[1] = as_u16x2((uint32_t)a.y | ((uint32_t)b.y << 16));
    v[2] = as_u16x2((uint32_t)a.z | ((uint32_t)b.z << 16));
    v[3] = as_u16x2((uint32_t)a.w | ((uint32_t)b.w << 16));
  }
  __device__ __forceinline__ void corners8(int64_t rank, u16x2 v[8]) const {
    const uint4 a = t3[2 * rank], b = t3[2 * rank + 1];
    v[0] = as_u16x2(a.x); v[1] = as_u16x2(a.y); v[2] = as_u16x2(a.z); v[3] = as_u16x2(a.w);
    v[4] = as_u16x2(b.x); v[5] = as_u16x2(b.y); v[6] = as_u16x2(b.z); v[7] = as_u16x2(b.w);
  }
  // the 27 cells of the triplet (x, y, z)
  __device__ __forceinline__ void table27(int x, int y, int z, u16x2 t[27]) const {
    u16x2 n[8], pxy[4], pxz[4], pyz[4], mx[4], my[4], mz[4], fyz[9];
    corners8(lex_base(M, x, y) + z, n);
    pair4(x, y, pxy);
    pair4(x, z, pxz);
    pair4(y, z, pyz);
    pair4(x, x, mx);
    pair4(y, y, my);
    pair4(z, z, mz);
    const u16x2 my2[2] = {my[0], my[3]}, mz2[2] = {mz[0], mz[3]};
    pair_cells(pyz, my2, mz2, as_u16x2((uint32_t)N0 | ((uint32_t)N1 << 16)), fyz);
    const u16x2 pxy2[2] = {mx[0] - pxy[0] - pxy[1], mx[3] - pxy[2] - pxy[3]};
    complete27(n, fyz, pxy, pxy2, pxz, t);
  }
  // The tile's shared tables, by the 256 threads of its workgroup.
  __device__ __forceinline__ void fill(FinishQuadLds &sh, int ib, int j, int kb, int lb) const {
    if (threadIdx.x < 4 * kQKB) {
      const int x = threadIdx.x, i = 4 * ib + x / kQKB, k = kb * kQKB + x % kQKB;
      if (i < j && k > j && k < M) {
        u16x2 c[27];
        table27(i, j, k, c);
#pragma unroll
        for (int y = 0; y < 27; ++y) sh.ijk[x][y] = as_u32(c[y]);
        sh.ik[x] = lex_base(M, i, k);
        sh.jk[x % kQKB] = lex_base(M, j, k);  // (the four i write the same)
        sh.quad[x] = quad_rank(M, i, j, k, k + 1) - (k + 1);
      }
    } else if (threadIdx.x < 4 * kQKB + 4 * kQLB) {
      const int x = threadIdx.x - 4 * kQKB, i = 4 * ib + x / kQLB, l = lb * kQLB + x % kQLB;
      if (i < j && l > j && l < M) {
        u16x2 c[27];
        table27(i, j, l, c);
#pragma unroll
        for (int ab = 0; ab < 9; ++ab) {
          sh.ijl[x][2 * ab] = as_u32(c[3 * ab]);
          sh.ijl[x][2 * ab + 1] = as_u32(c[3 * ab + 1]);
        }
      }
    }
  }
};

// The fixed-point score of one quad from the cells (c, d < 2) of its rows
// (a, b) (counted for a, b < 2, the others completed here), the sub-triplets'
// cells and the pair (k, l).  Three rows per step, their lookups added two
// steps later.
template <typename At>
__device__ __forceinline__ uint32_t score_quad(u16x2 (&core)[9][4], const u16x2 ikl[8], const u16x2 jkl[8],
                                               const u16x2 pkl[4], const uint32_t *tijk,
                                               const uint32_t *tijl, uint32_t two, const At &at) {
          uint32_t up = 0u, down = 0u;
          QuadLookups in_flight[2];
          auto add_up = [&](int n) {
            const QuadLookups &f = in_flight[n & 1];
            up += f.u[0] + f.u[1];
            up += f.u[2];
            down += f.d0[0] + f.d1[0];
            down += f.d0[1] + f.d1[1];
            down += f.d0[2] + f.d1[2];
            asm volatile("" : "+v"(up), "+v"(down));  // (keeps the additions of different steps apart)
          };
          auto step = [&](int n, u16x2 r0, u16x2 r1, u16x2 r2) {
            const uint32_t r[3] = {as_u32(r0), as_u32(r1), as_u32(r2)};
            uint32_t lo[3], hi[3];
  #pragma unroll
            for (int x = 0; x < 3; ++x) {
              lo[x] = lo_x4(r[x], two);
              hi[x] = hi_x4(r[x], two);
            }
            if (n >= 2) add_up(n - 2);
            QuadLookups &f = in_flight[n & 1];
  #pragma unroll
            for (int x = 0; x < 3; ++x) {
              f.u[x] = at(lo[x] + hi[x] + 4u);
              f.d0[x] = at(lo[x]);
              f.d1[x] = at(hi[x]);
            }
                  };
  #pragma unroll
          for (int ab = 0; ab < 9; ++ab) {
            u16x2 (&q)[4] = core[ab];
            if (ab == 2 || ab == 5) {
  #pragma unroll
              for (int x = 0; x < 4; ++x) q[x] = ikl[(ab == 2 ? 0 : 4) + x] - core[ab - 2][x] - core[ab - 1][x];
            } else if (ab == 6 || ab == 7) {
  #pragma unroll
              for (int x = 0; x < 4; ++x) q[x] = jkl[4 * (ab - 6) + x] - core[ab - 6][x] - core[ab - 3][x];
            } else if (ab == 8) {
  #pragma unroll
              for (int x = 0; x < 4; ++x) q[x] = (pkl[x] - ikl[x] - ikl[4 + x]) - core[6][x] - core[7][x];
            }
            const u16x2 e0 = as_u16x2(tijl[2 * ab]) - q[0] - q[2], e1 = as_u16x2(tijl[2 * ab + 1]) - q[1] - q[3];
            const u16x2 f0 = as_u16x2(tijk[3 * ab]) - q[0] - q[1], f1 = as_u16x2(tijk[3 * ab + 1]) - q[2] - q[3];
            const u16x2 f2 = as_u16x2(tijk[3 * ab + 2]) - e0 - e1;
            step(3 * ab, q[0], q[1], q[2]);
            step(3 * ab + 1, q[3], e0, e1);
            step(3 * ab + 2, f0, f1, f2);
          }
          add_up(25);
          add_up(26);
  return up - down;
}

// Completes the 81-row tables of every quad of the pass's tiles and scores them
// (workgroup per tile, round robin; thread = l and two of the k, four i each).
// Both classes are completed at once, two 16-bit counts per register.  The
// tables of the sub-triplets (i, j, k) and (i, j, l), which many quads share,
// are completed once per tile into LDS; (i, k, l) and (j, k, l) come from the
// triplet table (the latter once per four quads).  Rows are taken three at a
// time and their lookups added two steps later, so vector instructions (about
// 600 per quad and wave) and lookups (243) alternate: issue is what bounds it.
// It serves data sets above about 11900 samples, whose table and the 18.6 KB of
// shared tables leave two workgroups to a CU (123 registers would allow four
// waves per SIMD), one from about 16000 samples, and four again above 20478,
// where the table stays in global memory.  Against one class at a time in 32
// bits with all sub-triplets completed per quad (204 registers, all 243 lookups
// after the table, two workgroups per CU up to 20478 samples), whole scans: 128
// x 12500 2.71 -> 2.17 ms, 128 x 16384 3.19 -> 3.00, 128 x 18000 3.43 -> 3.14, 200
// x 18000 19.6 -> 16.0, 128 x 30000 6.57 -> 5.76 ms.
template <bool LDS>
__global__ void __launch_bounds__(256, 3) finish_quad_kernel(
    const uint2 *__restrict__ corners, const int64_t *__restrict__ pre_p,
    const uint4 *__restrict__ t3, const int32_t *__restrict__ pairs, int M, int Mp, int N0,
    int N1, int64_t tile_begin, int64_t n_tiles, const uint32_t *__restrict__ lfx,
    int lf_len, float scale, float *__restrict__ score, uint32_t *__restrict__ keyrange) {
  // the LDS table starts the kernel's dynamic LDS block, at LDS address 0
  // (no static LDS), so a lookup is one ds_read at the byte offset
  extern __shared__ __attribute__((aligned(16))) uint32_t qtab[];
  if (LDS) table_to_lds<256>(qtab, lfx, lf_len);
  FinishQuadLds &sh = *reinterpret_cast<FinishQuadLds *>(reinterpret_cast<unsigned char *>(qtab) +
                                                         (LDS ? (lf_len * 4 + 15) / 16 * 16 : 0));
  auto at = [&](uint32_t off) { return LDS ? fx_at_lds0((int)off) : fx_at(lfx, (int)off); };
  cptr<int64_t> pre = as_const(pre_p);
  const QuadTables tabs{t3, reinterpret_cast<const int4 *>(pairs), M, Mp, N0, N1};
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  uint32_t two = 2u;
  asm volatile("" : "+v"(two));
  int j = -1;
  int64_t jlo = 0, jhi = 0;
  for (int64_t slot = blockIdx.x; slot < n_tiles; slot += gridDim.x) {
    const int64_t t = tile_begin + slot;
    if (j < 0 || t < jlo || t >= jhi) {
      j = q_pivot(pre, M, t);
      jlo = pre[j];
      jhi = pre[j + 1];
    }
    int ib, kb, lb;
    q_decode(M, j, t - jlo, ib, kb, lb);
    __syncthreads();  // previous tile's readers are done (and the table is in)
    tabs.fill(sh, ib, j, kb, lb);
    __syncthreads();
    const int ll = threadIdx.x & (kQLB - 1), l = lb * kQLB + ll;
    const int ni = j - 4 * ib < 4 ? j - 4 * ib : 4;  // pivots i below j
    for (int half = 0; half < 2; ++half) {
      const int kk = (threadIdx.x >> 5) + 8 * half, k = kb * kQKB + kk;
      if (k <= j || l <= k || l >= M) continue;
      u16x2 jkl[8], pkl[4];
      tabs.corners8(lex_base(M, j, k) + l, jkl);
      tabs.pair4(k, l, pkl);
      const uint4 *rec = reinterpret_cast<const uint4 *>(corners + ((slot * 8) * kQKB + kk) * 128 + ll * 4);
      // one i ahead: the counted cells of both classes, and (i, k, l)
      uint4 next[4], nikl[2];
      auto fetch = [&](int w) {
        const uint4 *r0 = rec + (int64_t)w * (kQKB * 64), *r1 = r0 + 4 * kQKB * 64;
        next[0] = r0[0];
        next[1] = r0[1];
        next[2] = r1[0];
        next[3] = r1[1];
        const int64_t e = 2 * (sh.ik[w * kQKB + kk] + l);
        nikl[0] = t3[e];
        nikl[1] = t3[e + 1];
      };
      fetch(0);
      for (int w = 0; w < ni; ++w) {
        const uint4 v[2][2] = {{next[0], next[1]}, {next[2], next[3]}};  // [class][d]
        const u16x2 ikl[8] = {as_u16x2(nikl[0].x), as_u16x2(nikl[0].y), as_u16x2(nikl[0].z), as_u16x2(nikl[0].w),
                              as_u16x2(nikl[1].x), as_u16x2(nikl[1].y), as_u16x2(nikl[1].z), as_u16x2(nikl[1].w)};
        if (w + 1 < ni) fetch(w + 1);
        // cells (c, d < 2) of the rows (a, b): counted for a, b < 2
        u16x2 core[9][4];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int d = 0; d < 2; ++d) {
              const uint32_t w0 = a ? (cc ? v[0][d].w : v[0][d].y) : (cc ? v[0][d].z : v[0][d].x);
              const uint32_t w1 = a ? (cc ? v[1][d].w : v[1][d].y) : (cc ? v[1][d].z : v[1][d].x);
              core[3 * a][2 * cc + d] = as_u16x2(__builtin_amdgcn_perm(w1, w0, 0x05040100u));
              core[3 * a + 1][2 * cc + d] = as_u16x2(__builtin_amdgcn_perm(w1, w0, 0x07060302u));
            }
        const float k2 = fx_score(score_quad(core, ikl, jkl, pkl, sh.ijk[w * kQKB + kk],
                                             sh.ijl[w * kQLB + ll], two, at),
                                  scale);
        score[sh.quad[w * kQKB + kk] + l] = k2;
        const uint32_t key = f2key(k2);
        kmin = key < kmin ? key : kmin;
        kmax = key > kmax ? key : kmax;
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t a = __shfl_xor(kmin, off), b = __shfl_xor(kmax, off);
    kmin = a < kmin ? a : kmin;
    kmax = b > kmax ? b : kmax;
  }
  if ((threadIdx.x & 63) == 0 && kmax != 0u) {
    atomicMin(&keyrange[0], kmin);
    atomicMax(&keyrange[1], kmax);
  }
}

// Counts and scores the tiles in one kernel (the table and the staging in half a
// CU's LDS).  As the two kernels above, but the corner cells never leave the
// chip: both classes' samples are one sequence of chunks, the accumulators start
// at 2^23 (their low halves are the counts), at the class boundary each lane
// keeps its 128 class-0 cells as 16 KB of the workgroup's stash (L2), and after
// class 1 the wave of pivot i scores its 16 k x 32 l.  The four lanes that hold
// one (k, l)'s cells (genotype of k by lane half, genotype of l by lane parity)
// exchange them for four k at a time, so each scores one of the four: 8 lane-half
// swaps and 16 selects with a neighbour's register per four quads.  The shared
// tables lie in the idle staging buffers; (i, k, l), (j, k, l) and the pair (k, l)
// are loaded one quad ahead.
template <int SEL>
__device__ __forceinline__ uint32_t dpp_quad(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, SEL, 0xf, 0xf, true);
}

static_assert(sizeof(FinishQuadLds) <= 2 * kQStage, "shared tables in the staging buffers");
__host__ __device__ constexpr int quad_fused_lds(int lf_len) {
  return (lf_len * 4 + 15) / 16 * 16 + 2 * kQStage + 16;
}

__global__ void __launch_bounds__(256, 2) count_score_quad_kernel(
    const uint8_t *__restrict__ nib, const int64_t *__restrict__ pre_p, const uint4 *__restrict__ t3,
    const int32_t *__restrict__ pairs, int M, int Mp, int Sb, int Sb0, int Sb1, int N0, int N1,
    int64_t n_tiles, uint4 *__restrict__ stash_p, unsigned long long *__restrict__ queue,
    const uint32_t *__restrict__ lfx, int lf_len, float scale, float *__restrict__ score,
    uint32_t *__restrict__ keyrange) {
  extern __shared__ __attribute__((aligned(16))) uint32_t qtab[];
  uint8_t *stage = reinterpret_cast<uint8_t *>(qtab) + (lf_len * 4 + 15) / 16 * 16;
  FinishQuadLds &sh = *reinterpret_cast<FinishQuadLds *>(stage);
  int64_t *sTile = reinterpret_cast<int64_t *>(stage + 2 * kQStage);
  table_to_lds<256>(qtab, lfx, lf_len);
  auto at = [](uint32_t off) { return fx_at_lds0((int)off); };
  const QuadTables tabs{t3, reinterpret_cast<const int4 *>(pairs), M, Mp, N0, N1};
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  gptr<uint8_t> gv = (gptr<uint8_t>)nib;
  cptr<int64_t> pre = as_const(pre_p);
  uint4 *stash = stash_p + (int64_t)blockIdx.x * 4096 + wave * 1024;  // [16][lane]
  const int nch0 = (Sb0 + kQKC - 1) / kQKC, nch = nch0 + (Sb1 + kQKC - 1) / kQKC;
  const uint32_t cls1 = (uint32_t)Mp * 2u * (uint32_t)Sb;  // class 1's first row
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  int j = -1;
  int64_t jlo = 0, jhi = 0;
  // Workgroup b starts with tile b; the queue hands out those after them.  (The
  // next tile is drawn while one is counted: with every tile drawn, and few
  // tiles per workgroup, those launched first took two and the last ones none:
  // 48 SNPs x 1000 samples 208 -> 197 us per scan, 256 x 4096 unchanged.)
  int64_t slot = blockIdx.x;
  while (slot < n_tiles) {
    __builtin_amdgcn_s_setprio(0);
    // lane roles formed per tile (see the phenotype count kernel)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, r = lane & 31, g = lane >> 5;
    if (j < 0 || slot < jlo || slot >= jhi) {
      j = q_pivot(pre, M, slot);
      jlo = pre[j];
      jhi = pre[j + 1];
    }
    int ib, kb, lb;
    q_decode(M, j, slot - jlo, ib, kb, lb);
    const int i = 4 * ib + wave;  // may be >= j: then the wave's results are dropped
    const unsigned long long drawn = tid == 0 ? atomicAdd(queue, 1ull) : 0ull;  // the next tile
    // A row r of a row tile = (triplet r / 8, corner c = (r / 4) % 2, a, b)
    const int ta = r >> 3, rc = (r >> 2) & 1;
    const int prow = kQRowsL + kQRowsK + wave * 4 + (r & 3);
    const int xrow = kQRowsL + (4 * (r & 3) + ta) * 2 + rc;
    const int o_p = prow * kQRow + 16 * g, o_x = xrow * kQRow + 16 * g;
    const int o_b0 = r * kQRow + 16 * g, o_b1 = (32 + r) * kQRow + 16 * g;
    constexpr int kPc = kQKC / 16;
    constexpr int kMainU = 96 * kPc / 256;
    constexpr int kPairPieces = kQRowsP * kPc;
    uint32_t off[kMainU], offa = 0, offb = 0;
#pragma unroll
    for (int u = 0; u < kMainU; ++u) {
      const int c16 = tid + 256 * u;
      const int row = c16 / kPc, col = (c16 % kPc) * 16;
      const int snp = row < kQRowsL ? lb * kQLB + (row >> 1) : kb * kQKB + ((row - kQRowsL) >> 1);
      off[u] = (uint32_t)(((int64_t)snp * 2 + (row & 1)) * Sb + col);
    }
    if (tid < kPairPieces) {
      const int x = tid / kPc, col = (tid % kPc) * 16;  // pair row x: wave x >> 2, (a, b) = x & 3
      offa = (uint32_t)(((int64_t)(4 * ib + (x >> 2)) * 2 + ((x >> 1) & 1)) * Sb + col);
      offb = (uint32_t)(((int64_t)j * 2 + (x & 1)) * Sb + col);
    }
    v4i pf[kMainU], pa = {}, pb = {};
    auto fetch = [&](int ch) {
      const uint32_t c0 = ch < nch0 ? (uint32_t)ch * kQKC : cls1 + (uint32_t)(ch - nch0) * kQKC;
#pragma unroll
      for (int u = 0; u < kMainU; ++u) pf[u] = *reinterpret_cast<gptr<v4i>>(gv + (off[u] + c0));
      if (tid < kPairPieces) {
        pa = *reinterpret_cast<gptr<v4i>>(gv + (offa + c0));
        pb = *reinterpret_cast<gptr<v4i>>(gv + (offb + c0));
      }
    };
    auto store = [&](int buf) {
      uint8_t *dst = stage + buf * kQStage;
#pragma unroll
      for (int u = 0; u < kMainU; ++u) {
        const int c16 = tid + 256 * u;
        *reinterpret_cast<v4i *>(dst + (c16 / kPc) * kQRow + (c16 % kPc) * 16) = pf[u];
      }
      if (tid < kPairPieces)
        *reinterpret_cast<v4i *>(dst + (kQRowsL + kQRowsK + tid / kPc) * kQRow + (tid % kPc) * 16) = pa & pb;
    };
    v16f acc[4][2];
    auto clear = [&]() {
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[tt][0][v] = acc[tt][1][v] = 8388608.f;
    };
    // the low halves of row tile tt, column tile cb: word 2 t4 + a = (a, 0), (a, 1)
    auto words = [&](int tt, int cb, int h) {
      uint32_t w[4];
#pragma unroll
      for (int x = 0; x < 4; ++x)
        w[x] = __builtin_amdgcn_perm(__float_as_uint(acc[tt][cb][8 * h + 2 * x + 1]),
                                     __float_as_uint(acc[tt][cb][8 * h + 2 * x]), 0x05040100u);
      return make_uint4(w[0], w[1], w[2], w[3]);
    };
    auto keep = [&]() {
      uint32_t lo = (uint32_t)lane;  // opaque: the addresses are formed here
      asm volatile("" : "+v"(lo));
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int h = 0; h < 2; ++h) (stash + ((2 * tt + cb) * 2 + h) * 64)[lo] = words(tt, cb, h);
    };
    clear();
    fetch(0);
    store(0);
    __syncthreads();
#define EPI3_QLD(BB, STP, P, X, B0, B1)                                               \
    P = *reinterpret_cast<const v4i *>((BB) + o_p + 32 * (STP));                    \
    X = *reinterpret_cast<const v4i *>((BB) + o_x + 32 * (STP));                    \
    B0 = *reinterpret_cast<const v4i *>((BB) + o_b0 + 32 * (STP));                  \
    B1 = *reinterpret_cast<const v4i *>((BB) + o_b1 + 32 * (STP));
#define EPI3_QTILE(TT, P, X, B0, B1)                                                  \
    {                                                                               \
      const v4i a_ = (P) & qbcast<TT>(X);                                           \
      acc[TT][0] = qmma(a_, B0, acc[TT][0]);                                        \
      acc[TT][1] = qmma(a_, B1, acc[TT][1]);                                        \
    }
#define EPI3_QSTEP(P, X, B0, B1)                                                      \
    EPI3_QTILE(0, P, X, B0, B1)                                                     \
    EPI3_QTILE(1, P, X, B0, B1)                                                     \
    EPI3_QTILE(2, P, X, B0, B1)                                                     \
    EPI3_QTILE(3, P, X, B0, B1)
    // software pipeline over the four steps of a chunk, as in the count kernel
    v4i pX, xX, b0X, b1X, pY, xY, b0Y, b1Y;
    EPI3_QLD(stage, 0, pX, xX, b0X, b1X)
    for (int ch = 0; ch < nch; ++ch) {
      const bool more = ch + 1 < nch;
      if (ch == nch0) {
        keep();
        clear();
      }
      if (more) fetch(ch + 1);
      const uint8_t *buf = stage + (ch & 1) * kQStage;
      const uint8_t *nbuf = stage + ((ch + 1) & 1) * kQStage;
      EPI3_QLD(buf, 1, pY, xY, b0Y, b1Y)
      EPI3_QSTEP(pX, xX, b0X, b1X)
      __builtin_amdgcn_sched_barrier(0);
      EPI3_QLD(buf, 2, pX, xX, b0X, b1X)
      EPI3_QSTEP(pY, xY, b0Y, b1Y)
      __builtin_amdgcn_sched_barrier(0);
      EPI3_QLD(buf, 3, pY, xY, b0Y, b1Y)
      EPI3_QSTEP(pX, xX, b0X, b1X)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) asm volatile("" : "+v"(acc[tt][0]), "+v"(acc[tt][1]));
      if (more) store((ch + 1) & 1);
      __syncthreads();
      // after the last chunk this reads the other buffer's stale contents,
      // which no product uses
      EPI3_QLD(nbuf, 0, pX, xX, b0X, b1X)
      EPI3_QSTEP(pY, xY, b0Y, b1Y)
      __builtin_amdgcn_sched_barrier(0);
    }
#undef EPI3_QLD
#undef EPI3_QTILE
#undef EPI3_QSTEP
    if (nch == nch0) {
      keep();
      clear();
    }
    // class 1's cells, two per register (frees half of the accumulators)
    uint4 c1[4][2][2];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          c1[tt][cb][h] = words(tt, cb, h);
          asm volatile("" : "+v"(c1[tt][cb][h].x), "+v"(c1[tt][cb][h].y), "+v"(c1[tt][cb][h].z),
                            "+v"(c1[tt][cb][h].w));
        }
    __syncthreads();  // the staging buffers are idle from here to the next tile
    __builtin_amdgcn_s_setprio(1);  // scoring goes ahead of the other workgroup's counting
    tabs.fill(sh, ib, j, kb, lb);
    if (tid == 0) sTile[0] = (int64_t)(drawn + gridDim.x);
    __syncthreads();
    if (i < j) {  // wave-uniform
      int ln = threadIdx.x & 63;
      uint32_t two = 2u;
      asm volatile("" : "+v"(ln), "+v"(two));
      const bool odd = ln & 1;                 // genotype of l that this lane counted
      const int kr = 2 * (ln >> 5) + (ln & 1);  // its k of every four
      const int lr = (ln & 31) >> 1;           // its l of every 16
      struct Next {
        uint4 s[2], ikl[2], jkl[2];
        int4 pkl[2];
      } nx;
      auto valid = [&](int k, int l) { return k > j && l > k && l < M; };
      auto load = [&](int n) {
        const int tt = n >> 1, cb = n & 1;
        const int kk = 4 * tt + kr, k = kb * kQKB + kk, l = lb * kQLB + 16 * cb + lr;
        const bool ok = valid(k, l);
        nx.s[0] = (stash + 2 * n * 64)[ln];
        nx.s[1] = (stash + (2 * n + 1) * 64)[ln];
        const int64_t e = ok ? 2 * (sh.ik[wave * kQKB + kk] + l) : 0, f = ok ? 2 * (sh.jk[kk] + l) : 0;
        nx.ikl[0] = t3[e];
        nx.ikl[1] = t3[e + 1];
        nx.jkl[0] = t3[f];
        nx.jkl[1] = t3[f + 1];
        const int64_t p = (int64_t)k * Mp + l;  // k, l < M + 32: inside the padded tables
        nx.pkl[0] = tabs.pr[p];
        nx.pkl[1] = tabs.pr[(int64_t)Mp * Mp + p];
      };
      load(0);
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        const int tt = n >> 1, cb = n & 1;
        const Next cur = nx;
        if (n < 7) load(n + 1);
        const int k0 = kb * kQKB + 4 * tt, l0 = lb * kQLB + 16 * cb;
        if (k0 + 3 <= j || l0 + 15 <= k0 || l0 >= M) continue;  // wave-uniform: no quad here
        // x[t4][2 a + b]: both classes' counts
        u16x2 core[9][4];
        {
          const uint32_t s0[8] = {cur.s[0].x, cur.s[0].y, cur.s[0].z, cur.s[0].w,
                                  cur.s[1].x, cur.s[1].y, cur.s[1].z, cur.s[1].w};
          const uint32_t s1[8] = {c1[tt][cb][0].x, c1[tt][cb][0].y, c1[tt][cb][0].z, c1[tt][cb][0].w,
                                  c1[tt][cb][1].x, c1[tt][cb][1].y, c1[tt][cb][1].z, c1[tt][cb][1].w};
#pragma unroll
          for (int ab = 0; ab < 4; ++ab) {
            const uint32_t sel = ab & 1 ? 0x07060302u : 0x05040100u;
            uint32_t x[4];
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4)
              x[t4] = __builtin_amdgcn_perm(s1[2 * t4 + (ab >> 1)], s0[2 * t4 + (ab >> 1)], sel);
            // lane half h: triplets t4 = 2 h and 2 h + 1, genotypes c = 0, 1
            const auto e = __builtin_amdgcn_permlane32_swap(x[0], x[2], false, false);
            const auto o = __builtin_amdgcn_permlane32_swap(x[1], x[3], false, false);
            const int row = 3 * (ab >> 1) + (ab & 1);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              // even lanes take t4 = 2 h (own d = 0), odd lanes 2 h + 1 (own d = 1)
              const uint32_t pe = dpp_quad<0xB1>(e[c]), po = dpp_quad<0xB1>(o[c]);
              core[row][2 * c] = as_u16x2(odd ? po : e[c]);
              core[row][2 * c + 1] = as_u16x2(odd ? o[c] : pe);
            }
          }
        }
        const u16x2 ikl[8] = {as_u16x2(cur.ikl[0].x), as_u16x2(cur.ikl[0].y), as_u16x2(cur.ikl[0].z),
                              as_u16x2(cur.ikl[0].w), as_u16x2(cur.ikl[1].x), as_u16x2(cur.ikl[1].y),
                              as_u16x2(cur.ikl[1].z), as_u16x2(cur.ikl[1].w)};
        const u16x2 jkl[8] = {as_u16x2(cur.jkl[0].x), as_u16x2(cur.jkl[0].y), as_u16x2(cur.jkl[0].z),
                              as_u16x2(cur.jkl[0].w), as_u16x2(cur.jkl[1].x), as_u16x2(cur.jkl[1].y),
                              as_u16x2(cur.jkl[1].z), as_u16x2(cur.jkl[1].w)};
        const u16x2 pkl[4] = {as_u16x2((uint32_t)cur.pkl[0].x | ((uint32_t)cur.pkl[1].x << 16)),
                              as_u16x2((uint32_t)cur.pkl[0].y | ((uint32_t)cur.pkl[1].y << 16)),
                              as_u16x2((uint32_t)cur.pkl[0].z | ((uint32_t)cur.pkl[1].z << 16)),
                              as_u16x2((uint32_t)cur.pkl[0].w | ((uint32_t)cur.pkl[1].w << 16))};
        const int kk = 4 * tt + kr, k = kb * kQKB + kk, l = l0 + lr;
        if (valid(k, l)) {
          const float k2 = fx_score(score_quad(core, ikl, jkl, pkl, sh.ijk[wave * kQKB + kk],
                                               sh.ijl[wave * kQLB + 16 * cb + lr], two, at),
                                    scale);
          score[sh.quad[wave * kQKB + kk] + l] = k2;
          const uint32_t key = f2key(k2);
          kmin = key < kmin ? key : kmin;
          kmax = key > kmax ? key : kmax;
        }
      }
    }
    slot = rfl64x(sTile[0]);
    __syncthreads();  // this tile's readers of the shared tables and the slot are done
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t a = __shfl_xor(kmin, off), b = __shfl_xor(kmax, off);
    kmin = a < kmin ? a : kmin;
    kmax = b > kmax ? b : kmax;
  }
  if ((threadIdx.x & 63) == 0 && kmax != 0u) {
    atomicMin(&keyrange[0], kmin);
    atomicMax(&keyrange[1], kmax);
  }
}

template <bool LDS>
hipError_t launch_finish_quad_t(const epi3_dataset &d, const uint2 *corners, const int64_t *pre,
                                const uint4 *t3, int64_t tile_begin, int64_t n_tiles,
                                float *score, uint32_t *keyrange, int n_cu, hipStream_t s) {
  const int lf_len = d.n_samples + 2;
  const int lds = (LDS ? (lf_len * 4 + 15) / 16 * 16 : 0) + (int)sizeof(FinishQuadLds);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&finish_quad_kernel<LDS>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, finish_quad_kernel<LDS>, 256, lds);
  if (e != hipSuccess) return e;
  int64_t blocks = (int64_t)n_cu * (per_cu > 0 ? per_cu : 1);
  if (blocks > n_tiles) blocks = n_tiles;
  hipLaunchKernelGGL(finish_quad_kernel<LDS>, dim3((unsigned)blocks), dim3(256), lds, s, corners,
                     pre, t3, d.pairs, d.n_snps, d.snp_stride, d.n_controls, d.n_cases,
                     tile_begin, n_tiles, fx_table(d), lf_len, fx_scale(d.n_samples),
                     score, keyrange);
  return hipGetLastError();
}

}  // namespace

int64_t host_quad_tiles(int32_t M) {
  int64_t n = 0;
  for (int j = 0; j < M; ++j) n += q_tiles_of_j(M, j);
  return n;
}

hipError_t launch_quad_prefix(int32_t M, int64_t *jprefix, hipStream_t s) {
  hipLaunchKernelGGL(quad_prefix_kernel, dim3(1), dim3(1024), 0, s, (int)M, jprefix);
  return hipGetLastError();
}

hipError_t launch_count_mfma_quad(const epi3_dataset &d, const int64_t *jprefix,
                                  unsigned long long *queue, int64_t tile_begin, int64_t n_tiles,
                                  void *scratch, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  int dev = 0, n_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, count_mfma_quad_kernel, 256, 0);
  if (e != hipSuccess) return e;
  if (per_cu <= 0) per_cu = 1;
  int64_t blocks = (int64_t)n_cu * per_cu;
  if (blocks > n_tiles) blocks = n_tiles;
  const int Sb = d.byte_stride / 2;                 // FP4 bytes per row
  const int Sb0 = (d.n_controls + 127) / 128 * 64;  // bytes holding each class
  const int Sb1 = (d.n_cases + 127) / 128 * 64;
  hipLaunchKernelGGL(count_mfma_quad_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                     static_cast<const uint8_t *>(d.nibbles), jprefix, d.n_snps, d.snp_stride, Sb,
                     Sb0, Sb1, tile_begin, n_tiles, static_cast<uint2 *>(scratch), queue);
  return hipGetLastError();
}

bool quad_fused_ok(const epi3_dataset &d) { return quad_fused_lds(d.n_samples + 2) <= kLdsTableBytes; }

hipError_t launch_count_score_quad(const epi3_dataset &d, const int64_t *jprefix, const void *t3,
                                   unsigned long long *queue, void *stash, int64_t max_blocks, float *score,
                                   uint32_t *keyrange, hipStream_t s) {
  const int64_t n_tiles = host_quad_tiles(d.n_snps);
  if (n_tiles <= 0) return hipSuccess;
  if (!quad_fused_ok(d)) return hipErrorInvalidValue;
  int dev = 0, n_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int lds = quad_fused_lds(d.n_samples + 2);
  e = hipFuncSetAttribute(reinterpret_cast<const void *>(&count_score_quad_kernel),
                          hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, count_score_quad_kernel, 256, lds);
  if (e != hipSuccess) return e;
  int64_t blocks = (int64_t)n_cu * (per_cu > 0 ? per_cu : 1);
  blocks = std::min(blocks, std::min(n_tiles, max_blocks));
  if (blocks < 1) return hipErrorInvalidValue;
  const int Sb = d.byte_stride / 2;                 // FP4 bytes per row
  const int Sb0 = (d.n_controls + 127) / 128 * 64;  // bytes holding each class
  const int Sb1 = (d.n_cases + 127) / 128 * 64;
  hipLaunchKernelGGL(count_score_quad_kernel, dim3((unsigned)blocks), dim3(256), lds, s,
                     static_cast<const uint8_t *>(d.nibbles), jprefix, static_cast<const uint4 *>(t3), d.pairs,
                     d.n_snps, d.snp_stride, Sb, Sb0, Sb1, d.n_controls, d.n_cases, n_tiles,
                     static_cast<uint4 *>(stash), queue, fx_table(d), d.n_samples + 2, fx_scale(d.n_samples),
                     score, keyrange);
  return hipGetLastError();
}

hipError_t launch_finish_quad(const epi3_dataset &d, const void *scratch, const int64_t *jprefix,
                              const void *t3, int64_t tile_begin, int64_t n_tiles, float *score,
                              uint32_t *keyrange, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  int dev = 0, n_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const uint2 *cor = static_cast<const uint2 *>(scratch);
  const uint4 *t = static_cast<const uint4 *>(t3);
  return lf_in_lds(d.n_samples + 2)
             ? launch_finish_quad_t<true>(d, cor, jprefix, t, tile_begin, n_tiles, score, keyrange, n_cu, s)
             : launch_finish_quad_t<false>(d, cor, jprefix, t, tile_begin, n_tiles, score, keyrange, n_cu, s);
}

}  // namespace epi3
