// Count stage of the plain (two-class) scan on the matrix cores.
//
// For one class c, the corner cells of every triplet (i, j, k) are entries
// of matrix products over that class's samples:
//     C[(i, j, a, b), (k, g)] = sum_s (X_i[a][s] X_j[b][s]) X_k[g][s],
// rows (i, j, a, b), columns (k, g), K = the class's samples, 0/1 values
// (int8 bytes or FP4 nibbles) and exact accumulation.  This is the same
// integer table the paper fills with AND + POPCNT (Alg. 2); the other 19
// cells of each class follow from the pairwise tables as in the vector-ALU
// kernel.
//
// count_score_plain_kernel counts and scores (FP4 operands, tables of up to
// about 17600 entries): the corner cells never leave the workgroup but for
// one class's, kept in a small stash.  The two-kernel path below it serves
// int8 operands, longer tables, tiles of 2 pivots j and tables written out:
// counting writes the 8 corner cells of both classes of every triplet of a
// pass of tiles to a scratch buffer; a second kernel completes the tables and
// scores them (Eq. 1).
//
// Workgroup tile: 16 consecutive i, JB consecutive j, 256 / JB consecutive
// k (4096 triplets), so one staged sample chunk serves 16 + JB + 256 / JB
// SNPs instead of the 161 of a (32 i, one j, 128 k) slab.  Each of the 4
// waves owns 2 i-blocks of 8 x 2 j (four 32-row A tiles: 8 i x (a, b), the
// rows X_i[a] & X_j[b] formed in registers) and two 32-column B tiles.
// Operand rows are staged per chunk of 128 bytes (64 for JB = 2) in
// double-buffered LDS.
#include <algorithm>

#include "epi3_internal.h"

namespace epi3 {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

template <typename T>
using gptr = const __attribute__((address_space(1))) T *;

constexpr int kPI = kPlainI;   // i per workgroup tile

// Bytes per staged chunk of a row: 128 (four steps per barrier), 64 for
// JB = 2, whose 176 rows would otherwise take more than half of the LDS.
// Rows are padded by 16 bytes against bank conflicts.
__host__ __device__ constexpr int plain_chunk(int JB) { return JB == 2 ? 64 : 128; }

__host__ __device__ constexpr int plain_kt(int JB) { return 256 / JB; }

// Tiles of j-block J (j in [JB J, JB J + JB)): i-blocks of 16 below the
// block's last pivot, k-blocks of 256 / JB from JB J + 1 up to M - 1.
__host__ __device__ __forceinline__ int64_t plain_tiles_of_jb(int64_t M, int64_t J, int JB) {
  const int64_t j0 = J * JB;
  int64_t jmax = j0 + JB - 1;
  if (jmax > M - 2) jmax = M - 2;
  if (jmax < 1 || j0 > M - 2) return 0;
  const int KT = plain_kt(JB);
  return ((jmax + kPI - 1) / kPI) * ((M - 1 - j0 + KT - 1) / KT);
}

// i-block and k-block of tile rr of j-block J: bands of 8 i-blocks, k-block
// major within a band, so the tiles counted at a time on one XCD share the
// operand rows of 8 i-blocks and of a few k-blocks.
__host__ __device__ __forceinline__ void plain_tile_ib_kb(int rr, int64_t M, int64_t J, int JB,
                                                          int nkb, int &ib, int &kb) {
  int jmax = (int)J * JB + JB - 1;
  if (jmax > (int)M - 2) jmax = (int)M - 2;
  const int nib = (jmax + kPI - 1) / kPI;
  const int band = rr / (8 * nkb);
  const int rest = nib - 8 * band;
  const int bcnt = rest < 8 ? rest : 8;
  const int pos = rr - band * 8 * nkb;
  kb = pos / bcnt;
  ib = 8 * band + (pos - kb * bcnt);
}

__host__ __device__ __forceinline__ int64_t plain_jblocks(int64_t M, int JB) {
  return M < 3 ? 0 : (M - 1 + JB - 1) / JB;
}

// Lane n of every quad takes x from quad lane (SEL >> 2 n) & 3 (DPP
// quad_perm; the compiler folds it into the instruction that consumes it
// where it can).
template <int SEL>
__device__ __forceinline__ v4i quad_perm(v4i x) {
  v4i y;
  y.x = __builtin_amdgcn_update_dpp(0, x.x, SEL, 0xf, 0xf, true);
  y.y = __builtin_amdgcn_update_dpp(0, x.y, SEL, 0xf, 0xf, true);
  y.z = __builtin_amdgcn_update_dpp(0, x.z, SEL, 0xf, 0xf, true);
  y.w = __builtin_amdgcn_update_dpp(0, x.w, SEL, 0xf, 0xf, true);
  return y;
}

__device__ __forceinline__ int64_t rfl64q(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int rfl(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T *rflp(T *p) {
  return reinterpret_cast<T *>(rfl64q((int64_t)reinterpret_cast<uintptr_t>(p)));
}

// Job records and first tiles of a launch, passed by value.
constexpr int kPlainJobsPerLaunch = 24;
struct PlainJobs {
  PlainJob j[kPlainJobsPerLaunch];
  int64_t begin[kPlainJobsPerLaunch + 1];
};
static_assert(sizeof(PlainJobs) <= 3968, "kernel argument block");

// One workgroup per job: the record, its first global tile, the tiles before
// each of its j-blocks (jprefix[J]; jprefix[nJ] = all of them), and a clear
// tile queue.
__global__ void __launch_bounds__(1024) plain_setup_kernel(PlainJobs jobs, PlainJob *dst, int64_t *job_begin,
                                                           unsigned long long *queue) {
  const PlainJob *pj = &jobs.j[blockIdx.x];
  const int t = threadIdx.x;
  if (t == 0) {
    dst[blockIdx.x] = *pj;
    job_begin[blockIdx.x] = jobs.begin[blockIdx.x];
    if (blockIdx.x + 1 == gridDim.x) job_begin[gridDim.x] = jobs.begin[gridDim.x];
  }
  if (blockIdx.x == 0 && t < 8) queue[t] = 0ull;
  const int64_t M = pj->M;
  const int JB = pj->JB;
  const int64_t nJ = plain_jblocks(M, JB);
  int64_t *pre = const_cast<int64_t *>(pj->jprefix);
  __shared__ int64_t part[1024];
  const int64_t chunk = (nJ + 1023) / 1024;
  const int64_t a = t * chunk, b = (a + chunk < nJ) ? a + chunk : nJ;
  int64_t sum = 0;
  for (int64_t J = a; J < b; ++J) sum += plain_tiles_of_jb(M, J, JB);
  part[t] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int64_t v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int64_t run = part[t] - sum;
  for (int64_t J = a; J < b; ++J) {
    pre[J] = run;
    run += plain_tiles_of_jb(M, J, JB);
  }
  if (t == 1023) pre[nJ] = part[1023];
}

template <bool FP4>
struct PlainAcc {
  typedef v16i type;
  static __device__ __forceinline__ type mma(v4i a, v4i b, type c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t get(const type &c, int v) { return (uint32_t)c[v]; }
};
template <>
struct PlainAcc<true> {
  typedef v16f type;
  static __device__ __forceinline__ type mma(v4i a, v4i b, type c) {
    const v8i a8 = {a.x, a.y, a.z, a.w, 0, 0, 0, 0};
    const v8i b8 = {b.x, b.y, b.z, b.w, 0, 0, 0, 0};
    // FP4 operands; scale operands of constant 0 select the instruction form
    // without the scale prefix (unit scales), one issue slot less per product
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 4, 4, 0, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t get(const type &c, int v) { return (uint32_t)c[v]; }
};

// Decodes a tile index into its j-block through the prefix table.
struct TileDecoder {
  int J = -1;
  int64_t jlo = 0, jhi = 0;
  __device__ __forceinline__ void find(cptr<int64_t> pre, int nJ, int64_t t) {
    if (J < 0 || t < jlo || t >= jhi) {
      int lo = 0, hi = nJ - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= t) lo = mid; else hi = mid - 1;
      }
      J = lo;
      jlo = pre[J];
      jhi = pre[J + 1];
    }
  }
};

// (i0, j0, k0) of tile t of j-block J.
__device__ __forceinline__ void plain_tile_origin(const TileDecoder &dec, int64_t t, int M, int JB,
                                                  int &i0, int &j0, int &k0) {
  const int KT = 256 / JB;
  j0 = dec.J * JB;
  const int nkb = (M - 1 - j0 + KT - 1) / KT;
  int ib, kb;
  plain_tile_ib_kb((int)(t - dec.jlo), M, dec.J, JB, nkb, ib, kb);
  i0 = ib * kPI;
  k0 = j0 + 1 + kb * KT;
}

// Finds the job of global tile t: jobs own consecutive ranges of the tile
// order, job_begin[x] .. job_begin[x + 1] (uniform: scalar loads).
struct JobDecoder {
  int x = -1;
  int64_t lo = 0, hi = 0;
  __device__ __forceinline__ bool find(cptr<int64_t> job_begin, int n_jobs, int64_t t) {
    if (x >= 0 && t >= lo && t < hi) return false;
    int a = 0, b = n_jobs - 1;
    while (a < b) {
      const int mid = (a + b + 1) >> 1;
      if (job_begin[mid] <= t) a = mid; else b = mid - 1;
    }
    x = a;
    lo = job_begin[a];
    hi = job_begin[a + 1];
    return true;
  }
};

template <bool FP4, int JB>
__global__ void __launch_bounds__(256, 2) count_mfma_plain_kernel(
    const PlainJob *__restrict__ jobs, const int64_t *__restrict__ job_begin_p, int n_jobs,
    uint4 *__restrict__ corners, int64_t tile_begin, int64_t n_tiles, int64_t stride,
    unsigned long long *__restrict__ queue) {
  typedef PlainAcc<FP4> Acc;
  constexpr int KT = 256 / JB;
  constexpr int kPKC = plain_chunk(JB), kPRow = kPKC + 16;
  constexpr int kRowsI = 2 * kPI, kRowsJ = 2 * JB, kRowsK = 2 * KT;
  constexpr int kRows = kRowsI + kRowsJ + kRowsK;
  constexpr int kBuf = kRows * kPRow;
  constexpr int kChunks = kRows * (kPKC / 16);
  constexpr int kPer = (kChunks + 255) / 256;
  constexpr int NBP = KT / 32;  // pairs of B tiles; the 4 waves are (JB / 2) x NBP
  static_assert((JB / 2) * NBP == 4, "four waves per tile");
  __shared__ __attribute__((aligned(16))) unsigned char stage[2 * kBuf];
  __shared__ int64_t sTile[2];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wj = wave / NBP, wb = wave - wj * NBP;
  const int r = lane & 31, g = lane >> 5;
  cptr<int64_t> job_begin = as_const(job_begin_p);
  JobDecoder jd;
  int M = 0, Mp = 0, Sb = 0, Sb0 = 0, Sb1 = 0, nJ = 0;
  gptr<uint8_t> gv = nullptr;
  cptr<int64_t> pre = nullptr;
  TileDecoder dec;
  // lane roles: A row r = 4 i8 + 2 a + b; B column r = 2 k16 + g_k
  const int ri8 = r >> 2, ra = (r >> 1) & 1, rb = r & 1;
  const int ck16 = r >> 1, cpl = r & 1;
  // LDS byte offsets (within a buffer) of the rows this lane loads for its quad
  const int xi_off = (2 * (8 * rb + ri8) + ra) * kPRow;
  const int xj_off = (kRowsI + 2 * (2 * wj + ra) + rb) * kPRow;

  for (;;) {
    __syncthreads();
    if (tid == 0) sTile[0] = (int64_t)atomicAdd(queue, 1ull);
    __syncthreads();
    const int64_t slot = rfl64q(sTile[0]);  // scratch slot of this launch
    if (slot >= n_tiles) break;
    const int64_t tg = tile_begin + slot * stride;
    if (jd.find(job_begin, n_jobs, tg)) {
      const PlainJob &pj = jobs[jd.x];
      M = pj.M;
      Mp = pj.Mp;
      Sb = pj.Sb;
      Sb0 = pj.Sb0;
      Sb1 = pj.Sb1;
      nJ = (int)plain_jblocks(M, JB);
      gv = (gptr<uint8_t>)pj.vals;
      pre = as_const(pj.jprefix);
      dec.J = -1;
    }
    const int64_t t = tg - jd.lo;  // tile within its job
    dec.find(pre, nJ, t);
    int i0, j0, k0;
    plain_tile_origin(dec, t, M, JB, i0, j0, k0);

    for (int cls = 0; cls < 2; ++cls) {
      // the class's bytes rounded up to whole chunks (rows are zero-padded
      // to a multiple of 128 bytes)
      const int nch = ((cls ? Sb1 : Sb0) + kPKC - 1) / kPKC;
      const int64_t cbase = (int64_t)cls * Mp * 2;  // first row of this class
      // staging plan: rows [0, 32) X_i (i0 + x / 2, plane x % 2), then 2 JB
      // rows X_j, then 2 KT rows X_k (k0 + x / 2, plane x % 2)
      // 32-bit byte offsets of this thread's 16-byte pieces (the value planes
      // are far below 4 GB), so each load is a scalar base plus one VGPR
      constexpr int kPieces = kPKC / 16;
      uint32_t off[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int c16 = tid + 256 * u;
        const int row = c16 / kPieces < kRows ? c16 / kPieces : kRows - 1, col = (c16 % kPieces) * 16;
        int snp, pl;
        if (row < kRowsI) { snp = i0 + (row >> 1); pl = row & 1; }
        else if (row < kRowsI + kRowsJ) { const int x = row - kRowsI; snp = j0 + (x >> 1); pl = x & 1; }
        else { const int x = row - kRowsI - kRowsJ; snp = k0 + (x >> 1); pl = x & 1; }
        snp = snp < Mp ? snp : Mp - 1;  // rows past M read a zero row
        off[u] = (uint32_t)((cbase + (int64_t)snp * 2 + pl) * Sb + col);
      }
      v4i pf[kPer];
      auto fetch = [&](int ch) {
#pragma unroll
        for (int u = 0; u < kPer; ++u)
          if (tid + 256 * u < kChunks)
            pf[u] = *reinterpret_cast<gptr<v4i>>(gv + (off[u] + (uint32_t)ch * kPKC));
      };
      auto store = [&](int buf) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const int c16 = tid + 256 * u;
          if (c16 < kChunks)
            *reinterpret_cast<v4i *>(stage + buf * kBuf + (c16 / kPieces) * kPRow + (c16 % kPieces) * 16) = pf[u];
        }
      };
      typename Acc::type acc[2][2][2];  // [i-block][j of the pair][B tile]
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[x][y][z][v] = 0;
      if (nch > 0) {
        fetch(0);
        store(0);
      }
      __syncthreads();
      const int o_xi = xi_off + 16 * g, o_xj = xj_off + 16 * g;
      const int o_b0 = (kRowsI + kRowsJ + 2 * (16 * (2 * wb) + ck16) + cpl) * kPRow + 16 * g;
      const int o_b1 = (kRowsI + kRowsJ + 2 * (16 * (2 * wb + 1) + ck16) + cpl) * kPRow + 16 * g;
#define EPI3_PLD(BB, STP, XI, XJ, B0, B1)                                           \
      XI = *reinterpret_cast<const v4i *>((BB) + o_xi + 32 * (STP));              \
      XJ = *reinterpret_cast<const v4i *>((BB) + o_xj + 32 * (STP));              \
      B0 = *reinterpret_cast<const v4i *>((BB) + o_b0 + 32 * (STP));              \
      B1 = *reinterpret_cast<const v4i *>((BB) + o_b1 + 32 * (STP));
#define EPI3_PSTEP(XI, XJ, B0, B1)                                                  \
      {                                                                           \
        const v4i xi_[2] = {quad_perm<0xA0>(XI), quad_perm<0xF5>(XI)};            \
        _Pragma("unroll") for (int x = 0; x < 2; ++x) {                           \
          const v4i a0 = xi_[x] & quad_perm<0x44>(XJ);                            \
          acc[x][0][0] = Acc::mma(a0, B0, acc[x][0][0]);                          \
          acc[x][0][1] = Acc::mma(a0, B1, acc[x][0][1]);                          \
          const v4i a1 = xi_[x] & quad_perm<0xEE>(XJ);                            \
          acc[x][1][0] = Acc::mma(a1, B0, acc[x][1][0]);                          \
          acc[x][1][1] = Acc::mma(a1, B1, acc[x][1][1]);                          \
        }                                                                         \
      }                                                                           \
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (kPKC == 128) {
        // software pipeline over the four steps of a chunk (operand sets X
        // and Y in turn; the next chunk is stored before the last step)
        v4i xiX, xjX, b0X, b1X, xiY, xjY, b0Y, b1Y;
        EPI3_PLD(stage, 0, xiX, xjX, b0X, b1X)
        for (int ch = 0; ch < nch; ++ch) {
          const bool more = ch + 1 < nch;
          if (more) fetch(ch + 1);
          const uint8_t *buf = stage + (ch & 1) * kBuf;
          const uint8_t *nbuf = stage + ((ch + 1) & 1) * kBuf;
          EPI3_PLD(buf, 1, xiY, xjY, b0Y, b1Y)
          EPI3_PSTEP(xiX, xjX, b0X, b1X)
          EPI3_PLD(buf, 2, xiX, xjX, b0X, b1X)
          EPI3_PSTEP(xiY, xjY, b0Y, b1Y)
          EPI3_PLD(buf, 3, xiY, xjY, b0Y, b1Y)
          EPI3_PSTEP(xiX, xjX, b0X, b1X)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) asm volatile("" : "+v"(acc[x][y][0]), "+v"(acc[x][y][1]));
          if (more) store((ch + 1) & 1);
          __syncthreads();
          // after the last chunk this reads the other buffer's stale
          // contents, which no product uses
          EPI3_PLD(nbuf, 0, xiX, xjX, b0X, b1X)
          EPI3_PSTEP(xiY, xjY, b0Y, b1Y)
        }
      } else {
        for (int ch = 0; ch < nch; ++ch) {
          if (ch + 1 < nch) fetch(ch + 1);
          const uint8_t *buf = stage + (ch & 1) * kBuf;
  #pragma unroll 1
          for (int stp = 0; stp < kPKC / 32; ++stp) {
            const int off = stp * 32 + 16 * g;
            // the quad (a, b) loads X_i[a] of i-block b and X_j[b] of pivot a;
            // DPP hands each lane the two rows its A rows need
            const v4i xiq = *reinterpret_cast<const v4i *>(buf + xi_off + off);
            const v4i xjq = *reinterpret_cast<const v4i *>(buf + xj_off + off);
            v4i b[2];
  #pragma unroll
            for (int x = 0; x < 2; ++x)
              b[x] = *reinterpret_cast<const v4i *>(
                  buf + (kRowsI + kRowsJ + 2 * (16 * (2 * wb + x) + ck16) + cpl) * kPRow + off);
            const v4i xi[2] = {quad_perm<0xA0>(xiq), quad_perm<0xF5>(xiq)};  // [0,0,2,2], [1,1,3,3]
  #pragma unroll
            for (int x = 0; x < 2; ++x) {
              const v4i a0 = xi[x] & quad_perm<0x44>(xjq);  // [0,1,0,1]: X_j[b] of pivot 0
              acc[x][0][0] = Acc::mma(a0, b[0], acc[x][0][0]);
              acc[x][0][1] = Acc::mma(a0, b[1], acc[x][0][1]);
              const v4i a1 = xi[x] & quad_perm<0xEE>(xjq);  // [2,3,2,3]: X_j[b] of pivot 1
              acc[x][1][0] = Acc::mma(a1, b[0], acc[x][1][0]);
              acc[x][1][1] = Acc::mma(a1, b[1], acc[x][1][1]);
            }
          }
          if (ch + 1 < nch) store((ch + 1) & 1);
          __syncthreads();
        }
      }
#undef EPI3_PLD
#undef EPI3_PSTEP
      // corners out: lane (column, g) holds rows 8 u + 4 g + w, i.e. pivot
      // i8 = 2 u + g with cells (a, b) = w, for its column (k16, plane).
      // Record (i, j, k) of class cls is 16 bytes: plane-0 cells then plane-1
      // cells, each 4 x uint16 in (a, b) order.
      uint2 *cor = reinterpret_cast<uint2 *>(corners) + ((slot * 2 + cls) * (int64_t)kPI * 256) * 2;
      // record (il, jl, kl) = (8 x + 2 u + g, 2 wj + y, 16 (2 wb + z) + ck16)
      // sits at a constant per (x, y, z, u) plus one lane offset; the offset
      // is made opaque here so the 32 addresses are formed at the stores
      // instead of being held in registers through the tile
      uint32_t lo = (uint32_t)(((g * JB + 2 * wj) * KT + 32 * wb + ck16) * 2 + cpl);
      asm volatile("" : "+v"(lo));
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int c_off = (((8 * x + 2 * u) * JB + y) * KT + 16 * z) * 2;
              const uint32_t c0 = Acc::get(acc[x][y][z], 4 * u + 0), c1 = Acc::get(acc[x][y][z], 4 * u + 1);
              const uint32_t c2 = Acc::get(acc[x][y][z], 4 * u + 2), c3 = Acc::get(acc[x][y][z], 4 * u + 3);
              (cor + c_off)[lo] = make_uint2(c0 | (c1 << 16), c2 | (c3 << 16));
            }
    }
  }
}

// Lowest and highest key of the wave's lanes into keyrange[0..1].
__device__ __forceinline__ void flush_range(uint32_t kmin, uint32_t kmax, uint32_t *keyrange) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t a = __shfl_xor(kmin, off), b = __shfl_xor(kmax, off);
    kmin = a < kmin ? a : kmin;
    kmax = b > kmax ? b : kmax;
  }
  if ((threadIdx.x & 63) == 0 && kmax != 0u) {
    atomicMin(keyrange, kmin);
    atomicMax(keyrange + 1, kmax);
  }
}

// Three rows' lookups in the table at LDS address 0: L[r + 1], L[r_0], L[r_1]
// of rows held as (class-0 count | all << 16).
struct Lookups {
  uint32_t up[3], d0[3], d1[3];
};
__device__ __forceinline__ Lookups look_up(const uint32_t c[3], uint32_t two) {
  Lookups l;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const uint32_t r0 = lo_x4(c[a], two), r = (c[a] >> 16) << 2;
    l.up[a] = fx_at_lds0((int)r + 4);
    l.d0[a] = fx_at_lds0((int)r0);
    l.d1[a] = fx_at_lds0((int)(r - r0));
  }
  return l;
}
__device__ __forceinline__ void add_up(const Lookups &l, uint32_t &up, uint32_t &down) {
  up += l.up[0] + l.up[1];
  down += l.d0[0] + l.d1[0];
  down += l.d0[1] + l.d1[1];
  up += l.up[2];
  down += l.d0[2] + l.d1[2];
}

// Correction of a sum whose table in LDS ends after `lim` entries (it is
// complete at `lfx`).  An entry past those is needed only by a row of more
// than half of the samples, so by one row at most: `top`, the row with the
// largest count.  Its three lookups are replaced: what the LDS held at those
// addresses is subtracted again, so those words must not change between the
// two readings.  They lie in the staging buffers before their last
// kPairBytes (fused_ok_t), and from the barrier that ends the counts to the
// one that ends the scoring only the pair entries are written there, by each
// wave in its own time: they take the last kPairBytes.
__device__ __forceinline__ uint32_t fix_top(uint32_t sum, uint32_t top, const uint32_t *lfx,
                                            uint32_t lim) {
  const uint32_t r = top >> 16, r0 = top & 0xffffu;
  if (r + 1 >= lim) {
    sum += lfx[r + 1] - fx_at_lds0((int)(r + 1) << 2);
    sum -= lfx[r0] - fx_at_lds0((int)r0 << 2);
    sum -= lfx[r - r0] - fx_at_lds0((int)(r - r0) << 2);
  }
  return sum;
}

// Bytes between the two planes' k rows (half of the banks, for the stores).
constexpr int kPlanePad = 128;
// LDS of the count-and-score kernel: the log-factorial table at address 0,
// then the staging buffers and the tile slot.
template <int JB>
__host__ __device__ constexpr int plain_stage_bytes() {
  return 2 * ((2 * kPI + 2 * JB + 2 * plain_kt(JB)) * (plain_chunk(JB) + 16) + kPlanePad);
}
// Table entries that fit beside them with two workgroups per CU.
template <int JB>
constexpr int32_t plain_fused_entries() {
  return ((kLdsTableBytes - plain_stage_bytes<JB>() - 16) / 16) * 4;
}
// The four waves' pair entries while they score, at the end of the staging
// buffers: a cut table's lookups run past the table into those (fix_top).
constexpr int kPairBytes = 4 * 64 * 16;
// Longest table: the first entries in LDS, with a cover of 7/10 of it.
template <int JB>
constexpr int32_t plain_fused_longest() {
  return plain_fused_entries<JB>() * 10 / 7;
}
// Whether the lookups of a table of lf_len entries, cut to those that fit,
// end before the pair entries.
template <int JB>
constexpr bool plain_lookups_ok(int32_t lf_len) {
  return (int64_t)lf_len * 4 <=
         (int64_t)plain_fused_entries<JB>() * 4 + plain_stage_bytes<JB>() - kPairBytes;
}
static_assert(plain_lookups_ok<8>(plain_fused_longest<8>()) && plain_lookups_ok<4>(plain_fused_longest<4>()),
              "no lookup reaches words that a wave writes while another scores");

// Counts and scores the tiles in one kernel (FP4).  Both classes' samples are
// one sequence of chunks.  The accumulators start at 2^23, so an FP32 sum's
// low 16 bits are its count; at the class boundary each lane stores those of
// the 128 class-0 cells to the workgroup's 64 KB stash (L2-resident), the
// accumulators run on over class 1, and end with the all-sample cells.  The
// column tiles are the two planes of the same 32 k, so a lane holds all 8
// corner cells of its 16 triplets: half (g) of the 16 i, 2 j, one k.  Tables
// are completed for both classes at once, two 16-bit counts per register, from
// the pair table (j, k) completed once per j, (i, k) loaded once per i, and
// (i, j) of the wave's 32 pairs kept at the end of the idle staging buffers.  The next
// tile's slot is drawn while this one is counted and its first chunk loaded
// while this one is scored.
//
// Two waves per SIMD (229-235 registers), one of each workgroup, so one can
// count while the other scores.  A lone wave issues one vector instruction
// per 8 cycles and one lookup per 12 (measured with independent chains; two
// waves on a SIMD share 2.7 cycles per vector instruction), so with one
// scoring wave per SIMD the instructions of a triplet (206 vector, 83 LDS)
// cost about 2600 cycles per 64, whatever the LDS and the vector ALU could do
// together: at 3100 x 2500 the LDS is busy 66% of the time, the vector ALU 59%,
// the matrix cores 31%.  The scoring wave therefore goes first (priority 1).
// The X_i rows of both i-blocks are read from LDS instead of one read and
// eight lane permutations (16 vector instructions per 8 products instead of
// 24: 2048 x 16384 70.9 -> 69.4 ms).  Against the two-kernel path (32 bytes
// per triplet and class through HBM, the scoring waiting on them):
// 2048 x 16384 84.1 -> 69.4 ms, 3100 x 2500 112.5 -> 73.7 ms, 512 x 4096 1.06
// -> 0.87 ms, 1003 x 6007 6.07 -> 5.09 ms, 32 uneven data sets 72.6 -> 65.8 ms.
template <int JB, bool TRUNC, int MODE>
__global__ void __launch_bounds__(256, 2) count_score_plain_kernel(
    const PlainJob *__restrict__ jobs, const int64_t *__restrict__ job_begin_p, int n_jobs,
    uint4 *__restrict__ stash_p, int64_t tile_begin, int64_t n_tiles, int64_t stride,
    unsigned long long *__restrict__ queue, int tab_cap, PlainOut out) {
  typedef PlainAcc<true> Acc;
  constexpr int KT = 256 / JB;
  constexpr int kPKC = plain_chunk(JB), kPRow = kPKC + 16;
  constexpr int kRowsI = 2 * kPI, kRowsJ = 2 * JB, kRowsK = 2 * KT;
  constexpr int kRows = kRowsI + kRowsJ + kRowsK;
  constexpr int kBuf = kRows * kPRow + kPlanePad;
  constexpr int kPieces = kPKC / 16;
  constexpr int kPer = (kRows * kPieces + 255) / 256;
  constexpr int NBP = KT / 32;  // 32-wide k blocks; the 4 waves are (JB / 2) x NBP
  constexpr int kSteps = kPKC / 32;
  static_assert((JB / 2) * NBP == 4, "four waves per tile");
  static_assert(2 * kBuf == plain_stage_bytes<JB>() && 2 * kBuf % 16 == 0, "LDS layout");
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  uint8_t *stage = reinterpret_cast<uint8_t *>(lds + tab_cap);
  int64_t *sTile = reinterpret_cast<int64_t *>(stage + 2 * kBuf);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wj = wave / NBP, wb = wave - wj * NBP;
  const int r = lane & 31, g = lane >> 5;
  typedef int i4e __attribute__((ext_vector_type(4)));
  cptr<int64_t> job_begin = as_const(job_begin_p);
  JobDecoder jd;
  int M = 0, Mp = 0, nJ = 0, nch0 = 0, nch = 0;
  uint32_t Sb = 0, cls1 = 0, MpMp = 0, lim = 0, Npk = 0;
  gptr<uint8_t> gv = nullptr;
  cptr<int64_t> pre = nullptr;
  gptr<i4e> pr = nullptr;
  const uint32_t *lfx = nullptr;
  float scale = 1.f;
  float *score = nullptr;
  uint32_t *keyrange = nullptr;
  uint32_t kmin = 0xffffffffu, kmax = 0u;  // this thread's scores of the current job
  TileDecoder dec;
  const float ub = MODE == kPermOutBounded ? out.st->ub : 0.f;
  uint4 *stash = stash_p + (int64_t)blockIdx.x * (kPlainStash / 16) + wave * 1024;  // [16][lane]
  // lane roles: A row r = 4 i8 + 2 a + b; B column r = k (one plane per tile)
  const int ra = (r >> 1) & 1, rb = r & 1;
  const int o_xi = (r & ~1) * kPRow + 16 * g;  // i-block 0; block 1 is the next row
  const int o_xj = (kRowsI + 2 * (2 * wj + ra) + rb) * kPRow + 16 * g;
  const int o_b0 = (kRowsI + kRowsJ + 32 * wb + r) * kPRow + 16 * g;
  const int o_b1 = o_b0 + KT * kPRow + kPlanePad;

  // Consecutive tiles share operand rows: an XCD's slots are contiguous.  The
  // next tile is drawn between the classes and not ahead of the tile, so that it
  // goes to a workgroup that gets to it sooner: 590 -> 584 us at 512 x 4096,
  // 4.28 -> 4.25 ms at 1003 x 6007.
  TileSlots<unsigned> slots{queue, n_tiles, 0, (int)(blockIdx.x & 7)};
  // (i0, j0, k0) of tile t of the current job
  int i0 = 0, j0 = 0, k0 = 0;
  auto place = [&](int64_t t) {
    dec.find(pre, nJ, t);
    plain_tile_origin(dec, t, M, JB, i0, j0, k0);
    i0 = rfl(i0);
    j0 = rfl(j0);
    k0 = rfl(k0);
  };
  // Staged rows: [0, 32) X_i, then 2 JB rows X_j, then 2 KT rows X_k; SNP x's
  // planes are rows 2 x and 2 x + 1 of the value planes.  Piece u of a thread
  // is 16 bytes of row tid / kPieces + kStep u.  The i, j and k rows begin at
  // multiples of a wave's rows, so every piece is a wave-uniform base plus one
  // per-thread offset that is the same for all pieces.
  // In LDS the rows lie in the order in which consecutive lanes read them
  // (rows 36 words apart: no bank conflict among 16): X_i[a] of i-block b at
  // row 4 (i % 8) + 2 a + b, the k rows plane by plane.
  constexpr int kStep = 256 / kPieces, kWaveRows = 64 / kPieces;
  static_assert(kRowsI == kStep && kWaveRows == 8 && kRowsJ % 8 == 0 && kRowsK % 8 == 0,
                "a wave's 8 rows of a piece belong to one of i, j, k; piece 0 is i");
  uint32_t thr = 0;  // this thread's row and column within the staged rows, in bytes
  const int l_col = (lane & 7) * 16;
  const int l_i = (4 * (lane >> 4) + 2 * ((lane >> 3) & 1)) * kPRow + l_col;
  const int l_j = (lane >> 3) * kPRow + l_col;
  const int l_k = ((lane >> 3) & 1) * (KT * kPRow + kPlanePad) + (lane >> 4) * kPRow + l_col;
  auto has_piece = [&](int u) { return kWaveRows * wave + kStep * u < kRows; };  // wave-uniform
  v4i pf[kPer];
  auto fetch = [&](int ch) {
    const uint32_t c0 = ch < nch0 ? (uint32_t)ch * kPKC : cls1 + (uint32_t)(ch - nch0) * kPKC;
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if (has_piece(u)) {
        const int row = kWaveRows * wave + kStep * u;  // the wave's first row of this piece
        const int base = row < kRowsI ? 2 * i0 : row < kRowsI + kRowsJ ? 2 * j0 - kRowsI : 2 * k0 - kRowsI - kRowsJ;
        // (the row offset base + kStep u may be negative alone, never with thr's row)
        const int64_t o = (int64_t)(base + kStep * u) * Sb + c0;
        pf[u] = *reinterpret_cast<gptr<v4i>>(gv + o + thr);
      }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if (has_piece(u)) {
        const int row = kWaveRows * wave + kStep * u;  // the wave's first row of this piece
        uint8_t *dst = stage + buf * kBuf;
        if (u == 0)
          dst += (16 * (wave & 1) + (wave >> 1)) * kPRow + l_i;
        else if (row < kRowsI + kRowsJ)
          dst += row * kPRow + l_j;
        else
          dst += (kRowsI + kRowsJ + (row - kRowsI - kRowsJ) / 2) * kPRow + l_k;
        *reinterpret_cast<v4i *>(dst) = pf[u];
      }
  };

  if (wave == 0) slots.first(sTile);
  __syncthreads();
  int64_t slot = rfl64q(sTile[0]);
  bool loaded = false;  // the current tile's origin is set and its first chunk is in pf
  while (slot < n_tiles) {
    __builtin_amdgcn_s_setprio(0);
    if (!loaded) {
      const int64_t tg = tile_begin + slot * stride;
      if (jd.find(job_begin, n_jobs, tg)) {
        if (keyrange) flush_range(kmin, kmax, keyrange);
        kmin = 0xffffffffu;
        kmax = 0u;
        const PlainJob &pj = jobs[jd.x];
        M = rfl(pj.M);
        Mp = rfl(pj.Mp);
        Sb = (uint32_t)rfl(pj.Sb);
        nch0 = (rfl(pj.Sb0) + kPKC - 1) / kPKC;
        nch = nch0 + (rfl(pj.Sb1) + kPKC - 1) / kPKC;
        cls1 = (uint32_t)Mp * 2u * Sb;
        thr = (uint32_t)(tid / kPieces) * Sb + (uint32_t)(tid % kPieces) * 16u;
        MpMp = (uint32_t)Mp * (uint32_t)Mp;
        Npk = (uint32_t)rfl(pj.N0) | ((uint32_t)rfl(pj.N0 + pj.N1) << 16);
        nJ = (int)plain_jblocks(M, JB);
        gv = (gptr<uint8_t>)rflp(pj.vals);
        pre = as_const(rflp(pj.jprefix));
        pr = (gptr<i4e>)rflp(pj.pairs);
        lfx = rflp(pj.lfx);
        scale = __int_as_float(rfl(__float_as_int(pj.scale)));
        score = rflp(pj.score);
        keyrange = MODE == kPermOutSample ? out.range : rflp(pj.keyrange);
        lim = (uint32_t)(pj.lf_len < tab_cap ? pj.lf_len : tab_cap);
        dec.J = -1;
        table_to_lds<256>(lds, lfx, (int)lim);  // barrier below
      }
      place(tg - jd.lo);
      fetch(0);
    }
    unsigned drawn = 0u;  // thread 0: for the next tile, drawn between the classes
    typename Acc::type acc[2][2][2];  // [i-block][j of the pair][plane of k]
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[x][y][z][v] = 8388608.f;
    // the low halves of triplet (x, y, u)'s 8 accumulators: words 4 (a, b) of
    // plane 0, of plane 1
    auto cells = [&](int x, int y, int u) {
      uint32_t w[4];
#pragma unroll
      for (int h = 0; h < 4; ++h)
        w[h] = __builtin_amdgcn_perm(__float_as_uint(acc[x][y][h >> 1][4 * u + 2 * (h & 1) + 1]),
                                     __float_as_uint(acc[x][y][h >> 1][4 * u + 2 * (h & 1)]),
                                     0x05040100u);
      return make_uint4(w[0], w[1], w[2], w[3]);
    };
    auto keep = [&]() {
      uint32_t lo = (uint32_t)lane;  // opaque: the addresses are formed here, not held through the tile
      asm volatile("" : "+v"(lo));
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int y = 0; y < 2; ++y) (stash + (8 * x + 2 * u + y) * 64)[lo] = cells(x, y, u);
    };
    store(0);
    __syncthreads();
#define EPI3_PLD(BB, STP, XI, XJ, B0, B1)                                           \
    XI = *reinterpret_cast<const v4i *>((BB) + o_xi + 32 * (STP));                \
    XI##1 = *reinterpret_cast<const v4i *>((BB) + o_xi + kPRow + 32 * (STP));     \
    XJ = *reinterpret_cast<const v4i *>((BB) + o_xj + 32 * (STP));                \
    B0 = *reinterpret_cast<const v4i *>((BB) + o_b0 + 32 * (STP));                \
    B1 = *reinterpret_cast<const v4i *>((BB) + o_b1 + 32 * (STP));
#define EPI3_PSTEP(XI, XJ, B0, B1)                                                  \
    {                                                                             \
      const v4i xi_[2] = {XI, XI##1};                                         \
      _Pragma("unroll") for (int x = 0; x < 2; ++x) {                             \
        const v4i a0 = xi_[x] & quad_perm<0x44>(XJ);                              \
        acc[x][0][0] = Acc::mma(a0, B0, acc[x][0][0]);                            \
        acc[x][0][1] = Acc::mma(a0, B1, acc[x][0][1]);                            \
        const v4i a1 = xi_[x] & quad_perm<0xEE>(XJ);                              \
        acc[x][1][0] = Acc::mma(a1, B0, acc[x][1][0]);                            \
        acc[x][1][1] = Acc::mma(a1, B1, acc[x][1][1]);                            \
      }                                                                           \
    }
    __builtin_amdgcn_sched_barrier(0);
    // software pipeline over the steps of a chunk (operand sets X and Y in
    // turn; the next chunk is stored before the last step)
    v4i xiX, xiX1, xjX, b0X, b1X, xiY, xiY1, xjY, b0Y, b1Y;
    EPI3_PLD(stage, 0, xiX, xjX, b0X, b1X)
    for (int ch = 0; ch < nch; ++ch) {
      const bool more = ch + 1 < nch;
      if (ch == nch0) {
        keep();
        if (tid == 0) drawn = slots.draw();
      }
      if (more) fetch(ch + 1);
      const uint8_t *buf = stage + (ch & 1) * kBuf;
      const uint8_t *nbuf = stage + ((ch + 1) & 1) * kBuf;
      EPI3_PLD(buf, 1, xiY, xjY, b0Y, b1Y)
      EPI3_PSTEP(xiX, xjX, b0X, b1X)
      if constexpr (kSteps == 4) {
        __builtin_amdgcn_sched_barrier(0);
        EPI3_PLD(buf, 2, xiX, xjX, b0X, b1X)
        EPI3_PSTEP(xiY, xjY, b0Y, b1Y)
        __builtin_amdgcn_sched_barrier(0);
        EPI3_PLD(buf, 3, xiY, xjY, b0Y, b1Y)
        EPI3_PSTEP(xiX, xjX, b0X, b1X)
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) asm volatile("" : "+v"(acc[x][y][0]), "+v"(acc[x][y][1]));
      if (more) store((ch + 1) & 1);
      __syncthreads();
      // after the last chunk this reads the other buffer's stale contents,
      // which no product uses
      EPI3_PLD(nbuf, 0, xiX, xjX, b0X, b1X)
      EPI3_PSTEP(xiY, xjY, b0Y, b1Y)
    }
#undef EPI3_PLD
#undef EPI3_PSTEP
    if (nch == nch0) {
      keep();
      if (tid == 0) drawn = slots.draw();
    }
    if (wave == 0) slots.find(drawn, sTile);
    __syncthreads();  // the staging buffers are idle from here to the next tile
    // a scoring wave issues ahead of the other workgroup's counting waves: its
    // lookups keep the LDS busy, and the products still fit between
    __builtin_amdgcn_s_setprio(1);

    const int64_t sslot = slot;
    const int si0 = i0, jb = j0 + 2 * wj, kb = k0 + 32 * wb;
    slot = rfl64q(sTile[0]);
    // the next tile's first chunk, loaded towards the end of the scoring
    auto next = [&]() {
      loaded = false;
#pragma unroll
      for (int u = 0; u < kPer; ++u) pf[u] = v4i{};  // (ends the old chunk's live range)
      if (slot < n_tiles) {
        const int64_t tg = tile_begin + slot * stride;
        if (tg >= jd.lo && tg < jd.hi) {  // (another job needs its own table first)
          place(tg - jd.lo);
          fetch(0);
          loaded = true;
        }
      }
    };

    // ---- tables and scores ----
    // lane values made opaque again: what is derived from them below is formed
    // here and not held in registers through the counts
    int ln = lane;
    uint32_t two = 2u;
    asm volatile("" : "+v"(ln), "+v"(two));
    const int r = ln & 31, g = ln >> 5;
    const int k = kb + r, kc = k < Mp ? k : Mp - 1;
    const int i_end = kb < M ? jb + 1 - si0 : 0;  // first i (from si0) without a triplet here
    if (i_end > 0) {  // wave-uniform
    struct Raw { i4e a, b; };       // a pair's entries of both classes
    auto load2 = [&](uint32_t row, uint32_t col) {
      const uint32_t e = row * (uint32_t)Mp + col;
      return Raw{pr[e], pr[MpMp + e]};
    };
    // -> (class 0 | all << 16) per cell
    auto pack2 = [&](const Raw &w, u16x2 v[4]) {
      v[0] = as_u16x2((uint32_t)w.a.x | ((uint32_t)(w.a.x + w.b.x) << 16));
      v[1] = as_u16x2((uint32_t)w.a.y | ((uint32_t)(w.a.y + w.b.y) << 16));
      v[2] = as_u16x2((uint32_t)w.a.z | ((uint32_t)(w.a.z + w.b.z) << 16));
      v[3] = as_u16x2((uint32_t)w.a.w | ((uint32_t)(w.a.w + w.b.w) << 16));
    };
    auto pair4 = [&](uint32_t row, uint32_t col, u16x2 v[4]) { pack2(load2(row, col), v); };
    // the all-sample cells, two per register (frees half of the accumulators)
    uint4 all[2][4][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          all[x][u][y] = cells(x, y, u);
          asm volatile("" : "+v"(all[x][u][y].x), "+v"(all[x][u][y].y), "+v"(all[x][u][y].z),
                            "+v"(all[x][u][y].w));
        }
    // the next (i, k) entry and the next class-0 cells are loaded one triplet ahead
    Raw pik_n = load2((uint32_t)(si0 + g), (uint32_t)kc);
    uint4 q_n[2] = {stash[ln], (stash + 64)[ln]};
    // lane = pair (si0 + lane / 2, jb + lane % 2): its four counted cells, the
    // two (a, 2) cells and its lexicographic base, 32 bytes each, in this
    // wave's part of the buffers' end
    uint4 *pij_s = reinterpret_cast<uint4 *>(stage + 2 * kBuf - kPairBytes) + wave * 64;
    if (ln < 32) {
      u16x2 p[4], m[4];
      const int i = si0 + (ln >> 1);
      pair4((uint32_t)i, (uint32_t)(jb + (ln & 1)), p);
      pair4((uint32_t)i, (uint32_t)i, m);
      pij_s[2 * ln] = make_uint4(as_u32(p[0]), as_u32(p[1]), as_u32(p[2]), as_u32(p[3]));
      const uint64_t base = (uint64_t)lex_base(M, i, jb + (ln & 1));
      pij_s[2 * ln + 1] = make_uint4(as_u32(m[0] - p[0] - p[1]), as_u32(m[3] - p[2] - p[3]),
                                     (uint32_t)base, (uint32_t)(base >> 32));
    }
    u16x2 fjk[2][9];
    {
      u16x2 mk4[4];
      pair4((uint32_t)kc, (uint32_t)kc, mk4);
      const u16x2 mk[2] = {mk4[0], mk4[3]};
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        u16x2 p[4], m[4];
        pair4((uint32_t)(jb + y), (uint32_t)kc, p);
        pair4((uint32_t)(jb + y), (uint32_t)(jb + y), m);
        const u16x2 mj[2] = {m[0], m[3]};
        pair_cells(p, mj, mk, as_u16x2(Npk), fjk[y]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int il = 8 * x + 2 * u;
        if (il == 10) next();
        if (il >= i_end) continue;  // wave-uniform
        const int i = si0 + il + g;
        u16x2 pik[4];
        pack2(pik_n, pik);
        const uint4 q[2] = {q_n[0], q_n[1]};
        if (il + 2 < kPI) {
          pik_n = load2((uint32_t)(i + 2), (uint32_t)kc);
          q_n[0] = (stash + (il + 2) * 64)[ln];
          q_n[1] = (stash + (il + 3) * 64)[ln];
        }
        // Two triplets (j = jb, jb + 1), three rows (genotypes of i) of one
        // (b, c) at a time: completed, looked up, and added two steps later, so
        // vector instructions and lookups alternate and none waits for its
        // own result (all lookups of a triplet at once leave the LDS idle
        // while tables are completed and the vector ALU while it reads).
        uint32_t up[2] = {0u, 0u}, down[2] = {0u, 0u}, top[2] = {0u, 0u};
        uint4 pb[2];
        Lookups in_flight[2];
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const uint4 pa = pij_s[2 * (2 * (il + g) + y)], qa = all[x][u][y];
          pb[y] = pij_s[2 * (2 * (il + g) + y) + 1];
          const uint32_t pij[4] = {pa.x, pa.y, pa.z, pa.w}, pij2[2] = {pb[y].x, pb[y].y};
          const uint32_t qs[4] = {q[y].x, q[y].y, q[y].z, q[y].w}, as[4] = {qa.x, qa.y, qa.z, qa.w};
          u16x2 t[2][9];  // rows a = 0, 1: [a][3 b + c]
#pragma unroll
          for (int st = 0; st < 9; ++st) {
            constexpr int order[9] = {0, 1, 3, 4, 2, 5, 6, 7, 8};  // cells with a 2 after their parts
            const int bc = order[st], bb = bc / 3, cc = bc % 3;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
              if (bb < 2 && cc < 2) {  // counted: class 0 from the stash, all from the accumulators
                const int w = 2 * a + bb;
                t[a][bc] = as_u16x2(__builtin_amdgcn_perm(as[2 * cc + (w >> 1)], qs[2 * cc + (w >> 1)],
                                                          w & 1 ? 0x07060302u : 0x05040100u));
              } else if (bb < 2) {
                t[a][bc] = as_u16x2(pij[2 * a + bb]) - t[a][3 * bb] - t[a][3 * bb + 1];
              } else if (cc < 2) {
                t[a][bc] = pik[2 * a + cc] - t[a][cc] - t[a][3 + cc];
              } else {
                t[a][bc] = as_u16x2(pij2[a]) - t[a][6] - t[a][7];
              }
            }
            const uint32_t c[3] = {as_u32(t[0][bc]), as_u32(t[1][bc]),
                                   as_u32(fjk[y][bc] - t[0][bc] - t[1][bc])};
            if (TRUNC) {
#pragma unroll
              for (int a = 0; a < 3; ++a) top[y] = c[a] > top[y] ? c[a] : top[y];
            }
            const int n = 9 * y + st;
            if (n >= 2) {
              add_up(in_flight[n & 1], up[(n - 2) / 9], down[(n - 2) / 9]);
              // (keeps the additions of different steps apart)
              asm volatile("" : "+v"(up[(n - 2) / 9]), "+v"(down[(n - 2) / 9]));
            }
            in_flight[n & 1] = look_up(c, two);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        add_up(in_flight[0], up[1], down[1]);
        add_up(in_flight[1], up[1], down[1]);
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          uint32_t sum = up[y] - down[y];
          if (TRUNC) sum = fix_top(sum, top[y], lfx, lim);
          const float k2 = fx_score(sum, scale);
          const int j = jb + y;
          if (i < j && j < k && k < M) {
            const int64_t rank = (int64_t)(((uint64_t)pb[y].w << 32) | pb[y].z) + k;
            if (MODE == kPermOutPlane) score[rank] = k2;
            if (MODE == kPermOutSample)  // slot: the tile's triplet order (i, j, k)
              out.sample[(out.sample_base + sslot) * (int64_t)(kPI * 256) + (il + g) * 256 +
                         (2 * wj + y) * KT + 32 * wb + r] = k2;
            if (MODE == kPermOutBounded && k2 <= ub) {
              // rare (a few thousand of the C(M,3) scores): one atomic per append
              const unsigned long long pos = atomicAdd(&out.st->cn, 1ull);
              if ((int64_t)pos < out.ccap) {
                out.ckey[pos] = f2key(k2);
                out.crank[pos] = rank;
              }
            }
            const uint32_t key = f2key(k2);
            kmin = key < kmin ? key : kmin;
            kmax = key > kmax ? key : kmax;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      next();
    }
    __syncthreads();  // this tile's readers of the staging buffers and the table are done
  }
  if (keyrange) flush_range(kmin, kmax, keyrange);
}

// Completes both tables of every triplet of a pass and scores it; workgroup
// per tile (persistent, round robin).  The 256 threads are the tile's (j, k)
// and walk its 16 i, so the pair table (j, k) is completed once per tile and
// the per-SNP counts of i are wave-uniform.  Cells are carried as 4 x count
// (byte offsets into the log-factorial table, which sits at LDS address 0:
// the kernel declares no static LDS), so each of the 81 lookups per triplet
// needs at most one add.  The table is the job's own (its fixed-point step
// depends on its samples) and reloaded when the job changes.
template <int JB, bool LDS, bool COUNTS, int MODE>
__global__ void __launch_bounds__(256) finish_plain_kernel(const PlainJob *__restrict__ jobs,
                                                           const int64_t *__restrict__ job_begin_p,
                                                           int n_jobs,
                                                           const uint4 *__restrict__ corners,
                                                           int64_t tile_begin, int64_t n_tiles,
                                                           PlainOut out) {
  constexpr int KT = 256 / JB;
  constexpr int kTile = kPI * JB * KT;  // 4096 triplets
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  typedef int i4e __attribute__((ext_vector_type(4)));
  typedef unsigned u4e __attribute__((ext_vector_type(4)));
  cptr<int64_t> job_begin = as_const(job_begin_p);
  JobDecoder jd;
  int M = 0, Mp = 0, nJ = 0, Nx4[2] = {0, 0};
  uint32_t MpMp = 0;  // pair tables < 4 G entries
  cptr<int64_t> pre = nullptr;
  gptr<i4e> pr = nullptr;
  cptr<i4e> prc = nullptr;
  const uint32_t *lfx = nullptr;
  float scale = 1.f;
  float *score = nullptr;
  uint32_t *counts = nullptr, *keyrange = nullptr;
  // key range of this thread's scores of the current job (flushed per job)
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  TileDecoder dec;
  // bounded: this launch's append bound (set before the launch)
  const float ub = MODE == kPermOutBounded ? out.st->ub : 0.f;
  const int kl = threadIdx.x % KT, jl = threadIdx.x / KT;
  for (int64_t slot = blockIdx.x; slot < n_tiles; slot += gridDim.x) {
    const int64_t tg = tile_begin + slot * out.stride;
    if (jd.find(job_begin, n_jobs, tg)) {
      if (keyrange) flush_range(kmin, kmax, keyrange);
      kmin = 0xffffffffu;
      kmax = 0u;
      const PlainJob &pj = jobs[jd.x];
      M = pj.M;
      Mp = pj.Mp;
      nJ = (int)plain_jblocks(M, JB);
      Nx4[0] = pj.N0 << 2;
      Nx4[1] = pj.N1 << 2;
      MpMp = (uint32_t)Mp * (uint32_t)Mp;
      pre = as_const(pj.jprefix);
      pr = (gptr<i4e>)pj.pairs;
      prc = as_const(reinterpret_cast<const i4e *>(pj.pairs));
      lfx = pj.lfx;
      scale = pj.scale;
      score = pj.score;
      counts = pj.counts;
      keyrange = MODE == kPermOutSample ? out.range : pj.keyrange;
      dec.J = -1;
      if (LDS) {
        __syncthreads();  // the previous job's lookups are done
        table_to_lds<256>(lds, lfx, pj.lf_len);
        __syncthreads();
      }
    }
    const int64_t t = tg - jd.lo;  // tile within its job
    dec.find(pre, nJ, t);
    int i0, j0, k0;
    plain_tile_origin(dec, t, M, JB, i0, j0, k0);
    i0 = __builtin_amdgcn_readfirstlane(i0);
    gptr<u4e> cor = (gptr<u4e>)(corners + slot * 2 * (int64_t)kTile);
    const int j = j0 + jl, k = k0 + kl;
    const bool pair = j < k && k < M;
    if (!COUNTS && !pair) continue;
    int fjk[2][9];
    if (pair) {  // (tiles of 128 k reach past the padded stride)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const uint32_t cb = (uint32_t)c * MpMp;
        const i4e c4 = pr[cb + (uint32_t)j * Mp + k];
        const i4e jj = pr[cb + (uint32_t)j * Mp + j], kk = pr[cb + (uint32_t)k * Mp + k];
        const int pjk[4] = {c4.x << 2, c4.y << 2, c4.z << 2, c4.w << 2};
        const int mj[2] = {jj.x << 2, jj.w << 2}, mk[2] = {kk.x << 2, kk.w << 2};
        pair_cells(pjk, mj, mk, Nx4[c], fjk[c]);
      }
    }
    for (int il = 0; il < kPI; ++il) {
      const int i = i0 + il;
      if (COUNTS) {
        // Tables out: the waves stay together.  Each writes 216-byte tables a few
        // bytes at a time, and where they drift apart the parts of neighbouring
        // tables no longer meet in L2 (512 x 4096, whole call: 3.10 to 3.31 ms without
        // a barrier, with one to three workgroups per CU, 2.88 with one per tile, 2.58
        // with one per two i).
        if (il % 2 == 0) __syncthreads();
        if (!pair || i >= j) continue;
      } else if (i >= j) {
        break;
      }
      const int x = il * 256 + threadIdx.x;
      int tab[2][27];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const u4e q = cor[c * kTile + x];
        // record order: [plane of k][a][b] -> corner index 4 a + 2 b + plane; x 4
        const uint32_t n[8] = {(q.x << 2) & 0x3fffcu, (q.z << 2) & 0x3fffcu,
                               (q.x >> 14) & 0x3fffcu, (q.z >> 14) & 0x3fffcu,
                               (q.y << 2) & 0x3fffcu, (q.w << 2) & 0x3fffcu,
                               (q.y >> 14) & 0x3fffcu, (q.w >> 14) & 0x3fffcu};
        const uint32_t cb = (uint32_t)c * MpMp + (uint32_t)i * Mp;
        const i4e a4 = pr[cb + j], b4 = pr[cb + k], ii = prc[cb + i];
        const int pij[4] = {a4.x << 2, a4.y << 2, a4.z << 2, a4.w << 2};
        const int pij2[2] = {(ii.x << 2) - pij[0] - pij[1], (ii.w << 2) - pij[2] - pij[3]};
        const int pik[4] = {b4.x << 2, b4.y << 2, b4.z << 2, b4.w << 2};
        complete27(n, fjk[c], pij, pij2, pik, tab[c]);
      }
      const float k2 = fx_score(fx_sum<27, LDS>(tab[0], tab[1], lfx), scale);
      const int64_t rank = lex_base(M, i, j) + k;
      if (MODE == kPermOutPlane) score[rank] = k2;
      if (MODE == kPermOutSample) out.sample[(out.sample_base + slot) * kTile + x] = k2;
      if (MODE == kPermOutBounded && k2 <= ub) {
        // rare (a few thousand of the C(M,3) scores): one atomic per append
        const unsigned long long pos = atomicAdd(&out.st->cn, 1ull);
        if ((int64_t)pos < out.ccap) {
          out.ckey[pos] = f2key(k2);
          out.crank[pos] = rank;
        }
      }
      if (COUNTS) {
        uint32_t *o = counts + rank * 54;
        for (int x2 = 0; x2 < 27; ++x2) {
          o[x2] = (uint32_t)tab[0][x2] >> 2;
          o[27 + x2] = (uint32_t)tab[1][x2] >> 2;
        }
      }
      const uint32_t key = f2key(k2);
      kmin = key < kmin ? key : kmin;
      kmax = key > kmax ? key : kmax;
    }
  }
  if (keyrange) flush_range(kmin, kmax, keyrange);
}

}  // namespace

int64_t host_plain_tiles(int64_t M, int JB) {
  int64_t n = 0;
  const int64_t nJ = plain_jblocks(M, JB);
  for (int64_t J = 0; J < nJ; ++J) n += plain_tiles_of_jb(M, J, JB);
  return n;
}

hipError_t launch_plain_setup(const PlainJob *h, const int64_t *begin, int32_t n, PlainJob *dst_dev,
                              int64_t *job_begin_dev, unsigned long long *queue, hipStream_t s) {
  for (int x = 0; x < n; x += kPlainJobsPerLaunch) {
    PlainJobs jobs{};
    const int m = n - x < kPlainJobsPerLaunch ? n - x : kPlainJobsPerLaunch;
    for (int y = 0; y < m; ++y) jobs.j[y] = h[x + y];
    for (int y = 0; y <= m; ++y) jobs.begin[y] = begin[x + y];
    hipLaunchKernelGGL(plain_setup_kernel, dim3(m), dim3(1024), 0, s, jobs, dst_dev + x,
                       job_begin_dev + x, queue);
  }
  return hipGetLastError();
}

static hipError_t cu_count(int *n_cu) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return hipDeviceGetAttribute(n_cu, hipDeviceAttributeMultiprocessorCount, dev);
}

template <bool FP4, int JB>
static hipError_t launch_plain_count_t(const PlainJob *jobs, const int64_t *job_begin, int n_jobs,
                                       uint4 *corners, int64_t tile_begin, int64_t n,
                                       int64_t stride, unsigned long long *queue, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int n_cu = 0;
  hipError_t e = cu_count(&n_cu);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, count_mfma_plain_kernel<FP4, JB>, 256, 0);
  if (e != hipSuccess) return e;
  if (per_cu <= 0) per_cu = 1;
  int64_t blocks = (int64_t)n_cu * per_cu;
  if (blocks > n) blocks = n;
  hipLaunchKernelGGL((count_mfma_plain_kernel<FP4, JB>), dim3((unsigned)blocks), dim3(256), 0, s,
                     jobs, job_begin, n_jobs, corners, tile_begin, n, stride, queue);
  return hipGetLastError();
}

hipError_t launch_count_mfma_plain(const PlainJob *jobs, const int64_t *job_begin, int32_t n_jobs,
                                   int JB, bool fp4, uint4 *corners, int64_t tile_begin,
                                   int64_t n_tiles, int64_t stride, unsigned long long *queue,
                                   hipStream_t s) {
  if (stride < 1) return hipErrorInvalidValue;
  switch (JB) {
    case 2:
      return fp4 ? launch_plain_count_t<true, 2>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, stride, queue, s)
                 : launch_plain_count_t<false, 2>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, stride, queue, s);
    case 4:
      return fp4 ? launch_plain_count_t<true, 4>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, stride, queue, s)
                 : launch_plain_count_t<false, 4>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, stride, queue, s);
    case 8:
      return fp4 ? launch_plain_count_t<true, 8>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, stride, queue, s)
                 : launch_plain_count_t<false, 8>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, stride, queue, s);
  }
  return hipErrorInvalidValue;
}

template <int JB, bool TRUNC, int MODE>
static hipError_t launch_fused_t(const PlainJob *jobs, const int64_t *job_begin, int n_jobs,
                                 void *stash, int64_t max_blocks, int64_t tile_begin, int64_t n,
                                 int64_t stride, unsigned long long *queue, int32_t lf_len,
                                 const PlainOut &out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int n_cu = 0;
  hipError_t e = cu_count(&n_cu);
  if (e != hipSuccess) return e;
  auto kern = count_score_plain_kernel<JB, TRUNC, MODE>;
  const int32_t cap = TRUNC ? plain_fused_entries<JB>() : (lf_len + 3) / 4 * 4;
  const size_t lds = (size_t)cap * 4 + plain_stage_bytes<JB>() + 16;
  e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, lds);
  if (e != hipSuccess) return e;
  if (per_cu <= 0) per_cu = 1;
  int64_t blocks = (int64_t)n_cu * per_cu;
  if (blocks > n) blocks = n;
  if (blocks > max_blocks) blocks = max_blocks;
  if (blocks < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), lds, s, jobs, job_begin, n_jobs,
                     static_cast<uint4 *>(stash), tile_begin, n, stride, queue, cap, out);
  return hipGetLastError();
}

// Tables longer than the LDS holds beside the staging keep their first
// entries there: at most one row of a triplet's table can need another as
// long as those cover half of the samples; the cover of 7/10 taken here keeps
// the lookups clear of what the waves write.  The corrected rows cost little,
// also where nearly every triplet has one (rare alleles): 2048 x 16384 with
// minor allele frequencies of 0.01 to 0.5, 0.01 to 0.05 and 0.001 to 0.01 67.7,
// 66.1 and 65.8 ms (two kernels with the whole table: 85.7, 82.4, 82.0), 512 x
// 12400 1.13, 1.09, 1.09 ms (1.51, 1.45, 1.45).  16-bit counts.  The lookups
// that a longer table would need end before the words that the waves write
// while scoring.
template <int JB>
static bool fused_ok_t(int32_t lf_len) {
  return lf_len - 2 <= 65535 && lf_len <= plain_fused_longest<JB>() && plain_lookups_ok<JB>(lf_len);
}

bool plain_fused_ok(int JB, int32_t lf_len) {
  return JB == 8 ? fused_ok_t<8>(lf_len) : JB == 4 && fused_ok_t<4>(lf_len);
}

template <int JB, bool TRUNC>
static hipError_t launch_fused_m(const PlainJob *jobs, const int64_t *job_begin, int n_jobs,
                                 void *stash, int64_t max_blocks, int64_t tile_begin, int64_t n,
                                 int64_t stride, unsigned long long *queue, int32_t lf_len,
                                 const PlainOut &out, hipStream_t s) {
  switch (out.mode) {
    case kPermOutPlane:
      return launch_fused_t<JB, TRUNC, kPermOutPlane>(jobs, job_begin, n_jobs, stash, max_blocks, tile_begin, n, stride, queue, lf_len, out, s);
    case kPermOutSample:
      return launch_fused_t<JB, TRUNC, kPermOutSample>(jobs, job_begin, n_jobs, stash, max_blocks, tile_begin, n, stride, queue, lf_len, out, s);
    case kPermOutBounded:
      return launch_fused_t<JB, TRUNC, kPermOutBounded>(jobs, job_begin, n_jobs, stash, max_blocks, tile_begin, n, stride, queue, lf_len, out, s);
  }
  return hipErrorInvalidValue;
}

template <int JB>
static hipError_t launch_fused_j(const PlainJob *jobs, const int64_t *job_begin, int n_jobs,
                                 void *stash, int64_t max_blocks, int64_t tile_begin, int64_t n,
                                 int64_t stride, unsigned long long *queue, int32_t lf_len,
                                 const PlainOut &out, hipStream_t s) {
  return lf_len <= plain_fused_entries<JB>()
             ? launch_fused_m<JB, false>(jobs, job_begin, n_jobs, stash, max_blocks, tile_begin, n, stride, queue, lf_len, out, s)
             : launch_fused_m<JB, true>(jobs, job_begin, n_jobs, stash, max_blocks, tile_begin, n, stride, queue, lf_len, out, s);
}

hipError_t launch_count_score_plain(const PlainJob *jobs, const int64_t *job_begin, int32_t n_jobs,
                                    int JB, void *stash, int64_t max_blocks, int64_t tile_begin,
                                    int64_t n_tiles, int64_t stride, unsigned long long *queue,
                                    int32_t lf_len, const PlainOut &out, hipStream_t s) {
  if (stride < 1 || !plain_fused_ok(JB, lf_len)) return hipErrorInvalidValue;
  switch (JB) {
    case 4: return launch_fused_j<4>(jobs, job_begin, n_jobs, stash, max_blocks, tile_begin, n_tiles, stride, queue, lf_len, out, s);
    case 8: return launch_fused_j<8>(jobs, job_begin, n_jobs, stash, max_blocks, tile_begin, n_tiles, stride, queue, lf_len, out, s);
  }
  return hipErrorInvalidValue;
}

template <int JB, bool LDS, bool COUNTS, int MODE>
static hipError_t launch_finish_plain_t(const PlainJob *jobs, const int64_t *job_begin, int n_jobs,
                                        const uint4 *corners, int64_t tile_begin, int64_t n,
                                        int32_t lf_len, const PlainOut &out,
                                        hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int n_cu = 0;
  hipError_t e = cu_count(&n_cu);
  if (e != hipSuccess) return e;
  const size_t lds = LDS ? (size_t)(lf_len * 4 + 15) / 16 * 16 : 0;
  auto kern = finish_plain_kernel<JB, LDS, COUNTS, MODE>;
  e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, lds);
  if (e != hipSuccess) return e;
  if (per_cu <= 0) per_cu = 1;
  int64_t blocks = (int64_t)n_cu * per_cu;
  if (blocks > n) blocks = n;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), lds, s, jobs, job_begin, n_jobs,
                     corners, tile_begin, n, out);
  return hipGetLastError();
}

template <int JB, bool LDS>
static hipError_t launch_finish_plain_l(const PlainJob *jobs, const int64_t *job_begin, int n_jobs,
                                        const uint4 *corners, int64_t tile_begin, int64_t n,
                                        int32_t lf_len, bool counts,
                                        const PlainOut &out, hipStream_t s) {
  switch (out.mode) {
    case kPermOutPlane:
      return counts ? launch_finish_plain_t<JB, LDS, true, kPermOutPlane>(jobs, job_begin, n_jobs, corners, tile_begin, n, lf_len, out, s)
                    : launch_finish_plain_t<JB, LDS, false, kPermOutPlane>(jobs, job_begin, n_jobs, corners, tile_begin, n, lf_len, out, s);
    case kPermOutSample:
      return launch_finish_plain_t<JB, LDS, false, kPermOutSample>(jobs, job_begin, n_jobs, corners, tile_begin, n, lf_len, out, s);
    case kPermOutBounded:
      return launch_finish_plain_t<JB, LDS, false, kPermOutBounded>(jobs, job_begin, n_jobs, corners, tile_begin, n, lf_len, out, s);
  }
  return hipErrorInvalidValue;
}

template <int JB>
static hipError_t launch_finish_plain_j(const PlainJob *jobs, const int64_t *job_begin, int n_jobs,
                                        const uint4 *corners, int64_t tile_begin, int64_t n,
                                        int32_t lf_len, bool counts,
                                        const PlainOut &out, hipStream_t s) {
  return lf_in_lds(lf_len)
             ? launch_finish_plain_l<JB, true>(jobs, job_begin, n_jobs, corners, tile_begin, n, lf_len, counts, out, s)
             : launch_finish_plain_l<JB, false>(jobs, job_begin, n_jobs, corners, tile_begin, n, lf_len, counts, out, s);
}

hipError_t launch_finish_plain(const PlainJob *jobs, const int64_t *job_begin, int32_t n_jobs,
                               int JB, const uint4 *corners, int64_t tile_begin, int64_t n_tiles,
                               int32_t lf_len, bool counts, const PlainOut &out,
                               hipStream_t s) {
  if (out.stride < 1 || (counts && out.mode != kPermOutPlane)) return hipErrorInvalidValue;
  switch (JB) {
    case 2: return launch_finish_plain_j<2>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, lf_len, counts, out, s);
    case 4: return launch_finish_plain_j<4>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, lf_len, counts, out, s);
    case 8: return launch_finish_plain_j<8>(jobs, job_begin, n_jobs, corners, tile_begin, n_tiles, lf_len, counts, out, s);
  }
  return hipErrorInvalidValue;
}

int64_t host_plain_sample_valid(int64_t M, int JB, int64_t stride, int64_t *n_sample) {
  const int KT = 256 / JB;
  const int64_t nJ = plain_jblocks(M, JB);
  int64_t t0 = 0, valid = 0, ns = 0;
  for (int64_t J = 0; J < nJ; ++J) {
    const int64_t nt = plain_tiles_of_jb(M, J, JB);
    if (nt == 0) continue;
    const int64_t j0 = J * JB;
    const int64_t nkb = (M - 1 - j0 + KT - 1) / KT;
    // sampled tiles of this j-block: the multiples of stride in [t0, t0 + nt)
    for (int64_t t = (t0 + stride - 1) / stride * stride; t < t0 + nt; t += stride) {
      ++ns;
      int ib = 0, kb = 0;
      plain_tile_ib_kb((int)(t - t0), M, J, JB, (int)nkb, ib, kb);
      const int64_t i0 = (int64_t)ib * kPI, k0 = j0 + 1 + kb * KT;
      for (int64_t j = j0; j < j0 + JB && j < M; ++j) {
        const int64_t ni = std::max<int64_t>(0, std::min<int64_t>(i0 + kPI, j) - i0);
        const int64_t klo = std::max<int64_t>(k0, j + 1), khi = std::min<int64_t>(k0 + KT, M);
        valid += ni * std::max<int64_t>(0, khi - klo);
      }
    }
    t0 += nt;
  }
  if (n_sample) *n_sample = ns;
  return valid;
}

}  // namespace epi3
