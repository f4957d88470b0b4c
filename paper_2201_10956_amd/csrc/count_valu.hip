// Count stage on the vector ALU: AND + popcount over bit-planes, fused with
// the K2 score.
//
// Paper, Alg. 2 and the GPU approaches section: every combination i < j < k
// gets a private frequency table in registers, filled over all samples of
// both classes, then scored.  Differences from the paper's kernel:
//   * a wave owns P pivot pairs (i, j) with j wave-uniform and 64 lanes own
//     64 consecutive k > j, so the pair words X_i[a] & X_j[b] are formed once
//     per 32 samples on the scalar unit and shared by all lanes;
//   * only the 8 cells with genotypes in {0,1}^3 are counted (8 AND + 8
//     v_bcnt per triplet and 32 samples); the other 19 cells of each class
//     follow exactly from the pairwise tables and the class size (every
//     sample falls in exactly one of the 27 rows), so the table is the same
//     integer table the paper fills with 27 AND/POPCNT per word;
//   * a persistent grid pulls tiles (job, j, i-block, k-block) from an atomic
//     queue, which also serves batches of data sets of different shape.
#include "epi3_internal.h"

namespace epi3 {

__device__ __forceinline__ int64_t rfl64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Tiles of pivot j: ceil(j / P) i-blocks x ceil((M - 1 - j) / 64) k-blocks.
__host__ __device__ __forceinline__ int64_t tiles_of_j(int64_t M, int64_t j, int P) {
  if (j < 1 || j > M - 2) return 0;
  return ((j + P - 1) / P) * ((M - 1 - j + 63) / 64);
}

// The job records (by value), jprefix[j] = job-local tiles before pivot j,
// jprefix[M] = total, one block per job, and a clear tile queue.
struct Jobs {
  Job j[kJobsPerLaunch];
};
static_assert(sizeof(Jobs) <= 3968, "kernel argument block");
__global__ void __launch_bounds__(1024) valu_setup_kernel(Jobs jobs, Job *dst, unsigned long long *queue) {
  const Job &J = jobs.j[blockIdx.x];
  if (threadIdx.x == 0) dst[blockIdx.x] = J;
  if (blockIdx.x == 0 && threadIdx.x == 0) *queue = 0ull;
  const int64_t M = J.M;
  const int P = J.P;
  int64_t *pre = const_cast<int64_t *>(J.jprefix);
  __shared__ int64_t part[1024];
  const int t = threadIdx.x;
  const int64_t chunk = (M + 1023) / 1024;
  const int64_t a = t * chunk, b = (a + chunk < M) ? a + chunk : M;
  int64_t sum = 0;
  for (int64_t j = a; j < b; ++j) sum += tiles_of_j(M, j, P);
  part[t] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int64_t v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int64_t run = part[t] - sum;  // exclusive prefix of this chunk
  for (int64_t j = a; j < b; ++j) {
    pre[j] = run;
    run += tiles_of_j(M, j, P);
  }
  if (t == 1023) pre[M] = part[1023];
}

// acc + popcount(x) as one v_bcnt_u32_b32.  Written out because the compiler
// may otherwise reassociate the sums of an unrolled loop into v_bcnt(x, 0)
// plus v_add3, one more VALU op per two counts.
__device__ __forceinline__ uint32_t bcnt_acc(uint32_t x, uint32_t acc) {
  uint32_t r;
  asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
  return r;
}

// Accumulate the 8 corner cells of P pairs over words [w0, w1).
// acc[t][4a + 2b + c] += popcount(X_{i0+t}[a] & X_j[b] & X_k[c]).
template <int P>
__device__ __forceinline__ void accumulate(uint32_t (&acc)[P][8], const uint32_t *planes,
                                           int64_t Mp, int w0, int w1, int i0, int j, int k) {
  cptr<uint32_t> pc = as_const(planes);
  const uint2 *pv = reinterpret_cast<const uint2 *>(planes);
#pragma unroll 2
  for (int w = w0; w < w1; ++w) {
    const int64_t rowbase = (int64_t)w * Mp;
    const uint2 xk = pv[rowbase + k];
    const uint32_t xj0 = pc[(rowbase + j) * 2], xj1 = pc[(rowbase + j) * 2 + 1];
#pragma unroll
    for (int t = 0; t < P; ++t) {
      const uint32_t xi0 = pc[(rowbase + i0 + t) * 2], xi1 = pc[(rowbase + i0 + t) * 2 + 1];
      const uint32_t p00 = xi0 & xj0, p01 = xi0 & xj1, p10 = xi1 & xj0, p11 = xi1 & xj1;
      acc[t][0] = bcnt_acc(p00 & xk.x, acc[t][0]);
      acc[t][1] = bcnt_acc(p00 & xk.y, acc[t][1]);
      acc[t][2] = bcnt_acc(p01 & xk.x, acc[t][2]);
      acc[t][3] = bcnt_acc(p01 & xk.y, acc[t][3]);
      acc[t][4] = bcnt_acc(p10 & xk.x, acc[t][4]);
      acc[t][5] = bcnt_acc(p10 & xk.y, acc[t][5]);
      acc[t][6] = bcnt_acc(p11 & xk.x, acc[t][6]);
      acc[t][7] = bcnt_acc(p11 & xk.y, acc[t][7]);
    }
  }
}

// One tile: P pivots i0 .. i0 + P - 1, pivot j, 64 lanes = 64 consecutive k.
template <int P, bool COUNTS, bool LDS>
__device__ __forceinline__ void valu_tile(cptr<Job> cj, int job, int j, int r, int lane) {
  const uint32_t *planes = cj[job].planes;
  const int32_t *pairs = cj[job].pairs;
  const int M = cj[job].M, Mp = cj[job].Mp;
  const int W0 = cj[job].W0, W1 = cj[job].W1;
  const int nkb = (M - 1 - j + 63) >> 6;
  const int ib = r / nkb, kb = r - ib * nkb;
  const int i0 = ib * P;
  const int k = j + 1 + kb * 64 + lane;

  uint32_t acc0[P][8], acc1[P][8];
#pragma unroll
  for (int x = 0; x < P; ++x)
#pragma unroll
    for (int y = 0; y < 8; ++y) acc0[x][y] = acc1[x][y] = 0u;
  accumulate<P>(acc0, planes, Mp, 0, W0, i0, j, k);
  accumulate<P>(acc1, planes, Mp, W0, W0 + W1, i0, j, k);

  // ---- epilogue: complete the tables, K2, write ----
  // Cells are carried as 4 x count (byte offsets into the log-factorial
  // table).  The nine cells of the pair (j, k) are completed once per tile;
  // those of (i, j) are wave-uniform, so they stay on the scalar unit.
  const int N0 = cj[job].N0, N1 = cj[job].N1;
  const uint32_t *lfx = cj[job].lfx;
  const float scale = cj[job].scale;
  float *score = cj[job].score;
  uint32_t *counts = cj[job].counts;
  const int64_t MpMp = (int64_t)Mp * Mp;
  const int4 *pr = reinterpret_cast<const int4 *>(pairs);
  typedef int i4v __attribute__((ext_vector_type(4)));
  cptr<i4v> prc = as_const(reinterpret_cast<const i4v *>(pairs));
  const bool kvalid = k < M;
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  int fjk[2][9];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int4 kk = pr[c * MpMp + (int64_t)k * Mp + k];
    const int4 jk = pr[c * MpMp + (int64_t)j * Mp + k];
    const i4v mjj = prc[c * MpMp + (int64_t)j * Mp + j];
    const int ajk[4] = {jk.x << 2, jk.y << 2, jk.z << 2, jk.w << 2};
    const int mj[2] = {mjj.x << 2, mjj.w << 2}, mk[2] = {kk.x << 2, kk.w << 2};
    pair_cells(ajk, mj, mk, (c == 0 ? N0 : N1) << 2, fjk[c]);
  }
#pragma unroll
  for (int tt = 0; tt < P; ++tt) {
    const int i = i0 + tt;
    int tab[2][27];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const i4v pij = prc[c * MpMp + (int64_t)i * Mp + j];
      const i4v mii = prc[c * MpMp + (int64_t)i * Mp + i];
      const int4 pik = pr[c * MpMp + (int64_t)i * Mp + k];
      const int aij[4] = {pij.x << 2, pij.y << 2, pij.z << 2, pij.w << 2};
      const int aij2[2] = {(mii.x - pij.x - pij.y) << 2, (mii.w - pij.z - pij.w) << 2};
      const int aik[4] = {pik.x << 2, pik.y << 2, pik.z << 2, pik.w << 2};
      uint32_t n[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) n[x] = (c == 0 ? acc0[tt][x] : acc1[tt][x]) << 2;
      complete27(n, fjk[c], aij, aij2, aik, tab[c]);
    }
    const float k2 = fx_score(fx_sum<27, LDS>(tab[0], tab[1], lfx), scale);
    if (i < j && kvalid) {
      const int64_t rank = lex_base(M, i, j) + k;
      score[rank] = k2;
      const uint32_t key = f2key(k2);
      kmin = key < kmin ? key : kmin;
      kmax = key > kmax ? key : kmax;
      if (COUNTS) {
        uint32_t *o = counts + rank * 54;
#pragma unroll
        for (int x = 0; x < 27; ++x) {
          o[x] = (uint32_t)tab[0][x] >> 2;
          o[27 + x] = (uint32_t)tab[1][x] >> 2;
        }
      }
    }
  }
  // wave-reduce the key range, one atomic per tile
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t a = __shfl_xor(kmin, off), b = __shfl_xor(kmax, off);
    kmin = a < kmin ? a : kmin;
    kmax = b > kmax ? b : kmax;
  }
  if (lane == 0 && kmax != 0u) {
    atomicMin(cj[job].keyrange, kmin);
    atomicMax(cj[job].keyrange + 1, kmax);
  }
}

// Persistent grid over the tiles of every job; a job's tiles use its own P
// (PA or PB: one kernel serves a batch whose data sets prefer different P).
// Dynamic LDS only: the log-factorial table (LDS) starts at LDS address 0,
// followed by the workgroup's tile slot (MULTI).
// One job (MULTI = false): each wave draws its own tiles.  Several jobs: each
// has a log-factorial table of its own fixed-point step, so the workgroup
// draws four consecutive tiles of one job at a time (job tile ranges start at
// multiples of four) and reloads the table when the job changes.  That waits for
// the slowest of the four waves per draw; whole batches on the vector ALUs against
// one table for all jobs and a draw per wave (with this library's shorter
// selection): 16 sets of 300 x 3000 6.37 -> 5.68 ms, 4 sets of 500 x 6000 to 30 x
// 100 2.92 -> 2.75 ms, 200 sets of 40 to 59 SNPs x 500 5.93 -> 0.96 ms.
template <int PA, int PB, bool COUNTS, bool LDS, bool MULTI>
__global__ void __launch_bounds__(256) count_valu_kernel(const Job *__restrict__ jobs, int n_jobs,
                                                         int64_t total_tiles,
                                                         unsigned long long *__restrict__ queue,
                                                         int lf_len) {
  extern __shared__ __attribute__((aligned(16))) uint32_t sLds[];
  unsigned long long *sTile =
      reinterpret_cast<unsigned long long *>(sLds + (LDS ? (lf_len + 3) / 4 * 4 : 0));
  const int lane = threadIdx.x & 63;
  cptr<Job> cj = as_const(jobs);
  int job = -1;
  int64_t jb_begin = 0, jb_end = 0;
  int j = -1;
  int64_t jlo = 0, jhi = 0;
  if (LDS && !MULTI) {
    table_to_lds<256>(sLds, cj[0].lfx, lf_len);
    __syncthreads();
  }

  for (;;) {
    int64_t t;
    if (MULTI) {
      __syncthreads();  // the previous draw's readers of sTile are done
      if (threadIdx.x == 0) sTile[0] = atomicAdd(queue, 4ull);
      __syncthreads();
      t = rfl64((int64_t)sTile[0]);  // first of the four
    } else {
      unsigned long long got = 0;
      if (lane == 0) got = atomicAdd(queue, 1ull);
      t = rfl64((int64_t)got);
    }
    if (t >= total_tiles) break;
    if (job < 0 || t < jb_begin || t >= jb_end) {
      int lo = 0, hi = n_jobs - 1;  // last job whose first tile is <= t
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (cj[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
      }
      job = lo;
      jb_begin = cj[job].tile_begin;
      jb_end = jb_begin + cj[job].n_tiles;
      jlo = jhi = 0;
      j = -1;
      if (LDS && MULTI) {  // workgroup-uniform: t is
        table_to_lds<256>(sLds, cj[job].lfx, cj[job].lf_len);
        __syncthreads();
      }
    }
    if (MULTI) {
      t += __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      if (t >= jb_end) continue;  // padding of the job's tile range
    }
    const int M = cj[job].M;
    const int64_t local = t - jb_begin;
    if (j < 0 || local < jlo || local >= jhi) {
      cptr<int64_t> pre = as_const(cj[job].jprefix);
      int lo = 0, hi = M - 1;  // last pivot whose first tile is <= local
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= local) lo = mid; else hi = mid - 1;
      }
      j = lo;
      jlo = pre[j];
      jhi = pre[j + 1];
    }
    const int r = (int)(local - jlo);
    if (PA == PB || cj[job].P == PA)
      valu_tile<PA, COUNTS, LDS>(cj, job, j, r, lane);
    else
      valu_tile<PB, COUNTS, LDS>(cj, job, j, r, lane);
  }
}

hipError_t launch_valu_setup(const Job *h, int32_t n, Job *dst_dev, unsigned long long *queue,
                             hipStream_t s) {
  for (int x = 0; x < n; x += kJobsPerLaunch) {
    Jobs jobs{};
    const int m = n - x < kJobsPerLaunch ? n - x : kJobsPerLaunch;
    for (int y = 0; y < m; ++y) jobs.j[y] = h[x + y];
    hipLaunchKernelGGL(valu_setup_kernel, dim3(m), dim3(1024), 0, s, jobs, dst_dev + x, queue);
  }
  return hipGetLastError();
}

template <int PA, int PB, bool C, bool LDS, bool MULTI>
static hipError_t launch_valu_l(const Job *jobs_dev, int32_t n_jobs, int64_t total_tiles,
                                unsigned long long *queue, int32_t lf_len, hipStream_t s) {
  int dev = 0, n_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  auto kern = count_valu_kernel<PA, PB, C, LDS, MULTI>;
  const size_t lds = (LDS ? (size_t)(lf_len + 3) / 4 * 16 : 0) + (MULTI ? 16 : 0);
  e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, lds);
  if (e != hipSuccess) return e;
  if (per_cu <= 0) per_cu = 1;
  int64_t blocks = (int64_t)n_cu * per_cu;
  const int64_t need = (total_tiles + 3) / 4;
  if (blocks > need) blocks = need > 0 ? need : 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), lds, s, jobs_dev, n_jobs, total_tiles,
                     queue, lf_len);
  return hipGetLastError();
}

template <int PA, int PB, bool C, bool MULTI>
static hipError_t launch_valu_t(const Job *jobs_dev, int32_t n_jobs, int64_t total_tiles,
                                unsigned long long *queue, int32_t lf_len, hipStream_t s) {
  return lf_in_lds(lf_len)
             ? launch_valu_l<PA, PB, C, true, MULTI>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s)
             : launch_valu_l<PA, PB, C, false, MULTI>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s);
}

hipError_t launch_count_valu(const Job *jobs_dev, int32_t n_jobs, int64_t total_tiles,
                             unsigned long long *queue, int32_t lf_len, int32_t P_lo, int32_t P_hi,
                             bool counts, hipStream_t s) {
  if (n_jobs > 1) {  // batch (never with tables)
    if (counts) return hipErrorInvalidValue;
    if (P_lo != P_hi)
      return launch_valu_t<8, 4, false, true>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s);
    return P_lo == 4
               ? launch_valu_t<4, 4, false, true>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s)
               : launch_valu_t<8, 8, false, true>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s);
  }
  if (P_lo != P_hi) return hipErrorInvalidValue;
  if (P_lo == 4)
    return counts
               ? launch_valu_t<4, 4, true, false>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s)
               : launch_valu_t<4, 4, false, false>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s);
  return counts ? launch_valu_t<8, 8, true, false>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s)
                : launch_valu_t<8, 8, false, false>(jobs_dev, n_jobs, total_tiles, queue, lf_len, s);
}

int64_t host_tiles(int64_t M, int P) {
  int64_t n = 0;
  for (int64_t j = 0; j < M; ++j) n += tiles_of_j(M, j, P);
  return n;
}

int tile_P_default(int32_t M, int32_t N) {
  (void)N;
  return M >= 256 ? 8 : 4;
}

}  // namespace epi3
