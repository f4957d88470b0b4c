// Second-order scan: K2 of every pair of SNPs.
//
// Eq. 1 holds for any number of interacting SNPs (I = 3^k rows); for pairs
// the table has 9 rows per class.  Its four cells with both genotypes in
// {0, 1} are the pairwise tables that encoding counts for the triplet scan
// (products of the SNPs' planes over the class's samples), and the other five follow from the per-SNP counts (the diagonal of the pairwise
// tables) and the class size.  So scoring a pair is table completion and 27
// lookups; the counting itself happened at encoding.
#include "epi3_internal.h"

namespace epi3 {
namespace {

// K2 by lexicographic pair rank (summed in fixed point, stored as FP32) and the
// scores' key range.  Persistent workgroups; an item is 256 consecutive j
// (thread = j) by R rows i, so a thread loads its SNP's counts (a strided
// diagonal entry) once per item and the rows' come as wave-uniform loads, eight
// rows in flight at a time: with the table of many samples in LDS only a few
// waves fit a CU, and a row at a time waits for memory.  LDS: the log-factorial
// table, loaded once per workgroup.  Whole scans, a row per workgroup with the
// diagonal read per pair -> this: 512 x 4096 127 -> 96 us, 1003 x 6007 196 ->
// 134 us (four rows: 157, two: 206), 2048 x 16384 250 -> 228 us, 4096 x 1000
// 341 -> 235 us.
constexpr int kRowsAhead = 8;
template <bool LDS>
__global__ void __launch_bounds__(256) pair_scores_kernel(const int32_t *__restrict__ pairs,
                                                          int32_t M, int32_t Mp, int32_t N0,
                                                          int32_t N1, const uint32_t *__restrict__ lfx,
                                                          int32_t lf_len, float scale, int32_t R,
                                                          float *__restrict__ score,
                                                          uint32_t *__restrict__ keyrange) {
  extern __shared__ uint32_t tab[];  // no static LDS: the table starts at LDS address 0
  if (LDS) {
    table_to_lds<256>(tab, lfx, lf_len);
    __syncthreads();
  }
  const int4 *pr = reinterpret_cast<const int4 *>(pairs);
  cptr<int32_t> ps = as_const(pairs);
  const int64_t MpMp = (int64_t)Mp * Mp;
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  const int n_jt = (M + 255) / 256;
  int jt = 0;
  int64_t item = blockIdx.x;  // within j-tile jt: rows i < its last j
  for (;;) {
    for (; jt < n_jt; ++jt) {
      const int rows = 256 * jt + 255 < M - 1 ? 256 * jt + 255 : M - 1;
      const int n = (rows + R - 1) / R;
      if (item < n) break;
      item -= n;
    }
    if (jt >= n_jt) break;
    const int j = 256 * jt + threadIdx.x, jc = j < M ? j : M - 1;
    const int i0 = (int)item * R, i1 = i0 + R < M - 1 ? i0 + R : M - 1;
    const int4 jj[2] = {pr[(int64_t)jc * Mp + jc], pr[MpMp + (int64_t)jc * Mp + jc]};
    for (int ib = i0; ib < i1; ib += kRowsAhead) {
      int4 p[kRowsAhead][2];
      int mi[kRowsAhead][2][2];
#pragma unroll
      for (int y = 0; y < kRowsAhead; ++y)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int i = ib + y < M ? ib + y : M - 1;
          p[y][c] = pr[c * MpMp + (int64_t)i * Mp + jc];
          const int64_t ii = (c * MpMp + (int64_t)i * Mp + i) * 4;
          mi[y][c][0] = ps[ii] << 2;
          mi[y][c][1] = ps[ii + 3] << 2;
        }
#pragma unroll
      for (int y = 0; y < kRowsAhead; ++y) {
        const int i = ib + y;
        int t[2][9];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int n[4] = {p[y][c].x << 2, p[y][c].y << 2, p[y][c].z << 2, p[y][c].w << 2};
          const int mj[2] = {jj[c].x << 2, jj[c].w << 2};
          pair_cells(n, mi[y][c], mj, (c ? N1 : N0) << 2, t[c]);
        }
        if (i >= j || j >= M || i >= i1) continue;
        const float k2 = fx_score(fx_sum<9, LDS>(t[0], t[1], lfx), scale);
        score[pair_rank(M, i, j)] = k2;
        const uint32_t key = f2key(k2);
        kmin = key < kmin ? key : kmin;
        kmax = key > kmax ? key : kmax;
      }
    }
    item += gridDim.x;
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
hipError_t launch_pair_scores_t(const epi3_dataset &d, float *score, uint32_t *keyrange,
                                hipStream_t s) {
  const int M = d.n_snps;
  const int lf_len = d.n_samples + 2;
  const int lds = LDS ? lf_len * 4 : 0;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&pair_scores_kernel<LDS>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  int dev = 0, n_cu = 0;
  e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pair_scores_kernel<LDS>, 256, lds);
  if (e != hipSuccess) return e;
  int64_t blocks = (int64_t)n_cu * (per_cu > 0 ? per_cu : 1);
  // rows per item: one group of kRowsAhead, more once there are two items per workgroup
  const int64_t n_jt = (M + 255) / 256, rows = n_jt * M / 2;
  int64_t R = rows / (2 * blocks) / kRowsAhead * kRowsAhead;
  R = std::max<int64_t>(kRowsAhead, std::min<int64_t>(32, R));
  blocks = std::min(blocks, n_jt * ((M + R - 1) / R));
  hipLaunchKernelGGL(pair_scores_kernel<LDS>, dim3((unsigned)blocks), dim3(256), lds, s, d.pairs,
                     M, d.snp_stride, d.n_controls, d.n_cases, fx_table(d), lf_len,
                     fx_scale(d.n_samples), (int32_t)R, score, keyrange);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pair_scores(const epi3_dataset &d, float *score, uint32_t *keyrange,
                              hipStream_t s) {
  if (d.n_snps < 2) return hipSuccess;
  return lf_in_lds(d.n_samples + 2) ? launch_pair_scores_t<true>(d, score, keyrange, s)
                                    : launch_pair_scores_t<false>(d, score, keyrange, s);
}

}  // namespace epi3
