// Fourth-order scan: K2 of every quad of SNPs.
//
// Eq. 1 holds for any number of interacting SNPs; for quads the table has
// 3^4 = 81 rows per class.  The 8 corner cells of each of a quad's four
// sub-triplets come from a table counted once per triplet beforehand on the
// matrix cores (triplet_corners_kernel; they do not depend on the fourth SNP;
// classes of more than 65535 samples: counted per quad).  Data sets without
// value planes are scored here: per class and quad the 16 cells with all four
// genotypes in {0, 1} are counted by AND + POPCNT over the class's words (the
// paper's table filling, Alg. 2, with one more SNP), and the rest follow by
// inclusion-exclusion (quad_cells).  One thread per quad, quads by
// lexicographic rank, so the lanes of a wave share (i, j, k) and read
// consecutive l.
#include "epi3_internal.h"

namespace epi3 {
namespace {

// Corner cells of every triplet: t3[2 rank + x / 4] word x % 4 = the counts of
// cell x = 4 a + 2 b + c (a, b, c in {0, 1}) in both classes, class 1 in the
// high half.
//
// A product over each class's samples, on the bit planes themselves (a word
// becomes 32 E2M1 nibbles by shifts and masks, as for the pairwise tables): wave
// = i, 8 j and 64 k, rows (j, a, b) = X_i[a] & X_j[b], columns (k, c), a step is
// two words.  Neighbouring lanes hold c = 0 and 1 and exchange two cells each, so
// a lane writes 16 bytes.  A thread per triplet with popcounts took 490 us for 256
// x 4096, this 185.
__global__ void __launch_bounds__(256) triplet_corners_kernel(const uint32_t *__restrict__ planes,
                                                              int32_t M, int32_t Mp, int32_t W0,
                                                              int32_t W1, uint4 *__restrict__ t3) {
  typedef int v8 __attribute__((ext_vector_type(8)));
  typedef float v16 __attribute__((ext_vector_type(16)));
  constexpr int kAhead = 2;  // steps loaded ahead of the products
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.z * 4 + (threadIdx.x >> 6));
  const int j0 = blockIdx.y * 8, k0 = blockIdx.x * 64;
  if (i >= M - 2 || j0 + 7 <= i || k0 + 63 <= j0 || j0 >= M - 1) return;
  auto nibbles = [](uint32_t w) {
    const uint32_t m = 0x22222222u;
    return v8{(int)((w << 1) & m), (int)(w & m), (int)((w >> 1) & m), (int)((w >> 2) & m), 0, 0, 0, 0};
  };
  // A row r = 4 (j % 8) + 2 a + b; B column r = 2 (k % 16) + c
  const uint32_t *pi = planes + 2 * i + ((r >> 1) & 1), *pj = planes + 2 * (j0 + (r >> 2)) + (r & 1);
  const uint32_t *pk = planes + 2 * k0 + r;
  uint32_t n[4][16];  // class 0 in the low halves
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int wb = c ? W0 : 0, we = c ? W0 + W1 : W0;
    v16 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    uint32_t ni[kAhead], nj[kAhead], nk[kAhead][4];
    auto load = [&](int w) {
#pragma unroll
      for (int s = 0; s < kAhead; ++s) {
        const int wl = w + 2 * s + h < we ? w + 2 * s + h : we - 1;
        const int64_t o = (int64_t)wl * Mp * 2;
        ni[s] = pi[o];
        nj[s] = pj[o];
#pragma unroll
        for (int t = 0; t < 4; ++t) nk[s][t] = pk[o + 32 * t];
      }
    };
    if (wb < we) load(wb);
    for (int w = wb; w < we; w += 2 * kAhead) {
      uint32_t a[kAhead], k[kAhead][4];
#pragma unroll
      for (int s = 0; s < kAhead; ++s) {
        a[s] = w + 2 * s + h < we ? ni[s] & nj[s] : 0u;
#pragma unroll
        for (int t = 0; t < 4; ++t) k[s][t] = nk[s][t];
      }
      if (w + 2 * kAhead < we) load(w + 2 * kAhead);
#pragma unroll
      for (int s = 0; s < kAhead; ++s) {
        const v8 fa = nibbles(a[s]);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc[t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa, nibbles(k[s][t]), acc[t], 4, 4, 0, 0, 0, 0);
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        n[t][v] = c ? n[t][v] | ((uint32_t)acc[t][v] << 16) : (uint32_t)acc[t][v];
  }
  // registers 4 g .. 4 g + 3: the cells (a, b) of j % 8 = 2 g + h
  const bool odd = r & 1;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const uint32_t *v = n[t] + 4 * g;
      const uint32_t r0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? v[0] : v[2]), 0xB1, 0xf, 0xf, true);
      const uint32_t r1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? v[1] : v[3]), 0xB1, 0xf, 0xf, true);
      const int j = j0 + 2 * g + h, k = k0 + 16 * t + (r >> 1);
      if (i < j && j < k && k < M)
        t3[2 * (lex_base(M, i, j) + k) + (odd ? 1 : 0)] =
            odd ? make_uint4(r0, v[2], r1, v[3]) : make_uint4(v[0], r0, v[1], r1);
    }
}

// Class c's corner cells of triplet `rank`.
__device__ __forceinline__ void unpack8(const uint4 *t3, int64_t rank, int c, uint32_t *n) {
  const uint4 v = t3[2 * rank], w = t3[2 * rank + 1];
  const int s = 16 * c;
  n[0] = (v.x >> s) & 0xffffu; n[1] = (v.y >> s) & 0xffffu; n[2] = (v.z >> s) & 0xffffu; n[3] = (v.w >> s) & 0xffffu;
  n[4] = (w.x >> s) & 0xffffu; n[5] = (w.y >> s) & 0xffffu; n[6] = (w.z >> s) & 0xffffu; n[7] = (w.w >> s) & 0xffffu;
}

// T3: sub-triplet corners from the triplet table (else counted per quad).
template <bool LDS, bool T3>
__global__ void __launch_bounds__(256) quad_scores_kernel(
    const uint32_t *__restrict__ planes, const int32_t *__restrict__ pairs, int32_t M, int32_t Mp,
    int32_t W0, int32_t W1, int32_t N0, int32_t N1, const uint32_t *__restrict__ lfx, int32_t lf_len,
    float scale, int64_t Q, const uint4 *__restrict__ t3, float *__restrict__ score,
    uint32_t *__restrict__ keyrange) {
  extern __shared__ uint32_t tab[];  // no static LDS: the table starts at LDS address 0
  if (LDS) {
    table_to_lds<256>(tab, lfx, lf_len);
    __syncthreads();
  }
  const int64_t MpMp4 = (int64_t)Mp * Mp * 4;
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < Q;
       r += (int64_t)gridDim.x * blockDim.x) {
    int i, j, k, l;
    decode_quad_rank(M, r, i, j, k, l);
    uint32_t cnt[48];
    int t0[81], t1[81];
    auto counts = [&](int c) {
      const int w0 = c ? W0 : 0, w1 = c ? W0 + W1 : W0;
      if (T3) {
        quad_corner_counts(planes, Mp, w0, w1, i, j, k, l, cnt);
        unpack8(t3, lex_base(M, i, j) + k, c, cnt + 16);
        unpack8(t3, lex_base(M, i, j) + l, c, cnt + 24);
        unpack8(t3, lex_base(M, i, k) + l, c, cnt + 32);
        unpack8(t3, lex_base(M, j, k) + l, c, cnt + 40);
      } else {
        quad_counts(planes, Mp, w0, w1, 1, i, j, k, l, cnt);
      }
#pragma unroll
      for (int x = 0; x < 48; ++x) cnt[x] <<= 2;  // byte offsets into the table
    };
    counts(0);
    quad_cells<2>(cnt, pairs, Mp, i, j, k, l, N0 << 2, t0);
    counts(1);
    quad_cells<2>(cnt, pairs + MpMp4, Mp, i, j, k, l, N1 << 2, t1);
    const float k2 = fx_score(fx_sum<81, LDS>(t0, t1, lfx), scale);
    score[r] = k2;
    const uint32_t key = f2key(k2);
    kmin = key < kmin ? key : kmin;
    kmax = key > kmax ? key : kmax;
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

template <bool LDS, bool T3>
hipError_t launch_quad_scores_t(const epi3_dataset &d, const uint4 *t3, float *score,
                                uint32_t *keyrange, hipStream_t s) {
  const int M = d.n_snps;
  const int64_t Q = c4(M);
  const int lf_len = d.n_samples + 2;
  const int lds = LDS ? lf_len * 4 : 0;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&quad_scores_kernel<LDS, T3>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  int dev = 0, n_cu = 0;
  e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (T3) {
    e = launch_triplet_corners(d, const_cast<uint4 *>(t3), s);
    if (e != hipSuccess) return e;
  }
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, quad_scores_kernel<LDS, T3>, 256, lds);
  if (e != hipSuccess) return e;
  int64_t blocks = (int64_t)n_cu * (per_cu > 0 ? per_cu : 1) * 4;
  const int64_t need = (Q + 255) / 256;
  if (blocks > need) blocks = need;
  hipLaunchKernelGGL((quad_scores_kernel<LDS, T3>), dim3((unsigned)blocks), dim3(256), lds, s,
                     static_cast<const uint32_t *>(d.planes), d.pairs, M, d.snp_stride, d.words[0],
                     d.words[1], d.n_controls, d.n_cases, fx_table(d), lf_len,
                     fx_scale(d.n_samples), Q, t3, score, keyrange);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_triplet_corners(const epi3_dataset &d, void *t3, hipStream_t s) {
  const int M = d.n_snps;
  if (M < 3) return hipSuccess;
  if (d.snp_stride < M + 64) return hipErrorInvalidValue;  // the tiles end in the padding
  hipLaunchKernelGGL(triplet_corners_kernel, dim3((M + 63) / 64, (M + 7) / 8, (M + 3) / 4), dim3(256), 0,
                     s, static_cast<const uint32_t *>(d.planes), M, d.snp_stride, d.words[0],
                     d.words[1], static_cast<uint4 *>(t3));
  return hipGetLastError();
}

hipError_t launch_quad_scores(const epi3_dataset &d, void *t3, float *score, uint32_t *keyrange,
                              hipStream_t s) {
  if (d.n_snps < 4) return hipSuccess;
  const uint4 *t = static_cast<const uint4 *>(t3);
  if (lf_in_lds(d.n_samples + 2))
    return t ? launch_quad_scores_t<true, true>(d, t, score, keyrange, s)
             : launch_quad_scores_t<true, false>(d, t, score, keyrange, s);
  return t ? launch_quad_scores_t<false, true>(d, t, score, keyrange, s)
           : launch_quad_scores_t<false, false>(d, t, score, keyrange, s);
}

}  // namespace epi3
