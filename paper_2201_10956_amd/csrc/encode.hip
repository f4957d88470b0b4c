// Encoding kernels: genotype bytes -> per-genotype sample bit-planes, byte
// planes for the matrix-core path, and pairwise tables.
//
// Binarized format (Problem Formulation section, Fig. 1 text): SNP x is held
// as one bit-plane per genotype value, one bit per sample.  Reduced format
// (CPU approaches section): plane 2 is never stored because a sample is in
// plane 2 exactly when it is in neither plane 0 nor plane 1, and samples are
// split into a controls array and a cases array.  32-bit words (start of the
// Approaches section).  SNP-minor order (GPU approaches section: consecutive
// SNPs adjacent in memory so that lanes owning consecutive SNPs coalesce).
#include "epi3_internal.h"

namespace epi3 {

// planes[w][m][0..1]: bit b of word w = sample list[w * 32 + b] has genotype
// 0 (plane 0) / 1 (plane 1).  list < 0 marks padding; padding bits stay 0 in
// both planes.  SNP slots m >= M are zero.  Words W0 .. W0 + W1 - 1 are class 1.
// VALUES: the same bits as 0/1 values for the matrix cores, a row of S
// positions per (class c, SNP m, genotype g): bytes[c][m][g][p] = 1 and
// nib[c][m][g][p / 2] nibble = 0x2 (E2M1 1.0) where bit p of the class is set;
// positions past the class's words are 0.
//
// One workgroup per 16 SNPs and WORDS words of a class.  A wave reads 64
// consecutive list positions (two words) of four SNPs per step: within a class
// the list is in sample order, so the byte loads fall in a few cache lines of
// each SNP's row; two ballots per SNP form both planes of both words.  All
// steps' list entries, then all genotypes, are in flight at once (a step alone
// waits for the list entry, then for the genotype), so the kernel needs many
// short workgroups rather than few long ones.  The bits are turned in LDS:
// planes leave as 128-byte runs (16 SNPs), value rows as runs of 16 WORDS and
// 32 WORDS bytes, and the genotypes are read once for all three.  WORDS = 8
// until that makes kEncWide workgroups, 16 from there on.  Whole encodes with
// value planes, one kernel per SNP and 64 words plus one per value plane ->
// this: 64 x 1024 47 -> 37 us, 512 x 4096 94 -> 57 us (WORDS 16: 59, 64: 76),
// 1003 x 6007 121 -> 75 us (80, 107), 2048 x 16384 306 -> 188 us (WORDS 8: 194).
constexpr int kEncSnps = 16;
constexpr int64_t kEncWide = 4096;  // workgroups

// The E2M1 nibbles of bits 8 t .. 8 t + 7 of w, low nibble first.
__device__ __forceinline__ uint32_t nibbles_of(uint32_t w, int t) {
  uint32_t x = (w >> (8 * t)) & 0xffu;
  x = (x | x << 12) & 0x000f000fu;
  x = (x | x << 6) & 0x03030303u;
  return ((x | x << 3) & 0x11111111u) << 1;
}

// The bytes of bits 4 t .. 4 t + 3 of w.
__device__ __forceinline__ uint32_t bytes_of(uint32_t w, int t) {
  return (((w >> (4 * t)) & 0xfu) * 0x00204081u) & 0x01010101u;
}

template <bool VALUES, int WORDS>
__global__ void __launch_bounds__(256) encode_kernel(const uint8_t *__restrict__ geno, int64_t ld,
                                                     const int32_t *__restrict__ list, int32_t M,
                                                     int32_t Mp, int32_t W0, int32_t W1, int32_t S,
                                                     uint32_t *__restrict__ planes,
                                                     uint32_t *__restrict__ bytes,
                                                     uint32_t *__restrict__ nib,
                                                     int32_t *__restrict__ status) {
  __shared__ uint2 bits[WORDS][kEncSnps + 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = blockIdx.z, W = c ? W1 : W0, off = c ? W0 : 0;
  const int w0 = blockIdx.y * WORDS, m0 = blockIdx.x * kEncSnps;
  uint32_t z0[4], z1[4], o0[4], o1[4];  // lane u: words 2 u and 2 u + 1 of the four SNPs
#pragma unroll
  for (int q = 0; q < 4; ++q) z0[q] = z1[q] = o0[q] = o1[q] = 0u;
  bool bad = false;
  if (w0 < W && m0 + 4 * wave < M) {
    int sidx[WORDS / 2];
#pragma unroll
    for (int u = 0; u < WORDS / 2; ++u) {
      const int w = w0 + 2 * u + (lane >> 5);  // this lane's word
      sidx[u] = w < W ? list[(int64_t)(off + w) * 32 + (lane & 31)] : -1;
    }
    int g[WORDS / 2][4];
#pragma unroll
    for (int u = 0; u < WORDS / 2; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + 4 * wave + q;
        g[u][q] = 3;  // no genotype: padding, SNP slot >= M, word >= W
        if (m < M && sidx[u] >= 0) {
          g[u][q] = geno[(int64_t)m * ld + sidx[u]];
          bad |= g[u][q] > 2;
        }
      }
#pragma unroll
    for (int u = 0; u < WORDS / 2; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned long long z = __ballot(g[u][q] == 0), o = __ballot(g[u][q] == 1);
        const bool mine = lane == u;
        z0[q] = mine ? (uint32_t)z : z0[q];
        z1[q] = mine ? (uint32_t)(z >> 32) : z1[q];
        o0[q] = mine ? (uint32_t)o : o0[q];
        o1[q] = mine ? (uint32_t)(o >> 32) : o1[q];
      }
  }
  if (__ballot(bad) != 0ull && lane == 0) atomicOr(status, 1);
  if (lane < WORDS / 2) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      bits[2 * lane][4 * wave + q] = make_uint2(z0[q], o0[q]);
      bits[2 * lane + 1][4 * wave + q] = make_uint2(z1[q], o1[q]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < WORDS * kEncSnps / 2; x += 256) {
    if (x + (int)threadIdx.x >= WORDS * kEncSnps / 2) break;
    const int w = (x + threadIdx.x) / (kEncSnps / 2), m = 2 * (threadIdx.x % (kEncSnps / 2));
    if (w0 + w >= W) continue;
    const uint2 a = bits[w][m], b = bits[w][m + 1];
    *reinterpret_cast<uint4 *>(planes + ((int64_t)(off + w0 + w) * Mp + m0 + m) * 2) =
        make_uint4(a.x, a.y, b.x, b.y);
  }
  if constexpr (VALUES) {
    const int WS = S / 32;  // words of a row; the last group may end early
    const int64_t row0 = ((int64_t)c * Mp + m0) * 2;
#pragma unroll
    for (int x = 0; x < WORDS * kEncSnps * 2; x += 256) {  // 16 bytes: a word's nibbles
      const int w = (x + threadIdx.x) % WORDS, row = (x + threadIdx.x) / WORDS;
      if (w0 + w >= WS) continue;
      const uint2 v = bits[w][row >> 1];
      const uint32_t b = row & 1 ? v.y : v.x;
      *reinterpret_cast<uint4 *>(nib + (row0 + row) * (S / 8) + 4 * (w0 + w)) =
          make_uint4(nibbles_of(b, 0), nibbles_of(b, 1), nibbles_of(b, 2), nibbles_of(b, 3));
    }
#pragma unroll
    for (int x = 0; x < WORDS * kEncSnps * 4; x += 256) {  // 16 bytes: half a word's
      const int h = (x + threadIdx.x) % (2 * WORDS), row = (x + threadIdx.x) / (2 * WORDS);
      if (w0 + (h >> 1) >= WS) continue;
      const uint2 v = bits[h >> 1][row >> 1];
      const uint32_t b = (row & 1 ? v.y : v.x) >> (16 * (h & 1));
      *reinterpret_cast<uint4 *>(bytes + (row0 + row) * (S / 4) + 8 * w0 + 4 * h) =
          make_uint4(bytes_of(b, 0), bytes_of(b, 1), bytes_of(b, 2), bytes_of(b, 3));
    }
  }
}

// Nibble planes of bit planes that were encoded without them: a thread per word
// of a row (16 bytes out), runs of 16 words by consecutive threads, so the
// stores are 256-byte runs and the scattered reads stay in L2.  300 x 3000: 3 us
// for 2.4 MB, against the 415 us of vector-ALU counting it avoids.
__global__ void __launch_bounds__(256) expand_nibbles_kernel(const uint32_t *__restrict__ planes,
                                                             int32_t Mp, int32_t W0, int32_t W1, int32_t S,
                                                             uint32_t *__restrict__ nib) {
  const int c = blockIdx.z, W = c ? W1 : W0, off = c ? W0 : 0;
  const int w = blockIdx.y * 16 + (threadIdx.x & 15);
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4);  // 2 m + genotype
  if (w >= S / 32) return;
  const uint32_t b = w < W ? planes[(int64_t)(off + w) * Mp * 2 + row] : 0u;
  *reinterpret_cast<uint4 *>(nib + ((int64_t)c * Mp * 2 + row) * (S / 8) + 4 * w) =
      make_uint4(nibbles_of(b, 0), nibbles_of(b, 1), nibbles_of(b, 2), nibbles_of(b, 3));
}

// Pairwise tables out[c][x][y] = (n00, n01, n10, n11), n_ab = number of
// samples of class c with genotype a at SNP x and b at SNP y (a, b in {0, 1}).
// The diagonal holds the per-SNP counts (n_x(0), 0, 0, n_x(1)).
//
// A product of the plane rows with themselves over the class's samples, on
// v_mfma_f32_32x32x64_f8f6f4: lane l supplies row l % 32 (SNP r / 2, plane
// r % 2; a word's planes of consecutive SNPs are contiguous, so a load is two
// 128-byte runs) and the 32 samples of word l / 32 of the step.  A word
// becomes its 32 E2M1 nibbles by three shifts and four masks: operand dword t
// takes the samples whose bit is t modulo 4, the same for both operands.  FP32
// accumulation is exact below 2^24: segments of kPairSegment words are added
// to the stored counts one after the other.
//
// Only tiles on or above the diagonal count; the others are written as
// mirrors, (y, x) = (n00, n10, n01, n11).  RT = 2: workgroup tile 64 x 64
// SNPs, wave 32 x 32 (four products per four operand loads).  RT = 1, where
// those tiles would leave most CUs idle: workgroup tile 16 x 16 SNPs, the
// words split over the four waves and the counts added through LDS.  Whole
// encodes without value planes, popcounts of 64 x 64 tiles -> products: 64 x
// 1024 56 -> 43 us, 512 x 4096 124 -> 80 us (RT = 2 there: 83), 1003 x 6007 169
// -> 96 us, 2048 x 16384 524 -> 219 us (RT = 1 there: 273; 1400 SNPs: 85 against
// 90).  At 2048 SNPs the products take about 35 us and writing the 134 MB of
// tables about 30 us.
constexpr int kPairSegment = 1 << 18;  // words: 2^23 samples
constexpr int64_t kPairSmall = 256;     // fewer 64 x 64 tiles: RT = 1
constexpr int kPairAhead = 4;          // steps loaded ahead of the products

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// The E2M1 nibbles (0 or 1.0) of a word's 32 samples.
__device__ __forceinline__ v8i fp4_of_bits(uint32_t w) {
  const uint32_t m = 0x22222222u;
  return v8i{(int)((w << 1) & m), (int)(w & m), (int)((w >> 1) & m), (int)((w >> 2) & m), 0, 0, 0, 0};
}

template <int RT>
__global__ void __launch_bounds__(256, 3) pairs_kernel(const uint32_t *__restrict__ planes, int32_t Mp,
                                                    int32_t W0, int32_t W1,
                                                    int32_t *__restrict__ pairs) {
  constexpr int kSnps = 16 * RT;             // SNPs of a wave's rows and columns
  constexpr int kTile = RT == 2 ? 64 : 16;   // SNPs of a workgroup's
  __shared__ float part[RT == 1 ? 4 : 1][RT == 1 ? 16 : 1][64];
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // tile of the upper triangle, column by column: blockIdx.x = yb (yb + 1) / 2 + xb
  int yb = (int)((sqrtf(8.f * (float)blockIdx.x + 1.f) - 1.f) * 0.5f);
  while (yb * (yb + 1) / 2 > (int)blockIdx.x) --yb;
  while ((yb + 1) * (yb + 2) / 2 <= (int)blockIdx.x) ++yb;
  const int xb = (int)blockIdx.x - yb * (yb + 1) / 2;
  const int x0 = xb * kTile + (RT == 2 ? kSnps * (wave >> 1) : 0);
  const int y0 = yb * kTile + (RT == 2 ? kSnps * (wave & 1) : 0);
  if (y0 < x0) return;  // RT = 2, diagonal tile: no barriers there
  const int c = blockIdx.y;
  const int wb = c == 0 ? 0 : W0, we = c == 0 ? W0 : W0 + W1;
  const int64_t stride = (int64_t)Mp * 2;  // dwords of a word's planes
  int4 *out = reinterpret_cast<int4 *>(pairs) + (int64_t)c * Mp * Mp;
  int seg = wb;
  do {
    const int seg_end = we - seg > kPairSegment ? seg + kPairSegment : we;
    // this wave's steps of two words
    int s = seg, e = seg_end;
    if (RT == 1) {
      const int per = (((seg_end - seg + 1) / 2 + 3) / 4) * 2;
      s = seg + wave * per;
      e = s + per < seg_end ? s + per : seg_end;
    }
    v16f acc[RT][RT];
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
      for (int b = 0; b < RT; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    uint32_t px[kPairAhead][RT], py[kPairAhead][RT];
    const uint32_t *bx = planes + 2 * x0 + r, *by = planes + 2 * y0 + r;
    auto load = [&](int w) {  // words w .. w + 2 kPairAhead - 1, zero past e
#pragma unroll
      for (int t = 0; t < kPairAhead; ++t) {
        const int wl = w + 2 * t + h;
        const int64_t o = (int64_t)(wl < e ? wl : e - 1) * stride;
#pragma unroll
        for (int a = 0; a < RT; ++a) {
          px[t][a] = bx[o + 32 * a];
          py[t][a] = by[o + 32 * a];
        }
      }
    };
    if (s < e) load(s);
    for (; s < e; s += 2 * kPairAhead) {
      uint32_t cx[kPairAhead][RT], cy[kPairAhead][RT];
#pragma unroll
      for (int t = 0; t < kPairAhead; ++t)
#pragma unroll
        for (int a = 0; a < RT; ++a) {
          cx[t][a] = s + 2 * t + h < e ? px[t][a] : 0u;
          cy[t][a] = py[t][a];
        }
      if (s + 2 * kPairAhead < e) load(s + 2 * kPairAhead);
#pragma unroll
      for (int t = 0; t < kPairAhead; ++t) {
        v8i fx[RT], fy[RT];
#pragma unroll
        for (int a = 0; a < RT; ++a) {
          fx[a] = fp4_of_bits(cx[t][a]);
          fy[a] = fp4_of_bits(cy[t][a]);
        }
#pragma unroll
        for (int a = 0; a < RT; ++a)
#pragma unroll
          for (int b = 0; b < RT; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fx[a], fy[b], acc[a][b], 4,
                                                                        4, 0, 0, 0, 0);
      }
    }
    // Registers 4 g .. 4 g + 3 of lane (column q = (y, b), half h): rows
    // (x, a = 0, 1), (x + 1, a = 0, 1) with x = 4 g + 2 h; the lanes of a
    // column pair exchange two of them, then each has one pair's four cells.
    auto put = [&](int a, int b, int g, float v0, float v1, float v2, float v3) {
      const bool odd = r & 1;
      const uint32_t u0 = (uint32_t)v0, u1 = (uint32_t)v1, u2 = (uint32_t)v2, u3 = (uint32_t)v3;
      const uint32_t k0 = odd ? u2 : u0, k1 = odd ? u3 : u1;
      const uint32_t r0 = __builtin_amdgcn_mov_dpp(odd ? u0 : u2, 0xB1, 0xf, 0xf, true);
      const uint32_t r1 = __builtin_amdgcn_mov_dpp(odd ? u1 : u3, 0xB1, 0xf, 0xf, true);
      const int x = x0 + 16 * a + 4 * g + 2 * h + (odd ? 1 : 0), y = y0 + 16 * b + (r >> 1);
      int4 n = odd ? make_int4((int)r0, (int)k0, (int)r1, (int)k1)
                   : make_int4((int)k0, (int)r0, (int)k1, (int)r1);
      int4 *o = out + (int64_t)x * Mp + y;
      if (seg != wb) {
        const int4 p = *o;
        n.x += p.x; n.y += p.y; n.z += p.z; n.w += p.w;
      }
      *o = n;
      if (x0 != y0) out[(int64_t)y * Mp + x] = make_int4(n.x, n.z, n.y, n.w);
    };
    if constexpr (RT == 1) {
#pragma unroll
      for (int v = 0; v < 16; ++v) part[wave][v][lane] = acc[0][0][v];
      __syncthreads();
      float t[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        t[v] = part[0][4 * wave + v][lane] + part[1][4 * wave + v][lane] +
               part[2][4 * wave + v][lane] + part[3][4 * wave + v][lane];
      put(0, 0, wave, t[0], t[1], t[2], t[3]);
      __syncthreads();
    } else {
#pragma unroll
      for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int b = 0; b < RT; ++b)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            put(a, b, g, acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2],
                acc[a][b][4 * g + 3]);
    }
    seg = seg_end;
  } while (seg < we);
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, int64_t n) {
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n;
       x += (int64_t)gridDim.x * blockDim.x)
    p[x] = v;
}

// See launch_tables.
__global__ void __launch_bounds__(256) tables_kernel(const double *src_lf64, const int32_t *src_list,
                                                     int64_t n_list, double *lf64,
                                                     float *__restrict__ lf32,
                                                     uint32_t *__restrict__ lfx, int64_t n,
                                                     double scale, int32_t *list,
                                                     int32_t *__restrict__ status) {
  if (blockIdx.x == 0 && threadIdx.x < kStatusWords) status[threadIdx.x] = 0;
  const int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (x < n) {
    const double v = src_lf64[x];
    if (src_lf64 != lf64) lf64[x] = v;
    lf32[x] = (float)v;
    lfx[x] = (uint32_t)(unsigned long long)rint(v * scale);
  }
  if (x < n_list && src_list != list) list[x] = src_list[x];
}

hipError_t launch_tables(const double *src_lf64, const int32_t *src_list, int64_t n_list, double *lf64,
                         float *lf32, uint32_t *lfx, int64_t n, int shift, int32_t *list,
                         int32_t *status, hipStream_t s) {
  const int64_t m = n > n_list ? n : n_list;
  hipLaunchKernelGGL(tables_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, src_lf64, src_list,
                     n_list, lf64, lf32, lfx, n, ldexp(1.0, shift), list, status);
  return hipGetLastError();
}

hipError_t launch_encode(const uint8_t *geno, int64_t ld, const int32_t *sample_list, int32_t M,
                         int32_t Mp, int32_t W0, int32_t W1, int32_t n_classes, int32_t S,
                         uint32_t *planes, uint8_t *bytes, uint8_t *nib, int32_t *status,
                         hipStream_t s) {
  if (Mp % kEncSnps != 0) return hipErrorInvalidValue;
  const int words = bytes ? S / 32 : (W0 > W1 ? W0 : W1);  // value rows run on to S
  if (words <= 0) return hipSuccess;
  const bool wide = (int64_t)(Mp / kEncSnps) * ((words + 7) / 8) * n_classes >= kEncWide;
  const int per = wide ? 16 : 8;
  auto *kernel = bytes ? (wide ? encode_kernel<true, 16> : encode_kernel<true, 8>)
                       : (wide ? encode_kernel<false, 16> : encode_kernel<false, 8>);
  hipLaunchKernelGGL(kernel, dim3(Mp / kEncSnps, (words + per - 1) / per, n_classes), dim3(256), 0, s,
                     geno, ld, sample_list, M, Mp, W0, W1, S, planes,
                     reinterpret_cast<uint32_t *>(bytes), reinterpret_cast<uint32_t *>(nib), status);
  return hipGetLastError();
}

hipError_t launch_expand_nibbles(const uint32_t *planes, int32_t Mp, int32_t W0, int32_t W1, int32_t S,
                                 uint8_t *nib, hipStream_t s) {
  if (Mp % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(expand_nibbles_kernel, dim3(Mp / 8, (S / 32 + 15) / 16, 2), dim3(256), 0, s, planes, Mp,
                     W0, W1, S, reinterpret_cast<uint32_t *>(nib));
  return hipGetLastError();
}

hipError_t launch_pairs(const uint32_t *planes, int32_t Mp, int32_t W0, int32_t W1,
                        int32_t n_classes, int32_t *pairs, hipStream_t s) {
  if (Mp % 64 != 0) return hipErrorInvalidValue;  // tiles cover the stride exactly
  const int64_t n = Mp / 64;
  if (n * (n + 1) / 2 * n_classes >= kPairSmall) {
    hipLaunchKernelGGL(pairs_kernel<2>, dim3((unsigned)(n * (n + 1) / 2), n_classes), dim3(256), 0, s,
                       planes, Mp, W0, W1, pairs);
  } else {
    const int64_t m = Mp / 16;
    hipLaunchKernelGGL(pairs_kernel<1>, dim3((unsigned)(m * (m + 1) / 2), n_classes), dim3(256), 0, s,
                       planes, Mp, W0, W1, pairs);
  }
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

}  // namespace epi3
