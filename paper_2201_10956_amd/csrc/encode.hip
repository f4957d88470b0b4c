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
// both planes.  SNP slots m >= M are zero.  One wave per SNP and group of 64
// words: per step the 64 lanes read the genotype bytes of 64 consecutive
// list positions (two words; within a class the list is in sample order, so
// the reads fall in a few cache lines of the SNP's row) and two ballots form
// both planes of both words.
constexpr int kEncWords = 64;  // words per wave

__global__ void __launch_bounds__(256) encode_kernel(const uint8_t *__restrict__ geno, int64_t ld,
                                                     const int32_t *__restrict__ list, int32_t M,
                                                     int32_t Mp, int32_t Wtot,
                                                     uint32_t *__restrict__ planes,
                                                     int32_t *__restrict__ status) {
  const int lane = threadIdx.x & 63;
  const int m = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (m >= Mp) return;
  const int w0 = blockIdx.y * kEncWords;
  const uint8_t *row = geno + (int64_t)(m < M ? m : 0) * ld;
  uint2 *out = reinterpret_cast<uint2 *>(planes);
  bool bad = false;
  for (int w = w0; w < w0 + kEncWords && w < Wtot; w += 2) {
    const int wl = w + (lane >> 5);  // this lane's word
    int g = 3;                       // no genotype: padding, SNP slot >= M, word >= Wtot
    if (m < M && wl < Wtot) {
      const int sidx = list[(int64_t)wl * 32 + (lane & 31)];
      if (sidx >= 0) {
        g = row[sidx];
        bad |= g > 2;
      }
    }
    const unsigned long long z = __ballot(g == 0), o = __ballot(g == 1);
    if (lane == 0) out[(int64_t)w * Mp + m] = make_uint2((uint32_t)z, (uint32_t)o);
    if (lane == 32 && w + 1 < Wtot)
      out[(int64_t)(w + 1) * Mp + m] = make_uint2((uint32_t)(z >> 32), (uint32_t)(o >> 32));
  }
  if (__ballot(bad) != 0ull && lane == 0) atomicOr(status, 1);
}

// bytes[m][p][s] = 1 if sample s of SNP m has genotype p (p = 0, 1), else 0;
// samples s >= N and SNPs m >= M are 0.  S is a multiple of 4.
__global__ void __launch_bounds__(256) encode_bytes_kernel(const uint8_t *__restrict__ geno,
                                                           int64_t ld, int32_t M, int32_t N,
                                                           int32_t Mp, int32_t S,
                                                           uint32_t *__restrict__ bytes) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;  // dword within a row
  const int S4 = S >> 2;
  if (q >= S4) return;
  for (int m = blockIdx.y; m < Mp; m += gridDim.y) {
    uint32_t v0 = 0, v1 = 0;
    if (m < M) {
      const uint8_t *row = geno + (int64_t)m * ld;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int s = 4 * q + b;
        if (s < N) {
          const uint32_t g = row[s];
          v0 |= (uint32_t)(g == 0u) << (8 * b);
          v1 |= (uint32_t)(g == 1u) << (8 * b);
        }
      }
    }
    bytes[((int64_t)m * 2 + 0) * S4 + q] = v0;
    bytes[((int64_t)m * 2 + 1) * S4 + q] = v1;
  }
}

// nib[m][p][s / 2]: E2M1 value 1.0 (nibble 0x2) if sample s of SNP m has
// genotype p, else 0.0; samples 2d and 2d + 1 share byte d (low nibble first).
__global__ void __launch_bounds__(256) encode_nibbles_kernel(const uint8_t *__restrict__ geno,
                                                             int64_t ld, int32_t M, int32_t N,
                                                             int32_t Mp, int32_t S,
                                                             uint32_t *__restrict__ nib) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;  // dword of a row: 8 samples
  const int S8 = S >> 3;
  if (q >= S8) return;
  for (int m = blockIdx.y; m < Mp; m += gridDim.y) {
    uint32_t v0 = 0, v1 = 0;
    if (m < M) {
      const uint8_t *row = geno + (int64_t)m * ld;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int s = 8 * q + b;
        if (s < N) {
          const uint32_t g = row[s];
          v0 |= (uint32_t)(g == 0u) << (4 * b + 1);
          v1 |= (uint32_t)(g == 1u) << (4 * b + 1);
        }
      }
    }
    nib[((int64_t)m * 2 + 0) * S8 + q] = v0;
    nib[((int64_t)m * 2 + 1) * S8 + q] = v1;
  }
}

// Per-class 0/1 value planes for the matrix cores, through the class sample
// list: position p of class c is sample list[off_c + p] (p < len_c), else
// padding.  bytes[c][m][g][p] = 1 and nib[c][m][g][p / 2] nibble = 0x2 (E2M1
// 1.0) when that sample has genotype g in {0, 1}; padding and SNPs m >= M
// are 0.  One thread per 8 positions.
__global__ void __launch_bounds__(256) encode_values_kernel(
    const uint8_t *__restrict__ geno, int64_t ld, const int32_t *__restrict__ list, int32_t off0,
    int32_t len0, int32_t off1, int32_t len1, int32_t M, int32_t Mp, int32_t S,
    uint32_t *__restrict__ bytes, uint32_t *__restrict__ nib) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;  // positions 8q .. 8q + 7
  if (q >= S / 8) return;
  const int c = blockIdx.z;
  const int off = c ? off1 : off0, len = c ? len1 : len0;
  for (int m = blockIdx.y; m < Mp; m += gridDim.y) {
    uint32_t b0[2] = {0, 0}, b1[2] = {0, 0}, n0 = 0, n1 = 0;
    if (m < M) {
      const uint8_t *row = geno + (int64_t)m * ld;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int p = 8 * q + b;
        if (p < len) {
          const uint32_t g = row[list[off + p]];
          const uint32_t is0 = g == 0u, is1 = g == 1u;
          b0[b >> 2] |= is0 << (8 * (b & 3));
          b1[b >> 2] |= is1 << (8 * (b & 3));
          n0 |= is0 << (4 * b + 1);
          n1 |= is1 << (4 * b + 1);
        }
      }
    }
    const int64_t rb = ((int64_t)c * Mp + m) * 2;  // row of (class, snp, plane 0)
    reinterpret_cast<uint2 *>(bytes)[(rb + 0) * (S / 8) + q] = make_uint2(b0[0], b0[1]);
    reinterpret_cast<uint2 *>(bytes)[(rb + 1) * (S / 8) + q] = make_uint2(b1[0], b1[1]);
    nib[(rb + 0) * (S / 8) + q] = n0;
    nib[(rb + 1) * (S / 8) + q] = n1;
  }
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

__global__ void __launch_bounds__(256) log_tables_kernel(const double *__restrict__ lf64,
                                                         float *__restrict__ lf32,
                                                         uint32_t *__restrict__ lfx, int64_t n,
                                                         double scale) {
  const int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (x >= n) return;
  const double v = lf64[x];
  lf32[x] = (float)v;
  lfx[x] = (uint32_t)(unsigned long long)rint(v * scale);
}

hipError_t launch_log_tables(const double *lf64, float *lf32, uint32_t *lfx, int64_t n, int shift,
                             hipStream_t s) {
  hipLaunchKernelGGL(log_tables_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, lf64,
                     lf32, lfx, n, ldexp(1.0, shift));
  return hipGetLastError();
}

hipError_t launch_encode(const uint8_t *geno, int64_t ld, const int32_t *sample_list, int32_t M,
                         int32_t Mp, int32_t W0, int32_t W1, uint32_t *planes, int32_t *status,
                         hipStream_t s) {
  const int Wtot = W0 + W1;
  if (Wtot <= 0) return hipSuccess;
  dim3 grid((Mp + 3) / 4, (Wtot + kEncWords - 1) / kEncWords);
  hipLaunchKernelGGL(encode_kernel, grid, dim3(256), 0, s, geno, ld, sample_list, M, Mp, Wtot,
                     planes, status);
  return hipGetLastError();
}

hipError_t launch_encode_bytes(const uint8_t *geno, int64_t ld, int32_t M, int32_t N, int32_t Mp,
                               int32_t S, uint8_t *bytes, hipStream_t s) {
  const int S4 = S / 4;
  dim3 grid((S4 + 255) / 256, Mp < 65535 ? Mp : 65535);
  hipLaunchKernelGGL(encode_bytes_kernel, grid, dim3(256), 0, s, geno, ld, M, N, Mp, S,
                     reinterpret_cast<uint32_t *>(bytes));
  return hipGetLastError();
}

hipError_t launch_encode_nibbles(const uint8_t *geno, int64_t ld, int32_t M, int32_t N, int32_t Mp,
                                 int32_t S, uint8_t *nib, hipStream_t s) {
  const int S8 = S / 8;
  dim3 grid((S8 + 255) / 256, Mp < 65535 ? Mp : 65535);
  hipLaunchKernelGGL(encode_nibbles_kernel, grid, dim3(256), 0, s, geno, ld, M, N, Mp, S,
                     reinterpret_cast<uint32_t *>(nib));
  return hipGetLastError();
}

hipError_t launch_encode_values(const uint8_t *geno, int64_t ld, const int32_t *list, int32_t off0,
                                int32_t len0, int32_t off1, int32_t len1, int32_t classes,
                                int32_t M, int32_t Mp, int32_t S, uint8_t *bytes, uint8_t *nib,
                                hipStream_t s) {
  dim3 grid((S / 8 + 255) / 256, Mp < 65535 ? Mp : 65535, classes);
  hipLaunchKernelGGL(encode_values_kernel, grid, dim3(256), 0, s, geno, ld, list, off0, len0, off1,
                     len1, M, Mp, S, reinterpret_cast<uint32_t *>(bytes),
                     reinterpret_cast<uint32_t *>(nib));
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
