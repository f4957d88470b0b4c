// Selection of the k lowest K2 (paper: the solution is the combination with
// the lowest K2, end of the Problem Formulation section; GPU approaches
// section: each thread keeps its best, the host picks the final one).
//
// Here, for k >= 1 and exactly:
//   1. a first bound on the k-th smallest FP32 score T32 from one histogram of
//      2048 bins over the score plane's key range: T32 lies in the bin that
//      holds the k-th value.  For large planes the bound comes instead from a
//      full radix select (3 passes of 2048 bins) on a sample, every 32nd block
//      of 1024 scores: the sample's k-th smallest value is at least T32 (its k
//      smallest are k scores of the plane), which reads the plane once instead
//      of twice.  Every score up to the bound plus 2 e(N) is compacted into a
//      short list, and one workgroup per job finishes the select and collects
//      the candidates from that list (kernels over the plane or a long list do
//      it where the list overflows its capacity or is long);
//   2. every triplet with K2_fp32 <= T32 + 2 e(N) is a candidate, where e(N)
//      bounds |K2_fp32 - K2_fp64| for any table of N samples, so the candidate
//      set contains every member of the FP64 top-k;
//   3. each candidate's table is recounted and K2 re-evaluated in FP64 with
//      Eq. 1's bracketing, rows summed in row order;
//   4. each candidate's position under (K2_fp64, i, j, k) is counted against
//      all others and the first k are written out.
#include <algorithm>

#include "epi3_internal.h"

namespace epi3 {

// ---------------------------------------------------------------- init ----
// A kernel's share of job records, passed by value.
struct SelJobs {
  SelJob j[kSelJobsPerLaunch];
};
static_assert(sizeof(SelJobs) <= 3968, "kernel argument block");

// One workgroup per job: the record, a fresh state and clear histograms.  (One
// thread per job clearing 2048 bins after one launch per record took 13 + 2 us
// of the smallest scans; this takes 2.)
__global__ void __launch_bounds__(256) init_select_kernel(SelJobs jobs, SelJob *dst) {
  const SelJob &J = jobs.j[blockIdx.x];
  for (int b = threadIdx.x; b < kHistBins; b += 256) {
    J.hist[b] = 0u;
    J.hist2[b] = 0u;
    J.hist2[kHistBins + b] = 0u;
  }
  if (threadIdx.x != 0) return;
  dst[blockIdx.x] = J;
  SelState *st = J.st;
  *st = SelState{};
  st->kmin = 0xffffffffu;
  st->T = J.T;
  st->k = J.k;
  st->keff = J.k < J.T ? J.k : J.T;
}

// ----------------------------------------------------------- windows ----
// The keys [lo, lo + span] as the window of a pass of 2048 bins.
__device__ __forceinline__ SelWindow window_of(uint32_t lo, uint32_t span, uint64_t krem) {
  SelWindow w{};
  w.lo = lo;
  w.whi = lo + span;
  w.krem = krem;
  if (span == 0u) {
    w.done = 1u;
    w.kth = lo;
  } else {
    const int bl = 32 - __builtin_clz(span);  // bits of span
    w.shift = bl > 11 ? bl - 11 : 0;
  }
  return w;
}

// First window over a whole key range.
__device__ __forceinline__ SelWindow first_window(const SelState *st) {
  if (st->keff <= 0) {
    SelWindow w{};
    w.done = 2u;  // nothing to select
    return w;
  }
  return window_of(st->kmin, st->kmax - st->kmin, (uint64_t)st->keff);
}

// Narrows w to the bin that holds its krem-th key (unchanged if no bin does),
// by one whole workgroup of NT threads: each thread sums 2048 / NT neighbouring
// bins, the sums are scanned by wave, and the thread that holds the key's bins
// walks them.
template <int NT>
__device__ SelWindow find_bin(const uint32_t *hist, SelWindow w) {
  if (w.done) return w;
  constexpr int B = kHistBins / NT;
  __shared__ uint64_t wave_total[NT / 64];
  __shared__ SelWindow out;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint32_t h[B];
  uint64_t sum = 0;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    h[b] = hist[t * B + b];
    sum += h[b];
  }
  uint64_t upto = sum;  // inclusive scan over the wave
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t v = __shfl_up(upto, off);
    if (lane >= off) upto += v;
  }
  if (lane == 63) wave_total[wave] = upto;
  if (t == 0) out = w;
  __syncthreads();
  uint64_t before = upto - sum;
  for (int x = 0; x < wave; ++x) before += wave_total[x];
  if (before < w.krem && before + sum >= w.krem) {  // exactly one thread, if any
    int b = 0;
    while (before + h[b] < w.krem) before += h[b++];
    const uint32_t lo = w.lo + ((uint32_t)(t * B + b) << w.shift);
    const uint32_t width = (1u << w.shift) - 1u;
    SelWindow n = w;
    n.lo = lo;
    n.whi = lo > 0xffffffffu - width ? 0xffffffffu : lo + width;
    n.krem = w.krem - before;
    if (w.shift == 0) {
      n.done = 1u;
      n.kth = lo;
    } else {
      n.shift = w.shift > 11 ? w.shift - 11 : 0;
    }
    out = n;
  }
  __syncthreads();
  const SelWindow r = out;
  __syncthreads();  // before the next call writes `out`
  return r;
}

// v + err2, rounded up to the next float (v >= 0).
__device__ __forceinline__ float bound_up(uint32_t key, double err2) {
  const double u = (double)key2f(key) + err2;
  float f = (float)u;
  if ((double)f < u) f = __uint_as_float(__float_as_uint(f) + 1u);
  return f;
}

// Plane index of element e of the sample (every kSampleStride-th block).
__device__ __forceinline__ int64_t sample_at(int64_t e) {
  return (e / kSampleBlock) * kSampleBlock * kSampleStride + e % kSampleBlock;
}
// Elements of the sample of a plane of T scores (the last block may be short).
__host__ __device__ __forceinline__ int64_t sample_len(int64_t T) {
  const int64_t nb = (T + kSampleBlock - 1) / kSampleBlock;          // blocks of the plane
  const int64_t ns = (nb + kSampleStride - 1) / kSampleStride;      // sampled blocks
  const int64_t last = (ns - 1) * kSampleStride;                    // index of the last one
  return ns <= 0 ? 0 : (ns - 1) * kSampleBlock + (T - last * kSampleBlock < kSampleBlock
                                                       ? T - last * kSampleBlock
                                                       : kSampleBlock);
}

// A plane's scores before the first that is aligned to 16 bytes (the planes of
// a phenotype batch start T scores apart).
__device__ __forceinline__ int64_t unaligned_head(const float *score, int64_t n) {
  const int64_t head = (int64_t)((16u - (reinterpret_cast<uintptr_t>(score) & 15u)) & 15u) >> 2;
  return head < n ? head : n;
}

__device__ __forceinline__ uint32_t *hist_of(const SelJob &J, int p) {
  return p == 0 ? J.hist : J.hist2 + (p - 1) * kHistBins;
}

// Histogram pass p of 2048 bins over the window that pass p - 1 left; every
// workgroup narrows that window itself (2048 counts, instead of a kernel
// between the passes) and workgroup 0 keeps it for the next pass.
enum { kPassPlane = 0,   // jobs without a sampled bound: the whole plane
       kPassSample = 1,  // sampling jobs: the plane's sample
       kPassRest = 2 };  // jobs that tail_kernel left: the list if it holds all keys, else the plane
__global__ void __launch_bounds__(256) hist_kernel(const SelJob *__restrict__ sj, int which, int p) {
  const SelJob &J = sj[blockIdx.y];
  SelState *st = J.st;
  if (which == kPassRest ? !st->pending : !J.score || (J.sample != 0) != (which == kPassSample)) return;
  const bool list = which == kPassRest && st->cmode == 1u && st->cn <= (unsigned long long)J.ccap;
  const int64_t n = which == kPassSample ? sample_len(J.T) : list ? (int64_t)st->cn : J.T;
  const float *score = J.score;
  const bool wide = !list && which != kPassSample;  // a plane: 16-byte loads
  if (blockIdx.x > 0 && (int64_t)blockIdx.x * 256 * (wide ? 4 : 1) >= n) return;
  SelWindow w;
  if (p > 0) w = find_bin<256>(hist_of(J, p - 1), st->win[p - 1]);
  else if (which == kPassRest) w = st->rest;
  else w = first_window(st);
  if (blockIdx.x == 0 && threadIdx.x == 0) st->win[p] = w;
  if (w.done) return;
  __shared__ uint32_t h[kHistBins];
  for (int b = threadIdx.x; b < kHistBins; b += 256) h[b] = 0u;
  __syncthreads();
  auto add = [&](uint32_t key) {
    if (key >= w.lo) {
      const uint32_t d = (key - w.lo) >> w.shift;
      if (d < (uint32_t)kHistBins) atomicAdd(&h[d], 1u);
    }
  };
  const int64_t t0 = blockIdx.x * (int64_t)256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  if (which == kPassSample) {
    for (int64_t x = t0; x < n; x += step) add(f2key(score[sample_at(x)]));
  } else if (list) {
    for (int64_t x = t0; x < n; x += step) add(J.ckey[x]);
  } else {
    const int64_t head = unaligned_head(score, n), n4 = (n - head) >> 2;
    const float4 *s4 = reinterpret_cast<const float4 *>(score + head);
    auto add4 = [&](float4 v) {
      add(f2key(v.x));
      add(f2key(v.y));
      add(f2key(v.z));
      add(f2key(v.w));
    };
    int64_t x = t0;
    for (; x + 3 * step < n4; x += 4 * step) {  // four loads in flight
      const float4 v0 = s4[x], v1 = s4[x + step], v2 = s4[x + 2 * step], v3 = s4[x + 3 * step];
      add4(v0);
      add4(v1);
      add4(v2);
      add4(v3);
    }
    for (; x < n4; x += step) add4(s4[x]);
    const int64_t past = head + 4 * n4;  // the first workgroup: the ends
    if (t0 < head) add(f2key(score[t0]));
    if (t0 < n - past) add(f2key(score[past + t0]));
  }
  __syncthreads();
  uint32_t *out = hist_of(J, p);
  for (int b = threadIdx.x; b < kHistBins; b += 256)
    if (h[b]) atomicAdd(&out[b], h[b]);
}

// Every score <= the bound goes to the compacted list (key, rank).  The bound
// is the last key of the bin (or the sample's k-th key) + 2 e(N), at least the
// final threshold, so the list holds every key that the rest of the selection
// looks at.  A workgroup gathers its entries in LDS and takes its places in the
// list with one atomic: one per wave and step on the job's counter took most
// of the time where thousands are found (512 SNPs: 50 -> 20 us for 89 MB).
constexpr uint32_t kHeld = 512;
__global__ void __launch_bounds__(256) compact_kernel(const SelJob *__restrict__ sj) {
  const SelJob &J = sj[blockIdx.y];
  SelState *st = J.st;
  const int64_t T = J.T, ccap = J.ccap;
  if (!J.score || st->keff <= 0) return;
  if (blockIdx.x > 0 && (int64_t)blockIdx.x * 256 * 4 >= T) return;
  const int last = J.sample ? kHistPasses - 1 : 0;
  const SelWindow win = find_bin<256>(hist_of(J, last), st->win[last]);
  const float ub = bound_up(win.done ? win.kth : win.whi, J.err2);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->ub = ub;
    st->cmode = 1u;
  }
  __shared__ uint32_t held, hkey[kHeld];
  __shared__ int64_t hrank[kHeld];
  __shared__ unsigned long long first;
  if (threadIdx.x == 0) held = 0u;
  __syncthreads();
  const float *score = J.score;
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  // appends the wave's scores with pred set (wave-uniform call) to the
  // workgroup's list in LDS, or past its end to the job's list
  auto emit = [&](bool pred, float v, int64_t x) {
    const unsigned long long m = __ballot(pred);
    if (m == 0ull) return;
    uint32_t pos0 = 0;
    if (lane == 0) pos0 = atomicAdd(&held, (uint32_t)__popcll(m));
    pos0 = __shfl(pos0, 0);
    const uint32_t pos = pos0 + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    if (pred && pos < kHeld) {
      hkey[pos] = f2key(v);
      hrank[pos] = x;
    }
    const unsigned long long over = __ballot(pred && pos >= kHeld);
    if (over == 0ull) return;
    unsigned long long g0 = 0;
    if (lane == 0) g0 = atomicAdd(&st->cn, (unsigned long long)__popcll(over));
    g0 = __shfl(g0, 0);
    const unsigned long long g = g0 + __popcll(over & ((1ull << lane) - 1ull));
    if (pred && pos >= kHeld && (int64_t)g < ccap) {
      J.ckey[g] = f2key(v);
      J.crank[g] = x;
    }
  };
  // 16-byte loads: four scores per lane and step; nearly every step holds no
  // candidate, so one ballot decides
  const int64_t head = unaligned_head(score, T), T4 = (T - head) >> 2;
  const float4 *s4 = reinterpret_cast<const float4 *>(score + head);
  auto test4 = [&](bool in, float4 v, int64_t x4) {
    const bool any = in && (v.x <= ub || v.y <= ub || v.z <= ub || v.w <= ub);
    if (__ballot(any) == 0ull) return;
    const int64_t x = head + 4 * x4;
    emit(in && v.x <= ub, v.x, x);
    emit(in && v.y <= ub, v.y, x + 1);
    emit(in && v.z <= ub, v.z, x + 2);
    emit(in && v.w <= ub, v.w, x + 3);
  };
  int64_t base = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~63);
  for (; base + 3 * stride + 63 < T4; base += 4 * stride) {  // four loads in flight
    const int64_t x4 = base + lane;
    const float4 v0 = s4[x4], v1 = s4[x4 + stride], v2 = s4[x4 + 2 * stride], v3 = s4[x4 + 3 * stride];
    test4(true, v0, x4);
    test4(true, v1, x4 + stride);
    test4(true, v2, x4 + 2 * stride);
    test4(true, v3, x4 + 3 * stride);
  }
  for (; base < T4; base += stride) {
    const int64_t x4 = base + lane;
    const bool in = x4 < T4;
    test4(in, in ? s4[x4] : make_float4(0.f, 0.f, 0.f, 0.f), x4);
  }
  if (blockIdx.x == 0 && threadIdx.x < 64) {  // the ends: at most three scores each
    const int64_t past = head + 4 * T4;
    const float v = lane < head ? score[lane] : 0.f, w = lane < T - past ? score[past + lane] : 0.f;
    emit(lane < head && v <= ub, v, lane);
    emit(lane < T - past && w <= ub, w, past + lane);
  }
  __syncthreads();
  const uint32_t n = held < kHeld ? held : kHeld;
  if (threadIdx.x == 0 && n > 0) first = atomicAdd(&st->cn, (unsigned long long)n);
  __syncthreads();
  for (uint32_t x = threadIdx.x; x < n; x += 256) {
    const int64_t pos = (int64_t)first + x;
    if (pos < ccap) {
      J.ckey[pos] = hkey[x];
      J.crank[pos] = hrank[x];
    }
  }
}

// The rest of a job's selection by one workgroup: the remaining passes and the
// candidate collection over the compacted list, or over a plane of at most
// kTailPlane scores whose list overflowed.  Longer lists and planes are left to
// the kernels that spread them over the chip (st->pending).  What bounds these
// steps is launches and barriers, not the few thousand keys: two passes,
// threshold and collection took six launches and 28 us of a 157-SNP scan, this
// takes 7 us (64 SNPs: 6; the launches that find nothing left, 13, are only
// made for planes and lists that may be left).
__global__ void __launch_bounds__(1024) tail_kernel(const SelJob *__restrict__ sj) {
  const SelJob &J = sj[blockIdx.x];
  SelState *st = J.st;
  const int t = threadIdx.x, lane = t & 63;
  const bool list = st->cmode == 1u && st->cn <= (unsigned long long)J.ccap;
  const int64_t n = list ? (int64_t)st->cn : J.T;
  const int64_t keff = st->keff;
  SelWindow w{};
  if (keff <= 0) {
    w.done = 2u;
  } else if (!J.score) {
    // list built under the bound: no plane to fall back on if it overflowed
    // (reported as a capacity error; every later kernel skips the job)
    if (!list) w.done = 3u;
    else {
      const uint32_t top = f2key(st->ub), hi = top < st->kmax ? top : st->kmax;
      w = window_of(st->kmin, hi > st->kmin ? hi - st->kmin : 0u, (uint64_t)keff);
    }
  } else {
    const int last = J.sample ? kHistPasses - 1 : 0;
    w = find_bin<1024>(hist_of(J, last), st->win[last]);
    if (J.sample) {
      const uint32_t hi = w.done == 1u ? w.kth : w.whi;
      w = window_of(st->kmin, hi - st->kmin, (uint64_t)keff);
    }
  }
  __syncthreads();  // every thread has read the state
  if (w.done > 1u) {
    if (t == 0) st->done = w.done;
    return;
  }
  if (n > (list ? kTailList : kTailPlane)) {
    for (int b = t; b < kHistBins; b += 1024) J.hist[b] = J.hist2[b] = J.hist2[kHistBins + b] = 0u;
    if (t == 0) {
      st->rest = w;
      st->pending = 1u;
    }
    return;
  }
  __shared__ uint32_t h[kHistBins];
  __shared__ uint32_t found;
  const float *score = J.score;
  auto key_at = [&](int64_t x) { return list ? J.ckey[x] : f2key(score[x]); };
  for (int p = 0; p < kHistPasses && !w.done; ++p) {
    for (int b = t; b < kHistBins; b += 1024) h[b] = 0u;
    __syncthreads();
    for (int64_t x = t; x < n; x += 1024) {
      const uint32_t key = key_at(x);
      if (key >= w.lo) {
        const uint32_t d = (key - w.lo) >> w.shift;
        if (d < (uint32_t)kHistBins) atomicAdd(&h[d], 1u);
      }
    }
    __syncthreads();
    w = find_bin<1024>(h, w);
  }
  if (w.done != 1u) return;  // fewer than keff keys in the range
  const float thr = bound_up(w.kth, J.err2);
  if (t == 0) found = 0u;
  __syncthreads();
  for (int64_t base = t & ~63; base < n; base += 1024) {
    const int64_t x = base + lane;
    const uint32_t key = x < n ? key_at(x) : 0u;
    const bool pred = x < n && key2f(key) <= thr;
    const unsigned long long m = __ballot(pred);
    if (m == 0ull) continue;
    uint32_t pos0 = 0;
    if (lane == 0) pos0 = atomicAdd(&found, (uint32_t)__popcll(m));
    pos0 = __shfl(pos0, 0);
    const int64_t pos = (int64_t)pos0 + __popcll(m & ((1ull << lane) - 1ull));
    if (pred && pos < J.cap) {
      J.cand[pos] = list ? J.crank[x] : x;
      J.candkey[pos] = key;
    }
  }
  __syncthreads();
  if (t == 0) {
    st->kth = w.kth;
    st->thr = thr;
    st->ncand = found;
    st->done = 1u;
  }
}

// The jobs that tail_kernel left, after their passes: threshold T32 + 2 e(N)
// (rounded up to the next float), and every score up to it is a candidate.
__global__ void __launch_bounds__(256) collect_kernel(const SelJob *__restrict__ sj, int passes) {
  const SelJob &J = sj[blockIdx.y];
  SelState *st = J.st;
  if (!st->pending) return;
  const SelWindow w = find_bin<256>(hist_of(J, passes - 1), st->win[passes - 1]);
  if (w.done != 1u) return;
  const float thr = bound_up(w.kth, J.err2);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->kth = w.kth;
    st->thr = thr;
    st->done = 1u;
  }
  const bool list = st->cmode == 1u && st->cn <= (unsigned long long)J.ccap;
  const float *score = J.score;
  const int64_t n = list ? (int64_t)st->cn : J.T, cap = J.cap;
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t base = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~63); base < n;
       base += stride) {
    const int64_t x = base + lane;
    const bool pred = x < n && (list ? key2f(J.ckey[x]) : score[x]) <= thr;
    const unsigned long long m = __ballot(pred);
    if (m == 0ull) continue;
    unsigned long long pos0 = 0;
    if (lane == 0) pos0 = atomicAdd(&st->ncand, (unsigned long long)__popcll(m));
    pos0 = __shfl(pos0, 0);
    const unsigned long long pos = pos0 + __popcll(m & ((1ull << lane) - 1ull));
    if (pred && (int64_t)pos < cap) {
      J.cand[pos] = list ? J.crank[x] : x;
      J.candkey[pos] = list ? J.ckey[x] : f2key(score[x]);
    }
  }
}

// ----------------------------------------------------- FP64 re-score ----
// Sums of sixteen values over the lanes of a wave, in every lane.  Exchange
// steps halve the values per lane (8 + 4 + 2 + 1 swaps), two more add up the
// rest: 17 lane exchanges instead of six per value.
__device__ __forceinline__ void wave_sum16(const uint32_t a[16], int out[16]) {
  const int lane = threadIdx.x & 63;
  uint32_t v[16];
#pragma unroll
  for (int x = 0; x < 16; ++x) v[x] = a[x];
#pragma unroll
  for (int half = 8; half >= 1; half >>= 1) {
    const bool up = lane & half;  // keeps the upper half of the values
#pragma unroll
    for (int x = 0; x < half; ++x) {
      const uint32_t send = up ? v[x] : v[x + half], keep = up ? v[x + half] : v[x];
      v[x] = keep + __shfl_xor(send, half);
    }
  }
  v[0] += __shfl_xor(v[0], 16);
  v[0] += __shfl_xor(v[0], 32);  // lane x % 16 holds value x
#pragma unroll
  for (int x = 0; x < 16; ++x) out[x] = __builtin_amdgcn_readlane((int)v[0], x);
}

// Corner cells n[c][4a + 2b + c] of the classes c = 0 and 1 (words [0, W0) and
// [W0, W0 + W1)), or with a mask, of all samples and of the mask's (words
// [0, W0)), by the lanes of one wave.
__device__ __forceinline__ void corners(const uint32_t *planes, int64_t Mp, int W0, int W1, int i,
                                        int j, int k, const uint32_t *mask, uint32_t n[2][8]) {
  const int lane = threadIdx.x & 63;
  uint32_t a[16] = {};
  auto count = [&](int w, int c, uint32_t mk) {
    const uint2 *row = reinterpret_cast<const uint2 *>(planes) + (int64_t)w * Mp;
    const uint2 xi = row[i], xj = row[j], xk = row[k];
    const uint32_t xiv[2] = {xi.x, xi.y}, xjv[2] = {xj.x, xj.y}, xkv[2] = {xk.x, xk.y};
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const uint32_t m = xiv[p >> 2] & xjv[(p >> 1) & 1] & xkv[p & 1];
      a[8 * c + p] += __builtin_popcount(m & mk);
      if (mask) a[p] += __builtin_popcount(m);
    }
  };
  if (mask) {
    for (int w = lane; w < W0; w += 64) count(w, 1, mask[w]);
  } else {
    for (int w = lane; w < W0; w += 64) count(w, 0, 0xffffffffu);
    for (int w = W0 + lane; w < W0 + W1; w += 64) count(w, 1, 0xffffffffu);
  }
  int out[16];
  wave_sum16(a, out);
#pragma unroll
  for (int p = 0; p < 16; ++p) n[p >> 3][p & 7] = (uint32_t)out[p];
}

__device__ __forceinline__ void pair_args(const int32_t *pairs, int64_t Mp, int i, int j, int k,
                                          int aij[4], int aik[4], int ajk[4], int mi[2], int mj[2],
                                          int mk[2], int64_t st = 1) {
  const int4 *pr = reinterpret_cast<const int4 *>(pairs);
  const int4 pij = pr[((int64_t)i * Mp + j) * st], pik = pr[((int64_t)i * Mp + k) * st],
             pjk = pr[((int64_t)j * Mp + k) * st];
  const int4 ii = pr[((int64_t)i * Mp + i) * st], jj = pr[((int64_t)j * Mp + j) * st],
             kk = pr[((int64_t)k * Mp + k) * st];
  aij[0] = pij.x; aij[1] = pij.y; aij[2] = pij.z; aij[3] = pij.w;
  aik[0] = pik.x; aik[1] = pik.y; aik[2] = pik.z; aik[3] = pik.w;
  ajk[0] = pjk.x; ajk[1] = pjk.y; ajk[2] = pjk.z; ajk[3] = pjk.w;
  mi[0] = ii.x; mi[1] = ii.w; mj[0] = jj.x; mj[1] = jj.w; mk[0] = kk.x; mk[1] = kk.w;
}

// Full table [2][27] of one triplet, computed by the lanes of one wave.
// SPLIT: class words [0, W0) and [W0, W0 + W1), pairs [2][Mp][Mp].
// MASKED: totals from all words and pairs[0]; cases with the mask and
// case_pairs; controls = totals - cases.
__device__ void triplet_table(const uint32_t *planes, const int32_t *pairs,
                              const int32_t *case_pairs, int64_t case_stride,
                              const uint32_t *mask, int layout, int64_t Mp, int W0, int W1,
                              int N0, int N1, int i, int j, int k, int tab[2][27]) {
  int aij[4], aik[4], ajk[4], mi[2], mj[2], mk[2];
  uint32_t n[2][8];
  corners(planes, Mp, W0, W1, i, j, k, layout == EPI3_LAYOUT_SPLIT ? nullptr : mask, n);
  if (layout == EPI3_LAYOUT_SPLIT) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      pair_args(pairs + (int64_t)c * Mp * Mp * 4, Mp, i, j, k, aij, aik, ajk, mi, mj, mk);
      complete_table(n[c], aij, aik, ajk, mi, mj, mk, c ? N1 : N0, tab[c]);
    }
  } else {
    int tot[27];
    pair_args(pairs, Mp, i, j, k, aij, aik, ajk, mi, mj, mk);
    complete_table(n[0], aij, aik, ajk, mi, mj, mk, N0 + N1, tot);
    // case pair tables: two 16-bit counts per word
    {
      const uint2 *cp = reinterpret_cast<const uint2 *>(case_pairs);
      auto unpack = [&](int x, int y, int v[4]) {
        const uint2 w = cp[((int64_t)x * Mp + y) * case_stride];
        v[0] = (int)(w.x & 0xffffu); v[1] = (int)(w.x >> 16);
        v[2] = (int)(w.y & 0xffffu); v[3] = (int)(w.y >> 16);
      };
      int d[4];
      unpack(i, j, aij); unpack(i, k, aik); unpack(j, k, ajk);
      unpack(i, i, d); mi[0] = d[0]; mi[1] = d[3];
      unpack(j, j, d); mj[0] = d[0]; mj[1] = d[3];
      unpack(k, k, d); mk[0] = d[0]; mk[1] = d[3];
    }
    complete_table(n[1], aij, aik, ajk, mi, mj, mk, N1, tab[1]);
#pragma unroll
    for (int x = 0; x < 27; ++x) tab[0][x] = tot[x] - tab[1][x];
  }
}

// Pair (i, j) of lexicographic rank `rank` among the pairs of M SNPs.
__device__ __forceinline__ void decode_pair_rank(int64_t M, int64_t rank, int &i, int &j) {
  int lo = 0, hi = (int)M - 2;  // last i whose first rank <= rank
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pair_rank(M, mid, mid + 1) <= rank) lo = mid; else hi = mid - 1;
  }
  i = lo;
  j = (int)(rank - pair_rank(M, i, i + 1)) + i + 1;
}

// Both 9-row tables of the pair (i, j) of a SPLIT data set, recounted from
// the planes by the lanes of one wave: the four cells with genotypes in
// {0, 1} and the per-SNP counts, then the rest by pair_cells.
__device__ void pair_table(const uint32_t *planes, int64_t Mp, int W0, int W1, int N0, int N1,
                           int i, int j, int tab[2][27]) {
  const int lane = threadIdx.x & 63;
  uint32_t a[16] = {};  // per class n[2a + b] (4), mi[a] (2), mj[b] (2)
  auto count = [&](int w, int c) {
    const uint2 *row = reinterpret_cast<const uint2 *>(planes) + (int64_t)w * Mp;
    const uint2 xi = row[i], xj = row[j];
    a[8 * c + 0] += __builtin_popcount(xi.x & xj.x);
    a[8 * c + 1] += __builtin_popcount(xi.x & xj.y);
    a[8 * c + 2] += __builtin_popcount(xi.y & xj.x);
    a[8 * c + 3] += __builtin_popcount(xi.y & xj.y);
    a[8 * c + 4] += __builtin_popcount(xi.x);
    a[8 * c + 5] += __builtin_popcount(xi.y);
    a[8 * c + 6] += __builtin_popcount(xj.x);
    a[8 * c + 7] += __builtin_popcount(xj.y);
  };
  for (int w = lane; w < W0; w += 64) count(w, 0);
  for (int w = W0 + lane; w < W0 + W1; w += 64) count(w, 1);
  int v[16];
  wave_sum16(a, v);
#pragma unroll
  for (int c = 0; c < 2; ++c) pair_cells(v + 8 * c, v + 8 * c + 4, v + 8 * c + 6, c ? N1 : N0, tab[c]);
}

// Rows x of both classes' tables by lane: row 64 p + lane in r[class][p].
template <int ROWS>
struct LaneRows {
  static constexpr int P = (ROWS + 63) / 64;
  int r[2][P];
  __device__ __forceinline__ explicit LaneRows(const int (*tab)[ROWS]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < P; ++p) {
        r[c][p] = 0;
#pragma unroll
        for (int x = 64 * p; x < ROWS && x < 64 * p + 64; ++x)
          r[c][p] = lane == x - 64 * p ? tab[c][x] : r[c][p];
      }
  }
  // Eq. 1 in FP64: each row L[r + 1] - (L[r_0] + L[r_1]), added up in row
  // order.  The lookups of all rows are in flight at once; one after the other
  // they took most of a candidate's time.
  __device__ __forceinline__ double k2(int rows, const double *L) const {
    const int lane = threadIdx.x & 63;
    double sum = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      double term = 0.0;
      if (64 * p + lane < rows) term = L[r[0][p] + r[1][p] + 1] - (L[r[0][p]] + L[r[1][p]]);
      for (int x = 64 * p; x < rows && x < 64 * p + 64; ++x) sum += __shfl(term, x - 64 * p);
    }
    return sum;
  }
};

// A candidate's record, by the lanes of one wave.
template <int ROWS>
__device__ __forceinline__ void put_record(const SelJob &J, int64_t c, int64_t rank, int i, int j, int k,
                                           int l, const int (*tab)[ROWS], int rows) {
  const int lane = threadIdx.x & 63;
  const LaneRows<ROWS> lr(tab);
  const double k2 = lr.k2(rows, J.lf64);
  CandRec &R = J.rec[c];
  if (lane == 0) {
    R.key = (uint64_t)__double_as_longlong(k2);
    R.rank = rank;
    R.i = i; R.j = j; R.k = k; R.l = l;
    R.k2f = key2f(J.candkey[c]);
    R.k2 = k2;
  }
#pragma unroll
  for (int cl = 0; cl < 2; ++cl)
#pragma unroll
    for (int p = 0; p < LaneRows<ROWS>::P; ++p)
      if (64 * p + lane < rows) R.counts[ROWS * cl + 64 * p + lane] = (uint32_t)lr.r[cl][p];
}

// QUADS: jobs of order 4, a kernel of its own (twice the registers).
template <bool QUADS>
__global__ void __launch_bounds__(256) rescore_kernel(const SelJob *__restrict__ sj) {
  const SelJob &J = sj[blockIdx.y];
  SelState *st = J.st;
  if (st->done != 1u) return;
  const int64_t n = (int64_t)st->ncand < J.cap ? (int64_t)st->ncand : J.cap;
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t c = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6); c < n;
       c += waves) {
    const int64_t rank = J.cand[c];
    if constexpr (QUADS) {
      int i, j, k, l;
      decode_quad_rank(J.M, rank, i, j, k, l);
      int q[2][81];
      const int64_t MpMp4 = (int64_t)J.Mp * J.Mp * 4;
      for (int cl = 0; cl < 2; ++cl) {
        uint32_t cnt[48];
        const int w0 = cl ? J.W0 : 0, w1 = cl ? J.W0 + J.W1 : J.W0;
        quad_counts(J.planes, J.Mp, w0 + lane, w1, 64, i, j, k, l, cnt);
        for (int x = 0; x < 48; x += 16) {
          int sum[16];
          wave_sum16(cnt + x, sum);
          for (int y = 0; y < 16; ++y) cnt[x + y] = (uint32_t)sum[y];
        }
        quad_cells(cnt, J.pairs + cl * MpMp4, J.Mp, i, j, k, l, cl ? J.N1 : J.N0, q[cl]);
      }
      put_record<81>(J, c, rank, i, j, k, l, q, 81);
    } else {
      int tab[2][27];
      if (J.order == 2) {
        int i, j;
        decode_pair_rank(J.M, rank, i, j);
        pair_table(J.planes, J.Mp, J.W0, J.W1, J.N0, J.N1, i, j, tab);
  #pragma unroll
        for (int x = 9; x < 27; ++x) tab[0][x] = tab[1][x] = 0;
        put_record<27>(J, c, rank, i, j, 0, 0, tab, 9);
        continue;
      }
      int i, j, k;
      decode_rank(J.M, rank, i, j, k);
      int N0 = J.N0, N1 = J.N1;
      if (J.n1_dev) {
        N1 = *J.n1_dev;
        N0 = J.N0 + J.N1 - N1;
      }
      triplet_table(J.planes, J.pairs, J.case_pairs, J.case_stride, J.case_mask, J.layout, J.Mp,
                    J.W0, J.W1, N0, N1, i, j, k, tab);
      put_record<27>(J, c, rank, i, j, k, 0, tab, 27);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && (int64_t)st->ncand > J.cap) st->overflow = 1u;
}

// Hit `pos` of the job's list from candidate record x, by the lanes of one wave.
__device__ __forceinline__ void emit_hit(const SelJob &J, int64_t x, int64_t pos) {
  const int lane = threadIdx.x & 63;
  const CandRec &R = J.rec[x];
  auto copy = [&](uint32_t *out, int rows, int off) {
    for (int q = lane; q < 2 * rows; q += 64) {
      const int c = q >= rows;
      out[q] = R.counts[off * c + q - rows * c];
    }
  };
  if (J.order == 4) {
    epi3_quad_hit &H = J.quad_hits[pos];
    if (lane == 0) {
      H.i = R.i; H.j = R.j; H.k = R.k; H.l = R.l;
      H.k2_f32 = R.k2f;
      H.reserved = 0u;
      H.k2 = R.k2;
    }
    copy(&H.counts[0][0], 81, 81);
  } else if (J.order == 2) {
    epi3_pair_hit &H = J.pair_hits[pos];
    if (lane == 0) {
      H.i = R.i; H.j = R.j;
      H.k2_f32 = R.k2f;
      H.reserved = 0u;
      H.k2 = R.k2;
    }
    copy(&H.counts[0][0], 9, 27);
  } else {
    epi3_hit &H = J.hits[pos];
    if (lane == 0) {
      H.i = R.i; H.j = R.j; H.k = R.k;
      H.k2_f32 = R.k2f;
      H.k2 = R.k2;
    }
    copy(&H.counts[0][0], 27, 27);
  }
}

// Rank of every candidate = number of candidates before it under
// (K2_fp64, rank); each workgroup takes 64 candidates (one per lane) and its
// 16 waves split the comparisons, so chains stay short for a few thousand
// candidates.  Jobs with sort buffers (sortP > 0) are ordered by the sort
// kernels below instead.
constexpr int kRankThreads = 1024;
__global__ void __launch_bounds__(kRankThreads) rank_kernel(const SelJob *__restrict__ sj) {
  const SelJob &J = sj[blockIdx.y];
  SelState *st = J.st;
  if (st->done != 1u || J.sortP > 0) return;
  const int64_t n = (int64_t)st->ncand < J.cap ? (int64_t)st->ncand : J.cap;
  const int64_t keff = st->keff;
  __shared__ uint64_t skey[kRankThreads];
  __shared__ int64_t srank[kRankThreads];
  __shared__ int32_t spos[kRankThreads / 64][64];
  __shared__ int64_t place[64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t xb = blockIdx.x; xb * 64 < n; xb += gridDim.x) {
    const int64_t x = xb * 64 + lane;
    uint64_t mykey = ~0ull;
    int64_t myrank = 0;
    if (x < n) {
      mykey = J.rec[x].key;
      myrank = J.rec[x].rank;
    }
    int32_t part = 0;
    for (int64_t yb = 0; yb < n; yb += kRankThreads) {
      const int64_t y = yb + threadIdx.x;
      __syncthreads();
      skey[threadIdx.x] = y < n ? J.rec[y].key : ~0ull;
      srank[threadIdx.x] = y < n ? J.rec[y].rank : INT64_MAX;
      __syncthreads();
      // wave w compares with every 16th entry of the chunk
      const int lim = n - yb < kRankThreads ? (int)(n - yb) : kRankThreads;
      for (int z = wave; z < lim; z += kRankThreads / 64) {
        const uint64_t kz = skey[z];
        part += (kz < mykey) || (kz == mykey && srank[z] < myrank);
      }
    }
    spos[wave][lane] = part;
    __syncthreads();
    if (wave == 0) {
      int64_t pos = 0;
      for (int w = 0; w < kRankThreads / 64; ++w) pos += spos[w][lane];
      place[lane] = x < n && pos < keff ? pos : -1;
    }
    __syncthreads();
    for (int q = wave; q < 64; q += kRankThreads / 64)  // a wave per hit
      if (place[q] >= 0) emit_hit(J, xb * 64 + q, place[q]);
  }
}

// ---- ordering of large candidate sets: bitonic sort of (key, index) ----
// Entries past the candidate count carry key ~0 (above every FP64 key, which
// is the bit pattern of a non-negative double); equal keys of candidates are
// ordered by their lexicographic rank, equal padding keys by index.
__device__ __forceinline__ bool sort_before(const SelJob &J, uint64_t ka, uint32_t ia, uint64_t kb,
                                            uint32_t ib) {
  if (ka != kb) return ka < kb;
  if (ka == ~0ull) return ia < ib;
  return J.rec[ia].rank < J.rec[ib].rank;
}

__global__ void __launch_bounds__(256) sort_init_kernel(const SelJob *__restrict__ sj) {
  const SelJob &J = sj[blockIdx.y];
  const SelState *st = J.st;
  if (J.sortP == 0 || st->done != 1u) return;
  const int64_t n = (int64_t)st->ncand < J.cap ? (int64_t)st->ncand : J.cap;
  for (int64_t x = blockIdx.x * 256 + threadIdx.x; x < J.sortP; x += (int64_t)gridDim.x * 256) {
    J.skey[x] = x < n ? J.rec[x].key : ~0ull;
    J.sidx[x] = (uint32_t)x;
  }
}

// One compare-exchange stage (block size k, distance j >= kSortLocal) over
// global memory: thread t handles the pair (lo, lo + j).
// The launches follow the job with the most entries (a batch's jobs differ where
// their triplets are fewer than the capacity): a job is sorted after the stages of
// k = sortP, and later ones would reach past its entries.
__global__ void __launch_bounds__(256) sort_global_kernel(const SelJob *__restrict__ sj, int64_t k,
                                                          int64_t j) {
  const SelJob &J = sj[blockIdx.y];
  if (k > J.sortP || J.st->done != 1u) return;
  for (int64_t t = blockIdx.x * 256 + threadIdx.x; t < J.sortP / 2; t += (int64_t)gridDim.x * 256) {
    const int64_t lo = ((t & ~(j - 1)) << 1) | (t & (j - 1)), hi = lo + j;
    const bool asc = (lo & k) == 0;
    const uint64_t ka = J.skey[lo], kb = J.skey[hi];
    const uint32_t ia = J.sidx[lo], ib = J.sidx[hi];
    if (asc ? sort_before(J, kb, ib, ka, ia) : sort_before(J, ka, ia, kb, ib)) {
      J.skey[lo] = kb; J.skey[hi] = ka;
      J.sidx[lo] = ib; J.sidx[hi] = ia;
    }
  }
}

// The stages of distance j < kSortLocal inside blocks of kSortLocal entries
// in LDS: every block size from 2 up (full = 1), or only block size k.
constexpr int kSortLocal = 2048;
__global__ void __launch_bounds__(1024) sort_local_kernel(const SelJob *__restrict__ sj, int64_t k,
                                                          int full) {
  const SelJob &J = sj[blockIdx.y];
  if (J.sortP == 0 || k > J.sortP || J.st->done != 1u) return;
  __shared__ uint64_t lk[kSortLocal];
  __shared__ uint32_t li[kSortLocal];
  for (int64_t base = (int64_t)blockIdx.x * kSortLocal; base < J.sortP;
       base += (int64_t)gridDim.x * kSortLocal) {
    __syncthreads();
    for (int x = threadIdx.x; x < kSortLocal; x += 1024) {
      lk[x] = J.skey[base + x];
      li[x] = J.sidx[base + x];
    }
    __syncthreads();
    for (int64_t kk = full ? 2 : k; kk <= (full ? (int64_t)kSortLocal : k); kk <<= 1) {
      for (int jj = (int)((kk < kSortLocal ? kk : kSortLocal) >> 1); jj > 0; jj >>= 1) {
        const int t = threadIdx.x;  // pair t of the block
        const int lo = ((t & ~(jj - 1)) << 1) | (t & (jj - 1)), hi = lo + jj;
        const bool asc = ((base + lo) & kk) == 0;
        const uint64_t ka = lk[lo], kb = lk[hi];
        const uint32_t ia = li[lo], ib = li[hi];
        if (asc ? sort_before(J, kb, ib, ka, ia) : sort_before(J, ka, ia, kb, ib)) {
          lk[lo] = kb; lk[hi] = ka;
          li[lo] = ib; li[hi] = ia;
        }
        __syncthreads();
      }
    }
    for (int x = threadIdx.x; x < kSortLocal; x += 1024) {
      J.skey[base + x] = lk[x];
      J.sidx[base + x] = li[x];
    }
  }
}

__global__ void __launch_bounds__(256) sort_emit_kernel(const SelJob *__restrict__ sj) {
  const SelJob &J = sj[blockIdx.y];
  const SelState *st = J.st;
  if (J.sortP == 0 || st->done != 1u) return;
  const int64_t keff = st->keff;
  for (int64_t pos = blockIdx.x * 4 + (threadIdx.x >> 6); pos < keff; pos += (int64_t)gridDim.x * 4)
    emit_hit(J, J.sidx[pos], pos);
}

hipError_t launch_init_select(const SelJob *h, int32_t n, SelJob *dst_dev, hipStream_t s) {
  for (int x = 0; x < n; x += kSelJobsPerLaunch) {
    SelJobs jobs{};
    const int m = n - x < kSelJobsPerLaunch ? n - x : kSelJobsPerLaunch;
    for (int y = 0; y < m; ++y) jobs.j[y] = h[x + y];
    hipLaunchKernelGGL(init_select_kernel, dim3(m), dim3(256), 0, s, jobs, dst_dev + x);
  }
  return hipGetLastError();
}

// After a batch's sample pass (see launch_sample_bound in the header).
__global__ void __launch_bounds__(256) sample_bound_kernel(const SelJob *main, const SelJob *smp) {
  const SelJob &J = main[blockIdx.x], &S = smp[blockIdx.x];
  const SelWindow w = find_bin<256>(hist_of(S, kHistPasses - 1), S.st->win[kHistPasses - 1]);
  if (threadIdx.x != 0) return;
  SelState *st = J.st;
  // the sample's k smallest are k scores of the whole set, so its k-th
  // smallest is at least the whole set's: every member of the FP64 top-k
  // has an FP32 score <= that + 2 e(N)
  st->ub = w.done == 1u ? bound_up(w.kth, J.err2) : __builtin_inff();
  st->cmode = 1u;
  st->cn = 0ull;
}

hipError_t launch_sample_bound(const SelJob *main_dev, const SelJob *sample_dev, int32_t n_jobs,
                               hipStream_t s) {
  hipLaunchKernelGGL(sample_bound_kernel, dim3(n_jobs), dim3(256), 0, s, main_dev, sample_dev);
  return hipGetLastError();
}

// Workgroups per job of a pass over n scores of each of n_jobs planes.  A
// workgroup adds about 1500 of its 2048 bins to the job's, so it takes 128
// scores per thread once 256 workgroups (over all jobs) are busy, and at least
// 16: 20 planes of 1.4 million scores 60 us with 16 per thread, 32 so.
static unsigned pass_blocks(int64_t n, unsigned n_jobs) {
  const int64_t most = (n + 256 * 16 - 1) / (256 * 16), wide = (n + 256 * 128 - 1) / (256 * 128);
  const int64_t b = std::min(most, std::max<int64_t>(wide, (256 + n_jobs - 1) / n_jobs));
  return (unsigned)(b > 2048 ? 2048 : b < 1 ? 1 : b);
}

hipError_t launch_select_kth(SelJob *sel_dev, int32_t n_jobs, int64_t max_T, hipStream_t s) {
  for (int p = 0; p < kHistPasses; ++p)
    hipLaunchKernelGGL(hist_kernel, dim3(pass_blocks(max_T, n_jobs), n_jobs), dim3(256), 0, s, sel_dev,
                       (int)kPassPlane, p);
  return hipGetLastError();
}

hipError_t launch_select(SelJob *sel_dev, int32_t n_jobs, const SelectSizes &z, hipStream_t s) {
  const unsigned nj = (unsigned)n_jobs;
  const int64_t max_cap = z.max_cap;
  if (z.sampled)
    for (int p = 0; p < kHistPasses; ++p)
      hipLaunchKernelGGL(hist_kernel, dim3(pass_blocks(sample_len(z.max_T), nj), nj), dim3(256), 0, s,
                         sel_dev, (int)kPassSample, p);
  if (z.unsampled)
    hipLaunchKernelGGL(hist_kernel, dim3(pass_blocks(z.max_T, nj), nj), dim3(256), 0, s, sel_dev,
                       (int)kPassPlane, 0);
  if (z.sampled || z.unsampled)
    hipLaunchKernelGGL(compact_kernel, dim3(pass_blocks(z.max_T, nj), nj), dim3(256), 0, s, sel_dev);
  hipLaunchKernelGGL(tail_kernel, dim3(nj), dim3(1024), 0, s, sel_dev);
  if (z.rest) {
    // jobs that the tail left (the others return at once): after the first
    // histogram 21 bits of the key are open, else 32
    const int passes = z.sampled || !z.unsampled ? kHistPasses : kHistPasses - 1;
    const unsigned rb = std::min(pass_blocks(z.max_T, nj), std::max(2048u / nj, 8u));
    for (int p = 0; p < passes; ++p)
      hipLaunchKernelGGL(hist_kernel, dim3(rb, nj), dim3(256), 0, s, sel_dev, (int)kPassRest, p);
    hipLaunchKernelGGL(collect_kernel, dim3(rb, nj), dim3(256), 0, s, sel_dev, passes);
  }
  // a wave per candidate; most capacities are far above the candidates found,
  // and a workgroup without one still takes its turn (20 jobs of 1024: 34 us)
  const unsigned cb = (unsigned)std::min<int64_t>((max_cap + 3) / 4, std::max(1024u / nj, 32u));
  hipLaunchKernelGGL(z.quads ? rescore_kernel<true> : rescore_kernel<false>, dim3(cb, nj), dim3(256), 0, s,
                     sel_dev);
  const unsigned kb = (unsigned)std::min<int64_t>((max_cap + 63) / 64, std::max(256u / nj, 8u));
  hipLaunchKernelGGL(rank_kernel, dim3(kb, nj), dim3(kRankThreads), 0, s, sel_dev);
  const int64_t P = sort_len(max_cap);  // jobs with sort buffers (each skips the other path)
  if (P > 0) {
    const unsigned gb = (unsigned)std::min<int64_t>(P / 512, 4096);
    const unsigned lb = (unsigned)std::min<int64_t>(P / kSortLocal, 1024);
    hipLaunchKernelGGL(sort_init_kernel, dim3(gb, nj), dim3(256), 0, s, sel_dev);
    hipLaunchKernelGGL(sort_local_kernel, dim3(lb, nj), dim3(1024), 0, s, sel_dev, (int64_t)0, 1);
    for (int64_t k2 = 2 * kSortLocal; k2 <= P; k2 <<= 1) {
      for (int64_t j = k2 >> 1; j >= kSortLocal; j >>= 1)
        hipLaunchKernelGGL(sort_global_kernel, dim3(gb, nj), dim3(256), 0, s, sel_dev, k2, j);
      hipLaunchKernelGGL(sort_local_kernel, dim3(lb, nj), dim3(1024), 0, s, sel_dev, k2, 0);
    }
    const unsigned eb = (unsigned)std::min<int64_t>((z.max_k + 3) / 4, 1024);
    hipLaunchKernelGGL(sort_emit_kernel, dim3(eb > 0 ? eb : 1, nj), dim3(256), 0, s, sel_dev);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------ results ----
struct StatusPtrs {
  const int32_t *p[256];
};
__global__ void __launch_bounds__(256) gather_results_kernel(const uint2 *st, int64_t n_st, StatusPtrs ptrs,
                                                             int n_status, int32_t *status_out,
                                                             const uint2 *hits, int64_t n_hits, uint2 *st_out,
                                                             uint2 *hits_out) {
  const int64_t x0 = blockIdx.x * (int64_t)256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  for (int64_t x = x0; x < n_st; x += step) st_out[x] = st[x];
  for (int64_t x = x0; x < n_status; x += step) status_out[x] = *ptrs.p[x];
  for (int64_t x = x0; x < n_hits; x += step) hits_out[x] = hits[x];
}

hipError_t launch_gather_results(const SelState *st, const int32_t *const *status, int32_t n,
                                 const void *hits, int64_t hit_bytes, void *dst, hipStream_t s) {
  static_assert(sizeof(SelState) % 8 == 0, "8-byte units");
  uint8_t *out = static_cast<uint8_t *>(dst);
  for (int32_t base = 0; base < n; base += 256) {
    StatusPtrs ptrs{};
    const int32_t m = n - base < 256 ? n - base : 256;
    for (int32_t x = 0; x < m; ++x) ptrs.p[x] = status[base + x];
    const int64_t units = base == 0 ? hit_bytes / 8 : 0;  // the hits with the first launch
    const unsigned blocks = (unsigned)std::min<int64_t>(std::max<int64_t>((units + 255) / 256, 1), 256);
    hipLaunchKernelGGL(gather_results_kernel, dim3(blocks), dim3(256), 0, s,
                       reinterpret_cast<const uint2 *>(st + base), m * (int64_t)(sizeof(SelState) / 8), ptrs,
                       (int)m, reinterpret_cast<int32_t *>(out + n * (int64_t)sizeof(SelState)) + base,
                       static_cast<const uint2 *>(hits), units,
                       reinterpret_cast<uint2 *>(out + base * (int64_t)sizeof(SelState)),
                       reinterpret_cast<uint2 *>(out + result_head_bytes(n)));
  }
  return hipGetLastError();
}

// ------------------------------------------------------- test hook ----
__global__ void __launch_bounds__(256) score_triplets_kernel(
    const uint32_t *__restrict__ planes, const int32_t *__restrict__ pairs,
    const double *__restrict__ lf64, const uint32_t *__restrict__ lfx, float scale, int M, int64_t Mp, int W0,
    int W1, int N0, int N1, const uint32_t *__restrict__ ijk, int64_t n,
    uint32_t *__restrict__ counts, float *__restrict__ k2f, double *__restrict__ k2d) {
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t c = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6); c < n;
       c += waves) {
    const uint32_t i = ijk[3 * c], j = ijk[3 * c + 1], k = ijk[3 * c + 2];
    if (!(i < j && j < k && k < (uint32_t)M)) {  // not a triplet of this data set
      if (lane == 0) {
        if (k2f) k2f[c] = __builtin_nanf("");
        if (k2d) k2d[c] = __builtin_nan("");
        if (counts)
          for (int x = 0; x < 54; ++x) counts[c * 54 + x] = 0xffffffffu;
      }
      continue;
    }
    int tab[2][27];
    triplet_table(planes, pairs, nullptr, 1, nullptr, EPI3_LAYOUT_SPLIT, Mp, W0, W1, N0, N1, i, j,
                  k, tab);
    const double k2 = k2d ? LaneRows<27>(tab).k2(27, lf64) : 0.0;
    if (lane == 0) {
      uint32_t f = 0u;
      for (int x = 0; x < 27; ++x) {
        const int r0 = tab[0][x], r1 = tab[1][x];
        f += lfx[r0 + r1 + 1] - (lfx[r0] + lfx[r1]);
      }
      if (k2f) k2f[c] = fx_score(f, scale);
      if (k2d) k2d[c] = k2;
      if (counts)
        for (int x = 0; x < 27; ++x) {
          counts[c * 54 + x] = (uint32_t)tab[0][x];
          counts[c * 54 + 27 + x] = (uint32_t)tab[1][x];
        }
    }
  }
}

hipError_t launch_score_triplets(const epi3_dataset &d, const uint32_t *ijk, int64_t n,
                                 uint32_t *counts, float *k2f, double *k2, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 3) / 4;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(score_triplets_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                     (const uint32_t *)d.planes, d.pairs, d.lf64, fx_table(d),
                     fx_scale(d.n_samples), d.n_snps, (int64_t)d.snp_stride,
                     d.words[0], d.words[1], d.n_controls, d.n_cases, ijk, n, counts, k2f, k2);
  return hipGetLastError();
}

}  // namespace epi3
