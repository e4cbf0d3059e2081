// K-Means codebook on standard-normal samples (Sec. 3.4, the K-Means baseline) and its
// fine-tuning for cosine distance.
//
// Lloyd iterations entirely on the device, deterministic, two launches each:
//   cb_accumulate_kernel  nearest centroid per sample (nsn_search.h) and, in the same pass over the samples, the sums of
//                         every cluster's members: one partial per workgroup
//   km_update_kernel      adds the partials in a fixed order (fp64): the new centroids
// (fine-tuning: cb_ordered_kernel and ft_update_kernel; K-Means of samples with a range that fixed-point sums do not
// cover takes cb_ordered_kernel too)
#include <cmath>
#include <cstring>
#include <type_traits>

#include "nsn_host.h"
#include "nsn_search.h"

namespace nsn {

constexpr int kSumBlocks = 256;   // workgroups of the accumulation (and partial sums per cluster)
// four waves per SIMD (128 registers) for 4-dim codewords, two (256) for 8-dim ones: with three (168 registers) those spilled 16
// to 43 of them, and a kernel that needs scratch memory starts later: 2^20 8-dim samples 39 -> 36 us per K-Means iteration,
// 2^14 samples 17 -> 15 us (the ordered 4-dim kernels spill about 20: in lists and addresses).  Of an accumulation of 2^20
// 8-dim samples (27.5 us) set-up and the first samples take about 8, the merge of the waves' sums 3.
template <int SUB>
constexpr int kSumThreads = SUB == 4 ? 1024 : 512;
constexpr int kSumMost = 4096;  // samples added up in LDS at a time

// workspace: centroids, error sum of every workgroup, cosine sum of every cluster, the largest |sample| as fp32 bits, then
// per workgroup of the accumulation the member sums [256][SUB] and the member counts [256].  K-Means keeps the smallest
// |sample| but zero, less one, in the place of the cosine sums.
template <int SUB>
struct CodebookWs {
  double* centroids;
  double* block_err;
  double* cos_sum;
  uint32_t *least_bits, *most_bits;
  double* sums;
  double* counts;
  explicit CodebookWs(void* ws)
      : centroids(static_cast<double*>(ws)),
        block_err(centroids + kCodes * SUB),
        cos_sum(block_err + kSumBlocks),
        least_bits(reinterpret_cast<uint32_t*>(cos_sum)),
        most_bits(reinterpret_cast<uint32_t*>(cos_sum + kCodes)),
        sums(cos_sum + kCodes + 2),
        counts(sums + (size_t)kSumBlocks * kCodes * SUB) {}
  static size_t bytes() {
    return (size_t)(kCodes * SUB + kSumBlocks + kCodes + 2 + kSumBlocks * kCodes * (SUB + 1)) * sizeof(double);
  }
};

// start of a run: the centroids (the first samples, or the codebook at hand), no sample in the range yet
template <typename T>
__global__ void cb_start_kernel(const T* __restrict__ from, double* __restrict__ centroids, int n_elems,
                                uint32_t* __restrict__ least_bits, uint32_t* __restrict__ most_bits) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_elems) centroids[i] = (double)(float)from[i];
  if (i == 0) *least_bits = 0xffffffffu, *most_bits = 0u;
}

// Largest |sample| of the set and the smallest that is not zero, less one, as fp32 bits (their order is that of the values;
// infinities and NaN are above all of them, and zeros less one as well).  Two atomics per workgroup, on lines
// of their own that are served side by side: with one per wave of a 4096-wave launch they took 45 of 56 us.
constexpr int kRangeThreads = 1024, kRangeBlocks = 256;
typedef float row4 __attribute__((ext_vector_type(4), aligned(4)));  // (the samples are aligned as floats are)
__global__ __launch_bounds__(kRangeThreads) void cb_range_kernel(const float* __restrict__ samples, int64_t n_rows,
                                                                 uint32_t* __restrict__ least_bits,
                                                                 uint32_t* __restrict__ most_bits) {
  __shared__ uint32_t red[2][kRangeThreads / 64];
  uint32_t most = 0u, least = 0xffffffffu;
#pragma unroll 4
  for (int64_t i = (int64_t)blockIdx.x * kRangeThreads + threadIdx.x; i < n_rows; i += (int64_t)gridDim.x * kRangeThreads) {
    const row4 v = reinterpret_cast<const row4*>(samples)[i];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t bits = __float_as_uint(fabsf(v[k]));
      most = max(most, bits), least = min(least, bits - 1u);
    }
  }
  auto with_lane = [&](auto mask) {
    constexpr int M = decltype(mask)::value;
    most = max(most, (uint32_t)xor_lane_i32<M>((int)most));
    least = min(least, (uint32_t)xor_lane_i32<M>((int)least));
  };
  with_lane(std::integral_constant<int, 1>{}), with_lane(std::integral_constant<int, 2>{});
  with_lane(std::integral_constant<int, 4>{}), with_lane(std::integral_constant<int, 8>{});
  with_lane(std::integral_constant<int, 16>{}), with_lane(std::integral_constant<int, 32>{});
  if ((threadIdx.x & 63) == 0) red[0][threadIdx.x >> 6] = most, red[1][threadIdx.x >> 6] = least;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kRangeThreads / 64; ++w) most = max(most, red[0][w]), least = min(least, red[1][w]);
    atomicMax(most_bits, most);
    atomicMin(least_bits, least);
  }
}

__global__ void km_round_kernel(double* __restrict__ centroids, __half* __restrict__ out, int n_elems) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_elems) {
    const __half hv = f64_to_f16(centroids[i]);
    out[i] = hv;
    centroids[i] = (double)__half2float(hv);
  }
}

template <int SUB>
__device__ __forceinline__ double exact_dist(const double* __restrict__ centroid, const float (&x)[SUB]) {
  double d = 0.0;
#pragma unroll
  for (int i = 0; i < SUB; ++i) {
    const double t = (double)x[i] - centroid[i];
    d = __dadd_rn(d, __dmul_rn(t, t));  // no fused contraction: plain sum of squares
  }
  return d;
}

// Assignment and, in the same pass over the samples, member sums (ERR false) or the squared error (ERR true).
//
// The sums are formed in LDS by integer atomics on fixed-point values: integer addition is associative, so the result
// does not depend on the order in which lanes and waves arrive.  Every value enters exactly.  With 2^ex the power of two
// above the largest |sample|, values from 2^(ex - 27) on are multiples of 2^(ex - 50); the smaller ones (one normal value in
// twenty million) have sums of their own in units of 2^(ex - 77), which hold everything from 2^(ex - 54) on (sets with
// smaller values go to cb_ordered_kernel: sums_fit below).  At most kSumMost values are added before the LDS sums move
// to fp64 registers: no overflow of 63 bits.  Adding 1.5 * 2^52 puts the fixed-point value into the low bits of the fp64
// pattern; the patterns are added as they are and the member count times the constant's pattern comes off at the end.
// (The form this replaces wrote the assignments out and let one workgroup per cluster look through all of them:
// 270 us per iteration of 2^20 4-dim samples.)
template <int SUB, bool ERR>
__global__ __launch_bounds__(kSumThreads<SUB>) void cb_accumulate_kernel(const float* __restrict__ samples, int64_t n,
                                                                       CodebookWs<SUB> ws) {
  constexpr int NT = kSumThreads<SUB>;
  constexpr int kOwn = (kCodes * SUB + NT - 1) / NT;  // sums a thread carries in registers
  constexpr double kMagic = 6755399441055744.0;      // 1.5 * 2^52
  __shared__ SearchTables<SUB, false> T;
  __shared__ double cx[kCodes][SUB];
  __shared__ unsigned long long acc[ERR ? 1 : SUB][kCodes], acc_small[ERR ? 1 : SUB][kCodes];
  __shared__ uint32_t cnt[kCodes];
  __shared__ double red[NT / 64];
  const int tid = threadIdx.x;
  const int64_t per = ((n + kSumBlocks - 1) / kSumBlocks + 63) & ~(int64_t)63;
  const int64_t begin = (int64_t)blockIdx.x * per, end = min(n, begin + per);
  row4 ahead[SUB / 4];
  auto fetch = [&](int64_t idx) {  // (n >= 1)
    const row4* row = reinterpret_cast<const row4*>(samples) + min(idx, n - 1) * (SUB / 4);
#pragma unroll
    for (int q = 0; q < SUB / 4; ++q) ahead[q] = row[q];
  };
  double centroid[SUB] = {};  // of codeword `tid`
  if (tid < kCodes) {
#pragma unroll
    for (int i = 0; i < SUB; ++i) centroid[i] = ws.centroids[tid * SUB + i];
  }
  fetch(begin + tid);
  const uint32_t most = ERR ? 0u : *ws.most_bits, least = ERR ? 0u : *ws.least_bits;  // (on their way during the set-up)
  auto clear = [&](auto& sums) {
    for (int i = tid; i < kCodes * SUB; i += NT) (&sums[0][0])[i] = 0ull;
  };
  if constexpr (!ERR) {
    clear(acc);
    if (tid < kCodes) cnt[tid] = 0u;
  }
  if (tid < kCodes) {
#pragma unroll
    for (int i = 0; i < SUB; ++i) cx[tid][i] = centroid[i];
  }
  SearchRegs<SUB, false> R;
  search_setup<SUB, false, false>(T, R, tid, [&](int i) { return centroid[i]; });
  int ex = 0;
  uint32_t small = 0u;  // twice the bits of 2^(ex - 27) where the set holds smaller values (but zero)
  if constexpr (!ERR) {
    const float mx = __uint_as_float(most);
    if (mx > 0.f && mx < INFINITY) (void)frexpf(mx, &ex);  // mx < 2^ex
    ex = __builtin_amdgcn_readfirstlane(ex);
    // (from ex = -100 down every fp32 value is a multiple of the unit)
    const uint32_t from = ex > -100 ? (uint32_t)(ex - 27 + 127) << 23 : 0u;
    if (least + 1u < from && least != 0xffffffffu) small = 2u * from;
    small = __builtin_amdgcn_readfirstlane(small);
  }
  const double fixed = ldexp(1.0, 50 - ex);
  if constexpr (!ERR)
    if (small) clear(acc_small);
  double own[kOwn], own_n = 0.0, err = 0.0;
#pragma unroll
  for (int k = 0; k < kOwn; ++k) own[k] = 0.0;
  __syncthreads();
  for (int64_t base = begin; base < end; base += kSumMost) {
    const int64_t stop = min(end, base + kSumMost);
    for (int64_t w0 = base + (tid & ~63); w0 < stop; w0 += NT) {  // 64 samples per wave
      const bool valid = w0 + (tid & 63) < stop;
      float x[SUB];
#pragma unroll
      for (int i = 0; i < SUB; ++i) x[i] = ahead[i / 4][i % 4];
      // the next 64 are on their way while these are searched (the last one of the block again where there are none)
      const int64_t next = w0 + NT < stop ? w0 + NT : base + kSumMost + (tid & ~63);
      fetch(next + (tid & 63));
      float y[SUB];
#pragma unroll
      for (int i = 0; i < SUB; ++i) y[i] = x[i] * R.scale;
      const int code = search_nearest<SUB, false, SUB == 8, false>(T, R, y, [&](int c) { return exact_dist<SUB>(cx[c], x); });
      if constexpr (ERR) {
        if (valid) err += exact_dist<SUB>(cx[code], x);
      } else if (valid) {
        if (small) {
          uint32_t lowest = 0xffffffffu;
#pragma unroll
          for (int i = 0; i < SUB; ++i) lowest = min(lowest, __float_as_uint(x[i]) << 1);
          if (lowest < small) {
#pragma unroll
            for (int i = 0; i < SUB; ++i) {
              if ((__float_as_uint(x[i]) << 1) < small) {
                atomicAdd(&acc_small[i][code], (unsigned long long)(long long)((double)x[i] * (fixed * 0x1p27)));
                x[i] = 0.f;
              }
            }
          }
        }
#pragma unroll
        for (int i = 0; i < SUB; ++i)
          atomicAdd(&acc[i][code], (unsigned long long)__double_as_longlong(fma((double)x[i], fixed, kMagic)));
        atomicAdd(&cnt[code], 1u);
      }
    }
    if constexpr (!ERR) {
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kOwn; ++k) {  // dimension e % SUB of cluster e / SUB
        const int e = min(tid + k * NT, kCodes * SUB - 1);
        const unsigned long long s =
            acc[e % SUB][e / SUB] - (unsigned long long)cnt[e / SUB] * (unsigned long long)__double_as_longlong(kMagic);
        double t = (double)(long long)s;
        if (small) t += (double)(long long)acc_small[e % SUB][e / SUB] * 0x1p-27;
        own[k] += t;
      }
      if (tid < kCodes) own_n += (double)cnt[tid];
      if (base + kSumMost < end) {
        __syncthreads();
        clear(acc);
        if (small) clear(acc_small);
        if (tid < kCodes) cnt[tid] = 0u;
        __syncthreads();
      }
    }
  }
  if constexpr (ERR) {
    err = xor_sum(err, 64);
    if ((tid & 63) == 0) red[tid >> 6] = err;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int w = 0; w < NT / 64; ++w) t += red[w];
      ws.block_err[blockIdx.x] = t;
    }
  } else {
    const double unit = 1.0 / fixed;  // a power of two
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const int e = tid + k * NT;
      if (e < kCodes * SUB) ws.sums[(int64_t)blockIdx.x * kCodes * SUB + e] = own[k] * unit;
    }
    if (tid < kCodes) ws.counts[(int64_t)blockIdx.x * kCodes + tid] = own_n;
  }
}

// Assignment and sums over every codeword's samples in fp64 and in ONE order.  UNIT (fine-tuning): sums of x / |x| (zero
// samples add nothing).  Otherwise (K-Means of samples that fixed-point sums do not fit): sums of x and member counts.
// Fine-tuning needs the order: the steps are large (a rate of 2048 turns a small codeword by several times its error), so a
// difference in the last place of a sum grows to a different codebook within twenty of them, and the order is part of
// the result.  Runs of 16 samples are dealt out to 1024 chains, every chain adds the members of a codeword by
// ascending index, chains are added in pairs up to 64 and the sixteen results one after the other.
// A workgroup owns four neighbouring chains, i.e. 64 samples out of every 16384.  It searches 4096 of them at a time
// and leaves (chain, codeword) lists of positions in LDS, in whatever order the lanes arrive; then a thread per
// (chain, codeword) sorts its list (four entries on average) in registers and adds its samples.  A list that
// overflows is rebuilt from the codes.  (One workgroup per codeword looking through all codes: 0.9 ms per step of 2^20
// samples.)
constexpr int kChains = 1024, kRun = 16;
constexpr int kWgChains = kChains / kSumBlocks;             // 4
constexpr int kBlockPos = kSumMost / kWgChains;             // positions of a chain per block: 1024
constexpr int kPairs = kWgChains * kCodes, kListMost = 32;  // lists per workgroup, entries per list

// the first N of e in ascending order: odd-even merge sort, all indices known to the compiler
template <int N, int M>
__device__ __forceinline__ void sort_ascending(uint32_t (&e)[M]) {
#pragma unroll
  for (int a = 1; a < N; a *= 2)
#pragma unroll
    for (int k = a; k >= 1; k /= 2)
#pragma unroll
      for (int j = k % a; j + k < N; j += 2 * k)
#pragma unroll
        for (int i = 0; i < k; ++i)
          if (i + j + k < N && (i + j) / (2 * a) == (i + j + k) / (2 * a)) {
            const uint32_t lo = min(e[i + j], e[i + j + k]), hi = max(e[i + j], e[i + j + k]);
            e[i + j] = lo, e[i + j + k] = hi;
          }
}

template <int SUB, bool UNIT>
__global__ __launch_bounds__(kSumThreads<SUB>) void cb_ordered_kernel(const float* __restrict__ samples, int64_t n,
                                                                      CodebookWs<SUB> ws) {
  constexpr int NT = kSumThreads<SUB>, NWV = NT / 64, CPW = (kPairs / 64 + NWV - 1) / NWV;
  __shared__ SearchTables<SUB, false> T;
  __shared__ double cx[kCodes][SUB];
  __shared__ __attribute__((aligned(16))) uint16_t list[kPairs][kListMost];
  __shared__ uint32_t len[kPairs];
  __shared__ __attribute__((aligned(16))) uint16_t codes[kWgChains][kBlockPos];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  SearchRegs<SUB, false> R;
  {
    double centroid[SUB] = {};  // of codeword `tid`
    if (tid < kCodes) {
#pragma unroll
      for (int i = 0; i < SUB; ++i) centroid[i] = ws.centroids[tid * SUB + i];
#pragma unroll
      for (int i = 0; i < SUB; ++i) cx[tid][i] = centroid[i];
    }
    search_setup<SUB, false, false>(T, R, tid, [&](int i) { return centroid[i]; });
  }
  const int64_t n16 = n & ~(int64_t)(kRun - 1);
  double acc[CPW][SUB];
  uint32_t members[UNIT ? 1 : CPW] = {};
#pragma unroll
  for (int c = 0; c < CPW; ++c)
#pragma unroll
    for (int i = 0; i < SUB; ++i) acc[c][i] = 0.0;
  auto load = [&](int64_t idx, float (&x)[SUB]) {
    const row4* row = reinterpret_cast<const row4*>(samples) + idx * (SUB / 4);
#pragma unroll
    for (int q = 0; q < SUB / 4; ++q) {
      const row4 v = row[q];
      x[4 * q] = v.x, x[4 * q + 1] = v.y, x[4 * q + 2] = v.z, x[4 * q + 3] = v.w;
    }
  };
  auto add = [&](const float (&x)[SUB], double (&a)[SUB]) {
    if constexpr (!UNIT) {
#pragma unroll
      for (int i = 0; i < SUB; ++i) a[i] += (double)x[i];
      return;
    }
    double v[SUB], n2 = 0.0;
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      v[i] = (double)x[i];
      n2 += v[i] * v[i];
    }
    if (n2 > 0.0) {
      // v / nx with one reciprocal for all elements: two Newton steps for it, then the quotient corrected by its exact
      // remainder (Markstein's method), which rounds correctly
      const double nx = sqrt(n2);
      double r = __builtin_amdgcn_rcp(nx);
      r = fma(fma(-nx, r, 1.0), r, r);
      r = fma(fma(-nx, r, 1.0), r, r);
#pragma unroll
      for (int i = 0; i < SUB; ++i) {
        const double q = v[i] * r;
        a[i] += fma(fma(-q, nx, v[i]), r, q);
      }
    }
  };
  auto search = [&](const float (&x)[SUB]) {
    float y[SUB];
#pragma unroll
    for (int i = 0; i < SUB; ++i) y[i] = x[i] * R.scale;
    return search_nearest<SUB, false, false, false>(T, R, y, [&](int c) { return exact_dist<SUB>(cx[c], x); });
  };
  const int64_t blocks = (n16 + (int64_t)kSumMost * kSumBlocks - 1) / ((int64_t)kSumMost * kSumBlocks);
  for (int64_t blk = 0; blk < blocks; ++blk) {
    // sample of position p of chain `ch` (of the workgroup's four) in this block
    auto sample_of = [&](int ch, int p) -> int64_t {
      const int chain = blockIdx.x * kWgChains + ch;
      return ((blk * (kBlockPos / kRun) + (p >> 4)) * kChains + chain) * kRun + (p & 15);
    };
    for (int i = tid; i < kPairs; i += NT) len[i] = 0u;
    __syncthreads();
    for (int u = wave; u < kBlockPos / kRun; u += NWV) {
      const int ch = lane >> 4, p = u * kRun + (lane & 15);
      const int64_t idx = sample_of(ch, p);
      const bool valid = idx < n16;
      if (!__any(valid)) break;
      float x[SUB];
      load(min(idx, n - 1), x);
      const int code = search(x);
      if (valid) {
        const uint32_t at = atomicAdd(&len[code * kWgChains + ch], 1u);
        if (at < kListMost) list[code * kWgChains + ch][at] = (uint16_t)p;
      }
      codes[ch][p] = valid ? (uint16_t)code : (uint16_t)0xffff;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      const int pair = (wave + c * NWV) * 64 + lane;  // codeword pair / 4, chain pair % 4
      if (pair >= kPairs) break;  // (whole waves)
      const uint32_t count = len[pair];
      if constexpr (!UNIT) members[c] += count;
      if (count > kListMost) {
        for (int p0 = 0; p0 < kBlockPos; p0 += 8) {
          const uint4 w4 = *reinterpret_cast<const uint4*>(&codes[pair & 3][p0]);
          const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const uint32_t code = (k & 1) ? w[k / 2] >> 16 : w[k / 2] & 0xffffu;
            if (code == (uint32_t)(pair >> 2) && sample_of(pair & 3, p0 + k) < n16) {
              float x[SUB];
              load(sample_of(pair & 3, p0 + k), x);
              add(x, acc[c]);
            }
          }
        }
      }
      const uint32_t here = count > kListMost ? 0u : count;
      uint32_t e[kListMost];
#pragma unroll
      for (int q = 0; q < kListMost / 8; ++q) {
        const uint4 w4 = reinterpret_cast<const uint4*>(list[pair])[q];
        const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t v = (k & 1) ? w[k / 2] >> 16 : w[k / 2] & 0xffffu;
          e[8 * q + k] = 8 * q + k < (int)here ? v : 0xffffu;
        }
      }
      if (__any(here > kListMost / 2))
        sort_ascending<kListMost>(e);
      else
        sort_ascending<kListMost / 2>(e);
      // (back to LDS: a loop over registers would be unrolled to a body of its own per entry)
#pragma unroll
      for (int q = 0; q < kListMost / 8; ++q)
        reinterpret_cast<uint4*>(list[pair])[q] =
            make_uint4(e[8 * q] | e[8 * q + 1] << 16, e[8 * q + 2] | e[8 * q + 3] << 16, e[8 * q + 4] | e[8 * q + 5] << 16,
                       e[8 * q + 6] | e[8 * q + 7] << 16);
      // (four samples are asked for at a time: a trip to memory takes as long as six additions.  One ahead: 49.4
      // instead of 44.4 us per step of 2^20 8-dim samples)
      for (uint32_t k = 0; __any(k < here); k += 4) {
        float x[4][SUB];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {  // (position 0 of the block exists for every chain that has entries)
          const int64_t idx = sample_of(pair & 3, k + u < here ? list[pair][k + u] : 0);
          load(min(idx, n - 1), x[u]);
        }
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
          if (k + u < here) add(x[u], acc[c]);
      }
    }
    __syncthreads();
  }
  // the samples behind the last whole run: one for each of the first chains, the last of its order.  (As a block of their
  // own, with lists, they took 3 us a step.)
  if (n > n16 && blockIdx.x < kRun / kWgChains) {
    const int64_t tail0 = n16 + blockIdx.x * kWgChains;
    if (wave == 0) {
      float x[SUB];
      load(min(tail0 + (lane & 3), n - 1), x);
      const int code = search(x);
      if (lane < kWgChains) codes[lane][0] = tail0 + lane < n ? (uint16_t)code : (uint16_t)0xffff;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      const int pair = (wave + c * NWV) * 64 + lane;
      if (pair < kPairs && codes[pair & 3][0] == (uint32_t)(pair >> 2)) {
        float x[SUB];
        load(tail0 + (pair & 3), x);
        add(x, acc[c]);
        if constexpr (!UNIT) members[c] += 1u;
      }
    }
  }
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    const int pair = (wave + c * NWV) * 64 + lane;
    if (pair >= kPairs) break;
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      acc[c][i] += xor_lane<1>(acc[c][i]);
      acc[c][i] += xor_lane<2>(acc[c][i]);
      if ((lane & 3) == 0) ws.sums[((int64_t)blockIdx.x * kCodes + pair / kWgChains) * SUB + i] = acc[c][i];
    }
    if constexpr (!UNIT) {
      double m = (double)members[c];
      m += xor_lane<1>(m);
      m += xor_lane<2>(m);
      if ((lane & 3) == 0) ws.counts[(int64_t)blockIdx.x * kCodes + pair / kWgChains] = m;
    }
  }
}

// Adds the partial sums of kUpdateClusters<SUB> neighbouring clusters (128 consecutive bytes of every row of partials: one line)
// in a fixed order (fp64): kUpdateThreads = E sums x kUpdateThreads / E slices of the rows; for the counts, clusters x
// kUpdateThreads / clusters.  The first threads return with the sums and the member count of their cluster.  (Eight clusters per
// workgroup, i.e. 32 compute units at work: 5.3 us instead of 4.7; pieces of 32 bytes 10.7 us.)
template <int SUB>
constexpr int kUpdateClusters = 16 / SUB;
constexpr int kUpdateThreads = 128;
template <int SUB>
__device__ __forceinline__ void merge_partials(const CodebookWs<SUB>& ws, double (&sum)[SUB], double& count) {
  constexpr int UC = kUpdateClusters<SUB>, E = UC * SUB, SL = kUpdateThreads / E, PER = kSumBlocks / SL;
  constexpr int CSL = kUpdateThreads / UC, CPER = kSumBlocks / CSL;
  static_assert(PER * SL == kSumBlocks && CPER * CSL == kSumBlocks, "whole slices");
  __shared__ double part[SL][E], cpart[kUpdateThreads / 64][UC];
  const int e = threadIdx.x % E, sl = threadIdx.x / E;
  const int c = threadIdx.x % UC, cs = threadIdx.x / UC;
  double v[PER], n[CPER], t = 0.0, m = 0.0;
#pragma unroll
  for (int u = 0; u < PER; ++u) v[u] = ws.sums[((int64_t)(sl * PER + u) * kCodes + blockIdx.x * UC) * SUB + e];
#pragma unroll
  for (int u = 0; u < CPER; ++u) n[u] = ws.counts[(int64_t)(cs * CPER + u) * kCodes + blockIdx.x * UC + c];
#pragma unroll
  for (int u = 0; u < PER; ++u) t += v[u];
#pragma unroll
  for (int u = 0; u < CPER; ++u) m += n[u];
  part[sl][e] = t;
  if constexpr (UC < 4) m += xor_lane<2>(m);
  m += xor_lane<4>(m);
  m += xor_lane<8>(m);
  m += xor_lane<16>(m);
  m += xor_lane<32>(m);
  if ((threadIdx.x & 63) < UC) cpart[threadIdx.x >> 6][threadIdx.x & 63] = m;
  __syncthreads();
  if (threadIdx.x < UC) {
    count = 0.0;
#pragma unroll
    for (int w = 0; w < kUpdateThreads / 64; ++w) count += cpart[w][threadIdx.x];
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      sum[i] = 0.0;
#pragma unroll
      for (int k = 0; k < SL; ++k) sum[i] += part[k][threadIdx.x * SUB + i];
    }
  }
}

// an empty cluster keeps its centroid
template <int SUB>
__global__ __launch_bounds__(kUpdateThreads) void km_update_kernel(CodebookWs<SUB> ws) {
  double sum[SUB], count;
  merge_partials<SUB>(ws, sum, count);
  if (threadIdx.x < kUpdateClusters<SUB> && count > 0.0) {
#pragma unroll
    for (int i = 0; i < SUB; ++i) ws.centroids[(blockIdx.x * kUpdateClusters<SUB> + threadIdx.x) * SUB + i] = sum[i] / count;
  }
}

// Fine-tuning for cosine distance (Sec. 3.4): S = sum of x / |x| over a codeword's samples (fp64), then the
// codeword moves along the part of that sum that is orthogonal to it:
// c += lr / (N |c|) * (S - (S . c^) c^).   cos_sum[k] = S . c^ is the cluster's share of the summed cosine
// similarity BEFORE the move.
template <int SUB>
__global__ __launch_bounds__(kUpdateThreads) void ft_update_kernel(int64_t n, CodebookWs<SUB> ws, double lr) {
  constexpr int UC = kUpdateClusters<SUB>, E = UC * SUB, SL = kUpdateThreads / E;
  constexpr int kTrees = kSumBlocks / 16;  // sixteen workgroups = 64 chains: added in pairs, then the trees in order
  __shared__ double tree[kTrees][E];
  for (int g = threadIdx.x / E; g < kTrees; g += SL) {
    const int e = threadIdx.x % E;
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = ws.sums[((int64_t)(16 * g + u) * kCodes + blockIdx.x * UC) * SUB + e];
#pragma unroll
    for (int d = 1; d < 16; d *= 2)
#pragma unroll
      for (int u = 0; u < 16; u += 2 * d) v[u] += v[u + d];
    tree[g][e] = v[0];
  }
  __syncthreads();
  if (threadIdx.x < UC) {
    const int k = blockIdx.x * UC + threadIdx.x;
    double S[SUB], c[SUB], cn2 = 0.0;
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      S[i] = 0.0;
#pragma unroll
      for (int g = 0; g < kTrees; ++g) S[i] += tree[g][threadIdx.x * SUB + i];
      c[i] = ws.centroids[k * SUB + i];
      cn2 += c[i] * c[i];
    }
    double along = 0.0;
    if (cn2 > 0.0) {
      const double cn = sqrt(cn2);
#pragma unroll
      for (int i = 0; i < SUB; ++i) along += S[i] * (c[i] / cn);
#pragma unroll
      for (int i = 0; i < SUB; ++i)
        ws.centroids[k * SUB + i] = c[i] + lr * ((S[i] - along * (c[i] / cn)) / ((double)n * cn));
    }
    ws.cos_sum[k] = along;
  }
}

size_t codebook_workspace_bytes(int sub_dim, int64_t) {
  return sub_dim == 8 ? CodebookWs<8>::bytes() : CodebookWs<4>::bytes();
}

// Every sample enters the fixed-point sums exactly from 2^-54 of the power of two above the largest on; sets with
// smaller ones (but zero), infinities or NaN are added in fp64 instead.
static bool sums_fit(uint32_t least_less_one, uint32_t most_bits) {
  const uint32_t least_bits = least_less_one + 1u;  // (0: there are zeros only)
  float largest, least;
  memcpy(&largest, &most_bits, sizeof(largest));
  memcpy(&least, &least_bits, sizeof(least));
  if (!std::isfinite(largest)) return false;
  int ex = 0;
  (void)std::frexp(largest, &ex);
  return least_bits == 0u || (double)least >= std::ldexp(1.0, ex - 54);
}

template <int SUB>
static int codebook_run_t(const float* samples, int64_t n, int iters, void* codebook_out, double* mse_host,
                          void* workspace, hipStream_t stream) {
  const CodebookWs<SUB> ws(workspace);
  constexpr int n_elems = kCodes * SUB;
  struct {
    double err[kSumBlocks];
    uint32_t least_bits, unused[2 * kCodes - 1], most_bits, unused2;
  } host;
  auto run = [&](bool fixed) -> int {
    cb_start_kernel<<<(n_elems + 255) / 256, 256, 0, stream>>>(samples, ws.centroids, n_elems, ws.least_bits,
                                                               ws.most_bits);
    cb_range_kernel<<<kRangeBlocks, kRangeThreads, 0, stream>>>(samples, n * (SUB / 4), ws.least_bits, ws.most_bits);
    for (int it = 0; it < iters; ++it) {
      if (fixed)
        cb_accumulate_kernel<SUB, false><<<kSumBlocks, kSumThreads<SUB>, 0, stream>>>(samples, n, ws);
      else
        cb_ordered_kernel<SUB, false><<<kSumBlocks, kSumThreads<SUB>, 0, stream>>>(samples, n, ws);
      km_update_kernel<SUB><<<kCodes / kUpdateClusters<SUB>, kUpdateThreads, 0, stream>>>(ws);
    }
    km_round_kernel<<<(n_elems + 255) / 256, 256, 0, stream>>>(ws.centroids, static_cast<__half*>(codebook_out), n_elems);
    cb_accumulate_kernel<SUB, true><<<kSumBlocks, kSumThreads<SUB>, 0, stream>>>(samples, n, ws);
    if (hipGetLastError() != hipSuccess) return NSN_ERR_HIP;
    // error sums and the range lie next to each other
    if (hipMemcpyAsync(&host, ws.block_err, sizeof(host), hipMemcpyDeviceToHost, stream) != hipSuccess) return NSN_ERR_HIP;
    return hipStreamSynchronize(stream) == hipSuccess ? NSN_OK : NSN_ERR_HIP;
  };
  // (the range comes back with the error sums, so that ordinary samples pay nothing for the question)
  int rc = run(true);
  if (rc == NSN_OK && iters > 0 && !sums_fit(host.least_bits, host.most_bits)) rc = run(false);
  if (rc != NSN_OK) return rc;
  if (mse_host) {
    double tot = 0.0;
    for (int i = 0; i < kSumBlocks; ++i) tot += host.err[i];
    *mse_host = tot / ((double)n * SUB);
  }
  return NSN_OK;
}

template <int SUB>
static int finetune_run_t(const float* samples, int64_t n, int iters, double lr, void* codebook_io, double* cos_host,
                          void* workspace, hipStream_t stream) {
  const CodebookWs<SUB> ws(workspace);
  constexpr int n_elems = kCodes * SUB;
  double host_cos[kCodes];
  auto step = [&](double rate) {
    cb_ordered_kernel<SUB, true><<<kSumBlocks, kSumThreads<SUB>, 0, stream>>>(samples, n, ws);
    ft_update_kernel<SUB><<<kCodes / kUpdateClusters<SUB>, kUpdateThreads, 0, stream>>>(n, ws, rate);
  };
  auto mean_cos = [&](double* out) -> int {  // assignment + cosine sums of the current centroids (no move: rate 0)
    step(0.0);
    if (hipGetLastError() != hipSuccess) return NSN_ERR_HIP;
    if (hipMemcpyAsync(host_cos, ws.cos_sum, sizeof(host_cos), hipMemcpyDeviceToHost, stream) != hipSuccess)
      return NSN_ERR_HIP;
    if (hipStreamSynchronize(stream) != hipSuccess) return NSN_ERR_HIP;
    double tot = 0.0;
    for (int k = 0; k < kCodes; ++k) tot += host_cos[k];
    *out = tot / (double)n;
    return NSN_OK;
  };
  cb_start_kernel<<<(n_elems + 255) / 256, 256, 0, stream>>>(static_cast<const __half*>(codebook_io), ws.centroids, n_elems,
                                                             ws.least_bits, ws.most_bits);
  int rc = NSN_OK;
  double before = 0.0, after = 0.0;
  if (cos_host && (rc = mean_cos(&before)) != NSN_OK) return rc;
  for (int it = 0; it < iters; ++it) step(lr);
  km_round_kernel<<<(n_elems + 255) / 256, 256, 0, stream>>>(ws.centroids, static_cast<__half*>(codebook_io), n_elems);
  if (hipGetLastError() != hipSuccess) return NSN_ERR_HIP;
  if (cos_host) {
    if ((rc = mean_cos(&after)) != NSN_OK) return rc;
    cos_host[0] = before;
    cos_host[1] = after;
  } else if (hipStreamSynchronize(stream) != hipSuccess) {
    return NSN_ERR_HIP;
  }
  return NSN_OK;
}

int finetune_run(const float* samples, int64_t n_samples, int sub_dim, int iters, double lr, void* codebook_io,
                 double* cos_host, void* workspace, hipStream_t stream) {
  return sub_dim == 8 ? finetune_run_t<8>(samples, n_samples, iters, lr, codebook_io, cos_host, workspace, stream)
                      : finetune_run_t<4>(samples, n_samples, iters, lr, codebook_io, cos_host, workspace, stream);
}

int codebook_run(const float* samples, int64_t n_samples, int sub_dim, int iters, void* codebook_out,
                 double* mse_host, void* workspace, hipStream_t stream) {
  return sub_dim == 8 ? codebook_run_t<8>(samples, n_samples, iters, codebook_out, mse_host, workspace, stream)
                      : codebook_run_t<4>(samples, n_samples, iters, codebook_out, mse_host, workspace, stream);
}

// Codebook entries on 16 levels (Sec. 3.5): one workgroup; thread c owns codeword c.
template <int SUB>
__global__ __launch_bounds__(256) void cb_quantize_kernel(__half* __restrict__ codebook, uint8_t* __restrict__ codes,
                                                          __half* __restrict__ levels) {
  __shared__ float red_lo[4], red_hi[4];
  const int c = threadIdx.x, lane = c & 63, wave = c >> 6;
  float x[SUB], lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int i = 0; i < SUB; ++i) {
    x[i] = __half2float(codebook[c * SUB + i]);
    lo = fminf(lo, x[i]);
    hi = fmaxf(hi, x[i]);
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    lo = fminf(lo, __shfl_xor(lo, m, 64));
    hi = fmaxf(hi, __shfl_xor(hi, m, 64));
  }
  if (lane == 0) red_lo[wave] = lo, red_hi[wave] = hi;
  __syncthreads();
  lo = fminf(fminf(red_lo[0], red_lo[1]), fminf(red_lo[2], red_lo[3]));
  hi = fmaxf(fmaxf(red_hi[0], red_hi[1]), fmaxf(red_hi[2], red_hi[3]));
  const __half mn16 = f64_to_f16((double)lo), st16 = f64_to_f16(((double)hi - (double)lo) / 15.0);
  const double mn = (double)__half2float(mn16), st = (double)__half2float(st16);
#pragma unroll
  for (int i = 0; i < SUB; ++i) {
    int code = 0;
    if (st != 0.0) code = (int)fmin(fmax(floor(((double)x[i] - mn) / st + 0.5), 0.0), 15.0);
    codebook[c * SUB + i] = f64_to_f16(mn + st * (double)code);
    if (codes) codes[c * SUB + i] = (uint8_t)code;
  }
  if (levels && c == 0) levels[0] = mn16, levels[1] = st16;
}

int codebook_quantize(void* codebook_io, int sub_dim, uint8_t* codes_out, void* levels_out, hipStream_t stream) {
  if (sub_dim == 4)
    cb_quantize_kernel<4><<<1, 256, 0, stream>>>(static_cast<__half*>(codebook_io), codes_out, static_cast<__half*>(levels_out));
  else
    cb_quantize_kernel<8><<<1, 256, 0, stream>>>(static_cast<__half*>(codebook_io), codes_out, static_cast<__half*>(levels_out));
  return hipGetLastError() == hipSuccess ? NSN_OK : NSN_ERR_HIP;
}

}  // namespace nsn
