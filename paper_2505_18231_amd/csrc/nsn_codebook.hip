// K-Means codebook on standard-normal samples (Sec. 3.4, the K-Means baseline) and its
// fine-tuning for cosine distance.
//
// Lloyd iterations entirely on the device, deterministic, two launches each:
//   cb_accumulate_kernel  nearest centroid per sample (nsn_search.h) and, in the same pass over the samples, the sums of
//                         every cluster's members: one partial per workgroup
//   km_update_kernel /    adds the partials in a fixed order (fp64) and moves the centroids
//   ft_update_kernel
#include "nsn_host.h"
#include "nsn_search.h"

namespace nsn {

constexpr int kSumBlocks = 256;   // workgroups of the accumulation (and partial sums per cluster)
constexpr int kSumThreads = 512;
constexpr int kUpdateClusters = 8;  // clusters per workgroup of the update

// workspace: centroids, error sum of every workgroup, cosine sum of every cluster, largest |sample| (bits), then
// per workgroup of the accumulation 256 x SUB member sums and 256 member counts
template <int SUB>
struct CodebookWs {
  double* centroids;
  double* block_err;
  double* cos_sum;
  uint32_t* max_bits;
  double* sums;
  double* counts;
  explicit CodebookWs(void* ws)
      : centroids(static_cast<double*>(ws)),
        block_err(centroids + kCodes * SUB),
        cos_sum(block_err + kSumBlocks),
        max_bits(reinterpret_cast<uint32_t*>(cos_sum + kCodes)),
        sums(cos_sum + kCodes + 2),
        counts(sums + (size_t)kSumBlocks * kCodes * SUB) {}
  static size_t bytes() {
    return (size_t)(kCodes * SUB + kSumBlocks + kCodes + 2 + kSumBlocks * kCodes * (SUB + 1)) * sizeof(double);
  }
};

// start of a run: the centroids (the first samples, or the codebook at hand), no largest sample yet
template <typename T>
__global__ void cb_start_kernel(const T* __restrict__ from, double* __restrict__ centroids, int n_elems,
                                uint32_t* __restrict__ max_bits) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_elems) centroids[i] = (double)(float)from[i];
  if (i == 0) *max_bits = 0u;
}

// largest |sample| of the set, as fp32 bits (their order is that of the values)
__global__ __launch_bounds__(256) void cb_max_kernel(const float* __restrict__ samples, int64_t n_elems,
                                                     uint32_t* __restrict__ max_bits) {
  float m = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_elems; i += (int64_t)gridDim.x * 256)
    m = fmaxf(m, fabsf(samples[i]));
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) atomicMax(max_bits, __float_as_uint(m));
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

// Assignment and member sums in one pass over the samples.  WHAT: kSums adds the samples, kUnitSums adds x / |x|
// (zero samples add nothing), kError adds no members but the squared error.
//
// The sums are formed in LDS by integer atomics on fixed-point values: integer addition is associative, so the result
// does not depend on the order in which lanes and waves arrive.  A value enters with its last place at 2^-50 of the
// power of two above the largest |sample| and at most 4096 values are added before the LDS sums move to fp64
// registers: no overflow of 63 bits, and a rounding error per value that is below that of the fp64 running sum
// it stands for.  Adding 1.5 * 2^52 puts the fixed-point value into the low bits of the fp64 pattern;
// the patterns are added as they are and the member count times the constant's pattern comes off at the end.
// (The form this replaces wrote the assignments out and let one workgroup per cluster look through all of them:
// 270 us per iteration of 2^20 4-dim samples, 1.05 ms with x / |x|.)
enum { kSums, kUnitSums, kError };
template <int SUB, int WHAT>
__global__ __launch_bounds__(kSumThreads, 2) void cb_accumulate_kernel(const float* __restrict__ samples, int64_t n,
                                                                       CodebookWs<SUB> ws) {
  constexpr int kOwn = kCodes * SUB / kSumThreads;  // sums a thread carries in registers
  constexpr double kMagic = 6755399441055744.0;      // 1.5 * 2^52
  __shared__ SearchTables<SUB> T;
  __shared__ double cx[kCodes][SUB];
  __shared__ unsigned long long acc[WHAT == kError ? 1 : SUB][kCodes];
  __shared__ uint32_t cnt[kCodes];
  __shared__ double red[kSumThreads / 64];
  const int tid = threadIdx.x;
  SearchRegs<SUB, false> R;
  search_setup<SUB, false>(T, R, tid, [&](int c, int i) { return ws.centroids[c * SUB + i]; });
  for (int i = tid; i < kCodes * SUB; i += kSumThreads) (&cx[0][0])[i] = ws.centroids[i];
  double fixed = 0x1p50;  // values below 1
  if constexpr (WHAT == kSums) {
    int ex = 0;
    const float mx = __uint_as_float(*ws.max_bits);
    if (mx > 0.f && mx < INFINITY) (void)frexpf(mx, &ex);  // mx < 2^ex
    fixed = ldexp(1.0, 50 - ex);
  }
  auto clear = [&]() {
    if constexpr (WHAT != kError) {
      for (int i = tid; i < kCodes * SUB; i += kSumThreads) (&acc[0][0])[i] = 0ull;
      if (tid < kCodes) cnt[tid] = 0u;
    }
  };
  clear();
  double own[kOwn], own_n = 0.0, err = 0.0;
#pragma unroll
  for (int k = 0; k < kOwn; ++k) own[k] = 0.0;
  __syncthreads();
  const int64_t per = ((n + kSumBlocks - 1) / kSumBlocks + kSumThreads - 1) / kSumThreads * kSumThreads;
  const int64_t begin = (int64_t)blockIdx.x * per, end = min(n, begin + per);
  for (int64_t base = begin; base < end; base += 8 * kSumThreads) {
#pragma unroll 1
    for (int u = 0; u < 8; ++u) {
      const int64_t idx = base + u * kSumThreads + tid;
      if (base + u * kSumThreads >= end) break;  // uniform
      const bool valid = idx < end;
      float x[SUB];
      typedef float row4 __attribute__((ext_vector_type(4), aligned(4)));  // (the samples are aligned as floats are)
      const row4* row = reinterpret_cast<const row4*>(samples) + (valid ? idx : end - 1) * (SUB / 4);
#pragma unroll
      for (int q = 0; q < SUB / 4; ++q) {
        const row4 v = row[q];
        x[4 * q] = v.x, x[4 * q + 1] = v.y, x[4 * q + 2] = v.z, x[4 * q + 3] = v.w;
      }
      const int code = search_nearest<SUB, false>(T, R, x, [&](int c) { return exact_dist<SUB>(cx[c], x); });
      if constexpr (WHAT == kError) {
        if (valid) err += exact_dist<SUB>(cx[code], x);
      } else if (valid) {
        double v[SUB], n2 = 0.0;
#pragma unroll
        for (int i = 0; i < SUB; ++i) v[i] = (double)x[i];
        if constexpr (WHAT == kUnitSums) {
#pragma unroll
          for (int i = 0; i < SUB; ++i) n2 += v[i] * v[i];
          const double nx = sqrt(n2);
#pragma unroll
          for (int i = 0; i < SUB; ++i) v[i] = n2 > 0.0 ? v[i] / nx : 0.0;
        }
#pragma unroll
        for (int i = 0; i < SUB; ++i)
          atomicAdd(&acc[i][code], (unsigned long long)__double_as_longlong(fma(v[i], fixed, kMagic)));
        atomicAdd(&cnt[code], 1u);
      }
    }
    if constexpr (WHAT != kError) {
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kOwn; ++k) {
        const int e = tid + k * kSumThreads;
        const unsigned long long s =
            (&acc[0][0])[e] - (unsigned long long)cnt[e % kCodes] * (unsigned long long)__double_as_longlong(kMagic);
        own[k] += (double)(long long)s;
      }
      if (tid < kCodes) own_n += (double)cnt[tid];
      __syncthreads();
      clear();
      __syncthreads();
    }
  }
  if constexpr (WHAT == kError) {
    err = xor_sum(err, 64);
    if ((tid & 63) == 0) red[tid >> 6] = err;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int w = 0; w < kSumThreads / 64; ++w) t += red[w];
      ws.block_err[blockIdx.x] = t;
    }
  } else {
    double* out = ws.sums + (int64_t)blockIdx.x * kCodes * SUB;
    const double unit = 1.0 / fixed;  // a power of two
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const int e = tid + k * kSumThreads;  // dimension e / 256 of cluster e % 256
      out[(e % kCodes) * SUB + e / kCodes] = own[k] * unit;
    }
    if (tid < kCodes) ws.counts[(int64_t)blockIdx.x * kCodes + tid] = own_n;
  }
}

// Adds the partial sums of kUpdateClusters clusters: 1024 threads = 8 SUB sums x 1024 / (8 SUB) slices of the
// workgroups, slices added in order.  Thread e < 8 SUB returns the sum of dimension e % SUB of cluster e / SUB of
// the block's eight; cnt_s holds the eight member counts (a barrier has passed).
constexpr int kUpdateThreads = 1024;
template <int SUB>
__device__ __forceinline__ double merge_partials(const CodebookWs<SUB>& ws, double (&sum_s)[kUpdateThreads],
                                                 double (&cnt_s)[kUpdateClusters]) {
  constexpr int E = kUpdateClusters * SUB, SL = kUpdateThreads / E, PER = kSumBlocks / SL;
  const int e = threadIdx.x % E, sl = threadIdx.x / E;
  double v[PER], t = 0.0;
#pragma unroll
  for (int u = 0; u < PER; ++u) v[u] = ws.sums[((int64_t)(sl * PER + u) * kCodes + blockIdx.x * kUpdateClusters) * SUB + e];
#pragma unroll
  for (int u = 0; u < PER; ++u) t += v[u];
  sum_s[threadIdx.x] = t;
  // counts: whole numbers, any order of addition gives the same
  {
    const int c = threadIdx.x % kUpdateClusters, s2 = threadIdx.x / kUpdateClusters;
    double m = 0.0;
    for (int w = s2; w < kSumBlocks; w += kUpdateThreads / kUpdateClusters)
      m += ws.counts[(int64_t)w * kCodes + blockIdx.x * kUpdateClusters + c];
    m += __shfl_xor(m, 8, 64), m += __shfl_xor(m, 16, 64), m += __shfl_xor(m, 32, 64);
    __shared__ double cw[kUpdateThreads / 64][kUpdateClusters];
    if ((threadIdx.x & 63) < kUpdateClusters) cw[threadIdx.x >> 6][c] = m;
    __syncthreads();
    if (threadIdx.x < kUpdateClusters) {
      double tot = 0.0;
      for (int w = 0; w < kUpdateThreads / 64; ++w) tot += cw[w][threadIdx.x];
      cnt_s[threadIdx.x] = tot;
    }
  }
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x < E)
    for (int k = 0; k < SL; ++k) s += sum_s[k * E + threadIdx.x];
  return s;
}

// an empty cluster keeps its centroid
template <int SUB>
__global__ __launch_bounds__(kUpdateThreads) void km_update_kernel(CodebookWs<SUB> ws) {
  __shared__ double sum_s[kUpdateThreads], cnt_s[kUpdateClusters];
  const double s = merge_partials<SUB>(ws, sum_s, cnt_s);
  const int e = threadIdx.x;
  if (e < kUpdateClusters * SUB && cnt_s[e / SUB] > 0.0)
    ws.centroids[blockIdx.x * kUpdateClusters * SUB + e] = s / cnt_s[e / SUB];
}

// Fine-tuning for cosine distance (Sec. 3.4): S = sum of x / |x| over a codeword's samples (fp64), then the
// codeword moves along the part of that sum that is orthogonal to it:
// c += lr / (N |c|) * (S - (S . c^) c^).   cos_sum[k] = S . c^ is the cluster's share of the summed cosine
// similarity BEFORE the move.
template <int SUB>
__global__ __launch_bounds__(kUpdateThreads) void ft_update_kernel(int64_t n, CodebookWs<SUB> ws, double lr) {
  __shared__ double sum_s[kUpdateThreads], cnt_s[kUpdateClusters];
  const double mine = merge_partials<SUB>(ws, sum_s, cnt_s);
  __syncthreads();
  if (threadIdx.x < kUpdateClusters * SUB) sum_s[threadIdx.x] = mine;
  __syncthreads();
  if (threadIdx.x < kUpdateClusters) {
    const int k = blockIdx.x * kUpdateClusters + threadIdx.x;
    double S[SUB], c[SUB], cn2 = 0.0;
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      S[i] = sum_s[threadIdx.x * SUB + i];
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

template <int SUB>
static int codebook_run_t(const float* samples, int64_t n, int iters, void* codebook_out, double* mse_host,
                          void* workspace, hipStream_t stream) {
  const CodebookWs<SUB> ws(workspace);
  constexpr int n_elems = kCodes * SUB;
  cb_start_kernel<<<(n_elems + 255) / 256, 256, 0, stream>>>(samples, ws.centroids, n_elems, ws.max_bits);
  cb_max_kernel<<<1024, 256, 0, stream>>>(samples, n * SUB, ws.max_bits);
  for (int it = 0; it < iters; ++it) {
    cb_accumulate_kernel<SUB, kSums><<<kSumBlocks, kSumThreads, 0, stream>>>(samples, n, ws);
    km_update_kernel<SUB><<<kCodes / kUpdateClusters, kUpdateThreads, 0, stream>>>(ws);
  }
  km_round_kernel<<<(n_elems + 255) / 256, 256, 0, stream>>>(ws.centroids, static_cast<__half*>(codebook_out), n_elems);
  cb_accumulate_kernel<SUB, kError><<<kSumBlocks, kSumThreads, 0, stream>>>(samples, n, ws);
  if (hipGetLastError() != hipSuccess) return NSN_ERR_HIP;
  double host_err[kSumBlocks];
  if (hipMemcpyAsync(host_err, ws.block_err, sizeof(host_err), hipMemcpyDeviceToHost, stream) != hipSuccess)
    return NSN_ERR_HIP;
  if (hipStreamSynchronize(stream) != hipSuccess) return NSN_ERR_HIP;
  if (mse_host) {
    double tot = 0.0;
    for (int i = 0; i < kSumBlocks; ++i) tot += host_err[i];
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
    cb_accumulate_kernel<SUB, kUnitSums><<<kSumBlocks, kSumThreads, 0, stream>>>(samples, n, ws);
    ft_update_kernel<SUB><<<kCodes / kUpdateClusters, kUpdateThreads, 0, stream>>>(n, ws, rate);
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
                                                             ws.max_bits);
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
