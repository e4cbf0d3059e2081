// KV encoder kernels: Normalize - Shift - Normalize (Sec. 3.2), Hadamard rotation (Sec. 2),
// nearest-codeword search (Eq. 1), scale adjustment (Sec. 3.3).
//
// enc_kernel does all of it for a call whose Shift means are known before a token is quantised: append mode (stored means)
// and groups of 64 tokens (a workgroup holds a whole group).  Otherwise two launches form the means first:
//   enc_stats_kernel  per chunk: fp64 partial sums of x / b, b = fp16(||x|| / sqrt(d))
//   enc_means_kernel  per group: o = fp16(sum of partials / count)
// Double quantization (Sec. 3.5, side_bits = 4): the means are stored as 4-bit codes per 32 channels and subtracted in
// their dequantised form, s1 becomes 4-bit codes per 64-token block, and a' = fp16(s2 * alpha) is stored.
// Normalisation, rotation and the dot products that feed fp16 roundings run in fp64 (same rate as fp32 on this chip's
// vector units); the codeword search decides as an fp64 search would (nsn_search.h).
// NSN_VARIANT_ALT (a cross-check) runs the stages as separate kernels with an fp32 scan of all 256 distances.
#include "nsn_host.h"
#include <type_traits>

#include "nsn_search.h"
#include "nsn_vq.h"

namespace nsn {

// f(integral_constant<int, m>) for m = 1, 2, 4, ... < N
template <int N, int M = 1, typename F>
__device__ __forceinline__ void static_for_pow2(F&& f) {
  if constexpr (M < N) {
    f(std::integral_constant<int, M>{});
    static_for_pow2<N, M * 2>(f);
  }
}

// Square root and reciprocals from the hardware estimates (about 2^-26) and Newton steps, within an fp64 unit or two.  The
// arguments are sums of squares of moderate numbers or fp16 values: zero or far inside the fp64 range.
__device__ __forceinline__ double sqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g), h = fma(h, r, h);
  return x == 0.0 ? 0.0 : fma(fma(-g, g, x), h, g);
}
__device__ __forceinline__ double rcp_f64(double x) {  // 0 for 0
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return x == 0.0 ? 0.0 : r;
}
__device__ __forceinline__ double rsqrt_f64(double x) {  // 0 for 0
  double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  y = fma(y * e, fma(0.375, e, 0.5), y);
  return x == 0.0 ? 0.0 : y;
}

// the value of lane I of the caller's four lanes
template <int I>
__device__ __forceinline__ double quad_lane(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)dpp_mov_i32<I * 0x55, 0xf>((int)(u & 0xffffffffll));
  const unsigned hi = (unsigned)dpp_mov_i32<I * 0x55, 0xf>((int)(u >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)lo);
}

// ---------------------------------------------------------------------------------------
// Stage A: first Normalize scale per token, partial channel sums of the normalised tokens.
// grid (chunk, kv_head * 2 + tensor, sequence), block 256 = 4 waves; a wave takes four tokens at a
// time (sixteen lanes per token, a lane owns eight consecutive channels: one 16-byte load).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void enc_stats_kernel(Geometry g, const __half* __restrict__ k_in,
                                                        const __half* __restrict__ v_in, int max_new,
                                                        int max_len, const int32_t* __restrict__ seq_start,
                                                        const int32_t* __restrict__ n_new, CacheView kc,
                                                        CacheView vc, double* __restrict__ partial,
                                                        int chunk_tokens, int n_chunks, __half* __restrict__ ws_b,
                                                        int write_b) {
  const int chunk = blockIdx.x, h = blockIdx.y >> 1, tensor = blockIdx.y & 1, b = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane >> 4, col = lane & 15;  // token of the wave's four, channels [8 col, 8 col + 8)
  const CacheView& cv = tensor ? vc : kc;
  const __half* in = (tensor ? v_in : k_in) + ((int64_t)(b * g.n_kv_heads + h) * max_new) * kHeadDim;
  __half* wsb = ws_b + ((int64_t)(b * g.n_kv_heads + h) * 2 + tensor) * max_new;  // side_bits = 4 only
  const int start = seq_start[b];
  const int count = min(min(n_new[b], max_new), max_len - start);  // tokens that have a place in the cache
  const int t_end = min((chunk + 1) * chunk_tokens, count);

  double acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.0;
  // four steps of loads in flight; a token past the end is read from the last valid row (the chunk has at
  // least one: t_end > chunk start, or the loop below does not run) and its weight is set to zero
  auto fetch = [&](int t) -> uint4 {
    return *reinterpret_cast<const uint4*>(in + (int64_t)min(t, max(t_end - 1, 0)) * kHeadDim + 8 * col);
  };
  // where fp16(s1) of token t goes: one address that is linear in t, except for paged caches
  const bool linear = g.dq || !g.paged;  // uniform
  __half* const b_out = g.dq ? wsb
                             : reinterpret_cast<__half*>(cv.norms) +
                                   2 * ((int64_t)(b * g.n_kv_heads + h) * g.page_tokens + start) + 1;
  const int b_stride = g.dq ? 1 : 2;
  // Four steps to a round, their buffers refilled in place.  Bound by vector instructions (a plain read of the inputs takes
  // three quarters of the time), so what is done per token - square root, rounding, reciprocal - is done once for a
  // round's sixteen tokens and not once for every four: the sums over a token's sixteen lanes go apart as they are formed (five
  // additions in the order that sixteen had), lane `col` finishes step col & 3 and hands the reciprocal to the
  // other lanes.  8 x 8192 tokens x 8 heads: the whole call 553 -> 544 us with 4-dim codes, 443 -> 434 with 8-dim ones; 300
  // tokens 16.8 -> 14.7 us.  A wave's only step is a round of its own (four cost a call of 16 tokens 0.2 us).  Two or three are not:
  // their chains overlap in a round of four, and with it and the shorter search 17, 32 and 48 tokens of 8 sequences take 11.3, 11.7
  // and 13.5 us where step by step they took 12.7, 13.1 and 17.3.
  const int tw = chunk * chunk_tokens + 4 * wave;  // the wave's first token of a step (uniform)
  uint4 buf[4] = {fetch(tw + row), fetch(tw + row + 16), fetch(tw + row + 32), fetch(tw + row + 48)};
  auto round = [&](auto steps, int t0) {
    constexpr int N = decltype(steps)::value;
    double ss[N], x[N][8];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const __half* xh = reinterpret_cast<const __half*>(&buf[u]);
      ss[u] = 0.0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[u][i] = (double)__half2float(xh[i]);
        ss[u] = fma(x[u][i], x[u][i], ss[u]);
      }
      if constexpr (N == 4) buf[u] = fetch(t0 + 16 * u + row + 64);
    }
    double sum;
    if constexpr (N == 4) {
      const bool odd = lane & 1, upper = lane & 2;
      const double s01 = (odd ? ss[1] : ss[0]) + xor_lane<1>(odd ? ss[0] : ss[1]);
      const double s23 = (odd ? ss[3] : ss[2]) + xor_lane<1>(odd ? ss[2] : ss[3]);
      sum = (upper ? s23 : s01) + xor_lane<2>(upper ? s01 : s23);
      sum += xor_lane<4>(sum);
      sum += xor_lane<8>(sum);
    } else {
      sum = xor_sum_w<16>(ss[0]);
    }
    const int t = t0 + row + (N == 4 ? 16 * (lane & 3) : 0);
    const __half b16 = f64_to_f16(sqrt_f64(sum * (1.0 / kHeadDim)));
    const double rb = t < t_end ? rcp_f64((double)__half2float(b16)) : 0.0;  // (tokens past the end add nothing)
    double r[N] = {rb};
    if constexpr (N == 4) r[0] = quad_lane<0>(rb), r[1] = quad_lane<1>(rb), r[2] = quad_lane<2>(rb), r[3] = quad_lane<3>(rb);
#pragma unroll
    for (int u = 0; u < N; ++u) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = fma(x[u][i], r[u], acc[i]);
    }
    if (write_b && col < N && t < t_end) {
      if (linear) {
        b_out[(int64_t)t * b_stride] = b16;
      } else {
        const int pos = start + t;
        const int64_t base = unit_token_base(g, cv.block_table, b, h, pos);
        reinterpret_cast<__half*>(cv.norms)[2 * (base + token_in_unit(g, pos)) + 1] = b16;
      }
    }
  };
  for (int t0 = tw; t0 < t_end; t0 += 64) {
    if (t0 + 16 < t_end)
      round(std::integral_constant<int, 4>(), t0);
    else
      round(std::integral_constant<int, 1>(), t0);
  }
  // the wave's four token rows, then the four waves
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    acc[i] += xor_lane<16>(acc[i]);
    acc[i] += xor_lane<32>(acc[i]);
  }
  __shared__ double red[4][kHeadDim];
  if (row == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) red[wave][8 * col + i] = acc[i];
  }
  __syncthreads();
  if (threadIdx.x < kHeadDim) {
    const int c = threadIdx.x;
    const double s = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
    partial[((((int64_t)(b * g.n_kv_heads + h) * 2 + tensor) * n_chunks) + chunk) * kHeadDim + c] = s;
  }
}

// 4-bit round-to-nearest levels of one group (Sec. 3.5): minimum and step in fp16, the code of x taken
// against the rounded minimum and step
__device__ inline int rtn4_code(double x, double mn, double st) {
  if (st == 0.0) return 0;
  const double lvl = floor((x - mn) / st + 0.5);
  return (int)fmin(fmax(lvl, 0.0), 15.0);
}

// 4-bit codes of fp16(s1) of a 64-token block into its norms record; a lane owns one token (the block has at least one:
// lane 0 is valid)
__device__ __forceinline__ void quantize_s1(float x, bool valid, int lane, unsigned char* rec) {
  float lo = valid ? x : INFINITY, hi = valid ? x : -INFINITY;
  static_for_pow2<64>([&](auto mask) {
    constexpr int m = decltype(mask)::value;
    lo = fminf(lo, xor_lane<m>(lo)), hi = fmaxf(hi, xor_lane<m>(hi));
  });
  const __half mn16 = f64_to_f16((double)lo);  // exact: the minimum is one of the fp16 inputs
  const __half st16 = f64_to_f16(((double)hi - (double)lo) / 15.0);
  const int code = valid ? rtn4_code((double)x, (double)__half2float(mn16), (double)__half2float(st16)) : 0;
  const int other = xor_lane_i32<1>(code);
  if ((lane & 1) == 0 && valid) rec[kDqNormCodes + (lane >> 1)] = (unsigned char)(code | (other << 4));
  if (lane == 0) *reinterpret_cast<__half2*>(rec + kDqNormPar) = __halves2half2(mn16, st16);
}

// 16 levels per 32 channels (half a wave) of a mean; channel c of the calling thread.  Returns the dequantised value,
// stores the record where one is given.
__device__ __forceinline__ double quantize_mean(double mean, int c, unsigned char* rec) {
  double lo = mean, hi = mean;
  static_for_pow2<32>([&](auto mask) {
    constexpr int m = decltype(mask)::value;
    lo = fmin(lo, xor_lane<m>(lo)), hi = fmax(hi, xor_lane<m>(hi));
  });
  const __half mn16 = f64_to_f16(lo), st16 = f64_to_f16((hi - lo) / 15.0);
  const double mn = (double)__half2float(mn16), st = (double)__half2float(st16);
  const int code = rtn4_code(mean, mn, st);
  const int other = xor_lane_i32<1>(code);
  if (rec) {
    if ((c & 1) == 0) rec[c >> 1] = (unsigned char)(code | (other << 4));
    if ((c & 31) == 0) *reinterpret_cast<__half2*>(rec + kDqMeanPar + 4 * (c >> 5)) = __halves2half2(mn16, st16);
  }
  return mn + st * (double)code;
}

// ---------------------------------------------------------------------------------------
// Stage A1 (side_bits = 4, NSN_VARIANT_ALT): grid (64-token block of the call, kv_head * 2 + tensor, sequence), block 64.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void enc_brtn_kernel(Geometry g, int max_new, int max_len,
                                                      const int32_t* __restrict__ seq_start,
                                                      const int32_t* __restrict__ n_new, CacheView kc, CacheView vc,
                                                      const __half* __restrict__ ws_b) {
  const int h = blockIdx.y >> 1, tensor = blockIdx.y & 1, b = blockIdx.z;
  const int lane = threadIdx.x;
  const CacheView& cv = tensor ? vc : kc;
  const int start = seq_start[b];
  const int count = min(n_new[b], max_new);
  const int t = blockIdx.x * 64 + lane, pos = start + t;
  const bool valid = t < count && pos < max_len;
  if (blockIdx.x * 64 >= count || start + blockIdx.x * 64 >= max_len) return;  // uniform: lane 0 is valid below
  const float x = valid ? __half2float(ws_b[((int64_t)(b * g.n_kv_heads + h) * 2 + tensor) * max_new + t]) : 0.f;
  const int pos0 = start + blockIdx.x * 64;  // the block's first token (the record is chosen by it)
  quantize_s1(x, valid, lane, dq_norm_rec(cv, unit_token_base(g, cv.block_table, b, h, pos0), token_in_unit(g, pos0)));
}

// ---------------------------------------------------------------------------------------
// Stage A2: Shift vector of every new group.  grid (group-in-call, kv_head * 2 + tensor, sequence),
// block 128 (one thread per channel); partial sums are added in chunk order.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(128) void enc_means_kernel(Geometry g, int max_new, int max_len,
                                                        const int32_t* __restrict__ seq_start,
                                                        const int32_t* __restrict__ n_new, CacheView kc,
                                                        CacheView vc, const double* __restrict__ partial,
                                                        int chunk_tokens, int n_chunks) {
  const int gl = blockIdx.x, h = blockIdx.y >> 1, tensor = blockIdx.y & 1, b = blockIdx.z;
  const int c = threadIdx.x;
  const CacheView& cv = tensor ? vc : kc;
  const int start = seq_start[b];
  const int count = min(min(n_new[b], max_new), max_len - start);
  int first_chunk, last_chunk, tokens, g_abs;
  if (g.group_size > 0) {  // chunk_tokens == group_size
    first_chunk = gl;
    last_chunk = gl + 1;
    tokens = min(g.group_size, count - gl * g.group_size);
    g_abs = start / g.group_size + gl;
  } else {
    first_chunk = 0;
    last_chunk = (count + chunk_tokens - 1) / chunk_tokens;
    tokens = count;
    g_abs = 0;
  }
  if (tokens <= 0 || g_abs >= g.n_groups_max) return;
  const double* p = partial + (((int64_t)(b * g.n_kv_heads + h) * 2 + tensor) * n_chunks) * kHeadDim + c;
  double s = 0.0;
  // added in chunk order, loaded eight at a time (one load per addition would be one memory round
  // trip per chunk: 512 of them for a 131072-token sequence)
  for (int k0 = first_chunk; k0 < last_chunk; k0 += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = (k0 + u < last_chunk) ? p[(int64_t)(k0 + u) * kHeadDim] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (k0 + u < last_chunk) s += v[u];
  }
  const double mean = s / (double)tokens;
  const int64_t mean_index = (int64_t)(b * g.n_kv_heads + h) * g.n_groups_max + g_abs;
  if (!g.dq) {
    cv.means[mean_index * kHeadDim + c] = f64_to_f16(mean);
    return;
  }
  quantize_mean(mean, c, dq_mean_rec(cv, mean_index));
}

// ---------------------------------------------------------------------------------------
// The encoder.  grid (wg_tokens-token chunk of the call, kv_head * 2 + tensor, sequence), block 256.
//
// Bound by vector instructions.  A lane owns CPL channels of a token:
//   CPL = 16 (large calls): eight lanes per token, eight tokens per wave step.  Everything done once per token (square
//     roots, reciprocals, lane reductions) is shared by eight tokens, four of the seven butterfly stages stay
//     inside the lane and two more swap register halves between lanes (one instruction per register).  The rotated
//     token passes through LDS so that the search is a loop over the lane's sub-vectors (one copy of its code, its
//     registers free).
//   CPL = SUB (small calls): as many lanes as there are sub-vectors: the shortest chain of instructions per token.
//   CPL = 8 of 4-dim sub-vectors (calls between the two): sixteen lanes per token, two sub-vectors in each.
// (One sub-vector per lane for all sizes and a best-two search in one pass, the form this replaces, took 1147 vector
// instructions per two 4-dim tokens.)
// Lane layout for CPL = 16: bits 0, 4, 5 of the lane select channels 8 (l0 + 2 l4 + 4 l5) .. + 7 and the same plus 64,
// bits 1..3 the token of the step; after the rotation the lane holds channels 8 (l0 + 2 r + 4 l4 + 8 l5) .. + 7 for register
// halves r = 0, 1.  Channels i and i + 64, which the rotary embedding pairs, start out in one lane.
// ---------------------------------------------------------------------------------------
struct EncArgs {
  Geometry g;
  const __half *codebook, *k_in, *v_in;
  int max_new, max_len;
  const int32_t *seq_start, *n_new;
  CacheView kc, vc;
  int wg_tokens;  // tokens of a workgroup: 128 or 64 .. 8
  int own_means;  // 1: groups of 64 tokens, their means are formed here
};

__device__ __forceinline__ double swap_sum16(double v) {  // v + value of lane ^ 16
  uint2 a = __builtin_bit_cast(uint2, v), b = a;
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3"
      : "+v"(a.x), "+v"(b.x), "+v"(a.y), "+v"(b.y));
  return __builtin_bit_cast(double, a) + __builtin_bit_cast(double, b);
}
__device__ __forceinline__ double swap_sum32(double v) {  // v + value of lane ^ 32
  uint2 a = __builtin_bit_cast(uint2, v), b = a;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3"
      : "+v"(a.x), "+v"(b.x), "+v"(a.y), "+v"(b.y));
  return __builtin_bit_cast(double, a) + __builtin_bit_cast(double, b);
}
// sum over the lanes that share a token
template <int CPL>
__device__ __forceinline__ double token_sum(double v) {
  if constexpr (CPL == 16) {
    v += xor_lane<1>(v);
    return swap_sum32(swap_sum16(v));
  } else {
    v = xor_sum_w<16>(v);
    return CPL == 4 ? swap_sum16(v) : v;
  }
}
// Walsh-Hadamard butterflies over the token's 128 channels (unnormalised), in the lane layouts above
template <int CPL>
__device__ __forceinline__ void rotate_token(double (&v)[CPL], int lane) {
  auto inside = [&](int s) {
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      if ((i & s) == 0) {
        const double a0 = v[i], a1 = v[i | s];
        v[i] = a0 + a1;
        v[i | s] = a0 - a1;
      }
    }
  };
#pragma unroll
  for (int s = 1; s < CPL; s <<= 1) inside(s);
  auto across = [&](auto mc) {
    constexpr int m = decltype(mc)::value;
    const double sign = (lane & m) ? -1.0 : 1.0;
#pragma unroll
    for (int i = 0; i < CPL; ++i) v[i] = fma(v[i], sign, xor_lane<m>(v[i]));
  };
  if constexpr (CPL == 16) {
    // lane bit 5 (then 4) changes places with register bit 3, whose butterfly is then inside the lane
    uint2 w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = __builtin_bit_cast(uint2, v[i]);
#pragma unroll
    for (int i = 0; i < 8; i += 2)
      swap32x4(w[i].x, w[i + 8].x, w[i].y, w[i + 8].y, w[i + 1].x, w[i + 9].x, w[i + 1].y, w[i + 9].y);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = __builtin_bit_cast(double, w[i]);
    inside(8);
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = __builtin_bit_cast(uint2, v[i]);
#pragma unroll
    for (int i = 0; i < 8; i += 2)
      swap16x4(w[i].x, w[i + 8].x, w[i].y, w[i + 8].y, w[i + 1].x, w[i + 9].x, w[i + 1].y, w[i + 9].y);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = __builtin_bit_cast(double, w[i]);
    inside(8);
    across(std::integral_constant<int, 1>{});
  } else {
    static_for_pow2<16>(across);
    if constexpr (CPL == 4) across(std::integral_constant<int, 16>{});
  }
}

// WAVES: workgroups on a compute unit, i.e. waves per SIMD.  Three (CPL = 16) leave 168 registers and 53 KB of LDS to each: the
// search has its LEAN form, the Shift vector is unpacked in every step instead of held in 32 registers, and the sums of pass 1 lie
// where the tokens come later.  8-dim instances spill 8 to 20 registers, none in the loop over the search's tiles.  Calls back
// to back, 8 x 8192 tokens, 8 kv heads, 4-dim: 543 -> 517 us; 4 ragged sequences of up to 4096 tokens, 8-dim signs with the
// rotary embedding: 105 -> 93 us.
template <int SUB, int CPL, bool SIGN, bool ROPE, bool PASS1, int WAVES = 2>
__global__ __launch_bounds__(256, WAVES) void enc_kernel(EncArgs A) {
  static_assert(CPL == 16 || CPL == 8 || CPL == SUB, "lane layouts");
  static_assert(!SIGN || SUB == 8, "the sign + index format is defined on 8-dim sub-vectors");
  constexpr int J = kHeadDim / SUB, JB = SIGN ? 2 * J : J;  // sub-vectors, code bytes per token
  constexpr int NQ = CPL / SUB, LPT = kHeadDim / CPL;       // sub-vectors per lane, lanes per token
  constexpr int TPS = 64 * CPL / kHeadDim;                  // tokens per wave step
  __shared__ SearchTables<SUB, true, (WAVES > 2)> T;
  __shared__ double2 y_s[CPL == SUB ? 1 : 4][CPL == SUB ? 1 : CPL / 2][64];  // rotated tokens, per wave
  // the waves' sums of pass 1 (three workgroups to a compute unit: in the tokens' place, before there are any)
  __shared__ double own_red[WAVES > 2 ? 1 : 4][kHeadDim], mean_s[kHeadDim];
  double(*const red)[kHeadDim] = WAVES > 2 ? reinterpret_cast<double(*)[kHeadDim]>(y_s) : own_red;
  __shared__ __half b_s[64];
  const Geometry& g = A.g;
  const int h = blockIdx.y >> 1, tensor = blockIdx.y & 1, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // What a call of few tokens spends its time on is trips to memory one after the other, so everything goes out as early as it
  // can: the arguments in one go (fetched where they are first needed they are three trips), the codebook beside the
  // sequence's start, the first token's rows and Shift vector ahead of the set-up of the search.  One token: 5.7 -> 4.4 us; 64
  // tokens x 8 sequences x 8 heads 11.1 -> 8.9 us, of that 10.7 with the new order alone (the rest: nsn_search.h).  Workgroups without
  // tokens fetch the codebook for nothing; calls that are mostly empty places gained all the same: 64 sequences of 8192 places with
  // 64 tokens each 1579 -> 1485 us, 128 of 4096 with one token each 654 -> 588 us.
  asm volatile("" ::"s"(A.codebook), "s"(A.k_in), "s"(A.v_in), "s"(A.max_new), "s"(A.max_len), "s"(A.seq_start), "s"(A.n_new),
               "s"(A.kc.codes), "s"(A.vc.codes), "s"(A.kc.means), "s"(A.vc.means), "s"(A.kc.norms), "s"(A.vc.norms),
               "s"(A.wg_tokens), "s"(g.dq), "s"(g.n_kv_heads), "s"(g.n_groups_max), "s"(g.group_size));
  // (asked for in the step that turns the token, it was waited for there: one token x 1024 sequences x 8 kv heads, 4-dim 92.1 -> 88.3 us)
  if constexpr (ROPE) asm volatile("" ::"s"(g.rope));
  const CacheView cv = {tensor ? A.vc.codes : A.kc.codes, tensor ? A.vc.norms : A.kc.norms, tensor ? A.vc.means : A.kc.means,
                        tensor ? A.vc.block_table : A.kc.block_table};
  const __half* in = (tensor ? A.v_in : A.k_in) + (int64_t)(b * g.n_kv_heads + h) * A.max_new * kHeadDim;
  const int start_v = A.seq_start[b], n_new_v = A.n_new[b];
  // the whole codebook, four rows per lane (every wave finds the longest one), and the thread's own row
  typedef uint32_t words2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef uint32_t words4 __attribute__((ext_vector_type(4), aligned(4)));
  typedef typename std::conditional<SUB == 4, words2, words4>::type row_t;
  row_t rows[kCodes / 64], own_row = reinterpret_cast<const row_t*>(A.codebook)[tid];
#pragma unroll
  for (int k = 0; k < kCodes / 64; ++k) rows[k] = reinterpret_cast<const row_t*>(A.codebook)[lane + 64 * k];
  asm volatile("" ::: "memory");  // (or the compiler moves them behind the early return)
  const int start = __builtin_amdgcn_readfirstlane(start_v), n_new = __builtin_amdgcn_readfirstlane(n_new_v);
  const int count = min(min(n_new, A.max_new), A.max_len - start);  // tokens that have a place in the cache
  const int t_wg = blockIdx.x * A.wg_tokens, block0 = t_wg & ~63;
  if (t_wg >= count) return;  // (the whole workgroup)
  const int64_t mean_row = (int64_t)(b * g.n_kv_heads + h) * g.n_groups_max;

  // ---- the lane's token and channels --------------------------------------------------------------
  const int tok = CPL == 16 ? (lane >> 1) & 7 : lane / LPT;
  const int l0 = lane & 1, l4 = (lane >> 4) & 1, l5 = lane >> 5;
  const int jj = lane % LPT;
  const int ch0 = CPL == 16 ? 8 * (l0 + 2 * l4 + 4 * l5) : jj * CPL;
  const bool leader = CPL == 16 ? (lane & 0x31) == 0 : jj == 0;
  const int j_first = CPL == 16 ? (SUB == 4 ? 16 * l5 + 8 * l4 + 2 * l0 : 8 * l5 + 4 * l4 + l0) : jj * NQ;
  constexpr int kRaw = CPL == 4 ? 1 : CPL / 8;  // 16-byte (CPL = 4: 8-byte) pieces of the lane's inputs
  typedef typename std::conditional<CPL == 4, uint2, uint4>::type raw_t;
  const int wave_tokens = A.wg_tokens >> 2;
  const int t_begin = t_wg + wave * wave_tokens, t_end = min(t_begin + wave_tokens, count);
  raw_t xraw[kRaw];
  auto fetch = [&](int t) {  // (count >= 1; rows past the end are read from the last valid one)
    const __half* row = in + (int64_t)min(t, count - 1) * kHeadDim + ch0;
#pragma unroll
    for (int k = 0; k < kRaw; ++k) xraw[k] = *reinterpret_cast<const raw_t*>(row + 64 * k);
  };
  fetch(t_begin + tok);
  // pass 1 (groups of 64 tokens whose means are formed here, 4-bit side information; an instance of its own, so that no load is
  // under a condition): a wave's sixteen tokens of the 64-token block, four at a time (lane: token lane / 16, channels
  // 8 (lane % 16))
  const bool dq = PASS1 && g.dq, own_means = PASS1 && A.own_means;
  uint4 p1[4];
  if constexpr (PASS1) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      p1[u] = *reinterpret_cast<const uint4*>(
          in + (int64_t)min(block0 + 16 * wave + 4 * u + (lane >> 4), count - 1) * kHeadDim + 8 * (lane & 15));
  }
  // Shift vectors as they are stored: the first token's is on its way during the set-up.  (One form of loads for fp16 and 4-bit
  // means: with a branch the compiler waits for all earlier loads where the two meet.)
  typedef typename std::conditional<CPL == 4, words2, words4>::type mean_t;
  mean_t mraw[kRaw];    // fp16 channels, or their 4-bit codes from the first byte on (CPL = 4: from a multiple of four bytes)
  uint32_t mpar[kRaw];  // 4-bit: (min, step)
  auto fetch_mean = [&](int gi) {
    const unsigned char* rec = reinterpret_cast<const unsigned char*>(cv.means) + (mean_row + gi) * (dq ? kDqMeanRec : 2 * kHeadDim);
#pragma unroll
    for (int k = 0; k < kRaw; ++k) {
      const int c = ch0 + 64 * k, at = dq ? (c >> 1) & ~3 : 2 * c;
      mraw[k] = *reinterpret_cast<const mean_t*>(rec + at);
      mpar[k] = *reinterpret_cast<const uint32_t*>(rec + (dq ? kDqMeanPar + 4 * (c >> 5) : at));
    }
  };
  auto group_at = [&](int pos) { return min(group_of(g, min(pos, A.max_len - 1)), g.n_groups_max - 1); };
  int grp = -1;  // Shift group whose mean is in mraw
  if (!own_means) grp = group_at(start + t_begin + tok);
  fetch_mean(max(grp, 0));  // (where the means are formed here nothing of it is used)
  SearchRegs<SUB, true> R;
  {
    float n2 = 0.f;
#pragma unroll
    for (int k = 0; k < kCodes / 64; ++k) {
      const __half* c = reinterpret_cast<const __half*>(&rows[k]);
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < SUB; ++i) t = fmaf(__half2float(c[i]), __half2float(c[i]), t);
      n2 = fmaxf(n2, t);
    }
    // (a rotated token has norm sqrt(128): no sub-vector is longer than 11.4)
    search_setup<SUB, true, (WAVES > 2)>(T, R, tid, wave_max_lanes(n2),
                            [&](int i) { return __half2float(reinterpret_cast<const __half*>(&own_row)[i]); }, 4);
  }

  if constexpr (PASS1) {
    double acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int tb = 16 * wave + 4 * u + (lane >> 4);  // token of the block
      const __half* xh = reinterpret_cast<const __half*>(&p1[u]);
      double x[8], ss = 0.0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[i] = (double)__half2float(xh[i]);
        ss = fma(x[i], x[i], ss);
      }
      const __half b16 = f64_to_f16(sqrt_f64(xor_sum_w<16>(ss) * (1.0 / kHeadDim)));
      if ((lane & 15) == 0) b_s[tb] = b16;
      const double rb = block0 + tb < count ? rcp_f64((double)__half2float(b16)) : 0.0;
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = fma(x[i], rb, acc[i]);
    }
    if (own_means) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = swap_sum32(swap_sum16(acc[i]));
      if (lane < 16) {
#pragma unroll
        for (int i = 0; i < 8; ++i) red[wave][8 * lane + i] = acc[i];
      }
    }
    __syncthreads();
    const bool stores = t_wg == block0;  // one of the block's workgroups writes what belongs to the block
    if (own_means && tid < kHeadDim) {
      const int64_t mean_index = mean_row + (start + block0) / g.group_size;
      const double mean = (((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid]) / (double)min(64, count - block0);
      if (!dq) {
        const __half m16 = f64_to_f16(mean);
        mean_s[tid] = (double)__half2float(m16);
        if (stores) cv.means[mean_index * kHeadDim + tid] = m16;
      } else {
        mean_s[tid] = quantize_mean(mean, tid, stores ? dq_mean_rec(cv, mean_index) : nullptr);
      }
    }
    if (dq && stores && wave == 3) {
      const int pos0 = start + block0;
      quantize_s1(__half2float(b_s[lane]), block0 + lane < count, lane,
                  dq_norm_rec(cv, unit_token_base(g, cv.block_table, b, h, pos0), token_in_unit(g, pos0)));
    }
    __syncthreads();
  }

  // ---- pass 2 -----------------------------------------------------------------------------------
  constexpr bool kLate = WAVES > 2;
  double o[CPL];
  if (!kLate && own_means) {
#pragma unroll
    for (int i = 0; i < CPL; ++i) o[i] = mean_s[ch0 + (i & 7) + 64 * (i >> 3)];
  }
  auto unpack_mean = [&]() {
#pragma unroll
    for (int k = 0; k < kRaw; ++k) {
      constexpr int N = CPL == 4 ? 4 : 8;
      if (dq) {
        const __half2 par = __builtin_bit_cast(__half2, mpar[k]);
        const double mn = (double)__low2float(par), st = (double)__high2float(par);
        const uint32_t codes = CPL == 4 ? mraw[k].x >> (4 * (ch0 & 4)) : mraw[k].x;
#pragma unroll
        for (int i = 0; i < N; ++i) o[8 * k + i] = mn + st * (double)((codes >> (4 * i)) & 15u);
      } else {
        const __half* mh = reinterpret_cast<const __half*>(&mraw[k]);
#pragma unroll
        for (int i = 0; i < N; ++i) o[8 * k + i] = (double)__half2float(mh[i]);
      }
    }
  };
  if (!kLate && !own_means) unpack_mean();
  // (the rotated tokens are kept in the search's units; a table entry is -2 R.scale times the codeword's element.  All exact:
  // powers of two)
  const double y_scale = (double)R.scale;
  const double dot_scale = __builtin_ldexp(-0.5, -2 * (__builtin_amdgcn_frexp_expf(R.scale) - 1));  // -0.5 / y_scale^2
  // the lane's further codes lie at fixed distances from its first one (both layouts are linear in the bits of j)
  const int64_t dq1 = NQ > 1 ? code_offset(g.tiled, tensor != 0, JB, 0, CPL == 16 && SUB == 8 ? 2 : 1) : 0;
  const int64_t dq2 = NQ > 2 ? code_offset(g.tiled, tensor != 0, JB, 0, 4) : 0;
  const int64_t dsign = SIGN ? code_offset(g.tiled, tensor != 0, JB, 0, J) : 0;

  for (int t0 = t_begin; t0 < t_end; t0 += TPS) {  // (uniform over the wave)
    const int t = t0 + tok, pos = start + t;
    const bool valid = t < t_end;
    double v[CPL];
#pragma unroll
    for (int k = 0; k < kRaw; ++k) {
      const __half* xh = reinterpret_cast<const __half*>(&xraw[k]);
#pragma unroll
      for (int i = 0; i < (CPL == 4 ? 4 : 8); ++i) v[8 * k + i] = (double)__half2float(xh[i]);
    }
    if (t0 + TPS < t_end) fetch(t + TPS);
    if (!own_means) {
      const int want = group_at(pos);
      if (__any(want != grp)) {
        grp = want;
        fetch_mean(grp);
        if constexpr (!kLate) unpack_mean();
      }
    }
    __half b16;
    if constexpr (PASS1) {
      b16 = b_s[min(t - block0, 63)];
    } else {
      double ss = 0.0;
#pragma unroll
      for (int i = 0; i < CPL; ++i) ss = fma(v[i], v[i], ss);
      b16 = f64_to_f16(sqrt_f64(token_sum<CPL>(ss) * (1.0 / kHeadDim)));
    }
    const double bb = (double)__half2float(b16), rb = rcp_f64(bb);
    double ss = 0.0;
    if constexpr (kLate) {
      if (own_means) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) o[i] = mean_s[ch0 + (i & 7) + 64 * (i >> 3)];
      } else {
        unpack_mean();
      }
    }
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      v[i] = fma(v[i], rb, -o[i]);
      ss = fma(v[i], v[i], ss);
    }
    ss = token_sum<CPL>(ss);
    // second Normalize and the 1 / sqrt(d) of the rotation in one factor: v / s2 / sqrt(d) = v / ||v||
    const double rs = rsqrt_f64(ss), s2 = ss * rs * kInvSqrtD;
#pragma unroll
    for (int i = 0; i < CPL; ++i) v[i] *= rs * y_scale;
    if constexpr (ROPE) {
      if (tensor == 0) {  // keys only: channels c and c + 64 turn by position * inv_freq[c]
        // cos / sin from the fp64 table: block part and in-block part combined by the addition theorems
        const int pc = min(pos, A.max_len - 1), pair0 = ch0 & 63;
        const double2* blk = reinterpret_cast<const double2*>(g.rope + kRopeBlkOff + (int64_t)(pc >> 6) * kRopeBlkStride +
                                                              kRopeBlk64) + pair0;
        const double2* inb = reinterpret_cast<const double2*>(g.rope + kRopeInOff) + (pc & 63) * 64 + pair0;
        constexpr int NP = CPL == 4 ? 4 : 8;  // channel pairs of a lane
        const double side = (ch0 & 64) ? 1.0 : -1.0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const double2 c0 = blk[i], cj = inb[i];
          const double c = c0.x * cj.x - c0.y * cj.y, sn = c0.y * cj.x + c0.x * cj.y;
          if constexpr (CPL == 16) {
            const double x0 = v[i], x1 = v[i + 8];
            v[i] = x0 * c - x1 * sn;
            v[i + 8] = x1 * c + x0 * sn;
          } else {  // the partner channel lives in lane ^ (LPT / 2)
            const double other = xor_lane<LPT / 2>(v[i]);
            v[i] = v[i] * c + side * other * sn;
          }
        }
      }
    }
    rotate_token<CPL>(v, lane);
    if constexpr (NQ > 1) {
#pragma unroll
      for (int k = 0; k < CPL / 2; ++k) y_s[wave][k][lane] = make_double2(v[2 * k], v[2 * k + 1]);
    }
    const int64_t base = unit_token_base(g, cv.block_table, b, h, valid ? pos : start);
    const int tin = token_in_unit(g, pos);
    uint8_t* out = cv.codes + base * JB + code_offset(g.tiled, tensor != 0, JB, tin, j_first);
    double dot = 0.0;  // |y| . C[code] (y . C[code] without signs) in table units
#pragma unroll 1
    for (int q = 0; q < NQ; ++q) {
      double y[SUB];
      if constexpr (NQ > 1) {  // (this lane's own entries)
#pragma unroll
        for (int k = 0; k < SUB / 2; ++k) {
          const double2 p = y_s[wave][q * (SUB / 2) + k][lane];
          y[2 * k] = p.x, y[2 * k + 1] = p.y;
        }
      } else {
#pragma unroll
        for (int i = 0; i < SUB; ++i) y[i] = v[i];
      }
      // sign + index format: the nearest signed codeword has the signs of y and the magnitude codeword nearest to |y|
      // (the magnitudes are non-negative), and y . y_Q = |y| . C[code]
      uint32_t sign_byte = 0u;
      if constexpr (SIGN) {
#pragma unroll
        for (int i = 0; i < SUB; ++i) {
          if (y[i] < 0.0) sign_byte |= 1u << i;
          y[i] = fabs(y[i]);
        }
      }
      float yf[SUB];
#pragma unroll
      for (int i = 0; i < SUB; ++i) yf[i] = (float)y[i];
      const int code = search_nearest<SUB, true, (WAVES == 2), (WAVES > 2)>(T, R, yf, [&](int c) {
        double d = 0.0;
#pragma unroll
        for (int u = 0; u < SUB / 4; ++u) {
          const float4 e = T.n2c[u][SearchTables<SUB, true, (WAVES > 2)>::row(c)];
          const float ev[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double dd = y[4 * u + i] - (double)ev[i] * -0.5;
            d = __dadd_rn(d, __dmul_rn(dd, dd));  // plain sum of squares
          }
        }
        return d;
      });
#pragma unroll
      for (int u = 0; u < SUB / 4; ++u) {
        const float4 e = T.n2c[u][SearchTables<SUB, true, (WAVES > 2)>::row(code)];
        dot = fma(y[4 * u], (double)e.x, dot), dot = fma(y[4 * u + 1], (double)e.y, dot);
        dot = fma(y[4 * u + 2], (double)e.z, dot), dot = fma(y[4 * u + 3], (double)e.w, dot);
      }
      if (valid) {
        const int64_t at = NQ == 4 ? (q & 1) * dq1 + (q >> 1) * dq2 : q * dq1;
        out[at] = (uint8_t)code;
        if constexpr (SIGN) out[at + dsign] = (uint8_t)sign_byte;
      }
    }
    // scale adjustment: alpha = ||y||^2 / (y . y_Q), ||y||^2 = d
    dot = token_sum<CPL>(dot) * dot_scale;
    const double alpha = dot > 1e-12 * kHeadDim ? (double)kHeadDim * rcp_f64(dot) : 1.0;
    if (valid && leader) {
      if (dq)  // a' = fp16(s2 alpha); s1 is stored as a 4-bit code
        reinterpret_cast<__half*>(dq_norm_rec(cv, base, tin))[tin & 63] = f64_to_f16(s2 * alpha);
      else
        cv.norms[base + tin] = __halves2half2(f64_to_f16(bb * s2 * alpha), b16);
    }
  }
}

// ---------------------------------------------------------------------------------------
// NSN_VARIANT_ALT, last stage: shift, second Normalize, rotation, fp32 scan of the 256 distances, scale adjustment, stores.
// grid (64- or 16-token chunk, kv_head * 2 + tensor, sequence), block 256.  A lane owns one
// sub-vector (SUB channels) of one token; a wave covers 64 / J tokens at a time.
// ---------------------------------------------------------------------------------------
// FUSED: append mode - the first-Normalize scale is computed here instead of by the stats kernel
// SIGN:  the paper's 2-bit format (Sec. 3.4): the search runs on the absolute values against a
//        codebook of magnitudes; byte row jj holds the index, byte row 16 + jj the eight sign bits
template <int SUB, bool FUSED, bool SIGN = false>
__global__ __launch_bounds__(256) void enc_quant_kernel(Geometry g, const __half* __restrict__ codebook,
                                                        const __half* __restrict__ k_in,
                                                        const __half* __restrict__ v_in, int max_new,
                                                        int max_len, const int32_t* __restrict__ seq_start,
                                                        const int32_t* __restrict__ n_new, CacheView kc,
                                                        CacheView vc, int wave_tokens,
                                                        const __half* __restrict__ ws_b) {
  // wave_tokens: tokens per wave (16, or 4 when the call is too small to fill the chip with 64-token blocks)
  constexpr int J = kHeadDim / SUB;  // lanes per token
  constexpr int TPW = 64 / J;        // tokens per wave step
  constexpr int JB = SIGN ? 2 * J : J;  // code bytes per token
  static_assert(!SIGN || SUB == 8, "the sign + index format is defined on 8-dim sub-vectors");
  __shared__ VqTables<SUB> T;
  const int h = blockIdx.y >> 1, tensor = blockIdx.y & 1, b = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int jj = lane % J, tk = lane / J;
  const CacheView& cv = tensor ? vc : kc;
  const __half* in = (tensor ? v_in : k_in) + ((int64_t)(b * g.n_kv_heads + h) * max_new) * kHeadDim;
  const int start = seq_start[b];
  const int count = min(n_new[b], max_new);
  const int t_begin = blockIdx.x * (4 * wave_tokens) + wave * wave_tokens;

  // One token's inputs as this lane needs them (vector loads of SUB fp16 values); the first
  // token's loads are issued before the codebook tables are built, later ones one step ahead.
  typedef typename std::conditional<SUB == 4, uint2, uint4>::type vec_t;
  struct Tok {
    bool valid;
    int64_t base;
    int tin, pos;
    vec_t xraw, oraw;
    __half b16;
    uint32_t oq;  // side_bits = 4: the SUB 4-bit codes of this lane's channels of the mean
    __half2 op;   //                (min, step) of their 32-channel group
  };
  auto fetch = [&](int it) {
    Tok k;
    const int t = t_begin + it * TPW + tk;
    const int pos = start + t;
    k.valid = (t < count) && (pos < max_len);
    k.pos = pos;
    k.base = 0;
    k.tin = 0;
    k.xraw = vec_t{};
    k.oraw = vec_t{};
    k.b16 = __float2half(0.f);
    k.oq = 0u;
    k.op = __half2{};
    if (k.valid) {
      k.base = unit_token_base(g, cv.block_table, b, h, pos);
      k.tin = token_in_unit(g, pos);
      k.xraw = *reinterpret_cast<const vec_t*>(in + (int64_t)t * kHeadDim + jj * SUB);
      const int64_t mean_index =
          (int64_t)(b * g.n_kv_heads + h) * g.n_groups_max + min(group_of(g, pos), g.n_groups_max - 1);
      if (g.dq) {
        const unsigned char* rec = dq_mean_rec(cv, mean_index);
        if constexpr (SUB == 4)
          k.oq = *reinterpret_cast<const uint16_t*>(rec + jj * 2);
        else
          k.oq = *reinterpret_cast<const uint32_t*>(rec + jj * 4);
        k.op = *reinterpret_cast<const __half2*>(rec + kDqMeanPar + 4 * ((jj * SUB) >> 5));
        if constexpr (!FUSED) k.b16 = ws_b[((int64_t)(b * g.n_kv_heads + h) * 2 + tensor) * max_new + t];
      } else {
        k.oraw = *reinterpret_cast<const vec_t*>(cv.means + mean_index * kHeadDim + jj * SUB);
        if constexpr (!FUSED) k.b16 = reinterpret_cast<const __half*>(cv.norms)[2 * (k.base + k.tin) + 1];
      }
    }
    return k;
  };
  Tok nxt = fetch(0);

  vq_tables_fill<SUB>(T, [&](int c, int i) { return (double)__half2float(codebook[c * SUB + i]); });
  if (blockIdx.x * (4 * wave_tokens) >= count) return;

  const int n_it = wave_tokens / TPW;
  for (int it = 0; it < n_it; ++it) {
    if (t_begin + it * TPW >= count) break;  // wave-uniform: nothing left for this wave
    const Tok cur = nxt;
    if (it + 1 < n_it && t_begin + (it + 1) * TPW < count) nxt = fetch(it + 1);
    const bool valid = cur.valid;
    const int64_t base = cur.base;
    const int tin = cur.tin;
    const vec_t xraw = cur.xraw, oraw = cur.oraw;
    __half b16f = cur.b16;
    double xs[SUB], os[SUB];
    {
      const __half* xh = reinterpret_cast<const __half*>(&xraw);
      const __half* oh = reinterpret_cast<const __half*>(&oraw);
#pragma unroll
      for (int i = 0; i < SUB; ++i) {
        xs[i] = (double)__half2float(xh[i]);
        os[i] = (double)__half2float(oh[i]);
      }
      if (g.dq) {  // dequantised mean: min + step * code
        const double mn = (double)__low2float(cur.op), st = (double)__high2float(cur.op);
#pragma unroll
        for (int i = 0; i < SUB; ++i) os[i] = mn + st * (double)((cur.oq >> (4 * i)) & 15u);
      }
    }
    if constexpr (FUSED) {  // first Normalize here: b = fp16(||x|| / sqrt(d)), stored with the token
      double ssx = 0.0;
#pragma unroll
      for (int i = 0; i < SUB; ++i) ssx += xs[i] * xs[i];
      ssx = xor_sum_w<J>(ssx);
      b16f = f64_to_f16(sqrt(ssx) / kSqrtD);
      if (valid && jj == 0 && !g.dq) reinterpret_cast<__half*>(cv.norms)[2 * (base + tin) + 1] = b16f;
    }
    const double bb = (double)__half2float(b16f);
    // one division per token instead of one per channel: x * (1 / b) is within one fp64 unit of x / b, eight
    // decimal orders below anything the fp16 results and the code decisions can see
    const double rb = bb != 0.0 ? 1.0 / bb : 0.0;
    double v[SUB];
#pragma unroll
    for (int i = 0; i < SUB; ++i) v[i] = valid ? xs[i] * rb - os[i] : 0.0;
    // second Normalize
    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < SUB; ++i) ss += v[i] * v[i];
    ss = xor_sum_w<J>(ss);
    const double s2 = sqrt(ss) * kInvSqrtD;  // (feeds the stored scale a, compared to one fp16 unit)
    const double r2 = (s2 != 0.0) ? 1.0 / s2 : 0.0;
#pragma unroll
    for (int i = 0; i < SUB; ++i) v[i] *= r2;
    // Walsh-Hadamard butterflies: channel bits 0..log2(SUB)-1 in registers, the rest across lanes
#pragma unroll
    for (int s = 1; s < SUB; s <<= 1) {
#pragma unroll
      for (int i = 0; i < SUB; ++i) {
        if ((i & s) == 0) {
          const double a0 = v[i], a1 = v[i | s];
          v[i] = a0 + a1;
          v[i | s] = a0 - a1;
        }
      }
    }
    static_for_pow2<J>([&](auto mc) {
      constexpr int m = decltype(mc)::value;
      const bool upper = (jj & m) != 0;
#pragma unroll
      for (int i = 0; i < SUB; ++i) {
        const double other = xor_lane<m>(v[i]);
        v[i] = upper ? other - v[i] : v[i] + other;
      }
    });
    double y[SUB];
#pragma unroll
    for (int i = 0; i < SUB; ++i) y[i] = v[i] * kInvSqrtD;

    // sign + index format: the nearest signed codeword has the signs of y and the magnitude
    // codeword nearest to |y| (the magnitudes are non-negative), and y . y_Q = |y| . C[code]
    double ys[SUB];
    uint32_t sign_byte = 0u;
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      ys[i] = SIGN ? fabs(y[i]) : y[i];
      if (SIGN && y[i] < 0.0) sign_byte |= 1u << i;
    }
    const int code = vq_search<SUB>(T, ys);

    // scale adjustment: alpha = ||y||^2 / (y . y_Q)
    double dot = 0.0, nrm2 = 0.0;
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      dot += ys[i] * T.cx[code][i];
      nrm2 += y[i] * y[i];
    }
    dot = xor_sum_w<J>(dot);
    nrm2 = xor_sum_w<J>(nrm2);
    const double alpha = (dot > 1e-12 * kHeadDim) ? nrm2 / dot : 1.0;
    if (valid) {
      const int64_t off = code_offset(g.tiled, tensor != 0, JB, tin, jj);
      cv.codes[base * JB + off] = (uint8_t)code;
      if constexpr (SIGN) {
        const int64_t soff = code_offset(g.tiled, tensor != 0, JB, tin, J + jj);
        cv.codes[base * JB + soff] = (uint8_t)sign_byte;
      }
      if (jj == 0) {
        if (g.dq)  // a' = fp16(s2 alpha); s1 is stored separately as a 4-bit code
          reinterpret_cast<__half*>(dq_norm_rec(cv, base, tin))[tin & 63] = f64_to_f16(s2 * alpha);
        else
          reinterpret_cast<__half*>(cv.norms)[2 * (base + tin)] = f64_to_f16(bb * s2 * alpha);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
static int encode_chunk_tokens(const nsn_shape& s) { return s.group_size > 0 ? s.group_size : 256; }

static size_t encode_partial_bytes(const nsn_shape& s, int batch, int64_t max_new) {
  const int ct = encode_chunk_tokens(s);
  const int64_t n_chunks = (max_new + ct - 1) / ct;
  return (size_t)batch * s.n_kv_heads * 2 * n_chunks * kHeadDim * sizeof(double);
}

size_t encode_workspace_bytes(const nsn_shape& s, int batch, int64_t max_new) {
  // side_bits = 4 (NSN_VARIANT_ALT): fp16(s1) of every new token passes through the workspace
  const size_t b_bytes = s.side_bits == 4 ? (((size_t)batch * s.n_kv_heads * 2 * max_new * sizeof(__half)) + 255) & ~(size_t)255 : 0;
  return encode_partial_bytes(s, batch, max_new) + b_bytes;
}

// What a call takes in one lane layout, in us: a fixed part and so much per round of the chip, a workgroup on each of its 256
// compute units (two fit; the time grows by one step for every 256 of them all the same).  A round of workgroups with one wave
// at work is shorter.  Fitted to 6639 calls of 1 to 450 tokens a sequence and 128 to 150000 token places, 15 formats, each timed in
// every layout: the layout chosen is 0.3 % slower than the best one of a call in the geometric mean, where lines drawn at
// numbers of token places (8-dim 12288; 4-dim 4096, 6144 and 14336) made it 7.4 %, and for few tokens of many
// sequences up to twice as slow.  Small / eight / bulk, us: one token x 768 sequences x 8 kv heads, 8-dim 84 / - / 142; 4-dim, 8 kv
// heads: 5 tokens x 75 sequences 12.0 / 15.2 / 16.7, 9 x 65 19.4 / 15.6 / 21.9, 64 x 4 6.4 / 6.5 / 8.6, 64 x 9 12.1 / 11.0 / 11.7,
// 64 x 13 16.1 / 13.6 / 12.0, 64 x 30 31.7 / 24.7 / 21.4.
struct LayoutTime {
  float fixed, one_wave, round;
};
struct LayoutTimes {
  LayoutTime small, eight, bulk;
};
constexpr LayoutTimes kLayoutTimes[2][2][2] = {  // 4-dim, 8-dim | pass 1 | keys before the rotary embedding
    {{{{2.3f, 1.45f, 1.85f}, {2.4f, 1.5f, 2.6f}, {5.1f, 2.4f, 3.7f}}, {{2.6f, 1.4f, 2.2f}, {4.1f, 1.4f, 3.2f}, {5.4f, 2.8f, 3.85f}}},
     {{{3.4f, 2.65f, 2.75f}, {}, {5.1f, 4.4f, 4.6f}}, {{3.4f, 2.65f, 2.75f}, {}, {5.1f, 4.4f, 4.6f}}}},
    {{{{3.2f, 1.9f, 2.5f}, {}, {4.8f, 3.1f, 3.5f}}, {{3.6f, 1.7f, 3.1f}, {}, {4.2f, 3.5f, 4.3f}}},
     {{{4.2f, 3.0f, 3.25f}, {}, {4.7f, 4.05f, 4.6f}}, {{5.1f, 3.8f, 4.0f}, {}, {4.5f, 4.8f, 5.0f}}}}};

// The lane layout of a call: channels per lane (4, 8 or 16).  Tokens are counted by the workgroups that they take, not by their
// number: a call of many sequences with a few tokens each fills neither the waves nor the workgroups of the sixteen-channel layout.
int encode_layout(const nsn_shape& s, int batch, int max_new, bool pass1) {
  const LayoutTimes& times = kLayoutTimes[s.sub_dim == 8][pass1][s.rope_table != nullptr];
  auto workgroups = [&](int wg_tokens) {
    return (int64_t)s.n_kv_heads * 2 * batch * ((max_new + wg_tokens - 1) / wg_tokens);
  };
  auto estimate = [&](const LayoutTime& t, int wg_tokens) {
    return t.fixed + (float)((workgroups(wg_tokens) + 255) / 256) * (max_new <= wg_tokens / 4 ? t.one_wave : t.round);
  };
  const int small_tokens = s.sub_dim == 8 ? 16 : 8;
  if (workgroups(small_tokens) <= 512) return s.sub_dim;  // all of them are under way at once: the shortest chain
  const float small = estimate(times.small, small_tokens), bulk = estimate(times.bulk, 32);
  const float eight = s.sub_dim == 4 && !pass1 ? estimate(times.eight, 16) : INFINITY;
  return bulk < fminf(small, eight) ? 16 : eight < small ? 8 : s.sub_dim;
}

// Tokens per workgroup: one step per wave where that is what fills the chip, several where the workgroup's set-up (tables, operands:
// about a sixth of a step) is worth sharing; a 64-token block is the most that pass 1 holds.
int encode_wg_tokens(const nsn_shape& s, int batch, int max_new, bool pass1, int layout) {
  if (layout != 16) return layout > s.sub_dim ? 16 : s.sub_dim == 8 ? 16 : 8;
  const int64_t tokens = (int64_t)max_new * s.n_kv_heads * 2 * batch;
  return tokens < 32768 ? 32 : tokens >= 524288 && !pass1 ? 128 : 64;
}

// Three workgroups to a compute unit, of the 256, or two.  Three share their vector ALUs better, but their workgroups run without
// the tile requested ahead and unpack the Shift vector in every step, so each takes longer: worth it where the chip goes through
// fewer rounds, and always beyond four workgroups to a compute unit.  Two / three, us, batch 8 x 8 kv heads, formats 4-dim |
// 8-dim | 4-dim with the rotary embedding | 8-dim signs with it and means formed here (same results in all):
//    256 workgroups  17.2 / 18.3 | 15.9 / 16.6 | 18.7 / 19.3 | 13.9 / 15.7
//    512             26.0 / 27.7 | 22.8 / 24.1 | 28.9 / 30.0 | 21.4 / 23.3
//    640             34.8 / 34.4 | 30.2 / 29.1 | 37.5 / 36.4 | 30.4 / 28.3
//    768             34.9 / 34.8 | 30.2 / 29.5 | 39.4 / 36.0 | 33.3 / 29.3
//   1024             42.7 / 42.9 | 35.3 / 36.4 | 47.6 / 46.4 | 40.5 / 39.7
//   1280             52.2 / 51.4 | 44.5 / 43.2 | 58.5 / 56.3 | 50.7 / 45.7
//   2048             75.9 / 73.4 | 63.6 / 60.7 | 87.6 / 80.0 | 76.9 / 69.0
//   4096             143.6 / 136.5 | 119.7 / 112.1 | 156.8 / 144.2 | 138.8 / 127.9
// Those are sequences of one length.  Of a batch the host knows only the places, and workgroups without tokens leave holes: three
// that have some then lie on one compute unit and none on the next, where two to a unit leave the rest waiting for whichever is
// free.  16 sequences of 0.4 to 1 times 1088 tokens, one kv head, 544 places: 27.5 / 34.2, 24.0 / 28.6, 29.3 / 35.5, 21.1 / 28.4;
// 1280 to 1664 places with one long sequence among eight 0.75 to 0.87 times as fast.  Over 708 calls of 2 to 64 sequences, lengths from
// 0.03, 0.4 or 0.8 times the longest up, no one beyond 1900 places was slower with three (geometric mean 1.07 times as fast), and
// from 2048 on none of 480 more in which one sequence or half of them are long and the others a tenth of that.
int encode_per_unit(const nsn_shape& s, int batch, int max_new, int layout, int wg_tokens) {
  if (layout != 16) return 2;
  const int64_t places = (int64_t)s.n_kv_heads * 2 * batch * ((max_new + wg_tokens - 1) / wg_tokens);
  const bool three = batch > 1 ? places >= 2048 : places > 1024 || (places > 512 && places <= 768);
  return three ? 3 : 2;
}

int encode_launch(const nsn_shape& s, const void* codebook, const void* k_in, const void* v_in, int max_new,
                  const int32_t* seq_start, const int32_t* n_new, int batch, int freeze_means,
                  const nsn_cache& kc, const nsn_cache& vc, void* workspace, hipStream_t stream) {
  const Geometry g = make_geometry(s);
  const CacheView kv = make_view(kc), vv = make_view(vc);
  const int ct = encode_chunk_tokens(s);
  const int n_chunks = (max_new + ct - 1) / ct;
  double* partial = static_cast<double*>(workspace);
  __half* ws_b = reinterpret_cast<__half*>(static_cast<unsigned char*>(workspace) + encode_partial_bytes(s, batch, max_new));
  // the alternative is the vector-ALU scan (keys before the rotary embedding have the default form only)
  const bool alt = selected_variant(NSN_OP_ENCODE) == NSN_VARIANT_ALT && !g.rope;
  const bool own_means = !alt && !freeze_means && s.group_size == 64;
  if ((!freeze_means && !own_means) || (alt && g.dq)) {
    const dim3 grid_a(n_chunks, s.n_kv_heads * 2, batch);
    enc_stats_kernel<<<grid_a, 256, 0, stream>>>(g, (const __half*)k_in, (const __half*)v_in, max_new, s.max_len,
                                                 seq_start, n_new, kv, vv, partial, ct, n_chunks, ws_b, alt);
    if (alt && g.dq) {
      const dim3 grid_r((max_new + 63) / 64, s.n_kv_heads * 2, batch);
      enc_brtn_kernel<<<grid_r, 64, 0, stream>>>(g, max_new, s.max_len, seq_start, n_new, kv, vv, ws_b);
    }
  }
  if (!freeze_means && !own_means) {
    const int n_groups_new = s.group_size > 0 ? n_chunks : 1;
    const dim3 grid_m(n_groups_new, s.n_kv_heads * 2, batch);
    enc_means_kernel<<<grid_m, 128, 0, stream>>>(g, max_new, s.max_len, seq_start, n_new, kv, vv, partial, ct,
                                                 n_chunks);
  }
  const int64_t tokens = (int64_t)max_new * s.n_kv_heads * 2 * batch;
  if (alt) {
    // 64 tokens per workgroup; calls that would leave most compute units idle use 16 (4 per wave)
    const int wave_tokens = tokens >= 65536 ? 16 : 4;
    const dim3 grid_b((max_new + 4 * wave_tokens - 1) / (4 * wave_tokens), s.n_kv_heads * 2, batch);
    auto launch = [&](auto kernel) {
      kernel<<<grid_b, 256, 0, stream>>>(g, (const __half*)codebook, (const __half*)k_in, (const __half*)v_in, max_new,
                                         s.max_len, seq_start, n_new, kv, vv, wave_tokens, ws_b);
    };
    const bool fused = freeze_means && !g.dq;  // the quantiser computes s1 itself
    if (g.sign)
      fused ? launch(enc_quant_kernel<8, true, true>) : launch(enc_quant_kernel<8, false, true>);
    else if (s.sub_dim == 8)
      fused ? launch(enc_quant_kernel<8, true>) : launch(enc_quant_kernel<8, false>);
    else
      fused ? launch(enc_quant_kernel<4, true>) : launch(enc_quant_kernel<4, false>);
    return hipGetLastError() == hipSuccess ? NSN_OK : NSN_ERR_HIP;
  }
  const bool pass1 = own_means || g.dq;
  const int layout = encode_layout(s, batch, max_new, pass1), wg_tokens = encode_wg_tokens(s, batch, max_new, pass1, layout);
  const bool bulk = layout == 16, eight = layout > s.sub_dim && !bulk;
  const bool three = encode_per_unit(s, batch, max_new, layout, wg_tokens) == 3;
  const EncArgs a = {g, (const __half*)codebook, (const __half*)k_in, (const __half*)v_in, max_new, s.max_len, seq_start, n_new,
                     kv, vv, wg_tokens, own_means};
  const dim3 grid((max_new + wg_tokens - 1) / wg_tokens, s.n_kv_heads * 2, batch);
  auto launch = [&](auto kernel) { kernel<<<grid, 256, 0, stream>>>(a); };
  auto pick = [&](auto sub, auto sign, auto rope) {
    constexpr int kSub = decltype(sub)::value;
    constexpr bool kSign = decltype(sign)::value, kRope = decltype(rope)::value;
    if (pass1)
      three  ? launch(enc_kernel<kSub, 16, kSign, kRope, true, 3>)
      : bulk ? launch(enc_kernel<kSub, 16, kSign, kRope, true>)
             : launch(enc_kernel<kSub, kSub, kSign, kRope, true>);
    else if (eight)
      launch(enc_kernel<kSub, 8, kSign, kRope, false>);
    else
      three  ? launch(enc_kernel<kSub, 16, kSign, kRope, false, 3>)
      : bulk ? launch(enc_kernel<kSub, 16, kSign, kRope, false>)
             : launch(enc_kernel<kSub, kSub, kSign, kRope, false>);
  };
  auto with_format = [&](auto rope) {
    if (g.sign)
      pick(std::integral_constant<int, 8>{}, std::true_type{}, rope);
    else if (s.sub_dim == 8)
      pick(std::integral_constant<int, 8>{}, std::false_type{}, rope);
    else
      pick(std::integral_constant<int, 4>{}, std::false_type{}, rope);
  };
  g.rope ? with_format(std::true_type{}) : with_format(std::false_type{});
  return hipGetLastError() == hipSuccess ? NSN_OK : NSN_ERR_HIP;
}

}  // namespace nsn
