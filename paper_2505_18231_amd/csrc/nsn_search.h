// Nearest-codeword search (Eq. 1, squared Euclidean distance): one sub-vector per lane, 64 per call.
//
// Three steps, bound by vector instructions: per 64 searches of 256 4-dim codewords 265 of them (and 16 matrix instructions) up to
// the lists, then 60 for every group of the longest list among the 64, which holds one at least (LEAN: sixteen fewer and six more);
// 8-dim codewords 295 (and 32) and 95.  Settling two candidates takes 55 to 110 more.  (Keeping the best two indexed keys of every
// distance took about 740.)
//   1. matrix cores: D = ||c||^2 - 2 c . y + n for 32 codewords (rows) x 32 sub-vectors (columns) at a time, n slightly
//      above ||y||^2 (D > 0).  y, c and ||c||^2 enter as sums of fp16 parts, so D is good to about 2^-19 of
//      (|c| + |y|)^2.  A lane then holds 16 distances of one sub-vector per tile and keeps only the minima of two groups
//      of about eight: half an instruction per distance (three-operand minima), no index bookkeeping.  32 groups of codewords
//      leave 32 minima per sub-vector, sixteen in either half of the wave.
//   2. every group whose minimum lies within twice the error bound of the smallest is listed (almost always one).
//   3. the listed groups' codewords are gone through in fp32 on the vector ALUs (rows read from LDS).  Again
//      everything within the bound is listed: one candidate (all but about one sub-vector in two thousand) is the
//      nearest codeword for certain; several are settled by fp64 distances, lowest index on ties, so the code equals
//      an fp64 exhaustive search.  Where no sub-vector of the wave has more than two, they are noted on the way (one search in
//      thirty; going through the lists again for them held up the workgroup, and the launch waits for its slowest one:
//      64 tokens x 8 sequences x 8 heads 10.2 -> 8.9 us, 8 x 8192 tokens 580 -> 562 us, a K-Means iteration of 2^20
//      8-dim samples 3 us less).
// Groups of 8 against 16: twice the minima in step 2 (+56 instructions), half the rows in step 3 (-48 for 4-dim, -80 for
// 8-dim codewords, and half the LDS reads).
// LEAN is the form for three waves per SIMD (168 registers): no tile is requested ahead (the other waves fill the wait), the
// 8-dim second operands are read from LDS, the 4-dim rows of step 3 are fp16 (half the reads) and the first listed group needs
// no loop.
#pragma once

#include <type_traits>

#include "nsn_device.h"

namespace nsn {

typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));

// v_permlane32_swap: the upper half of `a` changes places with the lower half of `b` (v_permlane16_swap: odd 16-lane
// rows of `a` with even rows of `b`).  Written as instructions because the compiler's two-result builtins have
// returned the first result twice; they read other lanes' registers, which needs two idle cycles after the
// vector instruction that wrote them.  So does a matrix instruction that reads a swapped register: the compiler keeps that
// distance behind its own vector instructions but not behind asm, so the operand_ forms end with the two cycles.
__device__ __forceinline__ void operand_swap32(uint32_t& a, uint32_t& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
template <typename T>
__device__ __forceinline__ void swap32(T& a, T& b) {
  static_assert(sizeof(T) == 4, "one register each");
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// the largest of the wave's values, in every lane (no LDS traffic)
__device__ __forceinline__ float wave_max_lanes(float v) {
  v = fmaxf(v, xor_lane<1>(v)), v = fmaxf(v, xor_lane<2>(v)), v = fmaxf(v, xor_lane<4>(v)), v = fmaxf(v, xor_lane<8>(v));
  float a = v, b = v;
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  float c = fmaxf(a, b), d = c;
  swap32(c, d);
  return fmaxf(c, d);
}
// four pairs at a time: one wait for all of them
#define NSN_SWAP4(NAME, INSN, AFTER)                                                                              \
  template <typename T>                                                                                           \
  __device__ __forceinline__ void NAME(T& a0, T& b0, T& a1, T& b1, T& a2, T& b2, T& a3, T& b3) {                  \
    static_assert(sizeof(T) == 4, "one register each");                                                           \
    asm("s_nop 1\n\t" INSN " %0, %1\n\t" INSN " %2, %3\n\t" INSN " %4, %5\n\t" INSN " %6, %7" AFTER               \
        : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1), "+v"(a2), "+v"(b2), "+v"(a3), "+v"(b3));                        \
  }
NSN_SWAP4(swap32x4, "v_permlane32_swap_b32", "")
NSN_SWAP4(swap16x4, "v_permlane16_swap_b32", "")
NSN_SWAP4(operand_swap32x4, "v_permlane32_swap_b32", "\n\ts_nop 1")
#undef NSN_SWAP4

// Minima of the first N and of the other 16 - N results of a matrix instruction.  All results are positive, so their bit
// patterns order like integers: integer minima come without the operand canonicalisation that float minima have.
template <int N>
__device__ __forceinline__ void two_minima(const f16v& d, uint32_t& first, uint32_t& second) {
  auto u = [&](int i) { return __float_as_uint(d[i]); };
  auto min3 = [](uint32_t a, uint32_t b, uint32_t c) { return min(min(a, b), c); };
  first = u(0), second = u(N);
#pragma unroll
  for (int i = 1; i + 1 < N; i += 2) first = min3(first, u(i), u(i + 1));
  if (N % 2 == 0) first = min(first, u(N - 1));
#pragma unroll
  for (int i = N + 1; i + 1 < 16; i += 2) second = min3(second, u(i), u(i + 1));
  if (N % 2 == 0) second = min(second, u(15));
}

// A lane of half hf holds rows 8 (k / 4) + 4 hf + k % 4, k = 0..15, of 32 x 32 tile m: codewords 128 hf + 16 m + k.  Group
// 16 hf + 2 m is the first of them, the next group the others.
constexpr int kGroups = 32;
__host__ __device__ constexpr int row_codeword(int row) { return 128 * ((row >> 2) & 1) + 4 * (row >> 3) + (row & 3); }  // of tile 0

// LDS: -2 s c in fp32 (and, for codewords that are fp16 values, in fp16: half the reads of step 3; sixteen codewords and a
// gap, so that groups start in different banks) and ||s c||^2 group by group; s = the power of two that brings the longest
// codeword to norm [4, 8) (fp16 parts of any codebook then sit well inside the fp16 range).  `image`: the codeword-side operands
// of the matrix instructions, 16 bytes per codeword and lane half (without a gap between the halves' codewords: a 16-byte LDS
// read serves lanes 0..3 and 12..15 together, then the next eight such, and a gap of four made those collide).
template <int SUB, bool EXACT16, bool LEAN = false>
struct SearchTables {
  // 4-dim codewords: seven and nine to a group, which leaves no minimum with two operands (sixteen instructions fewer than
  // eight and eight, and six more for the ninth codeword, which a group of seven has from its neighbour: a candidate like all
  // others).  An 8-dim codeword takes ten.
  static constexpr int kFirst = SUB == 4 && LEAN ? 7 : 8, kGroupRows = 16 - kFirst;
  __host__ __device__ static constexpr int group_first(int g) { return 8 * g - (g & 1) * (8 - kFirst); }  // codeword
  __host__ __device__ static constexpr int row(int c) { return c + (c >> 4); }
  static constexpr int kNormStride = 12;  // floats per group
  static constexpr bool kHalfRows = EXACT16 && SUB == 4 && LEAN;
  static constexpr int kImages = SUB == 4 ? 2 : EXACT16 ? 1 : 3, kRows = kCodes + kCodes / 16;
  alignas(16) float4 n2c[SUB / 4][kRows];
  alignas(16) float cn[kGroups * kNormStride];  // (read sixteen bytes at a time: at eight-byte places 3 to 4 % of a small call)
  float n2max[4];
  alignas(16) _Float16 n2c16[kHalfRows ? kRows : 1][SUB];
  // 8-dim fp16 codewords: ||c||^2 in three parts and 1, and zeros for the upper half of the wave
  static constexpr int kZeros = kCodes;
  alignas(16) h4v norm_parts[EXACT16 && SUB == 8 ? kZeros + 7 * 16 + 1 : 1];
  alignas(16) h8 image[kImages][kCodes];
};

template <int SUB, bool EXACT16>
struct SearchRegs {
  h8 A[8];
  // SUB = 8: second operand; EXACT16 codewords (fp16 values) have no low part, ||c||^2 alone takes four slots.  (The other
  // form is read from LDS in every search: of the 256 registers at two waves per SIMD the ordered codebook kernels leave 18,
  // and this would take 32.)
  h4v A2[SUB == 8 && EXACT16 ? 8 : 1];
  float cm;     // largest norm of a scaled codeword, at least 4
  float scale;  // s
};

// Fills the tables and the operands of every wave of the workgroup (256 threads or more, all of them call it).
// get(i): element i of codeword `tid` (threads 0..255); n2: the largest squared norm of a codeword, in every thread (codewords that
// hold a NaN left out).  s is 2^ex_most at most: a caller that knows the longest sub-vector
// keeps it below 237 s this way.  Without that, sub-vectors 30 to 60 times as long as the longest codeword leave the fp16
// range and take 256 fp64 distances per wave (encoder, 4096 tokens x 8 heads with codewords a hundredth of the usual: 495 us
// instead of 54; K-Means of 2^20 samples whose first 256 are a fiftieth of the others: 100 to 270 us more in the first
// iteration; there the samples have no bound that one far value would not spoil).
template <int SUB, bool EXACT16, bool LEAN, typename F>
__device__ inline void search_setup(SearchTables<SUB, EXACT16, LEAN>& T, SearchRegs<SUB, EXACT16>& R, int tid, float n2, F get, int ex_most) {
  using Tables = SearchTables<SUB, EXACT16, LEAN>;
  typedef decltype(get(0)) real;
  const int lane = tid & 63;
  real own[SUB];
  if (tid < kCodes) {
#pragma unroll
    for (int i = 0; i < SUB; ++i) own[i] = get(i);
  }
  // s = 2^k with |c| s in [4, 8) for the longest codeword (1 for an empty or non-finite codebook)
  const float nm = sqrtf(n2);
  int ex = 0;
  if (nm > 0.f && nm < INFINITY) {
    (void)frexpf(nm, &ex);  // nm = f 2^ex, f in [1/2, 1)
    ex = min(max(3 - ex, -100), ex_most);
  }
  const float s = ldexpf(1.f, ex);
  R.scale = s;
  R.cm = nm * s * 1.0001f;
  if (R.cm < 4.f) R.cm = 4.f;  // (the error bound counts on 16 at least for (|c| + |y|)^2)
  if (tid < kCodes) {
    float cn = 0.f, f[SUB];
    h8 a0 = {}, a1 = {}, a2 = {};
    _Float16 hi[SUB], lo[SUB];
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      const real t = (real)-2 * (own[i] * (real)s);
      f[i] = (float)t;
      cn = fmaf(0.25f * f[i], f[i], cn);
      hi[i] = (_Float16)f[i];
      lo[i] = EXACT16 ? (_Float16)0.f : (_Float16)(float)(t - (real)(float)hi[i]);
    }
    // (the sum is pinned: folded into the conversion, one use of its fp16 value would be rounded from the unrounded sum
    // and the other from the fp32 one, and at a tie the parts would not add up)
    asm("" : "+v"(cn));
    _Float16 p[3];
    float rest = cn;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      p[k] = (_Float16)rest;
      rest -= (float)p[k];
    }
    if constexpr (SUB == 4) {  // k: -2c_hi (y_hi), -2c_hi (y_lo) | -2c_lo (y_hi), ||c||^2 in three parts, 1 (n)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a0[i] = a0[4 + i] = hi[i];
        a1[i] = lo[i];
        a1[4 + i] = i < 3 ? p[i < 3 ? i : 0] : (_Float16)1.f;
      }
      T.image[0][tid] = a0, T.image[1][tid] = a1;
    } else {  // -2c_hi (y_hi) | -2c_hi (y_lo); second operand: -2c_lo (y_hi) | parts of ||c||^2, 1 (n)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        a0[i] = hi[i], a1[i] = lo[i];
        a2[i] = i < 3 ? p[i < 3 ? i : 0] : (_Float16)(i == 3 ? 1.f : 0.f);
      }
      T.image[0][tid] = a0;
      if constexpr (EXACT16) {
        T.norm_parts[tid] = h4v{a2[0], a2[1], a2[2], a2[3]};
        if (tid <= 7 * 16) T.norm_parts[Tables::kZeros + tid] = h4v{};
      } else {
        T.image[1][tid] = a1, T.image[2][tid] = a2;
      }
    }
#pragma unroll
    for (int u = 0; u < SUB / 4; ++u)
      T.n2c[u][Tables::row(tid)] = make_float4(f[4 * u], f[4 * u + 1], f[4 * u + 2], f[4 * u + 3]);
    if constexpr (Tables::kHalfRows) {  // (a0 begins with them)
      typedef _Float16 row_t __attribute__((ext_vector_type(SUB)));
      row_t r;
#pragma unroll
      for (int i = 0; i < SUB; ++i) r[i] = a0[i];
      *reinterpret_cast<row_t*>(T.n2c16[Tables::row(tid)]) = r;
    }
    const int k = tid & 15;
    float* const cn_of = &T.cn[(tid >> 4) * 2 * Tables::kNormStride];
    const int in_first = k, in_second = Tables::kNormStride + k - Tables::kFirst;
    cn_of[k < Tables::kGroupRows ? in_first : in_second] = cn;
    if constexpr (Tables::kFirst == 7) cn_of[k >= 7 ? in_second : in_first] = cn;  // (7 and 8 are in both)
  }
  __syncthreads();
  const int row = row_codeword(lane & 31), half = lane >> 5;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    if constexpr (SUB == 4) {
      R.A[m] = T.image[half][16 * m + row];
    } else {
      R.A[m] = T.image[0][16 * m + row];
      if constexpr (EXACT16) R.A2[m] = T.norm_parts[16 * m + (half ? Tables::kZeros : row)];
    }
  }
}

// the same where a thread has only its own codeword at hand
template <int SUB, bool EXACT16, bool LEAN, typename F>
__device__ inline void search_setup(SearchTables<SUB, EXACT16, LEAN>& T, SearchRegs<SUB, EXACT16>& R, int tid, F get, int ex_most = 100) {
  float n2 = 0.f;
  if (tid < kCodes) {  // (whole waves)
#pragma unroll
    for (int i = 0; i < SUB; ++i) n2 = fmaf((float)get(i), (float)get(i), n2);
    n2 = wave_max_lanes(n2);
    if ((tid & 63) == 0) T.n2max[tid >> 6] = n2;
  }
  __syncthreads();
  search_setup<SUB, EXACT16, LEAN>(T, R, tid, fmaxf(fmaxf(T.n2max[0], T.n2max[1]), fmaxf(T.n2max[2], T.n2max[3])), get, ex_most);
}

__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, h2v));
}
__device__ __forceinline__ h8 words_h8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  typedef uint32_t u4v __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(h8, u4v{a, b, c, d});
}

// The codeword nearest to y / R.scale (this lane's sub-vector); all 64 lanes take part.  exact(c): fp64 squared
// distance of the lane's sub-vector to codeword c, in any unit.
// AHEAD: a tile's products are requested a whole tile before its minima are taken (32 more registers).
template <int SUB, bool EXACT16, bool AHEAD, bool LEAN, typename F>
__device__ __forceinline__ int search_nearest(const SearchTables<SUB, EXACT16, LEAN>& T, const SearchRegs<SUB, EXACT16>& R,
                                              const float (&y)[SUB], F exact) {
  using Tables = SearchTables<SUB, EXACT16, LEAN>;
  constexpr int NP = SUB / 2;
  float yn = 0.f;
#pragma unroll
  for (int i = 0; i < SUB; ++i) yn = fmaf(y[i], y[i], yn);
  uint32_t hi[NP], lo[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    hi[i] = pack_f16(y[2 * i], y[2 * i + 1]);
    const h2v h = __builtin_bit_cast(h2v, hi[i]);
    lo[i] = pack_f16(y[2 * i] - (float)h[0], y[2 * i + 1] - (float)h[1]);
  }
  const bool lower = (threadIdx.x & 32) == 0;
  // n: an fp16 value above ||y||^2 by more than any error of D (the same for all codewords: it decides nothing)
  const float n = fmaf(yn, 1.0f + 0x1p-8f, 0x1p-5f);
  constexpr uint32_t ONE1 = 0x3C003C00u;  // (1, 1)
  uint32_t one_n = pack_f16(1.f, n);
  // (by the instruction's own rounding: the value subtracted below is the one that was added)
  const float n16 = (float)__builtin_bit_cast(h2v, one_n)[1];
  // operands of the two column sets: a = the sub-vectors of lanes 0..31, b = those of lanes 32..63
  h8 ba, bb, ba2 = {}, bb2 = {};
  h4v na = {}, nb = {};
  if constexpr (SUB == 4) {
    uint32_t k0 = hi[0], k1 = hi[1], k2 = ONE1;
    operand_swap32x4(hi[0], k0, hi[1], k1, lo[0], k2, lo[1], one_n);
    ba = words_h8(hi[0], hi[1], lo[0], lo[1]);
    bb = words_h8(k0, k1, k2, one_n);
  } else {
    operand_swap32x4(hi[0], lo[0], hi[1], lo[1], hi[2], lo[2], hi[3], lo[3]);
    ba = words_h8(hi[0], hi[1], hi[2], hi[3]);
    bb = words_h8(lo[0], lo[1], lo[2], lo[3]);
    uint32_t one_nb = one_n;
    operand_swap32(one_n, one_nb);  // n of the set's column in either half of the wave
    if constexpr (EXACT16) {
      typedef uint32_t u2v __attribute__((ext_vector_type(2)));
      na = __builtin_bit_cast(h4v, u2v{ONE1, one_n}), nb = __builtin_bit_cast(h4v, u2v{ONE1, one_nb});
    } else {
      ba2 = words_h8(lower ? hi[0] : ONE1, lower ? hi[1] : one_n, lower ? hi[2] : 0u, lower ? hi[3] : 0u);
      bb2 = words_h8(lower ? lo[0] : ONE1, lower ? lo[1] : one_nb, lower ? lo[2] : 0u, lower ? lo[3] : 0u);
    }
  }
  uint32_t a0[8], a1[8], b0[8], b1[8];  // minima of the two groups of tile m held by this lane, sets a and b
  constexpr bool kFromLds = SUB == 8 && !EXACT16, kPartsFromLds = SUB == 8 && EXACT16 && LEAN;
  int second = row_codeword((int)(threadIdx.x & 31));
  if constexpr (EXACT16)
    second = lower ? second : Tables::kZeros;
  else
    second += kCodes * (1 + (int)((threadIdx.x >> 5) & 1));
  if constexpr (SUB == 8) asm volatile("" : "+v"(second));  // (keeps the reads of the second operand inside the search)
  auto second_operand = [&](int m) -> h8 {
    if constexpr (kFromLds) return (&T.image[0][0])[second + 16 * m];
    return h8{};
  };
  const f16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // a tile's product with 8-dim codewords is two matrix instructions, the second on the result of the first
  auto first_half = [&](int m, const h8& s2, const h8& y2, const h4v& nn) -> f16v {
    if constexpr (SUB == 8 && EXACT16)
      return __builtin_amdgcn_mfma_f32_32x32x8f16(kPartsFromLds ? T.norm_parts[second + 16 * m] : R.A2[m], nn, zero, 0, 0, 0);
    else if constexpr (SUB == 8)
      return __builtin_amdgcn_mfma_f32_32x32x16_f16(s2, y2, zero, 0, 0, 0);
    return zero;
  };
  auto second_half = [&](int m, const h8& y1, const f16v& d) -> f16v {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A[m], y1, d, 0, 0, 0);
  };
  auto tile = [&](int m, const h8& s2, const h8& y1, const h8& y2, const h4v& nn) -> f16v {
    return second_half(m, y1, first_half(m, s2, y2, nn));
  };
  // A result takes eleven issue slots, the minima of one set eight: left to itself the compiler puts them next to
  // each other and waits.
  if constexpr (AHEAD && kFromLds) {
    // The second operand of a tile is read a tile ahead of its products, and the first halves of both sets go out before
    // either's second, which would wait for it: a K-Means iteration of 2^20 8-dim samples 32.7 -> 31.2 us.  (In the encoder,
    // where the second operands are in registers, the longer lives cost as much as the waits.)
    h8 s_now = second_operand(0), s_next = second_operand(1);
    __builtin_amdgcn_sched_barrier(0);
    f16v ea = first_half(0, s_now, ba2, na), eb = first_half(0, s_now, bb2, nb);
    f16v da = second_half(0, ba, ea), db = second_half(0, bb, eb);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      s_now = s_next;
      __builtin_amdgcn_sched_barrier(0);
      if (m < 7) ea = first_half(m + 1, s_now, ba2, na), eb = first_half(m + 1, s_now, bb2, nb);
      __builtin_amdgcn_sched_barrier(0);
      if (m < 6) s_next = second_operand(m + 2);
      two_minima<Tables::kFirst>(da, a0[m], a1[m]);
      __builtin_amdgcn_sched_barrier(0);
      if (m < 7) da = second_half(m + 1, ba, ea);
      __builtin_amdgcn_sched_barrier(0);
      two_minima<Tables::kFirst>(db, b0[m], b1[m]);
      __builtin_amdgcn_sched_barrier(0);
      if (m < 7) db = second_half(m + 1, bb, eb);
    }
    __builtin_amdgcn_sched_barrier(0);
  } else if constexpr (AHEAD) {
    f16v da = tile(0, h8{}, ba, ba2, na), db = tile(0, h8{}, bb, bb2, nb);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      f16v da_next, db_next;
      __builtin_amdgcn_sched_barrier(0);
      if (m < 7) da_next = tile(m + 1, h8{}, ba, ba2, na);
      __builtin_amdgcn_sched_barrier(0);
      two_minima<Tables::kFirst>(da, a0[m], a1[m]);
      __builtin_amdgcn_sched_barrier(0);
      if (m < 7) db_next = tile(m + 1, h8{}, bb, bb2, nb);
      __builtin_amdgcn_sched_barrier(0);
      two_minima<Tables::kFirst>(db, b0[m], b1[m]);
      if (m < 7) da = da_next, db = db_next;
    }
    __builtin_amdgcn_sched_barrier(0);
  } else {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const h8 s2 = second_operand(m);
      two_minima<Tables::kFirst>(tile(m, s2, ba, ba2, na), a0[m], a1[m]);
      two_minima<Tables::kFirst>(tile(m, s2, bb, bb2, nb), b0[m], b1[m]);
    }
  }
  // The minima stay where they are: a lane holds those of its half's groups for one sub-vector of either column set.  What
  // crosses the halves is the smallest of each set, the thresholds and the lists (a swap each, against sixteen for all minima).
  uint32_t best_a = min(a0[0], a1[0]), best_b = min(b0[0], b1[0]);
#pragma unroll
  for (int m = 1; m < 8; ++m) best_a = min(min(best_a, a0[m]), a1[m]), best_b = min(min(best_b, b0[m]), b1[m]);
  swap32(best_a, best_b);
  const float best = __uint_as_float(min(best_a, best_b));
  // Error bound of either form of a distance, relative to M >= (|c| + |y|)^2, in units of 2^-24: the fp16 splits of
  // y and c leave 4 each (two roundings of 2^-11), the dropped low x low product 4, low parts below the normal fp16
  // range 2 (M >= 16), fp32 rounding of the inputs and of the threshold 3, the sum of at most 32 terms 24 (matrix cores)
  // or SUB + 3 (fp32).  (fp16 rows of step 3 are exact but for elements below the fp16 subnormal unit once scaled: at most
  // 2^-25 |y|_1, less than one unit of the bound.)  Anything that can be nearest lies within twice the bound of the computed
  // minimum.
  const float reach = R.cm + 1.0001f * __builtin_amdgcn_sqrtf(yn);
  // (beyond the fp16 range - ||y||^2 above 58000 -, a codebook that is not finite, or not a number: nothing is listed)
  const bool in_range = reach < 245.f;
  const float thr_n = in_range ? fmaf(2.f * 44.f * 5.9604645e-8f * reach, reach, best) : -INFINITY;  // for D (with n in it)
  const float thr = thr_n - n16;                                                                     // for the fp32 form
  float thr_a = thr_n, thr_b = thr_n;
  swap32(thr_a, thr_b);  // of sets a and b, in both halves
  uint32_t list_a = 0u, list_b = 0u;
  auto below = [](uint32_t t, float thr) { return __float_as_uint(__uint_as_float(t) - thr); };  // sign bit set: listed
#pragma unroll
  for (int m = 7; m >= 0; --m) {
    list_a = __builtin_amdgcn_alignbit(list_a, below(a1[m], thr_a), 31);
    list_b = __builtin_amdgcn_alignbit(list_b, below(b1[m], thr_b), 31);
    list_a = __builtin_amdgcn_alignbit(list_a, below(a0[m], thr_a), 31);
    list_b = __builtin_amdgcn_alignbit(list_b, below(b0[m], thr_b), 31);
  }
  swap32(list_a, list_b);  // of the own sub-vector: lower, upper half of the groups
  const uint32_t groups = in_range ? list_a | list_b << 16 : 0u;
  // rows of group g within the bound, as a bit mask
  auto rows_of = [&](int g) -> uint32_t {
    const int first = Tables::row(Tables::group_first(g));
    const float* n = &T.cn[g * Tables::kNormStride];
    const float4 n0 = reinterpret_cast<const float4*>(n)[0], n1 = reinterpret_cast<const float4*>(n)[1];
    float cnv[9] = {n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, n1.z, n1.w};
    if constexpr (Tables::kGroupRows == 9) cnv[8] = n[8];
    uint32_t mask = 0u;
#pragma unroll
    for (int k = Tables::kGroupRows - 1; k >= 0; --k) {
      float c[SUB];
      if constexpr (Tables::kHalfRows) {
        typedef _Float16 row_t __attribute__((ext_vector_type(SUB)));
        const row_t r = *reinterpret_cast<const row_t*>(T.n2c16[first + k]);
#pragma unroll
        for (int i = 0; i < SUB; ++i) c[i] = (float)r[i];
      } else {
#pragma unroll
        for (int u = 0; u < SUB / 4; ++u) {
          const float4 r = T.n2c[u][first + k];
          c[4 * u] = r.x, c[4 * u + 1] = r.y, c[4 * u + 2] = r.z, c[4 * u + 3] = r.w;
        }
      }
      float d = cnv[k] - thr;
#pragma unroll
      for (int i = 0; i < SUB; ++i) d = fmaf(c[i], y[i], d);
      mask = __builtin_amdgcn_alignbit(mask, __float_as_uint(d), 31);
    }
    return mask;
  };
  constexpr unsigned kListed = 32;  // candidates of a sub-vector that are settled by its lists
  int code = 0, code_before = 0, found = 0;  // the first candidate of the last group that holds any, and of the one before it
  uint32_t rows_at = 0u;                      // the candidates of the last such group
  auto take_group = [&](int g, uint32_t rows) {
    if (rows) code_before = code, rows_at = rows, code = Tables::group_first(g) + __builtin_ctz(rows);
    found += __builtin_popcount(rows);
  };
  uint32_t left = groups;
  if constexpr (LEAN) {  // every list holds a group, but for lanes out of range, where the last group stands in and nothing is taken
    const int g = __builtin_ctz(left | 0x80000000u);
    rows_at = rows_of(g);
    code = code_before = Tables::group_first(g) + __builtin_ctz(rows_at | 0x80000000u);
    found = left ? __builtin_popcount(rows_at) : 0;
    left &= left - 1u;
    for (; __any(left != 0u); left &= left - 1u) {
      const int gn = left ? __builtin_ctz(left) : 0;
      take_group(gn, left ? rows_of(gn) : 0u);
    }
  } else {
    do {
      const int g = left ? __builtin_ctz(left) : 0;
      take_group(g, left ? rows_of(g) : 0u);
      left &= left - 1u;
    } while (__any(left != 0u));
  }
  if (!__any(found != 1)) return code;
  if (!__any((unsigned)(found - 1) > 1u)) {
    // two candidates (one search of a wave in thirty holds such a sub-vector, mostly one): they are at hand
    if (found == 2) {
      const uint32_t other = rows_at & (rows_at - 1u);
      const int code2 = other ? code - __builtin_ctz(rows_at) + __builtin_ctz(other) : code_before;
      const double d = exact(code), d2 = exact(code2);
      // (a codeword that holds a NaN is listed with its group where the sign bit is set: it is never the nearest)
      if (d2 < d || d != d || (d2 == d && code2 < code)) code = code2;
    }
  } else {
    // None at all (not a number somewhere, or out of range): all codewords.  In the codebook's instances, whose samples have no
    // bound, more than kListed too, and then for the whole wave, which reads the rows together and not through lists that differ
    // from lane to lane.  (Samples a thousandth of the longest codeword list many groups: K-Means of 2^20 8-dim samples with an
    // outlier of 1000, twelve iterations, 5.2 -> 4.0 ms, 2^16 4-dim ones 0.74 -> 0.51 ms; with 8 or 16 for kListed an outlier of 300
    // takes up to 1.5 times as long.  The encoder's sub-vectors have a bound; there the wider condition cost 0.5 % of a prefill.)
    double e1 = INFINITY;
    int k1 = 0;
    const bool all = EXACT16 ? found < 1 : __any((unsigned)(found - 1) >= kListed);
    left = found > 1 && !all ? groups : 0u;
    while (__any(left != 0u)) {
      const int g = left ? __builtin_ctz(left) : 0;
      uint32_t rows = left ? rows_of(g) : 0u;
      while (__any(rows != 0u)) {
        if (rows) {
          const int c = Tables::group_first(g) + __builtin_ctz(rows);
          const double d = exact(c);
          if (d < e1 || (d == e1 && c < k1)) e1 = d, k1 = c;
        }
        rows &= rows - 1u;
      }
      left &= left - 1u;
    }
    if (all && found != 1) {
      auto take = [&](int c) {
        const double d = exact(c);
        if (d < e1) e1 = d, k1 = c;
      };
      if constexpr (EXACT16) {
        for (int c = 0; c < kCodes; ++c) take(c);
      } else {
#pragma unroll 2  // (four at once want registers that the ordered 4-dim kernel does not have)
        for (int c = 0; c < kCodes; ++c) take(c);
      }
    }
    if (found != 1) code = k1;
  }
  return code;
}

}  // namespace nsn
