// Nearest-codeword search (Eq. 1, squared Euclidean distance): one sub-vector per lane, 64 per call.
//
// Three steps, bound by vector instructions (about 300 per 64 searches of 256 codewords; keeping the best two
// indexed keys of every distance, the form this one replaced, took about 740):
//   1. matrix cores: D = ||c||^2 - 2 c . y for 32 codewords (rows) x 32 sub-vectors (columns) at a time.  y, c and
//      ||c||^2 enter as sums of fp16 parts, so D is good to about 2^-20 of (|c|^2 + 2 |c| |y|).  A lane
//      then holds 16 distances of one sub-vector per tile and keeps only their minimum: half an instruction per
//      distance (three-operand minima), no index bookkeeping.  16 groups of 16 codewords leave 16 minima per
//      sub-vector, brought to the lane that owns it by half-wave swaps.
//   2. every group whose minimum lies within twice the error bound of the smallest is listed (almost always one).
//   3. the listed groups' codewords are gone through in fp32 on the vector ALUs (rows read from LDS, padded so
//      that 16 different groups sit in 16 different bank quads: conflict-free for any choice of groups).  Again
//      everything within the bound is listed: one candidate (all but about one sub-vector in a thousand) is the
//      nearest codeword for certain; several are settled by fp64 distances, lowest index on ties, so the code equals
//      an fp64 exhaustive search.
// Groups of 16 balance the two sides: groups of 8 cost as much in step 2 as they save in step 3.
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
// vector instruction that wrote them.
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// four pairs at a time: one wait for all of them
#define NSN_SWAP4(NAME, INSN)                                                                                     \
  template <typename T>                                                                                           \
  __device__ __forceinline__ void NAME(T& a0, T& b0, T& a1, T& b1, T& a2, T& b2, T& a3, T& b3) {                  \
    static_assert(sizeof(T) == 4, "one register each");                                                           \
    asm("s_nop 1\n\t" INSN " %0, %1\n\t" INSN " %2, %3\n\t" INSN " %4, %5\n\t" INSN " %6, %7"                     \
        : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1), "+v"(a2), "+v"(b2), "+v"(a3), "+v"(b3));                        \
  }
NSN_SWAP4(swap32x4, "v_permlane32_swap_b32")
NSN_SWAP4(swap16x4, "v_permlane16_swap_b32")
#undef NSN_SWAP4

// The plain instruction: fminf() would add an operand canonicalisation per operand (no NaN can decide anything here:
// a sub-vector without exactly one candidate goes through the fp64 path).
__device__ __forceinline__ float min3f(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// Minimum of the sixteen results of a matrix instruction.  The first step is an instruction the compiler knows, so that
// it waits for the matrix pipe; every other one takes its result as an operand and so comes after it.
__device__ __forceinline__ float min16(const f16v& d) {
  const float x = __builtin_amdgcn_fmed3f(d[0], d[1], -INFINITY);
  float p = min3f(x, d[2], d[3]), q = min3f(x, d[8], d[9]);
  p = min3f(p, d[4], d[5]), q = min3f(q, d[10], d[11]);
  p = min3f(p, d[6], d[7]), q = min3f(q, d[12], d[13]);
  return min3f(min3f(q, d[14], d[15]), p, p);
}

// group g = 2 tile + half, row r of it <-> codeword (the rows a lane of that half holds of a 32 x 32 tile)
__host__ __device__ constexpr int group_codeword(int g, int r) {
  return 32 * (g >> 1) + 8 * (r >> 2) + 4 * (g & 1) + (r & 3);
}
__host__ __device__ constexpr int codeword_group(int c) { return 2 * (c >> 5) + ((c >> 2) & 1); }
__host__ __device__ constexpr int codeword_row(int c) { return 4 * ((c >> 3) & 3) + (c & 3); }

// LDS: -2 s c and ||s c||^2 in fp32, group by group; s = the power of two that brings the longest codeword to
// norm [4, 8) (fp16 parts of any codebook then sit well inside the fp16 range).
template <int SUB>
struct SearchTables {
  static constexpr int kRowStride = 17;   // 16-byte units per group of 16 rows
  static constexpr int kNormStride = 20;  // floats per group
  float4 n2c[SUB / 4][16 * kRowStride];
  float cn[16 * kNormStride];
};

template <int SUB, bool EXACT16>
struct SearchRegs {
  h8 A[8];
  // SUB = 8: second operand; EXACT16 codewords (fp16 values) have no low part, ||c||^2 alone takes four slots
  typename std::conditional<EXACT16, h4v, h8>::type A2[SUB == 8 ? 8 : 1];
  float cm;     // largest norm of a scaled codeword
  float scale;  // s
};

// Fills the tables and the operands of every wave of the workgroup (256 threads or more).  get(c, i): element i of
// codeword c.  No barrier inside: the caller puts one between this and the first search.
template <int SUB, bool EXACT16, typename F>
__device__ inline void search_setup(SearchTables<SUB>& T, SearchRegs<SUB, EXACT16>& R, int tid, F get) {
  typedef decltype(get(0, 0)) real;
  const int lane = tid & 63, row = lane & 31;
  real e[8][SUB];
#pragma unroll
  for (int m = 0; m < 8; ++m)
#pragma unroll
    for (int i = 0; i < SUB; ++i) e[m][i] = get(32 * m + row, i);
  real own[SUB];
  if (tid < kCodes) {
#pragma unroll
    for (int i = 0; i < SUB; ++i) own[i] = get(tid, i);
  }
  float n2max = 0.f;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    float n2 = 0.f;
#pragma unroll
    for (int i = 0; i < SUB; ++i) n2 = fmaf((float)e[m][i], (float)e[m][i], n2);
    n2max = fmaxf(n2max, n2);
  }
  n2max = wave_max(n2max);
  // s = 2^k with |c| s in [4, 8) for the longest codeword (1 for an empty or non-finite codebook)
  int ex = 0;
  const float nm = sqrtf(n2max);
  if (nm > 0.f && nm < INFINITY) {
    (void)frexpf(nm, &ex);  // nm = f 2^ex, f in [1/2, 1)
    ex = min(max(3 - ex, -100), 100);
  }
  const float s = ldexpf(1.f, ex);
  R.scale = s;
  R.cm = nm * s * 1.0001f;
  auto parts = [](float cn, _Float16 (&p)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      p[k] = (_Float16)cn;
      cn -= (float)p[k];
    }
  };
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    float cn = 0.f;
    _Float16 hi[SUB], lo[SUB];
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      const real c = e[m][i] * (real)s;
      cn = fmaf((float)c, (float)c, cn);
      const real t = (real)-2 * c;
      hi[i] = (_Float16)(float)t;
      lo[i] = EXACT16 ? (_Float16)0.f : (_Float16)(float)(t - (real)(float)hi[i]);
    }
    _Float16 p[3];
    parts(cn, p);
    const bool lower = lane < 32;
    h8 a;
    if constexpr (SUB == 4) {  // k: -2c_hi (y_hi), -2c_hi (y_lo) | -2c_lo (y_hi), ||c||^2 in three parts, 0
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = lower ? hi[i] : lo[i];
        a[4 + i] = lower ? hi[i] : (i < 3 ? p[i < 3 ? i : 0] : (_Float16)0.f);
      }
      R.A[m] = a;
    } else {  // -2c_hi (y_hi) | -2c_hi (y_lo); second operand: -2c_lo (y_hi) | parts of ||c||^2
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] = hi[i];
      R.A[m] = a;
      if constexpr (EXACT16) {
        h4v b;
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = (lower && i < 3) ? p[i < 3 ? i : 0] : (_Float16)0.f;
        R.A2[m] = b;
      } else {
        h8 b;
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = lower ? lo[i] : (i < 3 ? p[i < 3 ? i : 0] : (_Float16)0.f);
        R.A2[m] = b;
      }
    }
  }
  if (tid < kCodes) {
    const int g = codeword_group(tid), r = codeword_row(tid);
    float cn = 0.f, f[SUB];
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      const float c = (float)(own[i] * (real)s);
      cn = fmaf(c, c, cn);
      f[i] = -2.f * c;
    }
#pragma unroll
    for (int u = 0; u < SUB / 4; ++u)
      T.n2c[u][g * SearchTables<SUB>::kRowStride + r] = make_float4(f[4 * u], f[4 * u + 1], f[4 * u + 2], f[4 * u + 3]);
    T.cn[g * SearchTables<SUB>::kNormStride + r] = cn;
  }
}

__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, h2v));
}
__device__ __forceinline__ h8 words_h8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  typedef uint32_t u4v __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(h8, u4v{a, b, c, d});
}

// Index of the codeword nearest to y (this lane's sub-vector); all 64 lanes take part.  exact(c): fp64 squared
// distance of the lane's sub-vector to codeword c.
template <int SUB, bool EXACT16, typename F>
__device__ __forceinline__ int search_nearest(const SearchTables<SUB>& T, const SearchRegs<SUB, EXACT16>& R,
                                              const float (&y_in)[SUB], F exact) {
  constexpr int NP = SUB / 2;
  float y[SUB], yn = 0.f;
#pragma unroll
  for (int i = 0; i < SUB; ++i) {
    y[i] = y_in[i] * R.scale;
    yn = fmaf(y[i], y[i], yn);
  }
  uint32_t hi[NP], lo[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    hi[i] = pack_f16(y[2 * i], y[2 * i + 1]);
    const h2v h = __builtin_bit_cast(h2v, hi[i]);
    lo[i] = pack_f16(y[2 * i] - (float)h[0], y[2 * i + 1] - (float)h[1]);
  }
  const bool lower = (threadIdx.x & 32) == 0;
  constexpr uint32_t ONE1 = 0x3C003C00u, ONE0 = 0x00003C00u;  // (1, 1) and (1, 0)
  // operands of the two column sets: a = the sub-vectors of lanes 0..31, b = those of lanes 32..63
  h8 ba, bb, ba2, bb2;
  h4v ones4;
  if constexpr (SUB == 4) {
    uint32_t k0 = hi[0], k1 = hi[1], k2 = ONE1, k3 = ONE0;
    swap32x4(hi[0], k0, hi[1], k1, lo[0], k2, lo[1], k3);
    ba = words_h8(hi[0], hi[1], lo[0], lo[1]);
    bb = words_h8(k0, k1, k2, k3);
  } else {
    swap32x4(hi[0], lo[0], hi[1], lo[1], hi[2], lo[2], hi[3], lo[3]);
    ba = words_h8(hi[0], hi[1], hi[2], hi[3]);
    bb = words_h8(lo[0], lo[1], lo[2], lo[3]);
    if constexpr (EXACT16) {
      ones4 = h4v{(_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)0.f};
    } else {
      ba2 = words_h8(lower ? hi[0] : ONE1, lower ? hi[1] : ONE0, lower ? hi[2] : 0u, lower ? hi[3] : 0u);
      bb2 = words_h8(lower ? lo[0] : ONE1, lower ? lo[1] : ONE0, lower ? lo[2] : 0u, lower ? lo[3] : 0u);
    }
  }
  float ta[8], tb[8];
  const f16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    f16v da, db;
    if constexpr (SUB == 4) {
      da = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A[m], ba, zero, 0, 0, 0);
      db = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A[m], bb, zero, 0, 0, 0);
    } else if constexpr (EXACT16) {  // ||c||^2 is the same for every column: once for both sets
      const f16v d0 = __builtin_amdgcn_mfma_f32_32x32x8f16(R.A2[m], ones4, zero, 0, 0, 0);
      da = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A[m], ba, d0, 0, 0, 0);
      db = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A[m], bb, d0, 0, 0, 0);
    } else {
      da = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A2[m], ba2, zero, 0, 0, 0);
      db = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A2[m], bb2, zero, 0, 0, 0);
      da = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A[m], ba, da, 0, 0, 0);
      db = __builtin_amdgcn_mfma_f32_32x32x16_f16(R.A[m], bb, db, 0, 0, 0);
    }
    ta[m] = min16(da);
    tb[m] = min16(db);
  }
  // own sub-vector: ta[m] becomes the minimum of group 2m, tb[m] that of group 2m + 1
  swap32x4(ta[0], tb[0], ta[1], tb[1], ta[2], tb[2], ta[3], tb[3]);
  swap32x4(ta[4], tb[4], ta[5], tb[5], ta[6], tb[6], ta[7], tb[7]);
  float best = min3f(ta[0], tb[0], ta[1]);
  best = min3f(best, tb[1], ta[2]);
  best = min3f(best, tb[2], ta[3]);
  best = min3f(best, tb[3], ta[4]);
  best = min3f(best, tb[4], ta[5]);
  best = min3f(best, tb[5], ta[6]);
  best = min3f(best, tb[6], ta[7]);
  best = min3f(best, tb[7], tb[7]);
  // Error bound of either form of a distance, relative to M >= ||c||^2 + 2 |c| |y|, in units of 2^-24: the fp16 splits of
  // y and c leave 4 each (two roundings of 2^-11), the dropped low x low product 4, low parts below the normal fp16
  // range 2 (M >= 16), fp32 rounding of the inputs 2, the sum of at most 32 terms 24 (matrix cores) or SUB + 3
  // (fp32).  Anything that can be nearest lies within twice the bound of the computed minimum.
  const float M = R.cm * (R.cm + 2.0002f * __builtin_amdgcn_sqrtf(yn));
  const float thr = fmaf(2.f * 44.f * 5.9604645e-8f, M, best);
  uint32_t groups = 0u;
#pragma unroll
  for (int m = 7; m >= 0; --m) {
    groups = __builtin_amdgcn_alignbit(groups, __float_as_uint(tb[m] - thr), 31);
    groups = __builtin_amdgcn_alignbit(groups, __float_as_uint(ta[m] - thr), 31);
  }
  if (!(yn < 1e9f)) groups = 0u;  // beyond the fp16 range (or not a number): fp64 search below
  // rows of group g within the bound, as a bit mask
  auto rows_of = [&](int g) -> uint32_t {
    const float4* r0 = &T.n2c[0][g * SearchTables<SUB>::kRowStride];
    const float4* r1 = &T.n2c[SUB / 4 - 1][g * SearchTables<SUB>::kRowStride];
    const float4* n = reinterpret_cast<const float4*>(&T.cn[g * SearchTables<SUB>::kNormStride]);
    uint32_t mask = 0u;
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      const float4 cn4 = n[u];
      const float cnv[4] = {cn4.x, cn4.y, cn4.z, cn4.w};
#pragma unroll
      for (int k = 3; k >= 0; --k) {
        const float4 c = r0[4 * u + k];
        float d = cnv[k] - thr;
        d = fmaf(c.x, y[0], d), d = fmaf(c.y, y[1], d), d = fmaf(c.z, y[2], d), d = fmaf(c.w, y[3], d);
        if constexpr (SUB == 8) {
          const float4 e = r1[4 * u + k];
          d = fmaf(e.x, y[4], d), d = fmaf(e.y, y[5], d), d = fmaf(e.z, y[6], d), d = fmaf(e.w, y[7], d);
        }
        mask = __builtin_amdgcn_alignbit(mask, __float_as_uint(d), 31);
      }
    }
    return mask;
  };
  int code = 0, found = 0;
  {
    uint32_t left = groups;
    do {
      const int g = left ? __builtin_ctz(left) : 0;
      const uint32_t rows = left ? rows_of(g) : 0u;
      if (rows) code = group_codeword(g, __builtin_ctz(rows));
      found += __builtin_popcount(rows);
      left &= left - 1u;
    } while (__any(left != 0u));
  }
  if (__any(found != 1)) {  // (none at all: not a number somewhere, or out of range)
    double e1 = INFINITY;
    int k1 = 0;
    uint32_t left = found > 1 ? groups : 0u;
    while (__any(left != 0u)) {
      const int g = left ? __builtin_ctz(left) : 0;
      uint32_t rows = left ? rows_of(g) : 0u;
      while (__any(rows != 0u)) {
        if (rows) {
          const int c = group_codeword(g, __builtin_ctz(rows));
          const double d = exact(c);
          if (d < e1 || (d == e1 && c < k1)) e1 = d, k1 = c;
        }
        rows &= rows - 1u;
      }
      left &= left - 1u;
    }
    if (found < 1) {
      for (int c = 0; c < kCodes; ++c) {
        const double d = exact(c);
        if (d < e1) e1 = d, k1 = c;
      }
    }
    if (found != 1) code = k1;
  }
  return code;
}

}  // namespace nsn
