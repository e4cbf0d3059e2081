// Decode attention over the coded cache (App. B) for the tiled code layout: the gfx950 kernel.
//
// Arithmetic (per query head): score_t = scale (a^k_t HT(q) . C[codes^k_t] + b^k_t q . o^k_g),
// p = softmax(score), out = H^T sum_t p_t a^v_t C[codes^v_t] + sum_g (sum_{t in g} p_t b^v_t) o^v_g.
//
// How the 64 tokens of a group map onto a wave (lane = 16 c + n, c = 0..3, n = 0..15):
//   * scores: v_mfma_f32_16x16x32_f16 with the gathered KEY CODEWORDS as the A operand (row = token
//     16 tile + n of the group, the lane's eight k-slots = the eight channels it gathered: lane group c
//     owns channels [32 c, 32 c + 32)) and the rotated query as the B operand.  The sixteen columns carry
//     four heads x (fp16 hi part, fp16 lo part) x two tiles: tile parity p uses columns [4p, 4p+4) for hi
//     and [8+4p, 12+4p) for lo, all other columns of that B operand are zero, so two tiles accumulate
//     into one result and four k-steps x four tiles = sixteen matrix instructions give a group's scores
//     with ~22 significant bits of the query.  Adding column n and column n ^ 8 leaves, in lane
//     (rho = lane / 16, n): tile n / 4, head n % 4, tokens 16 tile + 4 rho + {0,1,2,3}.
//   * softmax per lane (one head, four tokens), running max kept lazily (rescale only when a score
//     exceeds it by 2^5), in log2 units.
//   * values: that register IS the A operand of v_mfma_f32_4x4x4_16B_f16 (block = lane / 4 holds four
//     tokens of one head row each), no transpose.  The B operand must hold four TOKENS of one channel
//     per lane, while a gathered codeword is four channels of one token: ds_read_b64_tr_b16 transposes
//     the gather on its way out of LDS (within 16 lanes, result lane 4 m + e, slot k <- source lane
//     4 k + m, element e).  With cbsz = 2 the four blocks of a 16-lane group share the weights of block
//     `abid` (= tile), each taking another sub-vector: 32 gathers + 32 matrix instructions per group, and
//     the accumulators are out_rot[head][channel] partial sums per 16-lane group.
//   * the fp16 weights are p a^v / A with A a power of two >= every a^v seen so far (rescaled lazily like
//     the running max), so the value contraction does not depend on the scale of V.
// One workgroup per (split, unit) - or, where decode_tile_splits prices it lower, one persistent
// workgroup per compute unit that takes an equal run of all groups (see the kernel's FLAT flag) - 8 waves,
// one 64 KiB codebook table replicated per LDS bank group (conflict-free gathers: one v_perm_b32 forms the
// address from a code byte).  Cache bytes are fetched two groups ahead into rotating register sets.  The fp16 residual (Sec. 3.2) is one more
// group whose four 16-token tiles are taken by waves 0..3 of the last split before their own groups (a
// quarter group each: a ninth wave would cap every wave at 168 registers, and a whole extra group on one
// wave would lengthen a four-group loop by a quarter).  Waves merge through LDS once; splits
// merge through fp32 partials in the workspace, the last wave to arrive (integer counter per query
// head) finishing the head: merge, one inverse Hadamard in registers, mean-vector term, output.
#pragma once

#include <algorithm>
#include <type_traits>

#include "nsn_host.h"

namespace nsn {
namespace tile {

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

constexpr int kPartialStride = 2 * kHeadDim + 2;  // rotated acc, mean-term acc, m (log2 units), l
constexpr float kLazyMaxLog2 = 5.0f;              // rescale only when a score beats the running max by 2^5
constexpr float kWeightScale = 1024.0f;           // fp16 weights carry 2^10 / A: small weights stay normal numbers
constexpr int kTableBytes = 65536;
constexpr int kRebase = 1 << 25;                  // tokens: 2^30 bytes of codes at most

template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }  // 2^-inf = 0
__device__ __forceinline__ uint32_t perm_b32(uint32_t s0, uint32_t s1, uint32_t sel) {
  return __builtin_amdgcn_perm(s0, s1, sel);
}
// (code byte k of `codes`) << 8 | lane offset: the LDS address of a table entry (the table starts at 0)
template <int K>
__device__ __forceinline__ uint32_t table_addr(uint32_t codes, uint32_t laneoff) {
  return perm_b32(codes, laneoff, 0x0c0c0400u + (K << 8));
}

#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ u2v lds_read64(uint32_t addr) { return *(const u2v __attribute__((address_space(3)))*)(addr); }
__device__ __forceinline__ u4v lds_read128(uint32_t addr) { return *(const u4v __attribute__((address_space(3)))*)(addr); }
__device__ __forceinline__ float lds_read32f(uint32_t addr) { return *(const float __attribute__((address_space(3)))*)(addr); }
__device__ __forceinline__ h4 lds_tr64(uint32_t addr) {
  return __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((s4v __attribute__((address_space(3)))*)(addr)));
}
__device__ __forceinline__ void lds_write128(uint32_t addr, u4v v) { *(u4v __attribute__((address_space(3)))*)(addr) = v; }
__device__ __forceinline__ void lds_write64(uint32_t addr, u2v v) { *(u2v __attribute__((address_space(3)))*)(addr) = v; }
__device__ __forceinline__ void lds_write32(uint32_t addr, uint32_t v) { *(uint32_t __attribute__((address_space(3)))*)(addr) = v; }
#else
__device__ __forceinline__ u2v lds_read64(uint32_t) { return u2v{0, 0}; }
__device__ __forceinline__ u4v lds_read128(uint32_t) { return u4v{0, 0, 0, 0}; }
__device__ __forceinline__ float lds_read32f(uint32_t) { return 0.f; }
__device__ __forceinline__ h4 lds_tr64(uint32_t) { return h4{}; }
__device__ __forceinline__ void lds_write128(uint32_t, u4v) {}
__device__ __forceinline__ void lds_write64(uint32_t, u2v) {}
__device__ __forceinline__ void lds_write32(uint32_t, uint32_t) {}
#endif

// Buffer descriptor: `bytes` bytes from p on; loads beyond them return zeros and do not access memory.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uint64_t)hi << 32 | lo), 0,
                                           __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
__device__ __forceinline__ u4v load128(rsrc_t r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }
__device__ __forceinline__ u2v load64(rsrc_t r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0); }
__device__ __forceinline__ uint32_t load32(rsrc_t r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0); }
__device__ __forceinline__ uint32_t load16(rsrc_t r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0); }

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// v_permlane16_swap / v_permlane32_swap exchange the odd 16-lane rows of `a` with the even rows of `b`
// (the upper half of `a` with the lower half of `b`).  Written as instructions: the compiler's two-result
// builtins for them were seen to return the first result twice.  The instruction reads other lanes'
// registers, which needs two idle cycles after a vector instruction wrote them (s_nop 1).
__device__ __forceinline__ void lane_swap16(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void lane_swap32(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void lane_swap16x2(uint32_t& a0, uint32_t& b0, uint32_t& a1, uint32_t& b1) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3" : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1));
}
__device__ __forceinline__ void lane_swap32x2(uint32_t& a0, uint32_t& b0, uint32_t& a1, uint32_t& b1) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3" : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1));
}
// 4 x 4 transpose between the four words and the wave's 16-lane groups: word t of group c <- word c of group t
__device__ __forceinline__ void group_transpose(uint32_t& w0, uint32_t& w1, uint32_t& w2, uint32_t& w3) {
  lane_swap16x2(w0, w1, w2, w3);
  lane_swap32x2(w0, w2, w1, w3);
}
// 4 x 4 transpose between the bytes of a word and bits 2, 3 of the lane number: byte x of lane k <- byte k of lane x
__device__ __forceinline__ uint32_t byte_transpose(uint32_t w, uint32_t sel_a, uint32_t sel_b) {
  w = __builtin_amdgcn_perm((uint32_t)xor_lane_i32<4>((int)w), w, sel_a);
  return __builtin_amdgcn_perm((uint32_t)xor_lane_i32<8>((int)w), w, sel_b);
}
// value of lane (lane ^ 16) / (lane ^ 32): a swap of two copies (no LDS traffic)
__device__ __forceinline__ float xor16(float v) {
  float a = v, b = v;
  lane_swap16(a, b);  // a: rows (0,0,2,2), b: rows (1,1,3,3)
  return ((threadIdx.x >> 4) & 1) ? a : b;
}
__device__ __forceinline__ float xor32(float v) {
  float a = v, b = v;
  lane_swap32(a, b);  // a: the lower half twice, b: the upper half twice
  return ((threadIdx.x >> 5) & 1) ? a : b;
}
// value of lane (lane ^ M): DPP inside a 16-lane row, register swaps across rows
template <int M>
__device__ __forceinline__ float xor_reg(float v) {
  if constexpr (M == 16)
    return xor16(v);
  else if constexpr (M == 32)
    return xor32(v);
  else
    return xor_lane<M>(v);
}
// max of finite or infinite values (never NaN here): the plain instruction, without the operand
// canonicalisation that fmaxf() adds under IEEE rules (one extra instruction per operand)
__device__ __forceinline__ float max3f(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float max2f(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// reductions over the sixteen lanes that share (lane % 4), i.e. one query head
__device__ __forceinline__ float head_max(float v) {
  v = max2f(v, dpp_mov<0x124>(v));  // row_ror:4
  v = max2f(v, dpp_mov<0x128>(v));  // row_ror:8
  v = max2f(v, xor16(v));
  v = max2f(v, xor32(v));
  return v;
}
__device__ __forceinline__ float head_sum(float v) {
  v += dpp_mov<0x124>(v);
  v += dpp_mov<0x128>(v);
  v += xor16(v);
  v += xor32(v);
  return v;
}
__device__ __forceinline__ float wave_max_all(float v) {
  v = max2f(v, dpp_mov<0xB1>(v));  // quad_perm [1,0,3,2]
  v = max2f(v, dpp_mov<0x4E>(v));  // quad_perm [2,3,0,1]
  return head_max(v);
}
__device__ __forceinline__ float wave_sum_all(float v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  return head_sum(v);
}
// value held by lane j of the caller's quad
template <int J>
__device__ __forceinline__ float quad_bcast(float v) {
  return dpp_mov<J | (J << 2) | (J << 4) | (J << 6)>(v);
}

__device__ __forceinline__ float half_lo_f(uint32_t u) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(u & 0xffffu)); }
__device__ __forceinline__ float half_hi_f(uint32_t u) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(u >> 16)); }
__device__ __forceinline__ void st_agent(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// LDS plan (dynamic block, starts at LDS address 0 because the gathers form absolute addresses):
//   [0, 64 KiB)   codebook table: entry (code c, copy p) at c * 256 + p * 8: 32 copies of 8 bytes (SUB = 4), or 16 of the
//                 first half of a codeword and, 128 bytes on, 16 of the second (SUB = 8: a lane's address serves both halves)
//   query block   fp16 hi / lo of the rotated, pre-scaled query [4][128] each; the same of the unrotated
//                 query (residual tiles); 128 zero bytes; q . o^k of the split's first Shift group (four
//                 heads); the unrotated query in fp32 [4][128]
//   merge block   per wave: rotated-domain sums [4][128] fp32, mean-term sums [4][128] fp32, (m, l) x 4
//   residual rows per wave 0..3: 16 fp16 key rows at a stride of 272 bytes, 16 value rows at 264
//                 (residual launches only)
// With keys normalised before the rotary embedding (ROPE), instead of the last two:
//   turn tables   fp16 hi and lo parts of (cos, sin)(j * inv_freq[i]), rows of 256 bytes whose 16-byte chunks are
//                 XOR-swizzled by the row number
//   per wave      4 KiB: q . RoPE_t(o^k) of the 64 tokens of the wave's next four groups, four heads each.  Its first
//                 life is the staging of the wave's residual rows (keys, then values), its last the merge block;
//                 (m, l) x 4 apart
template <int NW, bool ROPE>
struct Smem {
  static constexpr int kQhi = kTableBytes, kQlo = kQhi + 1024, kUhi = kQlo + 1024, kUlo = kUhi + 1024;
  static constexpr int kZero = kUlo + 1024, kQoFirst = kZero + 128, kQorig = kZero + 256;
  static constexpr int kTurn = kQorig + 2048;  // ROPE
  static constexpr int kMerge = ROPE ? kTurn + 32768 : kQorig + 2048;
  static constexpr int kMergeWave = ROPE ? 4096 : 2048 + 2048 + 256;
  static constexpr int kMl = ROPE ? kMerge + NW * kMergeWave : kMerge + 4096, kMlWave = ROPE ? 256 : kMergeWave;
  static constexpr int kBytes = ROPE ? kMl + NW * 256 : kMerge + NW * kMergeWave;
  // residual launches: 16 key rows (stride 272 bytes) and 16 value rows (stride 264) for each of four waves
  // (ROPE: 256 bytes, 16-byte chunks XOR-swizzled by the row number, one after the other in the wave's 4 KiB)
  static constexpr int kResKStride = ROPE ? 256 : 272, kResVStride = ROPE ? 256 : 264;
  static constexpr int kResWave = ROPE ? kMergeWave : 16 * 272 + 16 * 264;
  static constexpr int kRes = ROPE ? kMerge : kBytes;
  static constexpr int kBytesRes = ROPE ? kBytes : kRes + 4 * kResWave;
  static_assert(kBytesRes <= 160 * 1024, "LDS of one compute unit");
};

// one 64-token group's cache bytes as a lane needs them
// CW dwords per tensor; the sign + index format (SGN): [0, 4) index bytes, [4, 8) sign bytes, brought by arrange() to the
// byte order of the plain formats, the sign words as low address bytes of the first and (kx, vx) the second half of a codeword
template <int CW, bool SGN>
struct GroupRegs {
  uint32_t kc[CW], vc[CW];  // the lane's code bytes of the group
  uint32_t kx[SGN ? 4 : 1], vx[SGN ? 4 : 1];
  uint4 nk, nv;             // (a, b) fp16 pairs of the lane's four tokens
  uint32_t ok, ov;          // channels 2 lane, 2 lane + 1 of the group's Shift vectors (fp16 pairs)
  // 4-bit side information (DQ): nk / nv = {a' of the four tokens (two words), their four s1 nibbles, the
  // block's (min, step)}; ok / ov = the byte with the two channels' nibbles, okp / ovp = (min, step) of the
  // lane's 32-channel group
  uint32_t okp, ovp;
};
// min + step * code of a 4-bit level (par = fp16 pair (min, step))
__device__ __forceinline__ float dq_level(uint32_t par, uint32_t code) {
  return fmaf(half_hi_f(par), (float)code, half_lo_f(par));
}

// POW2: group_size (if any) and, for paged caches, page_size are powers of two: group and page indices are
// shifts (the other instance multiplies by reciprocals)
// PAGED: the caches are paged (block tables); the other instance never reads a block table and can
// fetch its first group before the sequence length is known
// FLAT: the launch is one persistent workgroup per compute unit.  All 64-token groups of all (sequence,
// kv head) units form one list (unit by unit, a unit without coded tokens counts as one group); workgroup c
// takes the c-th of n_splits equal runs of that list, which is a sequence of segments: (unit, first group,
// number of groups).  A unit that is cut by a run boundary is merged through partial results exactly as a
// split one is in the other instance.  Ragged batches and batches with more units than compute units keep
// every compute unit busy this way, and the codebook table is built once per workgroup.
// Every unit takes kSegCost list slots in front of its groups: a segment costs about as much as that many
// groups (query rotation, two barriers, the merge of the waves, a cold start of the loads), so that runs with
// many short units get fewer groups.  A run that ends inside those slots leaves the unit to the next run.
constexpr int kSegCost = 32;
// DQ: norms and means are stored in 4 bits (Sec. 3.5): 164-byte norm records per 64-token block, 80-byte mean records
// SGN: the sign + index format.  Its table holds every codeword's halves (four channels) under all sixteen sign patterns,
// [code][pattern] 16 bytes = low half, high half: one copy, gathered with random bank conflicts (about twice the
// cycles of the replicated table), but no instruction for the signs beyond the address; flipping the signs of
// conflict-free gathers on the vector ALUs costs about 300 instructions per group, which are the scarcer resource.
// ROPE: keys normalised before the rotary embedding: the mean term of the score is turned by the token's position
// (see rope_compute).
// SGN and ROPE caches keep the legacy code layout (K token-major, V blocks of J tokens, sub-vector-major).  The tokens of
// a group are dealt to the contraction's rows so that what a lane loads is contiguous: row 4 rho + k of tile t is token
// 16 rho + 4 t + k (tiled layout: 16 t + 4 rho + k), a lane loads token 16 rho + 4 c + k's key bytes and sixteen tokens of
// one value row, and arrange() exchanges words between 16-lane groups (four swaps) and bytes between lanes (twenty
// instructions), once per group.
// MANY: a kv head may have more than four query heads.  The others do without the unit arithmetic (with it at run time
// for all, four launches of the ragged paged batch of 24 sequences took 92.4 instead of 91.5 us, of 131072 1-bit tokens 0.5
// to 1 % more).
// Arguments: they fill four 64-byte lines, which no cache holds at the start of a launch.  Scalar loads are waited for all
// together: the lines that a prologue touches first cost one trip, and a line that it touches behind that wait costs another.
// What it needs ahead of the bulk loads lies in the first three (g to vc, seq_lens), the counts on the third and the fourth; the
// compiler reads four of them, from scale_log2e on, with one load that brings both lines in.  (With n_rep behind res, in the fourth
// line alone, and asked for behind the first wait: two launches of 56 units x 900 tokens on 32 caches in turn 15.49 instead of
// 15.19 us, four of 131072 1-bit tokens in HBM 88 to 86 instead of 87 to 85; on one cache, which the L2 holds, 14.56 instead of
// 14.63.  The legacy formats with the rotary embedding, which had all lines in one trip before, take 0.2 to 0.6 % longer.)
template <int SUB, int NW, bool POW2, bool PAGED, bool FLAT, bool DQ, bool SGN = false, bool ROPE = false,
          bool MANY = SGN || ROPE>
__global__ __launch_bounds__(NW * 64) void dec_tile_kernel(Geometry g, const __half* __restrict__ codebook,
                                                           const __half* __restrict__ q, CacheView kc, CacheView vc,
                                                           const int32_t* __restrict__ seq_lens,
                                                           float* __restrict__ out, int batch, float scale_log2e,
                                                           int n_splits, int per, int n_rep, float* partial,
                                                           int* counters, ResidualView res) {
  static_assert(NW == 8, "prologue work split: 512 threads fill the table, waves 0..3 rotate the query");
  constexpr int NSV = kHeadDim / SUB;  // sub-vectors per token
  constexpr bool LEGACY = SGN || ROPE;
  constexpr int J = SGN ? 2 * NSV : NSV;  // code bytes per token
  constexpr int CW = J / 4;               // code dwords per lane, group and tensor
  static_assert(!SGN || SUB == 8, "the sign + index format is defined on 8-dim sub-vectors");
  using SM = Smem<NW, ROPE>;
  using Regs = GroupRegs<CW, SGN>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

  // Five to eight query heads (n_rep) of a kv head are two units of up to four: unit head hu, kv head hu >> two
  const int two = MANY && n_rep > 4 ? 1 : 0;
  auto heads_of = [&](int hu) { return MANY ? min(4, n_rep - 4 * (hu & two)) : n_rep; };
  const int tid = threadIdx.x, lane0 = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cap_tokens = g.page_tokens * g.pages_per_seq;
  // the segment at hand (!FLAT: the launch's one (split, kv head, sequence))
  int split = FLAT ? 0 : blockIdx.x, hu = FLAT ? 0 : blockIdx.y, h = hu >> two, b = FLAT ? 0 : blockIdx.z;
  int t0 = split * per;
  int64_t mean_base = (int64_t)(b * g.n_kv_heads + h) * g.n_groups_max;

  // ---- loads that do not depend on the sequence length go out first ------------------------------
  // (all unconditional, so that the wait for the codebook can leave the later ones in flight)
  typedef typename std::conditional<SUB == 4, uint2, uint4>::type cw_t;
  const cw_t cw_reg = reinterpret_cast<const cw_t*>(codebook)[tid >> 1];  // two threads per code row

  // ---- FLAT: this workgroup's run of the group list (every wave computes the same numbers) --------
  const int hkv = g.n_kv_heads, n_units = hkv << two;  // kv heads, units per sequence
  int run_q = 0, run_pos = 0, run_end = 0, seg_g = 0;  // run length, list position, end of the run, slot inside the unit
  // codebook table: thread (code = tid / 2, half = tid % 2) fills eight 16-byte slots of its half row, starting
  // at a slot that depends on the code so that the 64 stores of a wave spread over all banks
  auto fill_table = [&]() {
    const int code = tid >> 1, half = tid & 1;
    u4v v;
    if constexpr (SUB == 4)
      v = u4v{cw_reg.x, cw_reg.y, cw_reg.x, cw_reg.y};
    else if constexpr (SGN)
      v = u4v{cw_reg.x, cw_reg.y, cw_reg.z, cw_reg.w};
    else
      v = half ? u4v{cw_reg.z, cw_reg.w, cw_reg.z, cw_reg.w} : u4v{cw_reg.x, cw_reg.y, cw_reg.x, cw_reg.y};
    const uint32_t row = code * 256 + half * 128;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if constexpr (SGN) {  // sign pattern n: bit i flips channel i of either half of the codeword
        const int n = 8 * half + ((u + code) & 7);
        const uint32_t s0 = ((n & 1) << 15) | ((uint32_t)(n & 2) << 30), s1 = ((n & 4) << 13) | ((uint32_t)(n & 8) << 28);
        lds_write128(code * 256 + n * 16, u4v{v.x ^ s0, v.y ^ s1, v.z ^ s0, v.w ^ s1});
      } else {
        lds_write128(row + (((u + code) & 7) << 4), v);
      }
    }
    if constexpr (ROPE) {  // turn tables: chunk i = part (hi / lo) i / 1024, row (i / 16) % 64, 16-byte chunk i % 16
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = tid + u * NW * 64, rw = (i >> 4) & 63;
        const uint4 t = reinterpret_cast<const uint4*>(g.rope + kRopeHiOff)[i];
        lds_write128(SM::kTurn + (i >> 10) * 16384 + rw * 256 + (((i & 15) ^ (rw & 15)) << 4), u4v{t.x, t.y, t.z, t.w});
      }
    }
  };
  if constexpr (FLAT) {
    auto groups_of = [](int len) { return max(1, (len + 63) >> 6); };
    // list positions taken by the sequences of one 64-sequence block: this lane's sequence, and the inclusive
    // prefix sums over the lanes
    auto block_sizes = [&](int b0, int& n, int& incl) {
      n = (b0 + lane0 < batch) ? (groups_of(seq_lens[b0 + lane0]) + kSegCost) * n_units : 0;
      incl = n;
      static_for<6>([&](auto kc_) {
        constexpr int d = 1 << decltype(kc_)::value;
        const int up = __shfl_up(incl, d);
        incl += (lane0 >= d) ? up : 0;
      });
    };
    int n0, incl0;
    block_sizes(0, n0, incl0);  // (the table is filled while these lengths are on their way)
    fill_table();
    int total = __builtin_amdgcn_readlane(incl0, 63);
    for (int b0 = 64; b0 < batch; b0 += 64) {
      int n, incl;
      block_sizes(b0, n, incl);
      total += __builtin_amdgcn_readlane(incl, 63);
    }
    run_q = (total + n_splits - 1) / n_splits;
    run_pos = (int)blockIdx.x * run_q;
    if (run_pos >= total) return;  // (all waves alike, before any barrier)
    run_end = min(total, run_pos + run_q);
    // the sequence that holds list position run_pos: sequences are laid out one after the other, each as
    // n_units units of its group count
    int before = 0;  // list positions in front of the 64-sequence block at hand
    for (int b0 = 0; b0 < batch; b0 += 64) {
      int n = n0, incl = incl0;
      if (b0 > 0) block_sizes(b0, n, incl);
      const int n_before = __popcll(__ballot(b0 + lane0 < batch && before + incl <= run_pos));  // sequences that end at or before it
      const int n_here = min(64, batch - b0);
      if (n_before < n_here) {
        b = b0 + n_before;
        const int incl_b = __builtin_amdgcn_readlane(incl, n_before), n_b = __builtin_amdgcn_readlane(n, n_before);
        const int off = run_pos - (before + incl_b - n_b);  // position inside the sequence's units
        const int slots = n_b / n_units;
        hu = off / slots;
        seg_g = off - hu * slots;  // (position among the unit's slots)
        break;
      }
      before += __builtin_amdgcn_readlane(incl, 63);
    }
  }

  bool first_segment = true;
  // FLAT: the next segment's sequence length, query row and first mean row are fetched a segment ahead
  int len_cur = 0, nb = 0, nh = 0;
  __half2 q2_next = __half2{};
  uint32_t okf_next = 0u, okfp_next = 0u;
  // PAGED: the wave's window of block-table entries (see load_window); the first group of a pass loads it
  int win0 = -(1 << 30), win_k = 0, win_v = 0, nwin_k = 0, nwin_v = 0;
  if constexpr (FLAT) len_cur = seq_lens[b];
  for (;;) {  // FLAT: one pass per segment of the run; otherwise a single pass
  // Everything a pass derives from the lane number is derived anew in each pass: values that the compiler
  // could compute once in front of the segment loop would stay in registers through all of it, and this
  // kernel has none to spare.
  int lane = lane0;
  if constexpr (FLAT || LEGACY) asm volatile("" : "+v"(lane));
  const int rho = lane >> 4, n16 = lane & 15, head = lane & 3, tile_of_lane = n16 >> 2;
  // ---- loads of one group (all unconditional: callers clamp the group index into the cache) ----
  // (legacy layout: the key row of token 16 (n / 4) + 4 rho + n % 4, sixteen tokens from 16 rho of value row n)
  const uint32_t lane_code_off = LEGACY ? (16 * (n16 >> 2) + 4 * rho + (n16 & 3)) * J : lane * NSV;
  const uint32_t lane_v_off = !LEGACY ? lane_code_off : J == 16 ? lane * 16 : (rho >> 1) * 1024 + n16 * 32 + (rho & 1) * 16;
  const int tok_of_lane = LEGACY ? 16 * rho + 4 * tile_of_lane : 16 * tile_of_lane + 4 * rho;  // its four tokens' first
  const uint32_t norm_off = tok_of_lane * 4;  // bytes
  const uint32_t lane_x4 = lane * 4;
  // Paged caches: the wave keeps 64 consecutive block-table entries of its sequence in two registers (lane i:
  // page win0 + i, clamped into the sequence's table row) and picks a group's entries with lane reads.  An
  // entry loaded right before its use would make the wave wait for every load it has in flight (loads return
  // in order); the window is loaded once per segment (the persistent instance asks for the next segment's
  // window when it leaves its main loop) and again only when a group lies beyond it.
  auto load_window = [&](int bb, int w0, int& wk, int& wv) {
    const int64_t e = (int64_t)bb * g.pages_per_seq + min(w0 + lane, g.pages_per_seq - 1);
    wk = kc.block_table[e], wv = vc.block_table[e];
  };
  // 64-token blocks of a page and of the whole buffer, whose number has 32 bits.  (With token indices in 64 bits, and the wait for
  // the window's entries where the paths with and without a reload meet - a wait for every load in flight, in every group -,
  // two launches of 32 ragged sequences took 87.4 instead of 86.4 us, 59 x 32 heads x 3232 tokens 113.1 instead of 111.1, four
  // launches of 12 x 16 heads x 11644 tokens in pages of 64 with 4-bit side information 216.8 instead of 208.9)
  const uint32_t page_blocks = (uint32_t)g.n_kv_heads * ((uint32_t)g.page_tokens >> 6);
  auto group_blocks = [&](uint32_t tg, bool real, uint32_t& kblock, uint32_t& vblock) {
    const int page = POW2 ? (int)(tg >> g.page_shift) : tokens_div((int)tg, g.page_div);
    const uint32_t tb = (POW2 ? tg & (g.page_tokens - 1) : tg - (uint32_t)page * g.page_tokens) >> 6;
    if (real && (unsigned)(page - win0) >= 64u) {  // wave-uniform
      win0 = page & ~63;
      load_window(b, win0, win_k, win_v);
      // (waited for here: where the two paths meet, the wait would be every group's, and for every load in flight)
      asm volatile("" : "+v"(win_k), "+v"(win_v));
    }
    // (a group that does not exist: the buffers' first block, which every wave reads then)
    const int at = (page - win0) & 63;
    const uint32_t in_page = (uint32_t)h * ((uint32_t)g.page_tokens >> 6) + tb;
    kblock = real ? (uint32_t)__builtin_amdgcn_readlane(win_k, at) * page_blocks + in_page : 0u;
    vblock = real ? (uint32_t)__builtin_amdgcn_readlane(win_v, at) * page_blocks + in_page : 0u;
  };
  const int gshift = g.group_size > 0 ? g.group_shift : 31;  // (no groups: index 0 for every token)
  auto shift_group = [&](int tg) -> int { return POW2 ? tg >> gshift : tokens_div(tg, g.group_div); };
  // Contiguous caches are read through buffer descriptors (the Shift vectors, which every group has, through plain pointers):
  // base and size in scalar registers, one vector addition per kind of array and group, and no address arithmetic on the scalar
  // unit, whose instructions a wave waits for one by one (about eight cycles each; 64-bit addresses of six arrays were thirty
  // of them per group).  Offsets count from token `base_tok` of the unit and have 32 bits: every kRebase tokens the
  // descriptors move on (in the branch that masked tokens take).  With the masked tokens' selects in a branch of their own and
  // one address for both halves of an 8-dim codeword a group with 1-bit codes takes 103 vector instructions instead of 144, 15
  // scalar ones instead of 55.  Persistent: 64 x 32 heads x 32768 tokens 916 -> 869 us; legacy formats: all options of the paper
  // 87.6 -> 77.9.  One workgroup per split, by machine: 131072 1-bit tokens, four launches 78 to 80 -> 75 to 77 on caches that
  // stay in the last-level cache, 80 to 88 -> 77 to 86 in HBM; 8 x 8192 tokens with residual 52.0 to 53.5 -> 50.0 to 52.1, and in
  // HBM 57.6 -> 56.4 on fast machines, 61 -> 61 to 62 on slow ones.  Its 4-bit instances go by block numbers as paged caches do:
  // setting up two sorts of descriptors ahead of the first load costs calls of a few groups per wave more than it saves (56
  // units x 900 4-dim tokens, two launches 15.6 against 15.45; 8-dim ones of 600 to 1300 tokens are 0.5 to 1 % above 64-bit
  // addresses either way).
  constexpr bool DESC = !PAGED && (FLAT || LEGACY || !DQ);
  const uint32_t unit_block = (uint32_t)(b * g.n_kv_heads + h) * ((uint32_t)g.page_tokens >> 6);  // (!DESC, contiguous)
  // (a split beyond the cache, which leaves at once, begins at its last group)
  int base_tok = min(t0, cap_tokens - 64), base_group = 0, last_tok = 0;  // base_tok's Shift group, the last group's first token
  rsrc_t kr_codes, vr_codes, kr_norms, vr_norms;
  const unsigned char *kp_means, *vp_means;
  constexpr uint32_t kMeanBytes = DQ ? kDqMeanRec : 2 * kHeadDim;
  auto describe = [&](int end_tok) {  // groups from end_tok on read as zeros, without a memory access
    base_group = shift_group(base_tok);
    if constexpr (DESC) {
      const uint32_t n = (uint32_t)min(end_tok - base_tok, 2 * kRebase);
      const int64_t tok = (int64_t)(b * g.n_kv_heads + h) * g.page_tokens + base_tok;
      kr_codes = make_rsrc(kc.codes + tok * J, n * J), vr_codes = make_rsrc(vc.codes + tok * J, n * J);
      const int64_t norms_at = DQ ? (tok >> 6) * kDqNormRec : tok * 4;
      const uint32_t norms_n = DQ ? (n >> 6) * kDqNormRec : n * 4;
      kr_norms = make_rsrc(reinterpret_cast<const unsigned char*>(kc.norms) + norms_at, norms_n);
      vr_norms = make_rsrc(reinterpret_cast<const unsigned char*>(vc.norms) + norms_at, norms_n);
    }
    last_tok = max(end_tok - 64, base_tok);
    const int64_t mean_at = (mean_base + base_group) * kMeanBytes;
    kp_means = reinterpret_cast<const unsigned char*>(kc.means) + mean_at;
    vp_means = reinterpret_cast<const unsigned char*>(vc.means) + mean_at;
  };
  // n: the group, counted from token t0.  One that does not exist (`real` false: the wave's list of groups has ended) is
  // loaded all the same: descriptors read zeros beyond their ends, the other form reads the first bytes of every array
  // (one cache line per instruction); nothing of it is used and any bytes are valid table indices.  With loads that are only
  // issued under a condition, the number of loads behind a given one depends on the path, the compiler's wait counts take the
  // smallest, and every wait for a group's bytes becomes a wait for all loads in flight, the groups requested ahead included.
  // Side information ahead of the codes: where the loop's first group meets its Shift vectors' and norms' first use, the wait is the
  // one that holds for every way there, also for one behind a group whose loads were the last ones (the compiler cannot know
  // that it is never taken), and counts only the loads that follow within a group.  Behind the codes, they made a wave with
  // one group wait for all of the second one's loads.  4-bit side information, eight loads of the fourteen: 56 units x 256
  // tokens, two launches 11.95 -> 11.45 us (4-dim), x 900 tokens 16.0 -> 15.5; all options of the paper, 8 x 8192 tokens, four
  // launches 69.6 -> 67.9.  Codes first: 8-dim fp16 calls on pages (1 % less) and the persistent fp16 instance on contiguous
  // caches (64 x 32 heads x 32768 tokens 869 instead of 876).  8-dim tiled instances are left to the scheduler within the order,
  // which gives them 0.5 %.
  auto load_group = [&](int n, bool real, Regs& G) {
    constexpr bool kCodesFirst = !LEGACY && !DQ && (PAGED ? SUB == 8 : FLAT), kOrdered = SUB == 4 || LEGACY;
    const uint32_t tg = token_of_group(t0, n);
    auto load_means = [&]() {
      const uint32_t mrec = (uint32_t)(shift_group(token_up_to(tg, last_tok)) - base_group) * kMeanBytes;
      if constexpr (DQ) {
        const uint32_t at_par = mrec + kDqMeanPar + 4 * ((uint32_t)lane >> 4);
        if constexpr (!ROPE) G.ok = kp_means[mrec + lane], G.okp = *reinterpret_cast<const uint32_t*>(kp_means + at_par);
        G.ov = vp_means[mrec + lane], G.ovp = *reinterpret_cast<const uint32_t*>(vp_means + at_par);
      } else {
        if constexpr (!ROPE) G.ok = *reinterpret_cast<const uint32_t*>(kp_means + (mrec + lane_x4));  // (ROPE: rope_load)
        G.ov = *reinterpret_cast<const uint32_t*>(vp_means + (mrec + lane_x4));
      }
    };
    uint32_t rel = 0u, kblock = 0u, vblock = 0u;  // DESC: the group's distance from base_tok; its 64-token blocks
    if constexpr (DESC) {
      rel = tg - (uint32_t)base_tok;
      asm("" : "+s"(rel));  // (or every offset gets a subtraction of its own)
    }
    auto load_norms = [&]() {
      if constexpr (DESC) {
        if constexpr (DQ) {  // one norm record per 64-token block
          const uint32_t rec = (rel >> 6) * kDqNormRec, tok0 = norm_off >> 2;  // (the lane's first token: a multiple of 4)
          const u2v ka = load64(kr_norms, rec + 2 * tok0), va = load64(vr_norms, rec + 2 * tok0);
          const uint32_t at_codes = rec + kDqNormCodes + (tok0 >> 1), at_par = rec + kDqNormPar;
          G.nk = make_uint4(ka.x, ka.y, load16(kr_norms, at_codes), load32(kr_norms, at_par));
          G.nv = make_uint4(va.x, va.y, load16(vr_norms, at_codes), load32(vr_norms, at_par));
        } else {
          const u4v nk = load128(kr_norms, norm_off + rel * 4), nv = load128(vr_norms, norm_off + rel * 4);
          G.nk = make_uint4(nk.x, nk.y, nk.z, nk.w), G.nv = make_uint4(nv.x, nv.y, nv.z, nv.w);
        }
      } else {
        constexpr int kBlockNorms = DQ ? kDqNormRec : 256;
        const uint32_t noff = real ? norm_off : 0u;
        const unsigned char* kn = reinterpret_cast<const unsigned char*>(kc.norms) + (uint64_t)kblock * kBlockNorms;
        const unsigned char* vn = reinterpret_cast<const unsigned char*>(vc.norms) + (uint64_t)vblock * kBlockNorms;
        if constexpr (DQ) {
          const uint32_t tok0 = noff >> 2;
          const uint2 ka = *reinterpret_cast<const uint2*>(kn + 2 * tok0), va = *reinterpret_cast<const uint2*>(vn + 2 * tok0);
          G.nk = make_uint4(ka.x, ka.y, *reinterpret_cast<const uint16_t*>(kn + (kDqNormCodes + (tok0 >> 1))),
                            *reinterpret_cast<const uint32_t*>(kn + kDqNormPar));
          G.nv = make_uint4(va.x, va.y, *reinterpret_cast<const uint16_t*>(vn + (kDqNormCodes + (tok0 >> 1))),
                            *reinterpret_cast<const uint32_t*>(vn + kDqNormPar));
        } else {
          G.nk = *reinterpret_cast<const uint4*>(kn + noff), G.nv = *reinterpret_cast<const uint4*>(vn + noff);
        }
      }
    };
    auto load_codes = [&]() {
      constexpr int VSTEP = LEGACY ? J : 1;  // 16-byte pieces; legacy: the lane's second value row is sixteen rows on
      const uint32_t lco = DESC ? lane_code_off + rel * J : real ? lane_code_off : 0u;
      const uint32_t lvo = DESC ? lane_v_off + rel * J : real ? lane_v_off : 0u;
      const unsigned char *kp = kc.codes + (uint64_t)kblock * (64 * J), *vp = vc.codes + (uint64_t)vblock * (64 * J);
#pragma unroll
      for (int w4 = 0; w4 < CW / 4; ++w4) {
        u4v kv4, vv4;
        if constexpr (DESC)
          kv4 = load128(kr_codes, lco + 16 * w4), vv4 = load128(vr_codes, lvo + 16 * w4 * VSTEP);
        else
          kv4 = *reinterpret_cast<const u4v*>(kp + (lco + 16 * w4)), vv4 = *reinterpret_cast<const u4v*>(vp + (lvo + 16 * w4 * VSTEP));
        G.kc[4 * w4] = kv4.x, G.kc[4 * w4 + 1] = kv4.y, G.kc[4 * w4 + 2] = kv4.z, G.kc[4 * w4 + 3] = kv4.w;
        G.vc[4 * w4] = vv4.x, G.vc[4 * w4 + 1] = vv4.y, G.vc[4 * w4 + 2] = vv4.z, G.vc[4 * w4 + 3] = vv4.w;
      }
    };
    if constexpr (kCodesFirst) {
      if constexpr (PAGED) group_blocks(tg, real, kblock, vblock);
      load_codes(), load_norms(), load_means();
    } else {
      load_means();
      if constexpr (kOrdered) __builtin_amdgcn_sched_barrier(0);
      if constexpr (PAGED)
        group_blocks(tg, real, kblock, vblock);
      else if constexpr (!DESC)
        kblock = vblock = real ? unit_block + (tg >> 6) : 0u;
      load_norms();
      if constexpr (kOrdered) __builtin_amdgcn_sched_barrier(0);
      load_codes();
    }
  };
  // legacy layout: a group's code bytes from the order they were loaded in to the order the gathers use
  auto arrange = [&](Regs& G) {
    if constexpr (LEGACY) {
      int ln = lane;
      asm volatile("" : "+v"(ln));  // (the selectors are formed anew each time: no registers to spare for them)
      const uint32_t bsel_a = (ln & 4) ? 0x03070105u : 0x06020400u, bsel_b = (ln & 8) ? 0x03020706u : 0x05040100u;
      const uint32_t ksh = (ln & 16) ? 0u : 4u, vsh = (ln & 1) ? 0u : 4u;  // SGN: which half of a codeword comes first
      const uint32_t k8 = (ln & 16) ? 0x08080808u : 0u, v8 = (ln & 1) ? 0x08080808u : 0u;
      if constexpr (SUB == 4) {
        group_transpose(G.kc[0], G.kc[2], G.kc[4], G.kc[6]);
        group_transpose(G.kc[1], G.kc[3], G.kc[5], G.kc[7]);
        // value rows n (words 0..3) and n + 16 (words 4..7), four tiles each -> word 2 tile + row / 16
        uint32_t w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = byte_transpose(G.vc[i], bsel_a, bsel_b);
#pragma unroll
        for (int t = 0; t < 4; ++t) G.vc[2 * t] = w[t], G.vc[2 * t + 1] = w[4 + t];
      } else {
        group_transpose(G.kc[0], G.kc[1], G.kc[2], G.kc[3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) G.vc[i] = byte_transpose(G.vc[i], bsel_a, bsel_b);
        if constexpr (SGN) {
          group_transpose(G.kc[4], G.kc[5], G.kc[6], G.kc[7]);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const uint32_t ks = G.kc[4 + t], vs = byte_transpose(G.vc[4 + t], bsel_a, bsel_b);
            // the low bytes of the gathers' addresses: sign pattern of a half << 4, offset of that half.  (Masked here, 32 words
            // instead of 64 addresses; with indices by reciprocals and not by branches over shifts and divisions: 16 ragged
            // sequences, two launches 54.7 -> 51.0 us, all options of the paper, four launches 82.8 -> 78.9)
            G.kc[4 + t] = ((ks << ksh) & 0xf0f0f0f0u) | k8, G.kx[t] = ((ks << (4u - ksh)) & 0xf0f0f0f0u) | (k8 ^ 0x08080808u);
            G.vc[4 + t] = ((vs << vsh) & 0xf0f0f0f0u) | v8, G.vx[t] = ((vs << (4u - vsh)) & 0xf0f0f0f0u) | (v8 ^ 0x08080808u);
          }
        }
      }
    }
  };
  // the lane's two channels of a Shift vector from its stored words
  auto mean_pair = [&](uint32_t w, uint32_t par, float& o0, float& o1) {
    if constexpr (DQ) {
      o0 = dq_level(par, w & 15u), o1 = dq_level(par, (w >> 4) & 15u);
    } else {
      o0 = half_lo_f(w), o1 = half_hi_f(w);
    }
  };

  int len, n_live, t1, n_grp, first_run = 0;
  bool res_here;  // this segment holds the unit's last group: it takes the residual rows
  if constexpr (FLAT) {
    len = len_cur;
    const int ng = max(1, (len + 63) >> 6);
    const int take_slots = min(ng + kSegCost - seg_g, run_end - run_pos);
    const int g0 = max(seg_g - kSegCost, 0), g1 = max(seg_g + take_slots - kSegCost, 0);  // the segment's groups
    if (g1 == g0) break;  // the run ends inside the unit's cost slots (all waves alike, no barrier pending)
    const int unit_pos = run_pos - seg_g + kSegCost;  // list position of the unit's first group
    first_run = unit_pos / run_q;
    n_live = (unit_pos + ng - 1) / run_q - first_run + 1;  // runs that hold groups of this unit
    split = (int)blockIdx.x - first_run;
    t0 = g0 << 6;
    t1 = min(len, g1 << 6);
    res_here = g1 == ng;
    h = hu >> two;
    mean_base = (int64_t)(b * hkv + h) * g.n_groups_max;
    // advance to the next segment's start (used at the end of the pass)
    run_pos += take_slots;
    seg_g = 0;  // (a run that goes on goes on with the next unit)
  }
  const int r = heads_of(hu);
  // (one workgroup per split: the quotient is formed here, in the shadow of the codebook row's load.  Taken from n_rep, the
  // compiler moves that load behind the shorter index arithmetic, among the bulk loads: four launches of 131072 1-bit
  // tokens 86.7 instead of 85.6 us.  The persistent instance, which would form it per segment, is as fast either way)
  const int q_per_kv = MANY || FLAT ? n_rep : g.n_q_heads / g.n_kv_heads;
  auto first_head = [&](int hv) { return (hv >> two) * q_per_kv + 4 * (hv & two); };
  const int hq0 = first_head(hu);
  // waves 0..3 rotate one query head each (the others load a valid row that they do not use)
  auto q_row = [&](int bb, int hv) {
    return *reinterpret_cast<const __half2*>(q + (int64_t)(bb * g.n_q_heads + first_head(hv) + min(wave & 3, heads_of(hv) - 1)) * kHeadDim +
                                             2 * lane);
  };
  auto mean_row_k = [&](int64_t base, int grp, uint32_t& w, uint32_t& par) {
    if constexpr (DQ) {
      const unsigned char* km = reinterpret_cast<const unsigned char*>(kc.means) + (base + grp) * kDqMeanRec;
      w = km[lane];
      par = *reinterpret_cast<const uint32_t*>(km + kDqMeanPar + 4 * (lane >> 4));
    } else {
      w = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const unsigned char*>(kc.means + (base + grp) * kHeadDim) +
                                             lane_x4);
      par = 0u;
    }
  };
  // the split's first Shift group: its q . o^k is formed once per workgroup (waves 4..7, one head each)
  const int grp_first = shift_group(min(t0, cap_tokens - 64));
  __half2 q2_raw = q2_next;
  uint32_t ok_first = okf_next, okp_first = okfp_next;
  if (!FLAT || first_segment) {
    q2_raw = q_row(b, hu);
    if constexpr (!ROPE) mean_row_k(mean_base, grp_first, ok_first, okp_first);
  }
  if constexpr (FLAT) {
    // the unit after this one (if the run goes on, this segment ends its unit and the next begins one)
    nb = b, nh = hu;
    if (run_pos < run_end && ++nh == n_units) {
      nh = 0;
      ++nb;
    }
    len_cur = seq_lens[nb];
    q2_next = q_row(nb, nh);
    if constexpr (!ROPE) mean_row_k((int64_t)(nb * hkv + (nh >> two)) * g.n_groups_max, 0, okf_next, okfp_next);
  }
  // (the three small loads stay ahead of the bulk ones: the waits for them then leave every later load in flight)
  __builtin_amdgcn_sched_barrier(0);
  Regs S0, S1, S2;  // each is loaded before it is read (with the bytes of a group that exists, or with any bytes)
  if constexpr (!FLAT) {
    // contiguous caches: the wave's first group is in bounds whatever the sequence length is (clamped into
    // the cache when the split lies beyond it: then it is never processed)
    if constexpr (!PAGED) {
      describe(cap_tokens);
      load_group(wave, DESC || token_of_group(t0, wave) < (uint32_t)cap_tokens, S0);  // (wslot == wave here)
    }
    len = seq_lens[b];
    // Splits that lie wholly beyond this sequence's end have nothing to do and leave at once (a ragged batch
    // is launched with the split count of its longest sequence); the others know how many of them there
    // are.  A sequence without coded tokens keeps split 0 (it may still have residual rows).
    n_live = len > 0 ? (len - 1) / per + 1 : 1;
    if (split >= n_live) return;
    t1 = split_end(t0, per, len);
    res_here = split == n_live - 1;
  }
  n_grp = (t1 > t0) ? (t1 - t0 + 63) >> 6 : 0;  // 64-token groups of this segment
  int t_whole = t1 - 64;                         // groups that begin later hold masked tokens (or are far from base_tok)
  if constexpr (FLAT || PAGED) base_tok = t0;
  describe(t0 + (n_grp << 6));
  t_whole = base_tok + min(t_whole - base_tok, kRebase);
  // FLAT: waves 4..7 take the segment's first groups: they are the ones that come out of the previous
  // segment early (waves 0..3 merge it), and a short segment then does not wait for the late ones
  const int wslot = FLAT ? (wave + 4) & 7 : wave;
  if constexpr (PAGED || FLAT) load_group(wslot, wslot < n_grp, S0);
  // ---- prologue: codebook table, query operands --------------------------------------------------
  if constexpr (!FLAT) fill_table();
  if (wave < 4) {  // d1: wave w rotates head w (zeros for a head that this launch does not have)
    const bool has_head = wave < r;
    const float x0 = has_head ? __low2float(q2_raw) : 0.f, x1 = has_head ? __high2float(q2_raw) : 0.f;
    const uint32_t e2 = wave * 128 + 2 * lane;  // element index of the pair in a [4][128] array
    {
      lds_write64(SM::kQorig + e2 * 4, u2v{__float_as_uint(x0), __float_as_uint(x1)});
      const float u0 = x0 * scale_log2e, u1 = x1 * scale_log2e;
      const _Float16 h0 = (_Float16)u0, h1 = (_Float16)u1;
      lds_write32(SM::kUhi + e2 * 2, __builtin_bit_cast(uint32_t, h2v{h0, h1}));
      lds_write32(SM::kUlo + e2 * 2,
                  __builtin_bit_cast(uint32_t, h2v{(_Float16)(u0 - (float)h0), (_Float16)(u1 - (float)h1)}));
    }
    float y0 = x0 + x1, y1 = x0 - x1;
    static_for<6>([&](auto kc_) {  // lane bit k <-> element bit k + 1
      constexpr int m = 1 << decltype(kc_)::value;
      const float p0 = xor_reg<m>(y0), p1 = xor_reg<m>(y1);
      const bool upper = (lane & m) != 0;
      y0 = upper ? p0 - y0 : y0 + p0;
      y1 = upper ? p1 - y1 : y1 + p1;
    });
    const float qscale = (float)kInvSqrtD * scale_log2e;
    y0 *= qscale, y1 *= qscale;
    const _Float16 h0 = (_Float16)y0, h1 = (_Float16)y1;
    lds_write32(SM::kQhi + e2 * 2, __builtin_bit_cast(uint32_t, h2v{h0, h1}));
    lds_write32(SM::kQlo + e2 * 2,
                __builtin_bit_cast(uint32_t, h2v{(_Float16)(y0 - (float)h0), (_Float16)(y1 - (float)h1)}));
  } else {
    if (first_segment && wave == 4 && lane < 32) lds_write32(SM::kZero + lane * 4, 0u);
    if constexpr (!ROPE) {
      const int hh = wave - 4;  // this wave loaded the query of head wave & 3 = hh
      const float x0 = hh < r ? __low2float(q2_raw) : 0.f, x1 = hh < r ? __high2float(q2_raw) : 0.f;
      float of0, of1;
      mean_pair(ok_first, okp_first, of0, of1);
      const float d = wave_sum_all(x0 * of0 + x1 * of1);
      if (lane == 0) lds_write32(SM::kQoFirst + hh * 4, __float_as_uint(d * scale_log2e));
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  // residual (Sec. 3.2): wave w < 4 of the last live split takes rows [16 w, 16 w + 16); a load instruction
  // covers four consecutive rows (16 lanes x 16 bytes each); rows beyond the capacity are clamped and masked later
  const bool res_wave = res.k != nullptr && res_here && wave < 4;
  uint4 rk[4], rv[4];
  int res_len = 0;
  auto load_residual_rows = [&]() {
    const int64_t unit_row = (int64_t)(b * g.n_kv_heads + h) * res.capacity;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = min(16 * wave + 4 * u + (lane >> 4), res.capacity - 1);
      rk[u] = *reinterpret_cast<const uint4*>(res.k + (unit_row + row) * kHeadDim + (lane & 15) * 8);
      rv[u] = *reinterpret_cast<const uint4*>(res.v + (unit_row + row) * kHeadDim + (lane & 15) * 8);
    }
  };
  if (res_wave) {
    // (the persistent instance fetches the rows where it stages them: thirty-two registers held from here
    // to there do not fit beside its other state; fetching and staging them at the segment's start through
    // waves 4..7, which reach a segment first, was measured and is no faster)
    if constexpr (!FLAT && !LEGACY) load_residual_rows();
    res_len = res.lens[b];
  }
  // The wave's second group goes out behind the first ones of all waves; every later group is requested when
  // the one before it is about to be needed (see process_group).  The compute unit's address pipeline takes
  // about 28 cycles per 1 KiB load instruction and a wave blocks at a load that cannot be accepted yet: a wave
  // that asks for more at once sits at its load instructions while the data of its first group is already in
  // its registers.  The per-split instance asks for the second group behind the first barrier and the residual
  // tile (the barrier then does not wait for eight waves' worth of load issue: 15.55 -> 15.17 us on the
  // 8 x 8192-token shape; behind the tile: 14.66 -> 14.38 us); the persistent instance, whose segments start
  // cold, in front of the barrier.
  // ROPE: operands of one batch of the mean term (four groups gi0, gi0 + NW, ...).  The four lanes of a quad own the four
  // heads of one group; for the loads they split the group's 16 pairs (i, i + 64) of this lane's channel range: lane c
  // of the quad takes four pairs of the mean row and of the block's (cos, sin) row.
  struct RopeIn {
    uint2 oa, ob;                // fp16 form: four channels from i0 and from 64 + i0
    uint32_t oaq, obq, oap, obp; // 4-bit form: their codes (two bytes each), (min, step) of their 32-channel groups
    float4 c01, c23;
  };
  RopeIn rin = {};
  auto rope_load = [&](int gi0) {
    const int bi = n16 >> 2, c = n16 & 3;
    // groups past the end are clamped into the tables (their results are never read)
    const int tg = token_up_to(token_of_group(t0, gi0 + NW * bi), cap_tokens - 64);
    const unsigned char* rec = g.rope + kRopeBlkOff + (int64_t)(tg >> 6) * kRopeBlkStride;
    const int i0 = 32 * (c >> 1) + 8 * rho + 4 * (c & 1);
    const int64_t row = mean_base + shift_group(tg);
    if constexpr (DQ) {
      const unsigned char* mr = reinterpret_cast<const unsigned char*>(kc.means) + row * kDqMeanRec;
      rin.oaq = *reinterpret_cast<const uint16_t*>(mr + (i0 >> 1));
      rin.obq = *reinterpret_cast<const uint16_t*>(mr + ((64 + i0) >> 1));
      rin.oap = *reinterpret_cast<const uint32_t*>(mr + kDqMeanPar + 4 * (i0 >> 5));
      rin.obp = *reinterpret_cast<const uint32_t*>(mr + kDqMeanPar + 4 * ((64 + i0) >> 5));
    } else {
      const __half* orow = kc.means + row * kHeadDim;
      rin.oa = *reinterpret_cast<const uint2*>(orow + i0);
      rin.ob = *reinterpret_cast<const uint2*>(orow + 64 + i0);
    }
    rin.c01 = reinterpret_cast<const float4*>(rec)[i0 >> 1];  // (cos, sin) of pairs i0, i0 + 1
    rin.c23 = reinterpret_cast<const float4*>(rec)[(i0 >> 1) + 1];
  };
  if constexpr (ROPE) rope_load(wslot);
  if constexpr (FLAT) load_group(wslot + NW, wslot + NW < n_grp, S1);
  __syncthreads();
  if constexpr (FLAT && !LEGACY) {
    // segments are short and start cold: three groups per wave go out before the first is used, and the set
    // that a group leaves takes the group three rounds on (see process_group)
    load_group(wslot + 2 * NW, wslot + 2 * NW < n_grp, S2);
  }

  // B operands of the score contraction (see the header): for tile parity p and k-step s the lane's eight
  // k-slots are channels [32 c + 8 s, +8) of head n % 4: hi part if n / 4 == p, lo part if n / 4 == p + 2,
  // zero otherwise
  const int nu = n16 >> 2;
  auto operand_addr = [&](int parity, uint32_t hi_arr, uint32_t lo_arr) -> uint32_t {
    const uint32_t off = head * 256 + rho * 64;
    return nu == parity ? hi_arr + off : nu == parity + 2 ? lo_arr + off : (uint32_t)SM::kZero;
  };
  h8 P0[4], P1[4];
  {
    const uint32_t a0 = operand_addr(0, SM::kQhi, SM::kQlo), a1 = operand_addr(1, SM::kQhi, SM::kQlo);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      P0[s] = __builtin_bit_cast(h8, lds_read128(a0 + 16 * s));
      P1[s] = __builtin_bit_cast(h8, lds_read128(a1 + 16 * s));
      if constexpr (SGN) {  // lanes of odd groups gather the codewords' high halves first
        const u4v x = __builtin_bit_cast(u4v, P0[s]), y = __builtin_bit_cast(u4v, P1[s]);
        const bool odd = rho & 1;
        P0[s] = __builtin_bit_cast(h8, u4v{odd ? x.z : x.x, odd ? x.w : x.y, odd ? x.x : x.z, odd ? x.y : x.w});
        P1[s] = __builtin_bit_cast(h8, u4v{odd ? y.z : y.x, odd ? y.w : y.y, odd ? y.x : y.z, odd ? y.y : y.w});
      }
    }
  }

  // ---- per-lane state: one head (lane % 4), partial sums over the lane's tokens -----------------
  float m_run = -INFINITY, l_run = 0.f, beta = 0.f, cf = 1.f;
  float qo[ROPE ? 4 : 1] = {};  // q . o^k (ROPE: of each of the lane's four tokens)
  float a_run = 0.f, w_scale = 0.f;  // A (power of two >= every a^v so far; 0 = none yet) and 2^10 / A
  f4 acc[8];                         // out_rot partial sums: component = head, see the epilogue for the channel
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = f4{0.f, 0.f, 0.f, 0.f};
  float accm[4][2];  // mean-vector term, channels 2 lane, 2 lane + 1 of the four heads
#pragma unroll
  for (int i = 0; i < 4; ++i) accm[i][0] = accm[i][1] = 0.f;
  int cur_group = -1;
  float ov0 = 0.f, ov1 = 0.f;
  const uint32_t laneoff = SUB == 4 ? (lane & 31) * 8 : (lane & 15) * 8;  // the lane's copy of the table

  auto half_lo = [](uint32_t u) -> float { return (float)__builtin_bit_cast(_Float16, (uint16_t)(u & 0xffffu)); };
  auto half_hi = [](uint32_t u) -> float { return (float)__builtin_bit_cast(_Float16, (uint16_t)(u >> 16)); };

  // mean-vector term of the Shift group that just ended: accm = accm * cf + (sum of beta) * o^v
  auto flush_group = [&]() {
    const float bs = head_sum(beta);
    const float bsum[4] = {quad_bcast<0>(bs), quad_bcast<1>(bs), quad_bcast<2>(bs), quad_bcast<3>(bs)};
    const float cfh[4] = {quad_bcast<0>(cf), quad_bcast<1>(cf), quad_bcast<2>(cf), quad_bcast<3>(cf)};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      accm[i][0] = accm[i][0] * cfh[i] + bsum[i] * ov0;
      accm[i][1] = accm[i][1] * cfh[i] + bsum[i] * ov1;
    }
    beta = 0.f;
    cf = 1.f;
  };

  // d4 for the lane's four tokens (scores s in log2 units); returns the fp16 weights p a^v 2^10 / A as the value-side A
  // operand.  Masked tokens come in with s = -inf and zero av, bv.
  auto softmax_step = [&](const float (&s)[4], const float (&av)[4], const float (&bv)[4]) -> h4 {
    const float smax = max3f(s[0], s[1], max2f(s[2], s[3]));
    const float amax = max3f(av[0], av[1], max2f(av[2], av[3]));
    const bool need = (smax - m_run > kLazyMaxLog2) || (amax > a_run);
    if (__any(need)) {
      const float m_new = max2f(m_run, head_max(smax));
      const float corr = (m_run == -INFINITY) ? 0.f : fast_exp2(m_run - m_new);
      l_run *= corr, beta *= corr, cf *= corr;
      m_run = m_new;
      // A: the next power of two >= the largest a^v of the wave (kept once it is large enough)
      const float amax_w = wave_max_all(amax);
      float a_new = a_run;
      if (amax_w > a_run) a_new = __uint_as_float((__float_as_uint(amax_w) + 0x007fffffu) & 0x7f800000u);
      const float a_inv = (a_new > 0.f) ? __builtin_amdgcn_rcpf(a_new) : 0.f;  // exact: a power of two
      const float a_ratio = a_run * a_inv;
      a_run = a_new;
      w_scale = kWeightScale * a_inv;
      const f4 c4 = {quad_bcast<0>(corr) * a_ratio, quad_bcast<1>(corr) * a_ratio, quad_bcast<2>(corr) * a_ratio,
                     quad_bcast<3>(corr) * a_ratio};
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] *= c4;
    }
    float w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float p = fast_exp2(s[k] - m_run);  // 0 for masked tokens
      l_run += p;
      beta = fmaf(p, bv[k], beta);
      w[k] = p * (av[k] * w_scale);
    }
    const h2v w01 = __builtin_convertvector(f2v{w[0], w[1]}, h2v), w23 = __builtin_convertvector(f2v{w[2], w[3]}, h2v);
    return h4{w01[0], w01[1], w23[0], w23[1]};
  };

  // The wave's sums over its four 16-lane groups: acc[X] of lane (rho, m, e) is a partial sum over the
  // tokens of group rho.  Two lane-swap rounds add the groups: afterwards red[j][head] of lane (rho, m, e)
  // is the wave's sum for accumulator X = j + 2 (rho & 1) + 4 (rho >> 1), times `factor`.
  auto reduce_acc = [&](float factor, float (&red)[2][4]) {
    // the swaps read registers that matrix instructions wrote: nothing may move across this point, and the
    // longest matrix instruction has drained after sixteen idle cycles
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    float red4[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float a = acc[x][i], b = acc[x + 4][i];
        lane_swap32(a, b);
        red4[x][i] = a + b;
      }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float a = red4[x][i], b = red4[x + 2][i];
        lane_swap16(a, b);
        red[x][i] = (a + b) * factor;
      }
  };
  const int m_res = n16 >> 2, e_res = n16 & 3;  // value-side result lane: block m, column e
  const uint32_t mbase = SM::kMerge + wave * SM::kMergeWave, mlbase = SM::kMl + wave * SM::kMlWave;

  // ---- residual: one 16-token tile of fp16 rows per wave, before the wave's coded groups -----------
  // fp16 key rows are the A operand as they are, the B operand is the UNROTATED query, and the value rows
  // accumulate in the original domain: their sum becomes the start value of the mean-vector term.
  if (res_wave) {
    const int rl = min(res_len, res.capacity);
    if (rl > 16 * wave) {  // wave-uniform
      const uint32_t sk = SM::kRes + wave * SM::kResWave, sv = ROPE ? sk : sk + 16 * SM::kResKStride;
      if constexpr (FLAT || LEGACY) load_residual_rows();
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = 4 * u + (lane >> 4);  // row of the tile; rows past the valid count are stored as zeros
        const bool live = 16 * wave + row < rl;
        const u4v kx = live ? u4v{rk[u].x, rk[u].y, rk[u].z, rk[u].w} : u4v{0u, 0u, 0u, 0u};
        const u4v vx = live ? u4v{rv[u].x, rv[u].y, rv[u].z, rv[u].w} : u4v{0u, 0u, 0u, 0u};
        if constexpr (ROPE) {
          lds_write128(sk + row * 256 + (((lane & 15) ^ row) << 4), kx);
          rv[u] = make_uint4(vx.x, vx.y, vx.z, vx.w);  // (they take the keys' place once the scores are there)
        } else {
          lds_write128(sk + row * SM::kResKStride + (lane & 15) * 16, kx);
          lds_write64(sv + row * SM::kResVStride + (lane & 15) * 16, u2v{vx.x, vx.y});
          lds_write64(sv + row * SM::kResVStride + (lane & 15) * 16 + 8, u2v{vx.z, vx.w});
        }
      }
      // written and read by different lanes of this one wave
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int par = wave & 1;
      const uint32_t ua = operand_addr(par, SM::kUhi, SM::kUlo);
      f4 D = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        // row = token n of the tile, channels [32 rho + 8 s, +8)
        const uint32_t chunk = 4 * rho + s;
        const h8 A = __builtin_bit_cast(h8, lds_read128(sk + n16 * SM::kResKStride + (ROPE ? chunk ^ n16 : chunk) * 16));
        const h8 B = __builtin_bit_cast(h8, lds_read128(ua + 16 * s));
        D = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, B, D, 0, 0, 0);
      }
      // hi + lo columns; the lanes of tile `wave` (n / 4 == wave) hold its scores, all others are masked
      float sc[4];
      const float zero[4] = {0.f, 0.f, 0.f, 0.f};
      float one[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool valid = tile_of_lane == wave && (16 * wave + 4 * rho + k) < rl;
        const float x = D[k] + dpp_mov<0x128>(D[k]);
        sc[k] = valid ? x : -INFINITY;
        one[k] = valid ? 1.f : 0.f;
      }
      const h4 wop = softmax_step(sc, one, zero);
      // value rows: source lane (rho, k = n / 4, m = n % 4) reads token 4 rho + k of the tile, channels
      // [4 (4 X + m), +4); the transposing read hands lane (rho, m, e) four tokens of channel 16 X + 4 m + e
      if constexpr (ROPE) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int row = 4 * u + (lane >> 4);
          lds_write128(sv + row * 256 + (((lane & 15) ^ row) << 4), u4v{rv[u].x, rv[u].y, rv[u].z, rv[u].w});
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      const int vr = 4 * rho + (n16 >> 2);
      const uint32_t vrow = sv + vr * SM::kResVStride + (ROPE ? (n16 & 1) : (n16 & 3)) * 8;
      auto vaddr = [&](int X) -> uint32_t {  // channels 4 (4 X + n % 4) .. + 3 of row vr
        return ROPE ? vrow + (((2 * X + ((n16 >> 1) & 1)) ^ vr) << 4) : vrow + X * 32;
      };
      static_for<4>([&](auto tc) {
        constexpr int T = decltype(tc)::value;
        if (wave == T) {  // `abid` is an immediate
          static_for<8>([&](auto xc) {
            constexpr int X = decltype(xc)::value;
            acc[X] = __builtin_amdgcn_mfma_f32_4x4x4f16(wop, lds_tr64(vaddr(X)), acc[X], 2, T, 0);
          });
        }
      });
      // the sums change domain: through the wave's own merge slot into the mean-term registers
      float red[2][4];
      reduce_acc(a_run * (1.0f / kWeightScale), red);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int ch = 16 * (j + 2 * (rho & 1) + 4 * (rho >> 1)) + 4 * m_res + e_res;
#pragma unroll
        for (int i = 0; i < 4; ++i) lds_write32(mbase + 2048 + (i * 128 + ch) * 4, __float_as_uint(red[j][i]));
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const u2v v2 = lds_read64(mbase + 2048 + (i * 128 + 2 * lane) * 4);
        accm[i][0] = __uint_as_float(v2.x), accm[i][1] = __uint_as_float(v2.y);
      }
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] = f4{0.f, 0.f, 0.f, 0.f};
      cf = 1.f;
    }
  }
  // (per-split instance: the wave's second group, see above; behind the residual tile, which needs no loads, so
  // that a wave with a tile asks out of the way of the other waves' load issue)
  if constexpr (!FLAT) load_group(wslot + NW, wslot + NW < n_grp, S1);

  // Gathers and contractions of one group, in batches.  Key side: sixteen matrix instructions in four
  // batches of four (tiles (0, 2) or (1, 3) x two k-steps, so that consecutive instructions alternate
  // between the two accumulators).  Value side: one batch per tile, eight transposed operands
  // (SUB = 4: sub-vectors 4 X + m; SUB = 8: sub-vectors 4 x + m as two halves, accumulator 2 x + hf).
  auto k_gather = [&](auto bc, const Regs& G, h8 (&A)[4]) {  // A[2 * sp + tp]: tile 2 tp + (B & 1), k-step 2 (B >> 1) + sp
    constexpr int B = decltype(bc)::value;
    static_for<4>([&](auto ec) {
      constexpr int E = decltype(ec)::value;
      constexpr int T = 2 * (E & 1) + (B & 1), S = 2 * (B >> 1) + (E >> 1);
      if constexpr (SGN) {
        constexpr uint32_t sel = 0x0c0c0000u | ((4 + S) << 8) | S;  // code byte << 8 | sign byte
        const u2v c0 = lds_read64(perm_b32(G.kc[T], G.kc[4 + T], sel)), c1 = lds_read64(perm_b32(G.kc[T], G.kx[T], sel));
        A[E] = __builtin_bit_cast(h8, u4v{c0.x, c0.y, c1.x, c1.y});
      } else if constexpr (SUB == 4) {
        const uint32_t w = G.kc[2 * T + (S >> 1)];
        const u2v c0 = lds_read64(table_addr<2 * (S & 1)>(w, laneoff));
        const u2v c1 = lds_read64(table_addr<2 * (S & 1) + 1>(w, laneoff));
        A[E] = __builtin_bit_cast(h8, u4v{c0.x, c0.y, c1.x, c1.y});
      } else {
        const uint32_t at = table_addr<S>(G.kc[T], laneoff);
        const u2v c0 = lds_read64(at), c1 = lds_read64(at + 128);
        A[E] = __builtin_bit_cast(h8, u4v{c0.x, c0.y, c1.x, c1.y});
      }
    });
  };
  auto k_contract = [&](auto bc, const h8 (&A)[4], f4& D0, f4& D1) {
    constexpr int B = decltype(bc)::value;
    static_for<4>([&](auto ec) {
      constexpr int E = decltype(ec)::value;
      constexpr int S = 2 * (B >> 1) + (E >> 1);
      if constexpr ((E & 1) == 0)  // tiles 0, 1 -> D0; tiles 2, 3 -> D1
        D0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[E], (B & 1) ? P1[S] : P0[S], D0, 0, 0, 0);
      else
        D1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[E], (B & 1) ? P1[S] : P0[S], D1, 0, 0, 0);
    });
  };
  auto v_gather = [&](auto tc, const Regs& G, h4 (&Bv)[8]) {
    constexpr int T = decltype(tc)::value;
    static_for<8>([&](auto xc) {
      constexpr int X = decltype(xc)::value;
      if constexpr (SGN) {
        constexpr uint32_t sel = 0x0c0c0000u | ((4 + (X >> 1)) << 8) | (X >> 1);
        Bv[X] = lds_tr64(perm_b32(G.vc[T], (X & 1) ? G.vx[T] : G.vc[4 + T], sel));
      } else if constexpr (SUB == 4)
        Bv[X] = lds_tr64(table_addr<X & 3>(G.vc[2 * T + (X >> 2)], laneoff));
      else
        Bv[X] = lds_tr64(table_addr<(X >> 1)>(G.vc[T], laneoff) + (X & 1) * 128);
    });
  };
  auto v_contract = [&](auto tc, const h4 (&Bv)[8], const h4& wop) {
    constexpr int T = decltype(tc)::value;
    static_for<8>([&](auto xc) {
      constexpr int X = decltype(xc)::value;
      acc[X] = __builtin_amdgcn_mfma_f32_4x4x4f16(wop, Bv[X], acc[X], 2, T, 0);
    });
  };
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  constexpr std::integral_constant<int, 2> c2{};
  constexpr std::integral_constant<int, 3> c3{};

  // ROPE: q . RoPE_t(o^k) (log2 units) for the 64 tokens of the batch of four groups whose operands are in `rin`.  With
  // t = 64 block + j and the channel pairs (i, i' = i + 64),   q . RoPE_t(o) = sum_i cos(j w_i) A'_i + sin(j w_i) B'_i,
  //   A'_i = q_i ro_i + q_i' ro_i',  B'_i = q_i' ro_i - q_i ro_i',  ro = RoPE_(64 block)(o):
  // a [64 tokens x 128] x [128 x heads] contraction whose token-side operand is the same for every group.  Rows =
  // (group, head), columns = 16 tokens; both sides in fp16 hi + lo parts, three products.  Lane (n, rho) supplies row
  // (group n / 4, head n % 4) at channels 32 ks + 8 rho + e and column n of the token-side table.
  auto rope_compute = [&]() {
    float rl[4], rh[4];  // the block's turned mean (times the score scale) at this lane's four pairs
    {
      const uint32_t oaw[2] = {rin.oa.x, rin.oa.y}, obw[2] = {rin.ob.x, rin.ob.y};
      const float cs[8] = {rin.c01.x, rin.c01.y, rin.c01.z, rin.c01.w, rin.c23.x, rin.c23.y, rin.c23.z, rin.c23.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float o0 = DQ ? dq_level(rin.oap, (rin.oaq >> (4 * e)) & 15u) : (e & 1) ? half_hi_f(oaw[e >> 1]) : half_lo_f(oaw[e >> 1]);
        const float o1 = DQ ? dq_level(rin.obp, (rin.obq >> (4 * e)) & 15u) : (e & 1) ? half_hi_f(obw[e >> 1]) : half_lo_f(obw[e >> 1]);
        const float cc = cs[2 * e] * scale_log2e, ss = cs[2 * e + 1] * scale_log2e;
        rl[e] = o0 * cc - o1 * ss;
        rh[e] = o1 * cc + o0 * ss;
      }
    }
    h8 AH[4], AL[4];
    static_for<4>([&](auto cc) {  // chunk c of the quad's lane c: four pairs from i0
      constexpr int c = decltype(cc)::value, ksp = c >> 1, hf = c & 1;
      const int i0 = 32 * ksp + 8 * rho + 4 * hf;
      const u4v a4 = lds_read128(SM::kQorig + (head * 128 + i0) * 4), b4 = lds_read128(SM::kQorig + (head * 128 + 64 + i0) * 4);
      const float qa[4] = {__uint_as_float(a4.x), __uint_as_float(a4.y), __uint_as_float(a4.z), __uint_as_float(a4.w)};
      const float qb[4] = {__uint_as_float(b4.x), __uint_as_float(b4.y), __uint_as_float(b4.z), __uint_as_float(b4.w)};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float xl = quad_bcast<c>(rl[e]), xh = quad_bcast<c>(rh[e]);
        const float Ap = qa[e] * xl + qb[e] * xh, Bp = qb[e] * xl - qa[e] * xh;
        const _Float16 ah = (_Float16)Ap, bh = (_Float16)Bp;
        AH[ksp][4 * hf + e] = ah;
        AL[ksp][4 * hf + e] = (_Float16)(Ap - (float)ah);
        AH[ksp + 2][4 * hf + e] = bh;
        AL[ksp + 2][4 * hf + e] = (_Float16)(Bp - (float)bh);
      }
    });
    // (the previous batch's entries, or the residual's, have been read: the values above depend on nothing of theirs,
    // but LDS accesses of one wave are served in order)
    static_for<4>([&](auto tc) {
      constexpr int tile = decltype(tc)::value;
      f4 d = {0.f, 0.f, 0.f, 0.f};
      const uint32_t row_addr = SM::kTurn + (16 * tile + n16) * 256;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const uint32_t a = row_addr + (((4 * ks + rho) ^ n16) << 4);
        const h8 th = __builtin_bit_cast(h8, lds_read128(a));
        const h8 tl = __builtin_bit_cast(h8, lds_read128(a + 16384));
        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(AH[ks], th, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(AL[ks], th, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(AH[ks], tl, d, 0, 0, 0);
      }
      // this lane holds group rho, token 16 tile + n, heads 0..3; entry [group][head][token], the token's 16-token
      // block XORed with the group (the four groups then write to different banks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        lds_write32(mbase + rho * 1024 + i * 256 + (16 * (tile ^ rho) + n16) * 4, __float_as_uint(d[i]));
    });
    // the entries are read back by other lanes of this wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  // One group: scores, softmax, value accumulation.  `G` holds the group's bytes, KA / KB the first two
  // key-side gather batches of it (issued while the previous group's value side was running); they are
  // refilled for `Gn`, the wave's next group, before this group's last matrix instructions are issued.
  // A gather batch is always issued two batches ahead of its matrix instructions; scheduling barriers keep
  // the compiler from sinking the gathers next to their uses, which would expose the LDS latency at
  // every one of the 48 matrix instructions of a group.
  // (inside a stage the matrix instructions go first: the operands they consume are dead before the next
  // gathers land, so a later batch can take over an earlier one's registers)
  h8 KA[4], KB[4];
  // it: position of the group in its batch of four (ROPE)
  auto process_group = [&](auto itc, int gi, Regs& G, Regs& Gn, Regs& Gnn) {
    constexpr int it = decltype(itc)::value;
    const int tg = t0 + (gi << 6);
    if constexpr (ROPE) {
      const u4v r4 = lds_read128(mbase + it * 1024 + head * 256 + (16 * (rho ^ it) + 4 * tile_of_lane) * 4);
      qo[0] = __uint_as_float(r4.x), qo[1] = __uint_as_float(r4.y), qo[2] = __uint_as_float(r4.z),
      qo[3] = __uint_as_float(r4.w);
    }
    // Shift group bookkeeping (wave-uniform)
    const int grp = shift_group(tg);
    if (grp != cur_group) {
      if (cur_group >= 0) flush_group();
      if constexpr (ROPE) {
        // the mean term is per token (below)
      } else if (grp == grp_first) {
        qo[0] = lds_read32f(SM::kQoFirst + head * 4);
      } else {
        float o0, o1;
        mean_pair(G.ok, G.okp, o0, o1);
        float qd[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const u2v q2u = lds_read64(SM::kQorig + (i * 128 + 2 * lane) * 4);
          qd[i] = wave_sum_all(__uint_as_float(q2u.x) * o0 + __uint_as_float(q2u.y) * o1);
        }
        const float lo01 = (head & 1) ? qd[1] : qd[0], hi23 = (head & 1) ? qd[3] : qd[2];
        qo[0] = ((head & 2) ? hi23 : lo01) * scale_log2e;
      }
      mean_pair(G.ov, G.ovp, ov0, ov1);
      cur_group = grp;
    }
    // d2/d3: HT(q) . C[codes] of the group's 64 tokens, four heads
    f4 D0 = {0.f, 0.f, 0.f, 0.f}, D1 = {0.f, 0.f, 0.f, 0.f};
    h8 KC[4], KD[4];
    h4 VA[8], VB[8], VC[8], VD[8];
    __builtin_amdgcn_sched_barrier(0);
    k_contract(c0, KA, D0, D1);
    __builtin_amdgcn_sched_barrier(0);
    k_gather(c2, G, KC);
    __builtin_amdgcn_sched_barrier(0);
    k_contract(c1, KB, D0, D1);
    __builtin_amdgcn_sched_barrier(0);
    k_gather(c3, G, KD);
    __builtin_amdgcn_sched_barrier(0);
    k_contract(c2, KC, D0, D1);
    __builtin_amdgcn_sched_barrier(0);
    v_gather(c0, G, VA);  // the first value-side gathers fly during the softmax arithmetic
    __builtin_amdgcn_sched_barrier(0);
    k_contract(c3, KD, D0, D1);
    __builtin_amdgcn_sched_barrier(0);
    v_gather(c1, G, VB);
    __builtin_amdgcn_sched_barrier(0);
    // hi + lo columns: lanes n < 8 take tiles 0, 1 from D0, lanes n >= 8 tiles 2, 3 from D1
    float sc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float x = D0[k] + dpp_mov<0x128>(D0[k]);
      const float y = D1[k] + dpp_mov<0x128>(D1[k]);
      sc[k] = (n16 < 8) ? x : y;
    }
    float ak[4], bk[4], av[4], bv[4];
    if constexpr (DQ) {  // b = min + step * code, a = b * a'
      const float apk[4] = {half_lo(G.nk.x), half_hi(G.nk.x), half_lo(G.nk.y), half_hi(G.nk.y)};
      const float apv[4] = {half_lo(G.nv.x), half_hi(G.nv.x), half_lo(G.nv.y), half_hi(G.nv.y)};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        bk[k] = dq_level(G.nk.w, (G.nk.z >> (4 * k)) & 15u), bv[k] = dq_level(G.nv.w, (G.nv.z >> (4 * k)) & 15u);
        ak[k] = bk[k] * apk[k], av[k] = bv[k] * apv[k];
      }
    } else {
      const uint32_t nkw[4] = {G.nk.x, G.nk.y, G.nk.z, G.nk.w}, nvw[4] = {G.nv.x, G.nv.y, G.nv.z, G.nv.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        ak[k] = half_lo(nkw[k]), bk[k] = half_hi(nkw[k]);
        av[k] = half_lo(nvw[k]), bv[k] = half_hi(nvw[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) sc[k] = fmaf(ak[k], sc[k], bk[k] * qo[ROPE ? k : 0]);
    if (tg > t_whole) {  // wave-uniform: only a sequence's last group has masked tokens (their bytes may be anything)
      asm volatile("");  // (or the compiler makes twelve selects of it that every group goes through)
      if (tg - base_tok > kRebase) {
        base_tok += kRebase;
        describe(t0 + (n_grp << 6));
        t_whole = base_tok + min(t1 - 64 - base_tok, kRebase);
      }
      const int tb0 = tg + tok_of_lane;  // the lane's first token
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool valid = (tb0 + k) < t1;
        sc[k] = valid ? sc[k] : -INFINITY, av[k] = valid ? av[k] : 0.f, bv[k] = valid ? bv[k] : 0.f;
      }
    }
    const h4 wop = softmax_step(sc, av, bv);

    // d5: out_rot[head][channel] += sum over tokens of weight * codeword channel
    __builtin_amdgcn_sched_barrier(0);
    v_contract(c0, VA, wop);
    __builtin_amdgcn_sched_barrier(0);
    v_gather(c2, G, VC);
    __builtin_amdgcn_sched_barrier(0);
    v_contract(c1, VB, wop);
    __builtin_amdgcn_sched_barrier(0);
    v_gather(c3, G, VD);
    __builtin_amdgcn_sched_barrier(0);
    // the group after the next one: requested just before the next one's bytes are first needed (below)
    // (this group's bytes have all been used by now)
    if constexpr (FLAT && !LEGACY)
      load_group(gi + 3 * NW, gi + 3 * NW < n_grp, G);
    else {
      // (the registers of the Shift vectors, which only a change of the Shift group reads, are nobody's temporaries: a write to
      // one would wait for every load in flight)
      if constexpr (!FLAT && !LEGACY) asm volatile("" ::"v"(Gnn.ok), "v"(Gnn.ov));
      load_group(gi + 2 * NW, gi + 2 * NW < n_grp, Gnn);
    }
    if constexpr (ROPE && it == 3) rope_load(gi + NW);  // the next batch
    __builtin_amdgcn_sched_barrier(0);
    v_contract(c2, VC, wop);
    __builtin_amdgcn_sched_barrier(0);
    arrange(Gn);
    __builtin_amdgcn_sched_barrier(0);
    // (any bytes are valid table indices: harmless when there is no next group; ROPE: the next batch's operands come
    // first, these gathers would only hold registers meanwhile)
    if constexpr (!(ROPE && it == 3)) k_gather(c0, Gn, KA);
    __builtin_amdgcn_sched_barrier(0);
    v_contract(c3, VD, wop);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!(ROPE && it == 3)) k_gather(c1, Gn, KB);
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- main loop: this wave's groups wave, wave + NW, ...; three register sets rotate (in use, next, in flight) ----
  if (wslot < n_grp) {
    int gi = wslot;
    arrange(S0);
    // Legacy layout: two register sets; the set that a group leaves takes the group after the next.  (One plain loop per
    // format: with the rotary batches as an outer loop of both, whose exit the inner one had taken already, the compiler
    // made three nested loops of it and spilled 61 to 79 registers in the split instances of sign codes with 4-bit side
    // information: 146.7 us for four launches of 8 x 8192 tokens, 82.2 so.)
    if constexpr (ROPE) {
      while (true) {
        rope_compute();
        k_gather(c0, S0, KA);
        k_gather(c1, S0, KB);
        process_group(c0, gi, S0, S1, S0);
        gi += NW;
        if (gi >= n_grp) break;
        process_group(c1, gi, S1, S0, S1);
        gi += NW;
        if (gi >= n_grp) break;
        process_group(c2, gi, S0, S1, S0);
        gi += NW;
        if (gi >= n_grp) break;
        process_group(c3, gi, S1, S0, S1);
        gi += NW;
        if (gi >= n_grp) break;
      }
    } else if constexpr (SGN) {
      k_gather(c0, S0, KA);
      k_gather(c1, S0, KB);
      while (true) {
        process_group(c0, gi, S0, S1, S0);
        gi += NW;
        if (gi >= n_grp) break;
        process_group(c1, gi, S1, S0, S1);
        gi += NW;
        if (gi >= n_grp) break;
      }
    } else {
      k_gather(c0, S0, KA);
      k_gather(c1, S0, KB);
      while (true) {
        process_group(c0, gi, S0, S1, S2);
        gi += NW;
        if (gi >= n_grp) break;
        process_group(c0, gi, S1, S2, S0);
        gi += NW;
        if (gi >= n_grp) break;
        process_group(c0, gi, S2, S0, S1);
        gi += NW;
        if (gi >= n_grp) break;
      }
    }
  }
  if (cur_group >= 0) flush_group();
  // the window of the unit that the next segment begins (pages 0..63), back before that segment asks for it
  if constexpr (FLAT && PAGED) load_window(nb, 0, nwin_k, nwin_v);

  // ---- epilogue: this wave's sums -> its merge slot ------------------------------------------------
  {
    float red[2][4];
    reduce_acc(a_run * (1.0f / kWeightScale), red);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int X = j + 2 * (rho & 1) + 4 * (rho >> 1);
      int ch;
      if constexpr (SUB == 4)
        ch = 16 * X + 4 * m_res + e_res;
      else  // X = 2 x + hf: sub-vector 4 x + m, half hf (sign codes: hf ^ (m & 1), odd lanes gather the other half first)
        ch = 8 * (4 * (X >> 1) + m_res) + 4 * ((X & 1) ^ (SGN ? m_res & 1 : 0)) + e_res;
#pragma unroll
      for (int i = 0; i < 4; ++i) lds_write32(mbase + (i * 128 + ch) * 4, __float_as_uint(red[j][i]));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      lds_write64(mbase + 2048 + (i * 128 + 2 * lane) * 4, u2v{__float_as_uint(accm[i][0]), __float_as_uint(accm[i][1])});
    const float l_tot = head_sum(l_run);
    if (lane < 4) lds_write64(mlbase + lane * 8, u2v{__float_as_uint(m_run), __float_as_uint(l_tot)});
  }
  __syncthreads();

  // ---- merge the waves: wave i takes head i, a lane channels 2 lane, 2 lane + 1 ------------------
  [&]() {
  if (wave >= r) return;
  const int hh = wave;
  float M = -INFINITY, L = 0.f, x0 = 0.f, x1 = 0.f, mm0 = 0.f, mm1 = 0.f;
  {
    float mw[NW], lw[NW];
    f2v rw[NW], qw[NW];
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      const uint32_t mb = SM::kMerge + wv * SM::kMergeWave;
      const u2v ml = lds_read64(SM::kMl + wv * SM::kMlWave + hh * 8);
      mw[wv] = __uint_as_float(ml.x), lw[wv] = __uint_as_float(ml.y);
      rw[wv] = __builtin_bit_cast(f2v, lds_read64(mb + (hh * 128 + 2 * lane) * 4));
      qw[wv] = __builtin_bit_cast(f2v, lds_read64(mb + 2048 + (hh * 128 + 2 * lane) * 4));
    }
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) M = fmaxf(M, mw[wv]);
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      const float e = (mw[wv] == -INFINITY) ? 0.f : fast_exp2(mw[wv] - M);
      L = fmaf(e, lw[wv], L);
      x0 = fmaf(e, rw[wv][0], x0), x1 = fmaf(e, rw[wv][1], x1);
      mm0 = fmaf(e, qw[wv][0], mm0), mm1 = fmaf(e, qw[wv][1], mm1);
    }
  }

  // ---- d6: merge the splits; the last wave to arrive for this query head finishes it -------------
  if (n_live > 1) {
    // !FLAT: partial [sequence][query head][split].  FLAT: [run][slot][query head of the unit]: slot 0 for
    // the segment that continues a unit begun in an earlier run, slot 1 for the one that begins a unit and
    // leaves its end to the next run (a run has at most one of each); run c of the unit's runs
    // first_run .. first_run + n_live - 1 therefore wrote slot 1 if c == first_run, else slot 0.
    auto partial_of = [&](int s) -> float* {
      if constexpr (FLAT)
        return partial + ((int64_t)((first_run + s) * 2 + (s == 0 ? 1 : 0)) * min(n_rep, 4) + hh) * kPartialStride;
      else
        return partial + ((int64_t)(b * g.n_q_heads + hq0 + hh) * n_splits + s) * kPartialStride;
    };
    float* P = partial_of(split);
    auto st2 = [](float* p, float lo, float hi) {  // 8-byte device-scope store (p is 8-byte aligned)
      __hip_atomic_store(reinterpret_cast<unsigned long long*>(p),
                         ((unsigned long long)__float_as_uint(hi) << 32) | __float_as_uint(lo), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    };
    auto ld2 = [](const float* p) -> float2 {
      const unsigned long long u = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
      return make_float2(__uint_as_float((uint32_t)u), __uint_as_float((uint32_t)(u >> 32)));
    };
    st2(P + 2 * lane, x0, x1);
    st2(P + kHeadDim + 2 * lane, mm0, mm1);
    if (lane == 0) st2(P + 2 * kHeadDim, M, L);
    // The partials are written with device-scope stores (they go through to memory: no cache holds them
    // back), the wave waits until every one has been acknowledged, and only then counts itself in; the
    // wave that reads n_live - 1 reads the other splits' partials with device-scope loads (they do not hit
    // in a cache that could hold older bytes).  The agent-scope release / acquire fences that would say
    // the same in the memory model make the compiler write back and invalidate the whole L2 around
    // the counter update: measured 7 us + 4 us per launch on the 8 x 8192-token shape.
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    int* cnt = counters + (b * g.n_q_heads + hq0 + hh) * kCounterStrideInts;
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old != n_live - 1) return;
    if (lane == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next call
    // chunks of SF splits, every load of a chunk issued before its first use (a chunk costs one trip to
    // memory); running max across chunks.  Up to eight live splits take one chunk of eight, more take chunks
    // of thirty-two (the loop's registers are free by now).
    M = -INFINITY, L = 0.f, x0 = x1 = mm0 = mm1 = 0.f;
    auto merge_chunks = [&](auto sfc) {
      constexpr int SF = decltype(sfc)::value;
      for (int s0 = 0; s0 < n_live; s0 += SF) {
        float2 pml[SF], pr[SF], pq[SF];
#pragma unroll
        for (int s = 0; s < SF; ++s) {
          pml[s] = make_float2(-INFINITY, 0.f);
          pr[s] = pq[s] = make_float2(0.f, 0.f);
          if (s0 + s < n_live) {  // uniform
            const float* ps = partial_of(s0 + s);
            pml[s] = ld2(ps + 2 * kHeadDim);
            pr[s] = ld2(ps + 2 * lane);
            pq[s] = ld2(ps + kHeadDim + 2 * lane);
          }
        }
        float Mn = M;
#pragma unroll
        for (int s = 0; s < SF; ++s) Mn = fmaxf(Mn, pml[s].x);
        if (Mn > -INFINITY) {
          const float corr = (M == -INFINITY) ? 0.f : fast_exp2(M - Mn);
          L *= corr, x0 *= corr, x1 *= corr, mm0 *= corr, mm1 *= corr;
#pragma unroll
          for (int s = 0; s < SF; ++s) {
            const float e = (s0 + s < n_live) ? fast_exp2(pml[s].x - Mn) : 0.f;
            L = fmaf(e, pml[s].y, L);
            x0 = fmaf(e, pr[s].x, x0), x1 = fmaf(e, pr[s].y, x1);
            mm0 = fmaf(e, pq[s].x, mm0), mm1 = fmaf(e, pq[s].y, mm1);
          }
          M = Mn;
        }
      }
    };
    if (n_live <= 8)
      merge_chunks(std::integral_constant<int, 8>{});
    else
      merge_chunks(std::integral_constant<int, 32>{});
  }
  // one inverse Hadamard per head (H is its own inverse), across the wave's lanes in registers
  {
    const float a0 = x0 + x1, a1 = x0 - x1;
    x0 = a0, x1 = a1;
  }
  static_for<6>([&](auto kc_) {
    constexpr int m = 1 << decltype(kc_)::value;
    const float p0 = xor_reg<m>(x0), p1 = xor_reg<m>(x1);
    const bool upper = (lane & m) != 0;
    x0 = upper ? p0 - x0 : x0 + p0;
    x1 = upper ? p1 - x1 : x1 + p1;
  });
  float2 o2 = make_float2(0.f, 0.f);
  if (L > 0.f) o2 = make_float2((x0 * (float)kInvSqrtD + mm0) / L, (x1 * (float)kInvSqrtD + mm1) / L);
  *reinterpret_cast<float2*>(out + (int64_t)(b * g.n_q_heads + hq0 + hh) * kHeadDim + 2 * lane) = o2;
  }();
  if constexpr (!FLAT) break;
  if (run_pos >= run_end) break;
  b = nb, hu = nh;  // the next unit (its first row and length are on their way or here)
  first_segment = false;
  if constexpr (PAGED) win0 = 0, win_k = nwin_k, win_v = nwin_v;
  }  // segments
}


// what one launch is given (host side)
struct Call {
  Geometry g;
  const void *codebook, *q;
  CacheView kc, vc;
  const int32_t* seq_lens;
  int batch, max_seq_len;
  float scale;
  int n_splits;  // resolved; kSplitsFlat: the persistent instance
  void* workspace;
  size_t counter_bytes;
  ResidualView res;
  float* out;
  hipStream_t stream;
};

template <int SUB, int NW, bool POW2, bool PAGED, bool FLAT, bool DQ, bool SGN = false, bool ROPE = false,
          bool MANY = SGN || ROPE>
static int launch_one(const Call& c) {
  const Geometry& g = c.g;
  int n_splits = c.n_splits;
  const int n_rep = g.n_q_heads / g.n_kv_heads, unit_heads = g.n_kv_heads * (n_rep > 4 ? 2 : 1);
  using SM = Smem<NW, ROPE>;
  const size_t smem = c.res.k != nullptr ? (size_t)SM::kBytesRes : (size_t)SM::kBytes;
  static const int attr_rc = [] {
    // the gathers address the codebook table by absolute LDS address: it must start at 0, i.e. the
    // kernel may not own any static LDS in front of its dynamic block
    hipFuncAttributes fa;
    const void* fn = reinterpret_cast<const void*>(dec_tile_kernel<SUB, NW, POW2, PAGED, FLAT, DQ, SGN, ROPE, MANY>);
    if (hipFuncGetAttributes(&fa, fn) != hipSuccess || fa.sharedSizeBytes != 0) return (int)NSN_ERR_HIP;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SM::kBytesRes) != hipSuccess)
      return (int)NSN_ERR_HIP;
    return (int)NSN_OK;
  }();  // initialised once, thread-safe
  if (attr_rc != NSN_OK) return attr_rc;
  int* counters = static_cast<int*>(c.workspace);
  float* partial = reinterpret_cast<float*>(static_cast<unsigned char*>(c.workspace) + c.counter_bytes);
  int per = 0;
  dim3 grid;
  if constexpr (FLAT) {
    // one workgroup per compute unit, never more runs than the workspace has partial slots for
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
      return NSN_ERR_HIP;
    const int64_t groups_max = (int64_t)c.batch * unit_heads * max(1, (c.max_seq_len + 63) / 64);
    n_splits = (int)std::min<int64_t>(std::min(n_cu, kFlatRunsMax), groups_max);
    grid = dim3(n_splits, 1, 1);
  } else {
    per = (((c.max_seq_len + n_splits - 1) / n_splits) + 63) & ~63;
    grid = dim3(n_splits, unit_heads, c.batch);
  }
  dec_tile_kernel<SUB, NW, POW2, PAGED, FLAT, DQ, SGN, ROPE, MANY><<<grid, NW * 64, smem, c.stream>>>(
      g, (const __half*)c.codebook, (const __half*)c.q, c.kc, c.vc, c.seq_lens, c.out, c.batch,
      c.scale * 1.44269504088896340736f, n_splits, per, n_rep, partial, counters, c.res);
  return hipGetLastError() == hipSuccess ? NSN_OK : NSN_ERR_HIP;
}

// the instance of the tiled code layout that fits the call
template <bool MANY>
static int launch_tiled(const Call& c, int sub_dim) {
  const Geometry& g = c.g;
  const bool pow2 = (g.group_size <= 0 || g.group_shift >= 0) && (!g.paged || g.page_shift >= 0);
  auto with_flags = [&](auto sub, auto flat, auto dq) {
    constexpr int kSub = decltype(sub)::value;
    constexpr bool kFlat = decltype(flat)::value, kDq = decltype(dq)::value;
    if (g.paged)
      return pow2 ? launch_one<kSub, 8, true, true, kFlat, kDq, false, false, MANY>(c)
                  : launch_one<kSub, 8, false, true, kFlat, kDq, false, false, MANY>(c);
    return pow2 ? launch_one<kSub, 8, true, false, kFlat, kDq, false, false, MANY>(c)
                : launch_one<kSub, 8, false, false, kFlat, kDq, false, false, MANY>(c);
  };
  auto with_sub = [&](auto flat) {
    if (g.dq)
      return sub_dim == 4 ? with_flags(std::integral_constant<int, 4>{}, flat, std::true_type{})
                          : with_flags(std::integral_constant<int, 8>{}, flat, std::true_type{});
    return sub_dim == 4 ? with_flags(std::integral_constant<int, 4>{}, flat, std::false_type{})
                        : with_flags(std::integral_constant<int, 8>{}, flat, std::false_type{});
  };
  // n_splits == kSplitsFlat: the persistent instance that cuts the list of all groups into equal runs
  return c.n_splits == kSplitsFlat ? with_sub(std::true_type{}) : with_sub(std::false_type{});
}

}  // namespace tile

int decode_many_heads_launch(const tile::Call& c, int sub_dim);  // tiled code layout, five to eight query heads per kv head
int decode_rows_launch(const tile::Call& c, int sub_dim);  // the instances of the legacy code layout

}  // namespace nsn
