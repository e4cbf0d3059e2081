// Host side of the matrix-core decode attention: workspace, split choice, and the kernel instances of the tiled code layout
// (index-only codes, keys taken as given) for up to four query heads per kv head.
#include "nsn_decode_tile.h"

namespace nsn {

// arrival counters sit at the head of the workspace: one per (sequence, query head), each on a 256-byte
// line of its own (atomic updates of one line are served one after the other, wherever in the line they fall)
size_t decode_counter_bytes(const nsn_shape& s, int batch) {
  return (size_t)batch * s.n_q_heads * kCounterStrideInts * sizeof(int);
}

// a unit is (sequence, kv head, up to four query heads of it)
static int decode_units(const nsn_shape& s, int batch) {
  return max(1, batch * s.n_kv_heads * (s.n_q_heads / s.n_kv_heads > 4 ? 2 : 1));
}

// Splits per unit of the one-workgroup-per-split instance.  A workgroup has a compute unit to itself
// (its LDS holds the codebook table) and the chip has 256 of them (the persistent launch, whose grid must not exceed
// them, asks the device), so the count is rounded down: one workgroup too many costs a whole second round
// (2-bit, 100 units x 8192 tokens: 17.3 us with two splits, 23.5 with three; with lengths of one kind and another, which the
// host does not know, the second round is not whole: 96 units of 818 to 3934 tokens 11.2 and 11.0 us).  Eight groups or fewer are one per wave
// and need no merge across workgroups (512 tokens: 6.2 us, 7.2 in four splits); beyond that a split gets eight groups,
// one per wave, but a unit at least four splits (the merge is paid by then: 1024 tokens in 2 / 4 splits 7.6 / 7.3 us,
// 8192 tokens in 16 / 32 splits 9.6 / 9.9 us).  More than 32 partials are read in two trips: only for very long contexts
// (32768 tokens in 32 / 64 splits 12.0 / 13.7 us, 131072 tokens 19.4 / 17.9 us).
int decode_tile_split_count(const nsn_shape& s, int batch, int max_seq_len) {
  const int units = decode_units(s, batch), groups = max(1, (max_seq_len + 63) / 64);
  const int useful = groups <= 8 ? 1 : min(groups > 1024 ? 64 : 32, max(4, (groups + 7) / 8));
  return max(1, min(useful, 256 / units));
}

// The persistent instance evens out ragged batches and unit counts that are no multiple of the compute units, but each
// segment of a run costs it more than a fresh workgroup does.  Both instances are priced in the time that eight waves
// take for one group each (1.1 to 3 us by format):
//   splits:      rounds of workgroups x (4 for the prologue and the merge + groups per wave)
//   persistent:  3 + 5 per segment of a run + an equal share of all groups (of about 0.7 of the longest sequence's, where
//                a batch has several: the lengths are on the device)
// Measured (us, splits / persistent), 2-bit: 256 units x 1000 tokens 8.5 / 11.2, 512 x 2000 21.2 / 25.4, 320 x 8192
// 57 / 47, 256 x 16384 62 / 64, the same with lengths from a quarter up 47 / 46; sign format, 320 x 4000 42 / 36.
int decode_tile_splits(const nsn_shape& s, int batch, int max_seq_len, int requested) {
  if (requested > 0) return min(requested, 64);
  const int splits = decode_tile_split_count(s, batch, max_seq_len);
  const int units = decode_units(s, batch), groups = max(1, (max_seq_len + 63) / 64);
  const int per_wave = (groups + 8 * splits - 1) / (8 * splits), rounds = (units * splits + 255) / 256;
  const double split_cost = (double)rounds * (4 + per_wave);
  const double flat_cost = 3 + 5 * (1 + units / 256.0) + (batch > 1 ? 0.7 : 1.0) * units * groups / (256.0 * 8);
  return flat_cost < split_cost ? kSplitsFlat : splits;
}

// one split: no partial results.  kSplitsFlat: two partials per run and query head of a unit, which is at least what
// an automatic split count takes (units x splits <= 256): the size for automatic splitting at any length
size_t decode_tile_workspace_bytes(const nsn_shape& s, int batch, int n_splits) {
  const size_t partials = n_splits == kSplitsFlat ? (size_t)kFlatRunsMax * 2 * min(4, s.n_q_heads / s.n_kv_heads)
                          : n_splits == 1         ? 0
                                                  : (size_t)batch * s.n_q_heads * n_splits;
  return decode_counter_bytes(s, batch) + partials * tile::kPartialStride * sizeof(float);
}

int decode_tile_launch(const nsn_shape& s, const void* codebook, const void* q, const nsn_cache& kc,
                       const nsn_cache& vc, const int32_t* seq_lens, int batch, int max_seq_len, float scale,
                       int n_splits, void* workspace, const nsn_residual* residual, float* out, hipStream_t stream) {
  const Geometry g = make_geometry(s);
  tile::Call c = {g, codebook, q, make_view(kc), make_view(vc), seq_lens, batch, max_seq_len, scale, n_splits, workspace,
                  decode_counter_bytes(s, batch), {nullptr, nullptr, nullptr, 0}, out, stream};
  if (residual)
    c.res = {static_cast<const __half*>(residual->k_fp16), static_cast<const __half*>(residual->v_fp16),
             residual->lens, residual->capacity};
  if (!g.tiled) return decode_rows_launch(c, s.sub_dim);
  return s.n_q_heads / s.n_kv_heads > 4 ? decode_many_heads_launch(c, s.sub_dim) : tile::launch_tiled<false>(c, s.sub_dim);
}

}  // namespace nsn
