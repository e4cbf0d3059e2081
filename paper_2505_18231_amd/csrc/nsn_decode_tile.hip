// Host side of the matrix-core decode attention: workspace, split choice, and the kernel instances of the tiled code layout
// (index-only codes, keys taken as given).
#include "nsn_decode_tile.h"

namespace nsn {

// arrival counters sit at the head of the workspace: one per (sequence, query head), each on a 256-byte
// line of its own (atomic updates of one line are served one after the other, wherever in the line they fall)
size_t decode_counter_bytes(const nsn_shape& s, int batch) {
  return (size_t)batch * s.n_q_heads * kCounterStrideInts * sizeof(int);
}

int decode_tile_splits(const nsn_shape& s, int batch, int max_seq_len, int requested) {
  const int cap = max(1, min(64, (max_seq_len + 255) / 256));
  if (requested > 0) return min(requested, 64);
  const int units = max(1, batch * s.n_kv_heads);
  // Half a chip's worth of units or more: splitting cannot even out a ragged batch any further (a split is a
  // workgroup with its own table and epilogue), the persistent instance can
  if (units >= 128) return kSplitsFlat;
  return max(1, min(cap, (256 + units - 1) / units));  // one 8-wave workgroup per compute unit
}

size_t decode_tile_workspace_bytes(const nsn_shape& s, int batch, int n_splits) {
  // kSplitsFlat: two partials per run and query head of a kv head
  const size_t partials = n_splits == kSplitsFlat ? (size_t)kFlatRunsMax * 2 * (s.n_q_heads / s.n_kv_heads)
                                                  : (size_t)batch * s.n_q_heads * n_splits;
  return decode_counter_bytes(s, batch) + partials * tile::kPartialStride * sizeof(float);
}

int decode_tile_launch(const nsn_shape& s, const void* codebook, const void* q, const nsn_cache& kc,
                       const nsn_cache& vc, const int32_t* seq_lens, int batch, int max_seq_len, float scale,
                       int n_splits, void* workspace, const nsn_residual* residual, float* out, hipStream_t stream) {
  const Geometry g = make_geometry(s);
  tile::Call c = {g, codebook, q, make_view(kc), make_view(vc), seq_lens, batch, max_seq_len, scale, n_splits, workspace,
                  decode_counter_bytes(s, batch), {nullptr, nullptr, nullptr, 0}, 0, 0, out, stream};
  if (residual)
    c.res = {static_cast<const __half*>(residual->k_fp16), static_cast<const __half*>(residual->v_fp16),
             residual->lens, residual->capacity};
  const int r_total = s.n_q_heads / s.n_kv_heads;
  // up to four query heads per kv head in one launch; five to eight as two launches on the same stream
  for (c.head_off = 0; c.head_off < r_total; c.head_off += 4) {
    c.r_pass = min(4, r_total - c.head_off);
    int rc;
    if (!g.tiled) {
      rc = decode_rows_launch(c, s.sub_dim);
    } else {
      const bool pow2 = (g.group_size <= 0 || g.group_shift >= 0) && (!g.paged || g.page_shift >= 0);
      auto with_flags = [&](auto sub, auto flat, auto dq) {
        constexpr int kSub = decltype(sub)::value;
        constexpr bool kFlat = decltype(flat)::value, kDq = decltype(dq)::value;
        if (g.paged)
          return pow2 ? tile::launch_one<kSub, 8, true, true, kFlat, kDq>(c) : tile::launch_one<kSub, 8, false, true, kFlat, kDq>(c);
        return pow2 ? tile::launch_one<kSub, 8, true, false, kFlat, kDq>(c) : tile::launch_one<kSub, 8, false, false, kFlat, kDq>(c);
      };
      auto with_sub = [&](auto flat) {
        if (g.dq)
          return s.sub_dim == 4 ? with_flags(std::integral_constant<int, 4>{}, flat, std::true_type{})
                                : with_flags(std::integral_constant<int, 8>{}, flat, std::true_type{});
        return s.sub_dim == 4 ? with_flags(std::integral_constant<int, 4>{}, flat, std::false_type{})
                              : with_flags(std::integral_constant<int, 8>{}, flat, std::false_type{});
      };
      // n_splits == kSplitsFlat: the persistent instance that cuts the list of all groups into equal runs
      rc = n_splits == kSplitsFlat ? with_sub(std::true_type{}) : with_sub(std::false_type{});
    }
    if (rc != NSN_OK) return rc;
  }
  return NSN_OK;
}

}  // namespace nsn
