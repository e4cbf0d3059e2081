// Kernel instances of the legacy code layout: the sign + index format, and every format with keys normalised before the rotary
// embedding.  (Group and page indices by reciprocals for all sizes, powers of two among them: half as many instances.)
// All but six rotary instances, all of them paged, fit in 256 registers; those spill 2 to 9 of them (persistent, sign codes and
// 4-bit side information most).
#include "nsn_decode_tile.h"

namespace nsn {

int decode_rows_launch(const tile::Call& c, int sub_dim) {
  const Geometry& g = c.g;
  auto run = [&](auto sub, auto sgn, auto rope) {
    constexpr int kSub = decltype(sub)::value;
    constexpr bool kSgn = decltype(sgn)::value, kRope = decltype(rope)::value;
    auto with_flat = [&](auto paged, auto dq) {
      constexpr bool kPaged = decltype(paged)::value, kDq = decltype(dq)::value;
      return c.n_splits == kSplitsFlat ? tile::launch_one<kSub, 8, false, kPaged, true, kDq, kSgn, kRope>(c)
                                       : tile::launch_one<kSub, 8, false, kPaged, false, kDq, kSgn, kRope>(c);
    };
    if (g.dq) return g.paged ? with_flat(std::true_type{}, std::true_type{}) : with_flat(std::false_type{}, std::true_type{});
    return g.paged ? with_flat(std::true_type{}, std::false_type{}) : with_flat(std::false_type{}, std::false_type{});
  };
  constexpr std::integral_constant<int, 4> four{};
  constexpr std::integral_constant<int, 8> eight{};
  if (g.sign) return g.rope ? run(eight, std::true_type{}, std::true_type{}) : run(eight, std::true_type{}, std::false_type{});
  return sub_dim == 4 ? run(four, std::false_type{}, std::true_type{}) : run(eight, std::false_type{}, std::true_type{});
}

}  // namespace nsn
