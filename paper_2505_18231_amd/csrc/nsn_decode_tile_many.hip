// Kernel instances of the tiled code layout for five to eight query heads per kv head.
#include "nsn_decode_tile.h"

namespace nsn {

int decode_many_heads_launch(const tile::Call& c, int sub_dim) { return tile::launch_tiled<true>(c, sub_dim); }

}  // namespace nsn
