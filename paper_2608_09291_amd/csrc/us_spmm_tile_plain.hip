// Instantiations of the tile kernel: 4-bit weights, rows in stored order.
#include "us_spmm_tile.h"

namespace us_spmm_detail {

hipError_t launch_tile_plain(int idx, const TileArgs &t, hipStream_t s) { return launch_tile_cfg<false, 4>(idx, t, s); }

}  // namespace us_spmm_detail
