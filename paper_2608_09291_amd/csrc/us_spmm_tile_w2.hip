// Instantiations of the tile kernel: 2-bit weights (the W2A4 setting of Section VII).
#include "us_spmm_tile.h"

namespace us_spmm_detail {

hipError_t launch_tile_w2(int idx, const TileArgs &t, hipStream_t s) { return launch_tile_cfg<false, 2>(idx, t, s); }

}  // namespace us_spmm_detail
