// Instantiations of the tile kernel: row-reordered 4-bit weights (Section V-B).
#include "us_spmm_tile.h"

namespace us_spmm_detail {

hipError_t launch_tile_perm(int idx, const TileArgs &t, hipStream_t s) { return launch_tile_cfg<true, 4>(idx, t, s); }

}  // namespace us_spmm_detail
