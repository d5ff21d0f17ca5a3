// The tiled similarity kernel for e4m3 rows.
#include "tile_kernel.h"

namespace apc {

hipError_t launch_tile_e4m3(int bq, const TileArgs& a, hipStream_t s) { return tile_dispatch<APC_E4M3>(bq, a, s); }

}  // namespace apc
