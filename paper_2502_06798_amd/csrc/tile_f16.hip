// The tiled similarity kernel for f16 rows.
#include "tile_kernel.h"

namespace apc {

hipError_t launch_tile_f16(int bq, const TileArgs& a, hipStream_t s) { return tile_dispatch<APC_F16>(bq, a, s); }

}  // namespace apc
