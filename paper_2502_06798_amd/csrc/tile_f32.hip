// The tiled similarity kernel for f32 rows.
#include "tile_kernel.h"

namespace apc {

hipError_t launch_tile_f32(int bq, const TileArgs& a, hipStream_t s) { return tile_dispatch<APC_F32>(bq, a, s); }

}  // namespace apc
