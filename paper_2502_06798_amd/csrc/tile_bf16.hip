// The tiled similarity kernel for bf16 rows.
#include "tile_kernel.h"

namespace apc {

hipError_t launch_tile_bf16(int bq, const TileArgs& a, hipStream_t s) { return tile_dispatch<APC_BF16>(bq, a, s); }

}  // namespace apc
