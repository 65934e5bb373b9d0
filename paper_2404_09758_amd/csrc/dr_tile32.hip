// dr_tile32.hip -- the opaque tile kernels of 32-pixel tiles.
#include "dr_tile.h"

template hipError_t launch_tile_t<32>(hipStream_t, const TileArgs&, int, dim3);
template hipError_t launch_batch_tile_t<32>(hipStream_t, const BatchArgs&, unsigned);
