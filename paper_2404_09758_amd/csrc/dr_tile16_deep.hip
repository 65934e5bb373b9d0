// dr_tile16_deep.hip -- the semi-transparent tile kernels of 16-pixel tiles.
#include "dr_tile.h"

template hipError_t launch_tile_deep_t<16>(hipStream_t, const TileArgs&, int, dim3);
