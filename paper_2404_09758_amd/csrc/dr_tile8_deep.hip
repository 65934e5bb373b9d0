// dr_tile8_deep.hip -- the semi-transparent tile kernels of 8-pixel tiles.
#include "dr_tile.h"

template hipError_t launch_tile_deep_t<8>(hipStream_t, const TileArgs&, int, dim3);
