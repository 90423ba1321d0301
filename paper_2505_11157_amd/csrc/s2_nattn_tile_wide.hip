// bf16 matrix-core tile kernels: staging mode kWide.
#include "s2_nattn_tile_impl.h"

template struct TileSet<kWide>;
