// bf16 matrix-core tile kernels: staging mode kRagged.
#include "s2_nattn_tile_impl.h"

template struct TileSet<kRagged>;
