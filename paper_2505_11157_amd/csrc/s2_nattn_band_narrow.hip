// fp32 band-tile kernels: rows staged column by column.
#include "s2_nattn_band_impl.h"

template struct BandSet<kNarrow>;
