// fp32 band-tile kernels: rows staged column by column, any channel count up to 64.
#include "s2_nattn_band_impl.h"

template struct BandSet<kRagged>;
