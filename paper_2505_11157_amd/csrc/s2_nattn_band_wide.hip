// fp32 band-tile kernels: rows staged four columns at a time.
#include "s2_nattn_band_impl.h"

template struct BandSet<kWide>;
