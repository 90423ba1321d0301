// fp32 band-tile kernels: bf16 tensors, rows staged four columns at a time.
#include "s2_nattn_band_impl.h"

template struct BandSet<bf16raw, kWide>;
