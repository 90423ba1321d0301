// fp32 band-tile kernels: bf16 tensors, rows staged column by column.
#include "s2_nattn_band_impl.h"

template struct BandSet<bf16raw, kNarrow>;
