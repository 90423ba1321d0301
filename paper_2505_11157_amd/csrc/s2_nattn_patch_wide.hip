// float32 patch kernels, staging mode kWide.
#include "s2_nattn_patch_impl.h"

template struct PatchSet<kWide>;
