// float32 patch kernels, staging mode kRagged.
#include "s2_nattn_patch_impl.h"

template struct PatchSet<kRagged>;
