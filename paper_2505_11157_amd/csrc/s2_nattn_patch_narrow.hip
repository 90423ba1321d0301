// float32 patch kernels, staging mode kNarrow.
#include "s2_nattn_patch_impl.h"

template struct PatchSet<kNarrow>;
