// Patch kernels of float32 tensors, staging mode kHalves.
#include "s2_nattn_patch_impl.h"

template struct PatchKernels<float, kHalves>;
