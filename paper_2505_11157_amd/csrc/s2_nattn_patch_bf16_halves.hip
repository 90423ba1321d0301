// Patch kernels of bf16 tensors, staging mode kHalves.
#include "s2_nattn_patch_impl.h"

template struct PatchKernels<unsigned short, kHalves>;
